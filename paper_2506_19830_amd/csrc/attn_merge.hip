// Merge of the split-prefix partials of verify attention (gfx950).
//
// Every (row tile, kv head, chunk) workgroup of the row-tile, streaming and
// general kernels leaves an unnormalised partial (O_s, m_s, l_s) per query row,
// m in log2 units.  The exact softmax over the union of the chunks is
//     M = max_s m_s,   w_s = 2^(m_s - M),   O = sum_s w_s O_s / sum_s w_s l_s,
//     lse = ln2 * (M + log2 sum_s w_s l_s).
// More than eight chunks: one wavefront owns one output row, lane s < n_s loads
// (m_s, l_s), the maximum and the denominator are reductions over the lanes on
// the vector ALU, the weights are then read lane by lane into scalar registers
// while each lane accumulates its D / 64 output columns.  Up to eight: D / 4 threads own a row (below).
#include "la_internal.hpp"

namespace la {
namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kWaves = 4;

// The grid is (row groups of a request, requests, batches of kMaxGridY requests), so that no division by the number of
// rows is needed; the number of partials comes from the kernel arguments where the host has put it there, so that the
// first loads of a wavefront are the partials themselves.
constexpr int kMaxGridY = 65535;
__device__ __forceinline__ int merge_request(const AttnParams &p) { return (int)(blockIdx.y + blockIdx.z * kMaxGridY); }
__device__ __forceinline__ int merge_chunks(const AttnParams &p, int b) {
  return p.n_inline ? p.req[b].n : attn_num_chunks(p.prefix_lens[b], p.chunk_len);
}

// Maximum and sum over a wavefront on the vector ALU, the same value in every lane.
template <int ROT>
__device__ __forceinline__ float row_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + ROT, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_rotate<8>(v));
  v = fmaxf(v, row_rotate<4>(v));
  v = fmaxf(v, row_rotate<2>(v));
  v = fmaxf(v, row_rotate<1>(v));
  return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
// (the halves and the rows first, then inside the rows: the order of a butterfly from lane ^ 32 down to lane ^ 1)
__device__ __forceinline__ float wave_sum(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const auto halves = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t h0 = halves[0], h1 = halves[1];
  const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1));
  const auto rows = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  const uint32_t r0 = rows[0], r1 = rows[1];
  v = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  return v + row_rotate<1>(v);
}

// kGroup: partial rows requested before the first is used.  Bound by the latency of the loads and what hangs on them:
// the first group is requested together with the (m, l) pairs, the reductions run on the vector ALU, and the weights are
// read lane by lane into scalar registers, so a wavefront of up to kGroup chunks waits for one round trip instead of two
// and sends nothing through the LDS (320 rows x 26 chunks: 4.5 -> 3.9 us, 5400 rows x 10: 7.6 -> 7.1 us).
template <int D, int kGroup>
__global__ __launch_bounds__(64 * kWaves) void attn_merge_kernel(const AttnParams p) {
  constexpr int E = D / 64;
  typedef __attribute__((ext_vector_type(E))) float fvec;
  typedef __attribute__((ext_vector_type(E))) __bf16 bvec;
  const int lane = threadIdx.x & 63;
  const int b = merge_request(p);
  const int r = (int)(blockIdx.x * kWaves + (threadIdx.x >> 6));
  if (b >= p.B || r >= p.n_rows) return;
  const size_t grow = (size_t)b * p.n_rows + r;   // row over all requests
  const int n_s = merge_chunks(p, b);
  const size_t slot0 = (size_t)b * p.s_max;
  const size_t stride = (size_t)p.n_rows * D;  // between the partials of consecutive chunks

  fvec acc = 0.f;
  float m_all = -INFINITY, denom = 0.f;
  // more than 64 chunks are folded 64 at a time with the usual running rescale
  for (int s0 = 0; s0 < n_s; s0 += 64) {
    const int cnt = min(64, n_s - s0);
    float m = -INFINITY, l = 0.f;
    if (lane < cnt) {
      const f32x2 ml = *(const f32x2 *)(p.part_ml + ((slot0 + s0 + lane) * p.n_rows + r) * 2);
      m = ml.x;
      l = ml.y;
    }
    const float *po = p.part_o + ((slot0 + s0) * p.n_rows + r) * D + E * lane;
    fvec o[kGroup];
    auto request = [&](int g) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < kGroup; ++j) {
        const int sj = g + j < cnt ? g + j : cnt - 1;   // surplus slots repeat the last chunk with weight zero
        o[j] = *(const fvec *)(po + (size_t)sj * stride);
      }
    };
    request(0);
    const float m_new = fmaxf(m_all, wave_max(m));
    const float w = (lane < cnt) ? __builtin_amdgcn_exp2f(m - m_new) : 0.f;
    const float rescale = __builtin_amdgcn_exp2f(m_all - m_new);  // 0 on the first pass (m_all = -inf)
    acc *= rescale;
    denom = denom * rescale + wave_sum(w * l);
    m_all = m_new;
    // with many chunks this loop is bound by the latency of its loads, so a whole group of partial rows is requested
    // before the first is used (32 rows: 64 registers)
#pragma unroll 1
    for (int g = 0;;) {
#pragma unroll
      for (int j = 0; j < kGroup; ++j) {
        const float ws = lane_value(w, g + j);   // (g + j <= 63; zero behind the last chunk)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = __builtin_fmaf(ws, o[j][e], acc[e]);
      }
      g += kGroup;
      if (g >= cnt) break;
      request(g);
    }
  }
  acc *= 1.0f / denom;
  const size_t orow = grow * D + E * lane;
  if (p.out_f32)
    *(fvec *)((float *)p.out + orow) = acc;
  else
    *(bvec *)((__bf16 *)p.out + orow) = __builtin_convertvector(acc, bvec);
  if (p.lse && lane == 0) p.lse[grow] = 0.69314718055994530942f * (m_all + __builtin_log2f(denom));
}

// Few chunks (at most kFew per request), the usual case with many query rows: D / 4 threads own one row, four output
// columns each.  Every thread forms the weights of its row itself (the (m, l) pairs are one broadcast load each) and
// has all its 16-byte partial loads in flight at once; nothing is exchanged between lanes.  Bound by the read of the
// partials: kFew is the next power of two, since a surplus load costs its issue slots and cache bandwidth although it
// hits (24576 rows x 10 chunks over 4 requests: 38.7 us with eight loads per row, 28.1 us with four; 5.2 TB/s).
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

template <int D, int kFew>
__global__ __launch_bounds__(256) void attn_merge_few_kernel(const AttnParams p) {
  constexpr int kPerRow = D / 4;
  const int b = merge_request(p);
  const int r = (int)(blockIdx.x * (256 / kPerRow) + threadIdx.x / kPerRow);
  if (b >= p.B || r >= p.n_rows) return;
  const size_t grow = (size_t)b * p.n_rows + r;   // row over all requests
  const int col = (threadIdx.x % kPerRow) * 4;
  const int n_s = merge_chunks(p, b);  // <= kFew (checked by the host)
  const size_t slot0 = (size_t)b * p.s_max;
  const size_t stride = (size_t)p.n_rows * D;
  const float *po = p.part_o + (slot0 * p.n_rows + r) * D + col;
  const float *pml = p.part_ml + (slot0 * p.n_rows + r) * 2;

  f32x4 o[kFew];
  float m[kFew], l[kFew];
#pragma unroll
  for (int s = 0; s < kFew; ++s) {
    const int sc = s < n_s ? s : n_s - 1;  // surplus slots repeat the last chunk with weight zero
    o[s] = *(const f32x4 *)(po + (size_t)sc * stride);
    const f32x2 ml = *(const f32x2 *)(pml + (size_t)sc * p.n_rows * 2);
    m[s] = s < n_s ? ml.x : -INFINITY;
    l[s] = ml.y;
  }
  float m_all = m[0];
#pragma unroll
  for (int s = 1; s < kFew; ++s) m_all = fmaxf(m_all, m[s]);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  float denom = 0.f;
#pragma unroll
  for (int s = 0; s < kFew; ++s) {
    const float w = __builtin_amdgcn_exp2f(m[s] - m_all);  // 0 for surplus slots
    denom = __builtin_fmaf(w, l[s], denom);
    acc += o[s] * w;
  }
  const float inv = 1.0f / denom;
  acc *= inv;
  const size_t orow = grow * D + col;
  if (p.out_f32)
    *(f32x4 *)((float *)p.out + orow) = acc;
  else
    *(bf16x4 *)((__bf16 *)p.out + orow) = __builtin_convertvector(acc, bf16x4);
  if (p.lse && col == 0) p.lse[grow] = 0.69314718055994530942f * (m_all + __builtin_log2f(denom));
}

template <int D>
hipError_t launch_merge(const AttnParams &p, hipStream_t stream) {
  auto grid = [&](int rows) {
    return dim3((unsigned)((p.n_rows + rows - 1) / rows), (unsigned)(p.B < kMaxGridY ? p.B : kMaxGridY),
                (unsigned)((p.B + kMaxGridY - 1) / kMaxGridY));
  };
  constexpr int kRows = 256 / (D / 4), kLong = D > 128 ? 16 : 32;
  if (p.s_max <= 2)
    hipLaunchKernelGGL((attn_merge_few_kernel<D, 2>), grid(kRows), dim3(256), 0, stream, p);
  else if (p.s_max <= 4)
    hipLaunchKernelGGL((attn_merge_few_kernel<D, 4>), grid(kRows), dim3(256), 0, stream, p);
  else if (p.s_max <= 8)
    hipLaunchKernelGGL((attn_merge_few_kernel<D, 8>), grid(kRows), dim3(256), 0, stream, p);
  else if (p.s_max <= 16)
    hipLaunchKernelGGL((attn_merge_kernel<D, 16>), grid(kWaves), dim3(64 * kWaves), 0, stream, p);
  else
    hipLaunchKernelGGL((attn_merge_kernel<D, kLong>), grid(kWaves), dim3(64 * kWaves), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_merge(const AttnParams &p, hipStream_t stream) {
  ProfileScope scope(SLOT_ATTN_MERGE, stream);
  switch (p.D) {
    case 64: return launch_merge<64>(p, stream);
    case 128: return launch_merge<128>(p, stream);
    case 256: return launch_merge<256>(p, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace la
