// Verify attention, the general path (gfx950): fp32 tensors (the small-case / reference-precision configuration), and
// bf16 / fp8-e4m3 storage at the head dimensions the MFMA kernels are not written for (64 and 256).  Results are
// fp32-accurate for every storage type: products are exact or fp32, sums fp32.
//
// Work unit: a workgroup owns RB x 16 query rows of one (request, kv head) -- rows that share a kv head, so a key is
// read once for all of them -- and walks their visible keys: the request's prefix through the block table, the part of
// the drafted chain / pool the rows' branches see, and the tokens of the rows' own branches (Algorithm 1: a branch sees
// the shared prefix, the drafted steps before it and only its own continuation).  The keys are dealt out to the
// wavefronts in blocks of kKeys; every wavefront keeps its own online softmax state and the NW states are folded through
// LDS at the end.  Where rows and heads alone leave the chip idle, and the caller brought the workspace, the prefix is cut
// into chunks reduced by workgroups of their own (make_general_plan), whose partials the merge kernel combines; without a
// workspace one workgroup walks a row block's whole prefix and writes its result.
//
// Both contractions run on the matrix cores, S^T = K Q^T and O^T += V^T P^T (16 x 16 tiles):
//   * bf16 / fp8 storage: K and V are bf16 operands as stored (fp8 widened, exact) and so is Q, unscaled -- the score
//     scale multiplies the fp32 scores, so nothing is rounded before the softmax.  A probability (fp32) is split into
//     three bf16 terms p = hi + mid + lo by truncation, which is exact (24 significand bits = 3 x 8): three MFMAs per
//     V operand, at the fp32 sum's precision and an eighth of the cost of fp32 matrix instructions.
//   * fp32 storage: v_mfma_f32_16x16x4_f32.
// A wavefront shares nothing until the fold, so the loop has no barrier.  K goes global -> LDS directly
// (global_load_lds_dwordx4: 1 KiB of consecutive key rows, so that the address unit sees whole cache lines; operands read
// straight from global memory would touch 16 rows per instruction, which measured three times slower) into a ring of the
// wavefront's own, a block ahead of its use, and is read back as 16-byte operand pieces; piece p of key k lies in slot
// p ^ swz(k), which makes those reads free of bank conflicts.  V^T, which wants several keys of one head-dim column per
// lane, comes straight into registers: a lane reads the same D/16 neighbouring columns of several key rows (contiguous
// over the 16 lanes of a group) and pairs the rows up with byte permutes.  The keys of a block are numbered so that the
// accumulator registers of S^T are the P^T operand.
//
// What bounds it: vector instruction issue (exponentials and the three-term split, about eleven issue slots per score)
// next to the matrix cores; at one row block per workgroup the K/V stream out of L2 as well, so bf16 / fp8 calls at
// head dimension 64 take two row blocks that share every operand (8190 keys, 8 kv heads, 512 rows each, bf16, unsplit:
// 33 us with one row block in 256 workgroups, 41 us with two in 128; split to fill the chip: 35 and 30 us with the
// merge).  Measured, MI355X, against one wavefront per query row (what this kernel replaces): that case 3610 -> 30 us;
// fp32, 256 keys, 64 rows, head dimension 64: 84 -> 9 us with launch; head dimension 256, bf16, 8192 keys, 16 rows x 4 kv
// heads: 87 us unsplit, 19.5 us in chunks.
#include <mutex>
#include <type_traits>

#include "attn_common.hpp"

namespace la {
namespace {

template <int T>
constexpr int kBytes = T == LA_F32 ? 4 : T == LA_BF16 ? 2 : 1;

// N consecutive 32-bit words (N a power of two, address aligned to min(16, 4N) bytes)
template <int N>
__device__ __forceinline__ void load_words(const uint8_t *at, uint32_t (&w)[N]) {
  if constexpr (N == 1) {
    w[0] = *(const uint32_t *)at;
  } else if constexpr (N == 2) {
    const u32x2 v = *(const u32x2 *)at;
    w[0] = v[0], w[1] = v[1];
  } else {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const u32x4 v = *(const u32x4 *)(at + 16 * i);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[4 * i + j] = v[j];
    }
  }
}

// How tokens of storage type T are held, D head dimensions.  Lane (m, kg) = (lane & 15, lane >> 4).
//   bf16 / fp8: blocks of 32 keys in two halves of 16.  K operand t of half h: key 16 h + m, eight head dims
//     from General::dim0; V: key rows 16 (e / 4) + 4 kg + e % 4, e = 0..7, columns m D/16 .. +D/16.
//   fp32: blocks of 16 keys.  K: key m, head dims kg D/4 .. +D/4.  V: key rows 4 kg + e, e = 0..3, the same columns.
template <int D, int T>
struct Store {
  static constexpr bool kF32 = T == LA_F32;
  static constexpr int kRow = D * kBytes<T>;            // bytes per key row
  static constexpr int kPieces = kRow / 16;
  static constexpr int kKeys = kF32 ? 16 : 32;
  static constexpr int kLoads = kKeys * kRow / 1024;    // direct loads per K block
  static constexpr int kVRows = kF32 ? 4 : 8;
  static constexpr int kVWords = D / 16 * kBytes<T> / 4;
  // slot of piece 0 of key row k: 16 consecutive keys at one piece must fall into 16 different slots of 256 bytes
  static __device__ __forceinline__ int swz(int k) {
    constexpr int rows = kPieces >= 16 ? 1 : 16 / kPieces;
    return (k / rows) & ((kPieces < 16 ? kPieces : 16) - 1);
  }
  // piece that holds K operand t (fp8: two operands per piece; fp32: four); see dim0
  static __device__ __forceinline__ int piece(int dim) { return dim * kBytes<T> / 16; }
};
template <int D, int T>
struct RawV {
  uint32_t v[Store<D, T>::kVRows][Store<D, T>::kVWords];
};

enum Segment { SEG_PREFIX = 0, SEG_CHAIN, SEG_BRANCH };

// eight stored elements as a bf16 operand (fp8: widened)
template <int T>
__device__ __forceinline__ bf16x8 operand8(const u32x4 &w, int half) {
  u32x4 v = w;
  if constexpr (T == LA_FP8_E4M3) {
    const uint32_t a = half ? w[2] : w[0], b = half ? w[3] : w[1];
    v = u32x4{fp8x2_to_bf16x2<false>(a), fp8x2_to_bf16x2<true>(a), fp8x2_to_bf16x2<false>(b), fp8x2_to_bf16x2<true>(b)};
  }
  return __builtin_bit_cast(bf16x8, v);
}

// 16 bytes per lane global -> LDS, the wavefront's 64 pieces landing at lds_addr + 16 lane (see attn_stream.hip); the
// caller waits for the vector memory counter and fences before it reads them
__device__ __forceinline__ void load_lds16(const uint8_t *src, uint32_t lds_addr) {
  lds_addr = __builtin_amdgcn_readfirstlane(lds_addr);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(lds_addr) : "m0");
}
// the compiler keeps LDS accesses on their side of this; no instruction
__device__ __forceinline__ void order_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
// Direct loads are ordered with LDS reads by nothing but counters: before a load may overwrite a stage, the reads of
// what it held have to have returned.  (Free where a result that depends on all of them is needed first anyway.)
__device__ __forceinline__ void wait_reads() {
  order_lds();
  __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0), the other counters left at their maxima
}
// The direct loads have landed, and the LDS reads before them have returned.
__device__ __forceinline__ void wait_loads() {
  order_lds();
  __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
  order_lds();
}

// high halves of two fp32 words = two bf16 by truncation
__device__ __forceinline__ uint32_t high_halves(float a, float b) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a), 0x07060302u);
}
__device__ __forceinline__ float trunc_bf16(float x) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & 0xffff0000u);
}

// Maximum and sum over the 16 lanes of a DPP row, in every lane of it.
template <int ROT>
__device__ __forceinline__ float row_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + ROT, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, row_rotate<8>(v));
  v = fmaxf(v, row_rotate<4>(v));
  v = fmaxf(v, row_rotate<2>(v));
  return fmaxf(v, row_rotate<1>(v));
}
__device__ __forceinline__ float row_sum(float v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  return v + row_rotate<1>(v);
}

// D: head dimension; KV, BR: storage type of the prefix cache and of the branch / chain / pool K and V; RB: blocks of
// 16 rows; NW: wavefronts.
template <int D, int KV, int BR, int RB, int NW>
struct General {
  static constexpr bool kF32 = KV == LA_F32;
  static constexpr int kKeys = kF32 ? 16 : 32;        // keys per block
  static constexpr int kTiles = kKeys / 16;           // S^T tiles per block
  static constexpr int kCols = D / 16;                // head-dim columns per lane = O^T tiles
  static constexpr int kQ = kF32 ? D / 4 : D / 32;    // Q operands per row block
  using QOp = typename std::conditional<kF32, float, bf16x8>::type;
  static constexpr bool kQLds = D == 256;             // Q operands in LDS (the registers hold O, K and V then)
  static constexpr int kRowPad = D + 4;               // fold buffer: floats per row
  static constexpr int kFoldBytes = NW * RB * 16 * (kRowPad + 2) * 4;
  static constexpr int kStageBytes = kKeys * D * (kBytes<KV> > kBytes<BR> ? kBytes<KV> : kBytes<BR>);   // of one wavefront
  static constexpr int kStages = D == 256 ? 1 : 2;
  static constexpr int kQBytes = kQLds ? RB * 16 * D * (kF32 ? 4 : 2) : 0;
  static constexpr int kLds = NW * kStages * kStageBytes + kQBytes > kFoldBytes ? NW * kStages * kStageBytes + kQBytes : kFoldBytes;

  // First head dim of operand t of lane group kg, for Q and for K of either storage type: neighbouring operands are the
  // two halves of an fp8 piece where the cache is fp8.
  static __device__ __forceinline__ int dim0(int t, int kg) {
    if constexpr (kF32) return kg * (D / 4) + t;
    else if constexpr (KV == LA_BF16) return 32 * t + 8 * kg;
    else return 64 * (t / 2) + 16 * kg + 8 * (t & 1);
  }

  const AttnParams &p;
  int lane, wave, m, kg, b, kvh, P, gl;
  const int32_t *table;
  QOp q[kQLds ? 1 : RB][kQLds ? 1 : kQ];
  uint8_t *q_lds;          // kQLds: 16-byte pieces [row block][piece][lane]
  uint8_t *ring;           // this wavefront's K stages
  uint32_t ring_lds;       // its LDS address
  f32x4 o[RB][kCols];      // O^T: column tile c, register i: head dim kCols (4 kg + i) + c, row m
  float m_run[RB], l_run[RB];
  int row_tok[RB], row_bstart[RB], vis[RB];
  uint64_t seen[RB];
  float c_pre, c_br, v_pre, v_br;  // score scale (log2 units) and value scale of the prefix and of the other tokens
  bool tree;

  __device__ __forceinline__ General(const AttnParams &params) : p(params) {}

  // element index of token `tok`'s row of this kv head
  template <int SEG>
  __device__ __forceinline__ size_t row_index(int tok) const {
    if constexpr (SEG == SEG_PREFIX) {
      const int lb = tok >> p.block_shift;
      const int blk = table ? table[lb] : b * p.max_blocks + lb;
      return (((size_t)blk * p.Hkv + kvh) * p.block_size + (tok & (p.block_size - 1))) * D;
    } else if constexpr (SEG == SEG_CHAIN) {
      return (((size_t)b * p.C + tok) * p.Hkv + kvh) * D;
    } else {
      return (((size_t)b * gl + tok) * p.Hkv + kvh) * D;
    }
  }
  // Where the 16 keys of a full half block (a multiple of 16 tokens into the prefix, so inside one cache block) start:
  // wavefront-uniform, read from the table by a scalar load.
  __device__ __forceinline__ size_t half_base(int tok) const {
    typedef const __attribute__((address_space(4))) int32_t *cint_ptr;
    tok = __builtin_amdgcn_readfirstlane(tok);
    const int lb = tok >> p.block_shift;
    const int blk = table ? ((cint_ptr)(uintptr_t)table)[lb] : b * p.max_blocks + lb;
    return (((size_t)blk * p.Hkv + kvh) * p.block_size + (tok & (p.block_size - 1))) * D;
  }

  // K of a full prefix block at element offsets base[half] -> stage
  __device__ __forceinline__ void load_k_full(const size_t (&base)[kTiles], int stage) const {
    using S = Store<D, KV>;
    constexpr int rows = 1024 / S::kRow;   // key rows per load: 1 .. 16, inside one half
#pragma unroll
    for (int j = 0; j < S::kLoads; ++j) {
      const int k = j * rows + lane / S::kPieces;
      const uint32_t off = (uint32_t)(k & 15) * S::kRow + (uint32_t)((lane % S::kPieces) ^ S::swz(k)) * 16;
      load_lds16((const uint8_t *)p.k_cache + base[j * rows / 16] * kBytes<KV> + off, ring_lds + stage * kStageBytes + j * 1024);
    }
  }
  __device__ __forceinline__ void load_v_full(const size_t (&base)[kTiles], RawV<D, KV> &r) const {
    using S = Store<D, KV>;
    constexpr int es = kBytes<KV>;
    const uint32_t off = (uint32_t)(4 * kg * D + m * kCols) * es;
#pragma unroll
    for (int e = 0; e < S::kVRows; ++e)
      load_words<S::kVWords>((const uint8_t *)p.v_cache + base[e / 4] * es + off + (e % 4) * D * es, r.v[e]);
  }
  // any block: tokens first .. of the segment, clamped to `last`
  template <int SEG, int T>
  __device__ __forceinline__ void load_any(int first, int last, RawV<D, T> &r) const {
    using S = Store<D, T>;
    constexpr int es = kBytes<T>;
    const uint8_t *kp = (const uint8_t *)(SEG == SEG_PREFIX ? p.k_cache : SEG == SEG_CHAIN ? p.k_chain : p.k_branch);
    const uint8_t *vp = (const uint8_t *)(SEG == SEG_PREFIX ? p.v_cache : SEG == SEG_CHAIN ? p.v_chain : p.v_branch);
    wait_reads();
#pragma unroll
    for (int j = 0; j < S::kLoads; ++j) {
      const int k = j * (1024 / S::kRow) + lane / S::kPieces;
      load_lds16(kp + row_index<SEG>(min(first + k, last)) * es + ((lane % S::kPieces) ^ S::swz(k)) * 16, ring_lds + j * 1024);
    }
#pragma unroll
    for (int e = 0; e < S::kVRows; ++e)
      load_words<S::kVWords>(vp + (row_index<SEG>(min(first + 16 * (e / 4) + 4 * kg + e % 4, last)) + m * kCols) * es, r.v[e]);
    wait_loads();
  }

  // S^T of one block (K in `stage`): tile h, register i is key 16 h + 4 kg + i of the block against row m of row block rb
  template <int T>
  __device__ __forceinline__ void scores(int stage, f32x4 (&s)[RB][kTiles]) const {
    using S = Store<D, T>;
    const uint8_t *kt = ring + stage * kStageBytes;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int h = 0; h < kTiles; ++h) s[rb][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    // (keys m and 16 + m share the swizzle)
    auto k_piece = [&](int h, int t) __attribute__((always_inline)) {
      return *(const u32x4 *)(kt + (16 * h + m) * S::kRow + (S::piece(dim0(t, kg)) ^ S::swz(m)) * 16);
    };
    // (an offset the compiler cannot see through keeps the LDS reads inside the loop)
    uint32_t q_off = lane * 16;
    if constexpr (kQLds) asm volatile("" : "+v"(q_off));
    if constexpr (kF32) {
#pragma unroll
      for (int t4 = 0; t4 < kQ / 4; ++t4)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          const u32x4 kw = k_piece(0, 4 * t4);
          f32x4 qv;
          if constexpr (kQLds) qv = *(const f32x4 *)(q_lds + (rb * (kQ / 4) + t4) * 1024 + q_off);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t w = kw[j];
            float qj;
            if constexpr (kQLds) qj = qv[j]; else qj = q[rb][4 * t4 + j];
            s[rb][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, w), qj, s[rb][0], 0, 0, 0);
          }
        }
    } else {
      u32x4 k_last[kTiles];
#pragma unroll
      for (int t = 0; t < kQ; ++t) {
        u32x4 kw[kTiles];
        if (T == LA_BF16 || (t & 1) == 0) {
#pragma unroll
          for (int h = 0; h < kTiles; ++h) k_last[h] = k_piece(h, t);
        }
#pragma unroll
        for (int h = 0; h < kTiles; ++h) kw[h] = k_last[h];
        bf16x8 qf[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          if constexpr (kQLds) qf[rb] = *(const bf16x8 *)(q_lds + (rb * kQ + t) * 1024 + q_off); else qf[rb] = q[rb][t];
        }
#pragma unroll
        for (int h = 0; h < kTiles; ++h) {
          const bf16x8 kf = operand8<T>(kw[h], t & 1);
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
            s[rb][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[rb], s[rb][h], 0, 0, 0);
        }
      }
    }
  }

  // The scores become probabilities against the running maximum, which a lane group raises only when a block exceeds
  // it by more than kRaise log2 units (probabilities up to 2^kRaise cost an fp32 sum nothing): the common path exchanges
  // nothing between lanes.  c: score scale.
  __device__ __forceinline__ void softmax(f32x4 (&s)[RB][kTiles], float c) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float mx = s[rb][0][0];
#pragma unroll
      for (int h = 0; h < kTiles; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[rb][h][i]);
      mx *= c;   // (c > 0)
      if (__builtin_amdgcn_ballot_w64(mx > m_run[rb] + kRaise)) {
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));   // the row's block maximum, the same in its four lanes
        const float m_new = fmaxf(m_run[rb], mx);
        const float alpha = __builtin_amdgcn_exp2f(m_run[rb] - (m_new == -INFINITY ? 0.f : m_new));
        m_run[rb] = m_new;
        l_run[rb] *= alpha;
#pragma unroll
        for (int cc = 0; cc < kCols; ++cc) o[rb][cc] *= alpha;
      }
      const float off = m_run[rb] == -INFINITY ? 0.f : -m_run[rb];
      float sum = 0.f;
#pragma unroll
      for (int h = 0; h < kTiles; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s[rb][h][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[rb][h][i], c, off));
          sum += s[rb][h][i];
        }
      l_run[rb] += sum;
    }
  }

  // O^T += V^T P^T; vs: value scale
  template <int T>
  __device__ __forceinline__ void accumulate(const RawV<D, T> &r, f32x4 (&s)[RB][kTiles], float vs) {
    if constexpr (KV == LA_FP8_E4M3) {
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int h = 0; h < kTiles; ++h) s[rb][h] *= vs;
    }
    if constexpr (kF32) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < kCols; ++c)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            const uint32_t w = r.v[e][c];
            o[rb][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, w), s[rb][0][e], o[rb][c], 0, 0, 0);
          }
    } else {
      bf16x8 pt[RB][3];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        u32x4 w[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float a = s[rb][j >> 1][2 * (j & 1)], d = s[rb][j >> 1][2 * (j & 1) + 1];
          w[0][j] = high_halves(a, d);
          a -= trunc_bf16(a), d -= trunc_bf16(d);
          w[1][j] = high_halves(a, d);
          a -= trunc_bf16(a), d -= trunc_bf16(d);
          w[2][j] = high_halves(a, d);
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) pt[rb][x] = __builtin_bit_cast(bf16x8, w[x]);
      }
#pragma unroll
      for (int cw = 0; cw < kCols / 2; ++cw) {   // two columns: the low and the high half of word cw of every key row
        uint32_t row[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if constexpr (T == LA_BF16) {
            row[e] = r.v[e][cw];
          } else {
            const uint32_t w = r.v[e][cw / 2];
            row[e] = (cw & 1) ? fp8x2_to_bf16x2<true>(w) : fp8x2_to_bf16x2<false>(w);
          }
        }
        u32x4 lo, hi;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          lo[j] = __builtin_amdgcn_perm(row[2 * j + 1], row[2 * j], 0x05040100u);
          hi[j] = __builtin_amdgcn_perm(row[2 * j + 1], row[2 * j], 0x07060302u);
        }
        const bf16x8 va = __builtin_bit_cast(bf16x8, lo), vb = __builtin_bit_cast(bf16x8, hi);
#pragma unroll
        for (int x = 2; x >= 0; --x)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            o[rb][2 * cw] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pt[rb][x], o[rb][2 * cw], 0, 0, 0);
            o[rb][2 * cw + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, pt[rb][x], o[rb][2 * cw + 1], 0, 0, 0);
          }
      }
    }
  }

  // a block of another kind than a full prefix block, start to end
  template <int SEG, int T>
  __device__ __forceinline__ void masked_block(int first, int last) {
    RawV<D, T> r;
    load_any<SEG, T>(first, last, r);
    f32x4 s[RB][kTiles];
    scores<T>(0, s);
#pragma unroll
    for (int h = 0; h < kTiles; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int key = first + 16 * h + 4 * kg + i;
        int seg = 0;
        if (SEG == SEG_CHAIN && tree) seg = p.pool_seg[(size_t)b * p.C + min(key, last)];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          bool hide = key > last;
          if constexpr (SEG == SEG_CHAIN) hide |= tree ? !((seen[rb] >> seg) & 1) : key >= vis[rb];
          if constexpr (SEG == SEG_BRANCH) hide |= key > row_tok[rb] || key < row_bstart[rb];
          if (hide) s[rb][h][i] = -INFINITY;
        }
      }
    softmax(s, SEG == SEG_PREFIX ? c_pre : c_br);
    accumulate<T>(r, s, SEG == SEG_PREFIX ? v_pre : v_br);
  }
};

template <int D, int KV, int BR, int RB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_general_kernel(const AttnParams p) {
  using G = General<D, KV, BR, RB, NW>;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float *fold = (float *)lds;   // (the K rings and Q are done with by then)
  G g(p);
  g.q_lds = lds + NW * G::kStages * G::kStageBytes;
  g.lane = threadIdx.x & 63, g.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  g.m = g.lane & 15, g.kg = g.lane >> 4;
  g.ring = lds + g.wave * (G::kStages * G::kStageBytes);
  g.ring_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)g.ring;
  int id = blockIdx.x + p.first_wg;
  g.kvh = __builtin_amdgcn_readfirstlane(id % p.Hkv);
  id = __builtin_amdgcn_readfirstlane(id / p.Hkv);
  const int row_tile = __builtin_amdgcn_readfirstlane(id % p.n_row_tiles);
  ChunkSel sel;
  if (G::kF32 || (p.s_max == 1 && !p.n_inline)) {   // not split: the unit is the request
    sel.b = __builtin_amdgcn_readfirstlane(id / p.n_row_tiles), sel.c = 0, sel.n_chunks = 1, sel.k_begin = 0;
    sel.P = sel.k_end = __builtin_amdgcn_readfirstlane(p.prefix_lens[sel.b]);
  } else {
    sel = attn_select_chunk<true>(p, __builtin_amdgcn_readfirstlane(id / p.n_row_tiles));
  }
  g.b = sel.b, g.P = sel.P;
  const bool last_chunk = sel.c == sel.n_chunks - 1;
  g.gl = p.gamma * p.L;
  g.table = p.block_tables ? p.block_tables + (size_t)g.b * p.max_blocks : nullptr;
  g.tree = p.pool_seg != nullptr;
  {
    float ks = 1.f, vs = 1.f;
    if (KV == LA_FP8_E4M3) ks = p.k_scale ? p.k_scale[g.kvh] : 1.f, vs = p.v_scale ? p.v_scale[g.kvh] : 1.f;
    g.c_pre = p.scale_log2 * ks, g.v_pre = vs;
    g.c_br = BR == LA_FP8_E4M3 ? g.c_pre : p.scale_log2, g.v_br = BR == LA_FP8_E4M3 ? vs : 1.f;
  }
  const int r0 = row_tile * 16 * RB, r1 = min(p.R, r0 + 16 * RB);
  int vis_max = 0;   // chain / pool tokens the tile has to look at
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = min(r0 + 16 * rb + g.m, p.R - 1);   // rows past the last repeat it and are not stored
    const int tok = r / p.G, br = tok / p.L;
    g.row_tok[rb] = tok, g.row_bstart[rb] = br * p.L;
    g.vis[rb] = 0, g.seen[rb] = 0;
    if (p.C > 0) {
      if (g.tree) {
        g.seen[rb] = p.seg_mask[g.b * p.gamma + br];
        vis_max = p.C;
      } else {
        g.vis[rb] = p.chain_vis[g.b * p.gamma + br];
        vis_max = max(vis_max, g.vis[rb]);
      }
    }
    const size_t qrow = (((size_t)g.b * g.gl + tok) * p.Hq + g.kvh * p.G + (r - tok * p.G)) * D;
    if constexpr (G::kF32) {
#pragma unroll
      for (int t = 0; t < G::kQ / 4; ++t) {
        const f32x4 v = *(const f32x4 *)((const float *)p.q + qrow + G::dim0(4 * t, g.kg));
        if constexpr (G::kQLds) {
          if (g.wave == 0) *(f32x4 *)(g.q_lds + (rb * (G::kQ / 4) + t) * 1024 + g.lane * 16) = v;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) g.q[rb][4 * t + j] = v[j];
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < G::kQ; ++t) {
        const bf16x8 v = *(const bf16x8 *)((const uint16_t *)p.q + qrow + G::dim0(t, g.kg));
        if constexpr (G::kQLds) {
          if (g.wave == 0) *(bf16x8 *)(g.q_lds + (rb * G::kQ + t) * 1024 + g.lane * 16) = v;
        } else {
          g.q[rb][t] = v;
        }
      }
    }
    g.m_run[rb] = -INFINITY, g.l_run[rb] = 0.f;
#pragma unroll
    for (int c = 0; c < G::kCols; ++c) g.o[rb][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  if (p.C > 0) {
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) vis_max = max(vis_max, __shfl_xor(vis_max, off));
    vis_max = __builtin_amdgcn_readfirstlane(vis_max);
  }
  if constexpr (G::kQLds) __syncthreads();
  const int t_lo = __builtin_amdgcn_readfirstlane(r0 / p.G), t_hi = __builtin_amdgcn_readfirstlane((r1 - 1) / p.G);
  const int tk0 = __builtin_amdgcn_readfirstlane((t_lo / p.L) * p.L);

  // ---- full prefix blocks: wave, wave + NW, ...
  constexpr int kKeys = G::kKeys;
  // A chunk may hold no prefix key at all (a short prefix beside long branches, attn_chunk_range): its range then starts
  // behind its end, and the blocks are counted from zero.
  const bool any_prefix = sel.k_end > sel.k_begin;
  const int n_full = any_prefix ? sel.k_end / kKeys : 0;   // (chunks start at multiples of 64 keys)
  int blk = (any_prefix ? sel.k_begin / kKeys : 0) + g.wave;
  {
    size_t base[G::kTiles], next[G::kTiles];
    auto bases = [&](int at, size_t (&out)[G::kTiles]) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < G::kTiles; ++h) out[h] = g.half_base(at * kKeys + 16 * h);
    };
    if (blk < n_full) {
      bases(blk, base);
      g.load_k_full(base, 0);
      bases(min(blk + NW, n_full - 1), next);
    }
    int stage = 0;
    for (; blk < n_full; blk += NW) {
      wait_loads();   // this block's K, requested a block ago
      const bool more = blk + NW < n_full;
      if (G::kStages > 1 && more) g.load_k_full(next, stage ^ 1);
      RawV<D, KV> r;
      g.load_v_full(base, r);
      f32x4 s[RB][G::kTiles];
      g.template scores<KV>(stage, s);
      if (G::kStages == 1 && more) {
        wait_reads();
        g.load_k_full(next, 0);
      }
      if (G::kStages > 1) stage ^= 1;
#pragma unroll
      for (int h = 0; h < G::kTiles; ++h) base[h] = next[h];
      bases(min(blk + 2 * NW, n_full - 1), next);
      g.softmax(s, g.c_pre);
      g.template accumulate<KV>(r, s, g.v_pre);
    }
  }
  // ---- the rest, dealt out in the same round: the prefix's last, partial block, chain / pool blocks, branch blocks
  const int n_tail = any_prefix && sel.k_end % kKeys ? 1 : 0, n_chain = last_chunk ? (vis_max + kKeys - 1) / kKeys : 0;
  const int n_own = last_chunk ? (t_hi - tk0 + 1 + kKeys - 1) / kKeys : 0;
  int i = blk - n_full;
  if (n_tail) {
    if (i == 0) {
      g.template masked_block<SEG_PREFIX, KV>(n_full * kKeys, g.P - 1);
      i += NW;
    }
    --i;
  }
  if (p.C > 0)
#pragma unroll 1
    for (; i < n_chain; i += NW) g.template masked_block<SEG_CHAIN, BR>(i * kKeys, vis_max - 1);
  i -= n_chain;
#pragma unroll 1
  for (; i < n_own; i += NW) g.template masked_block<SEG_BRANCH, BR>(tk0 + i * kKeys, t_hi);

  // ---- fold the wavefronts' states: all of them to LDS, then a wavefront per row (and again NW rows on).  The weights of a
  // row's states are formed once, a lane per state, and handed out by lane reads; a lane adds up D / 64 columns.  Measured
  // against a thread per element that forms all weights itself, the row blocks one after the other: head dimension 256,
  // bf16, 822 keys, 28 rows x 2 kv heads 16.2 -> 14.3 us (with the merge), fp32, 35 keys 11.4 -> 9.6 us; at head dimension
  // 64 within a percent.
  constexpr int kRows = RB * 16;
  float *f_m = fold + NW * kRows * G::kRowPad, *f_l = f_m + NW * kRows;   // [wave][row]
  __syncthreads();   // (the K rings and Q are done with)
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    float l = g.l_run[rb];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const int at = g.wave * kRows + 16 * rb + g.m;
    if (g.lane < 16) f_m[at] = g.m_run[rb], f_l[at] = l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // this lane's columns kCols (4 kg + i) .. +kCols of row m
      float *dst = fold + at * G::kRowPad + G::kCols * (4 * g.kg + i);
#pragma unroll
      for (int c = 0; c < G::kCols; c += 4) {
        const f32x4 v = {g.o[rb][c][i], g.o[rb][c + 1][i], g.o[rb][c + 2][i], g.o[rb][c + 3][i]};
        *(f32x4 *)(dst + c) = v;
      }
    }
  }
  __syncthreads();
  constexpr int kE = D / 64;   // columns per lane
  typedef __attribute__((ext_vector_type(kE))) float fvec;
  typedef __attribute__((ext_vector_type(kE))) __bf16 bvec;
#pragma unroll
  for (int row0 = 0; row0 < kRows; row0 += NW) {
    const int row = row0 + g.wave;
    if (kRows % NW && row >= kRows) break;
    static_assert(NW <= 16, "a state per lane of a DPP row");
    const int w_of = g.lane % 16;
    const float m = w_of < NW ? f_m[w_of * kRows + row] : -INFINITY, l = w_of < NW ? f_l[w_of * kRows + row] : 0.f;
    const float mm = row_max(m);
    const float m_use = mm == -INFINITY ? 0.f : mm;   // (a chunk may show a row nothing; its last one shows it itself)
    const float wt = __builtin_amdgcn_exp2f(m - m_use);
    const float den = row_sum(wt * l);
    fvec acc = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float ww = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wt), w));
      const fvec v = *(const fvec *)(fold + (w * kRows + row) * G::kRowPad + kE * g.lane);
#pragma unroll
      for (int e = 0; e < kE; ++e) acc[e] = __builtin_fmaf(ww, v[e], acc[e]);
    }
    const int r = r0 + row;
    if (r >= p.R) continue;
    const int tok = r / p.G;   // (wavefront-uniform)
    const size_t in_req = (size_t)tok * p.Hq + g.kvh * p.G + (r - tok * p.G);
    if (p.part_o) {
      const size_t prow = ((size_t)g.b * p.s_max + sel.c) * p.n_rows + in_req;
      *(fvec *)(p.part_o + prow * D + kE * g.lane) = acc;
      if (g.lane == 0) *(f32x2 *)(p.part_ml + prow * 2) = f32x2{mm, den};
      continue;
    }
    const size_t orow = (size_t)g.b * p.n_rows + in_req;
    const fvec v = acc / den;
    if (p.out_f32)
      *(fvec *)((float *)p.out + orow * D + kE * g.lane) = v;
    else
      *(bvec *)((__bf16 *)p.out + orow * D + kE * g.lane) = __builtin_convertvector(v, bvec);   // round to nearest even
    if (p.lse && g.lane == 0) p.lse[orow] = 0.69314718055994530942f * (mm + __builtin_log2f(den));
  }
}

template <int D, int KV, int BR, int RB, int NW>
hipError_t launch_shape(const AttnParams &p, hipStream_t stream) {
  using G = General<D, KV, BR, RB, NW>;
  auto kern = attn_general_kernel<D, KV, BR, RB, NW>;
  constexpr int kLds = G::kLds;
  static_assert(kLds <= 160 * 1024, "LDS of one CU");
  static std::once_flag once;
  static hipError_t configured = hipSuccess;
  std::call_once(once, [&] {
    configured = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
  });
  if (configured != hipSuccess) return configured;
  if (p.n_row_tiles != (p.R + 16 * RB - 1) / (16 * RB)) return hipErrorInvalidValue;
  const int64_t grid = (int64_t)p.Hkv * p.n_row_tiles * p.total_units;
  if (grid > INT32_MAX) return hipErrorInvalidValue;
  // (a launch holds less than 2^32 threads; the runtime drops what is beyond without an error)
  constexpr int64_t kMaxGrid = 1 << 21;
  AttnParams q = p;
  for (int64_t at = 0; at < grid; at += kMaxGrid) {
    q.first_wg = (int)at;
    const unsigned wgs = (unsigned)(grid - at < kMaxGrid ? grid - at : kMaxGrid);
    hipLaunchKernelGGL(kern, dim3(wgs), dim3(64 * NW), kLds, stream, q);
  }
  return hipGetLastError();
}

template <int KV, int BR>
hipError_t launch_typed(const AttnParams &p, int row_blocks, hipStream_t stream) {
  if constexpr (KV == LA_F32) {
    switch (p.D) {
      case 64: return launch_shape<64, KV, BR, 1, 16>(p, stream);
      case 128: return launch_shape<128, KV, BR, 1, 8>(p, stream);
      case 256: return launch_shape<256, KV, BR, 1, 8>(p, stream);
    }
  } else {
    switch (p.D) {
      case 64: return row_blocks == 2 ? launch_shape<64, KV, BR, 2, 8>(p, stream) : launch_shape<64, KV, BR, 1, 8>(p, stream);
      case 256: return launch_shape<256, KV, BR, 1, 8>(p, stream);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams &p, int row_blocks, hipStream_t stream) {
  ProfileScope scope(SLOT_ATTN_F32, stream);
  if (p.kv_type == LA_F32 && p.br_type == LA_F32) return launch_typed<LA_F32, LA_F32>(p, row_blocks, stream);
  if (p.kv_type == LA_BF16 && p.br_type == LA_BF16) return launch_typed<LA_BF16, LA_BF16>(p, row_blocks, stream);
  if (p.kv_type == LA_FP8_E4M3 && p.br_type == LA_FP8_E4M3) return launch_typed<LA_FP8_E4M3, LA_FP8_E4M3>(p, row_blocks, stream);
  if (p.kv_type == LA_FP8_E4M3 && p.br_type == LA_BF16) return launch_typed<LA_FP8_E4M3, LA_BF16>(p, row_blocks, stream);
  return hipErrorInvalidValue;
}

}  // namespace la
