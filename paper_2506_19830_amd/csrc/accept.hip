// Token-level speculative accept / resample over the vocabulary (gfx950).
//
// Section 2 ("Speculative Decoding"): the K drafted tokens of a branch are examined in
// order, x_i accepted with probability min(1, p_i(x_i)/q_i(x_i)); the first rejection n
// stops the walk and one token is drawn from norm(max(0, p_n - q_n)); with all K accepted
// a bonus token is drawn from p_K.
//
// Launches:
//   stats   one coalesced pass over every logit row (NB*(2K+1) rows x V): per (row, slice)
//           the exact maximum and sum 2^((x-max)*log2e/T), fp32.  This is the HBM-bound
//           part: each logit is read exactly once, 16-byte loads, eight in flight per lane.
//   sample  grid (fine slices, NB): every workgroup folds the slice statistics of its
//           branch, gathers p_i(x_i), q_i(x_i) and tests u*q < p in order (n); then the fp64
//           resampling path, one pass over target row n and draft row n (target row K alone
//           when n = K): the slice's sums of exp(z - max), and of the same over the tokens
//           whose residual max(0, p-q) is positive beyond doubt; tokens in doubt are listed.
//   pick    grid NB: the normalisers, each slice's residual mass (its listed tokens settled),
//           the slice in which the running sum first exceeds u_sample * total, then the lane
//           inside it (its tokens evaluated again, four or eight per lane), then the token.
//   warp    (only with top-k / top-p) one workgroup per target row: the smallest logit the row keeps and the
//           mass of the kept tokens.  Both filters are predicates on a token's value (keep v iff fewer than k
//           tokens are larger; keep v iff the mass of the larger kept tokens is below top_p * Z_k), so equal
//           logits are never split.  With top-p alone the threshold is searched among the candidates rowz listed.
//           With a small k, or where those fall short, a bound taken from the lanes' largest logits leaves a short
//           list of candidate tokens, which is sorted and walked in descending order; otherwise (and whenever such
//           a list overflows or falls short) two radix selections over an order-preserving key of the logit: the
//           k-th largest by count, then among those the value at which the descending cumulative mass reaches
//           top_p of the kept mass.  sample / pick then use
//           p(v) = [key(v) >= key_min] * exp((x_v - max)/T) / Z_kept for the target rows.
//   rowz    (only with top-p alone) grid (fine-slice groups, target rows): the fp64 mass of every target row in
//           fine slices, which warp folds: top-p's threshold is a share of the whole row's mass; and the tokens
//           heavy enough to be kept, for warp.
// The two resampling rows are re-read once (2 of the 2K+1 rows of a branch; cache hits).
// fp64 there makes the blocked running sum agree with a sequential one to ~1e-16, so the
// drawn token does not depend on the summation order.
#include <limits.h>

#include <type_traits>

#include "la_internal.hpp"

namespace la {
namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;

constexpr int kThreads = 256;
constexpr int kFinePer = 8;                 // tokens per lane in the fp64 kernels (FineWords holds eight)
constexpr int kFine = kThreads * kFinePer;  // 2048 tokens per fine slice
constexpr int kMaxFine = 1024;   // fine slices per row the fp64 kernels can stage in LDS (vocab <= 2M)

// (bit-casting a vector element in place, __builtin_bit_cast(float, w[k]), reads element 0 with this compiler;
// pass the element by value instead)
__device__ __forceinline__ float as_f32(uint32_t w) { return __builtin_bit_cast(float, w); }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }

template <bool BF16>
__device__ __forceinline__ float load_logit(const void *base, size_t idx) {
  if constexpr (BF16) return __builtin_bit_cast(float, (uint32_t)((const uint16_t *)base)[idx] << 16);
  return ((const float *)base)[idx];
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
// Maximum and sum over a wavefront on the vector ALU, for values whose order of summation does not matter.
template <int ROT>
__device__ __forceinline__ float row_rotate(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + ROT, 0xf, 0xf, false));
}
// over the 16 lanes of a DPP row
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
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_max_dpp(float v) {
  v = row_max(v);
  return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = row_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Sum over the 16 lanes of a DPP row, on the vector ALU (a shuffle goes through the LDS pipeline, two accesses per
// double and step, which the workgroups of the fp64 kernels were queueing for).  Every lane of a row ends with
// the same bits: each step adds the same pairs in all of them, in one order or the other.
template <int ROT>
__device__ __forceinline__ double row_rotate(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x120 + ROT, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x120 + ROT, 0xf, 0xf, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double row_sum(double v) {
  v += row_rotate<8>(v);
  v += row_rotate<4>(v);
  v += row_rotate<2>(v);
  return v + row_rotate<1>(v);
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// row rw of the stacked [target rows ; draft rows] list
template <bool BF16>
__device__ __forceinline__ const uint8_t *stacked_row(const AcceptParams &p, int rw) {
  constexpr size_t esz = BF16 ? 2 : 4;
  const int n_t = p.NB * (p.K + 1);
  if (rw < n_t) return (const uint8_t *)p.target + (size_t)rw * p.V * esz;
  return (const uint8_t *)p.draft + (size_t)(rw - n_t) * p.V * esz;
}

// exp(y) in fp64 for the arguments met here (y = (x - max)/T <= 0 up to rounding; the result only has to be the same
// function of y everywhere it is used, and within an ulp or two of the true value).  y = k ln2 + r with |r| <= ln2/2
// by a two-term reduction (k * ln2_hi is exact for |k| < 2^11), e^r by its Taylor polynomial of degree 13
// (remainder < 5e-18), then the scaling by 2^k, which also takes results below the normal range to denormals / zero.
// About 20 fp64 instructions, against several times that for the general library routine.
// a * b + c with the constant c read from scalar registers (left to itself the compiler copies every constant of the
// polynomial into a vector register pair first, two moves per step, to use the two-address form of the instruction)
__device__ __forceinline__ double fma_const(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

__device__ __forceinline__ double exp64(double y) {
  y = fmax(y, -750.0);   // (y <= 0 up to rounding: x never exceeds the row maximum)
  // k = nearest integer to y * log2(e): adding 1.5 * 2^52 leaves it in the low bits of the sum (as a double by taking
  // the constant off again, as an integer in the low word of the bit pattern); the rounding and conversion
  // instructions this replaces run at a quarter of the rate of an addition
  const double shifted = __builtin_fma(y, 1.4426950408889634074, 6755399441055744.0);
  const double k = shifted - 6755399441055744.0;
  const int ki = (int)(uint32_t)__builtin_bit_cast(uint64_t, shifted);
  double r = __builtin_fma(-k, 6.93147180369123816490e-01, y);
  r = __builtin_fma(-k, 1.90821492927058770002e-10, r);
  double q = fma_const(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);
  q = fma_const(q, r, 1.0 / 39916800.0);
  q = fma_const(q, r, 1.0 / 3628800.0);
  q = fma_const(q, r, 1.0 / 362880.0);
  q = fma_const(q, r, 1.0 / 40320.0);
  q = fma_const(q, r, 1.0 / 5040.0);
  q = fma_const(q, r, 1.0 / 720.0);
  q = fma_const(q, r, 1.0 / 120.0);
  q = fma_const(q, r, 1.0 / 24.0);
  q = fma_const(q, r, 1.0 / 6.0);
  q = __builtin_fma(q, r, 0.5);
  q = __builtin_fma(q, r, 1.0);
  q = __builtin_fma(q, r, 1.0);
  return __builtin_ldexp(q, ki);
}

// fp64 probability mass (unnormalised) of one logit: exp(x/T - max/T)
__device__ __forceinline__ double mass64(float x, double mx_over_t, double inv_temp) {
  return exp64((double)x * inv_temp - mx_over_t);
}

// ---------------------------------------------------------------------------------------------
// exp(x / T) of the bf16 logits 2^-12 <= |x| < 64, both signs, in the order of their bit patterns: a table in LDS that
// the kernels walking whole rows look their masses up in.  An exponential costs about 110 cycles of a SIMD, a lookup about
// 20 and an LDS read; with 4608 entries nearly every token of a row is in it (of normal logits of deviation 3 one
// token in 15000 is not; it takes the exponential).  The stats kernel's first workgroups write it to the workspace, to
// the last bit or two: the product x / T is carried in two terms.  Measured at V = 152064: sample 21.2 -> 14.6 us (32
// branches, draft rows), rowz 15.4 -> 12.5 us (54 rows; in slices of eight per workgroup 14.4, of four 13.4).
//
// The masses of such a row are in units of e^0, not of e^(max/T): nothing but their quotients leaves the call, and with
// |max| / T up to 300 no sum overflows and a token that vanishes weighs e^-445 of the row at most.  A row beyond that keeps
// the maximum as its unit and the exponential per token (mass_unit).  fp32 logits, calls of less than 64 slices, whose
// workspace has no room for it, and temperatures below 0.11 have no table: its largest entry is e^(64/T), which leaves the
// range of a double at T = 0.0902; at 0.11 it is e^582.  Nor do calls that it would cost more than it gives (worth_a_table).
// ---------------------------------------------------------------------------------------------
constexpr int kTabLo = 115 * 128;               // bit pattern of 2^-12
constexpr int kTabHalf = 18 * 128;              // up to 2^6
constexpr int kTab = 2 * kTabHalf + 2;          // a zero behind the positive values, the negative ones, a zero behind those
constexpr float kTabMaxExponent = 300.f;
constexpr float kTabMinTemperature = 0.11f;     // (as the descriptor holds it)

__device__ __forceinline__ double table_entry(int i, double inv_temp) {
  const int neg = i > kTabHalf, j = i - neg * (kTabHalf + 1);
  if (j == kTabHalf) return 0.0;
  const double x = (double)bf16_lo((uint32_t)(j + kTabLo + neg * 0x8000));
  const double y = x * inv_temp, rest = __builtin_fma(x, inv_temp, -y);
  const double e = exp64(y);
  return __builtin_fma(e, rest, e);
}

// max / T where that is the unit of a row's masses, else 0
__device__ __forceinline__ double mass_unit(const AcceptParams &p, float row_max) {
  const double m_t = (double)row_max * p.inv_temp;
  return p.exp_tab && fabs(m_t) <= (double)kTabMaxExponent ? 0.0 : m_t;
}
// what a mass in the row's unit is in units of e^(max/T)
__device__ __forceinline__ double unit_over_max(const AcceptParams &p, float row_max) {
  return exp64(mass_unit(p, row_max) - (double)row_max * p.inv_temp);
}

// The table from the workspace to LDS, by n_threads threads, with all loads in flight at once; barrier to follow.
template <int n_threads>
struct TableCopy {
  static constexpr int kLoads = (kTab / 2 + n_threads - 1) / n_threads;
  u32x4 w[kLoads];
  __device__ __forceinline__ void load(const double *from) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int i = threadIdx.x + j * n_threads;
      w[j] = ((const u32x4 *)from)[i < kTab / 2 ? i : 0];
    }
  }
  __device__ __forceinline__ void store(double *to) const {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int i = threadIdx.x + j * n_threads;
      if (i < kTab / 2) ((u32x4 *)to)[i] = w[j];
    }
  }
};

// The kFinePer consecutive logits of a row that a lane of the walking kernels owns, from token v (a multiple of kFinePer)
// on, as loaded (bf16: two to a word); tokens at or past V read as -inf.  vec: every row starts on a 16-byte boundary.
template <bool BF16>
struct FineWords {
  u32x4 w[BF16 ? 1 : 2];
  __device__ __forceinline__ void load(const void *base, size_t row_off, int v, int V, bool vec) {
    const uint8_t *at = (const uint8_t *)base + (row_off + v) * (BF16 ? 2 : 4);
    if (vec && v + 8 <= V) {
      w[0] = *(const u32x4 *)at;
      if constexpr (!BF16) w[1] = *(const u32x4 *)(at + 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (BF16) {
          const uint32_t lo = v + 2 * e < V ? ((const uint16_t *)at)[2 * e] : 0xFF80u;   // -inf
          const uint32_t hi = v + 2 * e + 1 < V ? ((const uint16_t *)at)[2 * e + 1] : 0xFF80u;
          w[0][e] = lo | hi << 16;
        } else {
          w[0][e] = v + e < V ? ((const uint32_t *)at)[e] : 0xFF800000u;
          w[1][e] = v + 4 + e < V ? ((const uint32_t *)at)[4 + e] : 0xFF800000u;
        }
      }
    }
  }
  // values below x_min become -inf
  __device__ __forceinline__ void keep(float x_min) {
    float x[8];
    get(x);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (BF16) {
        const uint32_t word = w[0][k];
        w[0][k] = (x[2 * k] >= x_min ? word & 0xFFFFu : 0xFF80u) | (x[2 * k + 1] >= x_min ? word & 0xFFFF0000u : 0xFF800000u);
      } else {
        const uint32_t a = w[0][k], b = w[1][k];
        w[0][k] = x[k] >= x_min ? a : 0xFF800000u;
        w[1][k] = x[4 + k] >= x_min ? b : 0xFF800000u;
      }
    }
  }
  __device__ __forceinline__ void get(float (&x)[8]) const {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (BF16) {
        const uint32_t word = w[0][k];
        x[2 * k] = bf16_lo(word);
        x[2 * k + 1] = bf16_hi(word);
      } else {
        const uint32_t a = w[0][k], b = w[1][k];
        x[k] = as_f32(a);
        x[4 + k] = as_f32(b);
      }
    }
  }
};

// The masses of eight logits in their row's unit (o_t = mass_unit).  TAB: by the table, and by the exponential for
// what is not in it.
template <bool BF16, bool TAB>
__device__ __forceinline__ void masses(const FineWords<BF16> &words, const double *tab, double o_t, const AcceptParams &p,
                                       double (&m)[8]) {
  if constexpr (!TAB) {
    float x[8];
    words.get(x);
#pragma unroll
    for (int e = 0; e < 8; ++e) m[e] = mass64(x[e], o_t, p.inv_temp);
  } else {
    // two tokens per instruction: their places in the table, kTabHalf (a zero) for what is not in it
    u16x2 most = {0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t word = words.w[0][k];
      const u16x2 u = __builtin_bit_cast(u16x2, word);
      u16x2 i = (u & (uint16_t)0x7FFF) - (uint16_t)kTabLo;
      most = __builtin_elementwise_max(most, i);
      i = __builtin_elementwise_min(i, (u16x2){kTabHalf, kTabHalf}) + (u >> 15) * (uint16_t)(kTabHalf + 1);
      m[2 * k] = tab[i.x];
      m[2 * k + 1] = tab[i.y];
    }
    if (__ballot(most.x >= kTabHalf || most.y >= kTabHalf) || o_t != 0.0) {
      float x[8];
      words.get(x);
      const float zero_below = (float)((o_t - 746.0) / p.inv_temp);   // (-inf among them)
      uint32_t rest = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t i = ((__builtin_bit_cast(uint32_t, x[e]) >> 16) & 0x7FFFu) - (uint32_t)kTabLo;
        if (i >= (uint32_t)kTabHalf || o_t != 0.0) {
          m[e] = 0.0;
          if (x[e] > zero_below) rest |= 1u << e;
        }
      }
      while (__ballot(rest != 0)) {   // one token per lane and round
        const int bit = __ffs((int)rest) - 1;
        float v = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) v = e == bit ? x[e] : v;
        const double mv = mass64(v, o_t, p.inv_temp);
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = e == bit ? mv : m[e];
        rest &= rest - 1;
      }
    }
  }
}

// The mass of one logit by the same rule and to the same bits, the table read from the workspace: what the pick kernel
// evaluates again has to agree with the sums it was chosen by.
template <bool BF16>
__device__ __forceinline__ double mass_again(float x, double o_t, const AcceptParams &p) {
  if constexpr (BF16) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x) >> 16, i = (u & 0x7FFFu) - (uint32_t)kTabLo;
    if (p.exp_tab && o_t == 0.0 && i < (uint32_t)kTabHalf) return p.exp_tab[i + (u >> 15) * (kTabHalf + 1)];
  }
  return mass64(x, o_t, p.inv_temp);
}

// ---------------------------------------------------------------------------------------------
// stats: grid (n_chunks, rows); a slice is 256 lanes x 8 16-byte loads (16384 bf16 / 8192 fp32 logits)
// ---------------------------------------------------------------------------------------------
template <bool BF16>
struct StatsShape {
  static constexpr int kLoads = 8;
  static constexpr int kPerVec = BF16 ? 8 : 4;
  static constexpr int kPer = kLoads * kPerVec;  // logits per lane
  static constexpr int kSlice = kThreads * kPer;
};

template <bool BF16, bool VEC>
__global__ __launch_bounds__(kThreads, 6) void accept_stats_kernel(const AcceptParams p) {
  using Sh = StatsShape<BF16>;
  __shared__ float red[2][kThreads / 64];
  const int c = blockIdx.x, rw = blockIdx.y;
  const int tid = threadIdx.x;
  const uint8_t *row = stacked_row<BF16>(p, rw);
  const int v0 = c * Sh::kSlice;
  const int v1 = min(p.V, v0 + Sh::kSlice);

  float x[Sh::kPer];
  if constexpr (VEC) {
    u32x4 w[Sh::kLoads];
#pragma unroll
    for (int e = 0; e < Sh::kLoads; ++e) {
      const int v = v0 + (e * kThreads + tid) * Sh::kPerVec;  // consecutive lanes read consecutive 16 B
      // V % kPerVec == 0 on this path, so a vector is all-in or all-out; out-of-range lanes re-read the row start
      w[e] = *(const u32x4 *)(row + (size_t)(v < v1 ? v : 0) * (BF16 ? 2 : 4));
    }
#pragma unroll
    for (int e = 0; e < Sh::kLoads; ++e) {
      const bool in = v0 + (e * kThreads + tid) * Sh::kPerVec < v1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t word = w[e][k];
        if constexpr (BF16) {
          x[e * 8 + 2 * k] = in ? bf16_lo(word) : -INFINITY;
          x[e * 8 + 2 * k + 1] = in ? bf16_hi(word) : -INFINITY;
        } else {
          x[e * 4 + k] = in ? as_f32(word) : -INFINITY;
        }
      }
    }
  } else {
#pragma unroll
    for (int e = 0; e < Sh::kPer; ++e) {
      const int v = v0 + e * kThreads + tid;
      x[e] = v < v1 ? load_logit<BF16>(row, v) : -INFINITY;
    }
  }
  float m = x[0];
#pragma unroll
  for (int e = 1; e < Sh::kPer; ++e) m = fmaxf(m, x[e]);
  m = wave_max(m);
  if ((tid & 63) == 0) red[0][tid >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));  // slice maximum
  // a slice whose logits are all -inf (a masked part of the vocabulary) has mass 0: the exponent offset is taken
  // from 0 instead of from -inf, which would turn -inf - (-inf) into a NaN; the slice is recorded as (-inf, 0) and
  // drops out of every fold (weight 2^(-inf - row maximum) = 0)
  const float cm = -((m == -INFINITY) ? 0.f : m) * p.inv_temp_log2;
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < Sh::kPer; ++e) s += __builtin_amdgcn_exp2f(__builtin_fmaf(x[e], p.inv_temp_log2, cm));
  s = wave_sum(s);
  if ((tid & 63) == 0) red[1][tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    f32x2 out = {m, (red[1][0] + red[1][1]) + (red[1][2] + red[1][3])};
    *(f32x2 *)(p.stats + ((size_t)rw * p.n_chunks + c) * 2) = out;
  }
  if (BF16 && p.exp_tab)
    for (int i = (rw * p.n_chunks + c) * kThreads; i < kTab; i += gridDim.x * gridDim.y * kThreads)
      if (i + tid < kTab) p.exp_tab[i + tid] = table_entry(i + tid, p.inv_temp);
}

// Fold the slice statistics of one row into its maximum and sum 2^((x-max)*c); called by a whole wavefront, lanes
// over slices, the same result in every lane.
__device__ __forceinline__ void wave_fold_row(const AcceptParams &p, int rw, int lane, float &m_out, float &z_out) {
  const float *st = p.stats + (size_t)rw * p.n_chunks * 2;
  float m = -INFINITY;
  for (int c = lane; c < p.n_chunks; c += 64) m = fmaxf(m, st[2 * c]);
  m = wave_max(m);
  float z = 0.f;
  for (int c = lane; c < p.n_chunks; c += 64)
    z += st[2 * c + 1] * __builtin_amdgcn_exp2f((st[2 * c] - m) * p.inv_temp_log2);
  m_out = m;
  z_out = wave_sum(z);
}

// Order-preserving key of an fp32 value: larger value <=> larger key (as unsigned).
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t b = __builtin_bit_cast(uint32_t, x + 0.0f);   // -0 and +0 are one value: (-0) + (+0) = +0
  return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

// The N (4 or 8) consecutive logits of a row that a lane owns, from token v (a multiple of N) on; tokens at or past V read as
// -inf.  vec: every row starts on a 16-byte boundary.
template <bool BF16, int N>
__device__ __forceinline__ void load_own(const void *base, size_t row_off, int v, int V, bool vec, float (&x)[N]) {
  if constexpr (N == 8) {
    FineWords<BF16> w;
    w.load(base, row_off, v, V, vec);
    w.get(x);
  } else {
    static_assert(N == 4, "tokens per lane of the pick kernel");
    if (vec && v + 4 <= V) {
      if constexpr (BF16) {
        const u32x2 w = *(const u32x2 *)((const uint16_t *)base + row_off + v);
        const uint32_t lo = w.x, hi = w.y;
        x[0] = bf16_lo(lo);
        x[1] = bf16_hi(lo);
        x[2] = bf16_lo(hi);
        x[3] = bf16_hi(hi);
      } else {
        const u32x4 w = *(const u32x4 *)((const float *)base + row_off + v);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t word = w[e];
          x[e] = as_f32(word);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) x[e] = v + e < V ? load_logit<BF16>(base, row_off + v + e) : -INFINITY;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// warp: grid NB*(K+1), one workgroup of 1024 lanes per target row (Section 4, Setup: temperature, top_k, top_p)
// ---------------------------------------------------------------------------------------------
constexpr int kWarpThreads = 1024;
constexpr int kRep = 16;   // histogram copies per workgroup
constexpr int kHist = 257; // elements between two copies: one more than the buckets, so that the same bucket of
                           // different copies lies in different LDS banks

// Calls f(x) for every logit of a row, the workgroup's lanes striding over it, with several loads in flight per
// lane (16-byte loads when the row allows: eight per lane and batch).
template <bool BF16, typename F>
__device__ __forceinline__ void row_foreach(const void *row, int V, F &&f) {
  constexpr int kPerVec = BF16 ? 8 : 4;
  constexpr int kInFlight = 8;   // 16-byte loads per lane and batch
  const int tid = threadIdx.x;
  if (V % kPerVec == 0) {   // then every row starts on a 16-byte boundary
    const int n_vec = V / kPerVec;
    for (int i0 = tid; i0 < n_vec; i0 += kInFlight * kWarpThreads) {
      u32x4 w[kInFlight];
#pragma unroll
      for (int j = 0; j < kInFlight; ++j) {
        const int i = i0 + j * kWarpThreads;
        w[j] = *(const u32x4 *)((const uint8_t *)row + (size_t)(i < n_vec ? i : i0) * 16);
      }
#pragma unroll
      for (int j = 0; j < kInFlight; ++j) {
        if (i0 + j * kWarpThreads >= n_vec) break;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t word = w[j][k];
          if constexpr (BF16) {
            f(bf16_lo(word));
            f(bf16_hi(word));
          } else {
            f(as_f32(word));
          }
        }
      }
    }
  } else {
    for (int v0 = tid; v0 < V; v0 += 8 * kWarpThreads) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int v = v0 + j * kWarpThreads;
        x[j] = load_logit<BF16>(row, v < V ? v : v0);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (v0 + j * kWarpThreads < V) f(x[j]);
    }
  }
}

// Radix selection over the keys of a set of values, 8 bits per round from the top.  BY_MASS = false: the k-th
// largest key (count{key > result} < k <= count{key >= result}).  BY_MASS = true: the key at which the descending
// cumulative mass first reaches target (mass{key > result} < target <= mass{key >= result}); if the whole mass
// stays below target, floor_key.  BF16 values have 16 significant key bits: two rounds instead of four.
// `each(f)` calls f(x) for every value of the set, the workgroup's lanes sharing the work; values with a key below
// floor_key take no part (the caller guarantees that the answer lies at or above it).
// The mass histogram is accumulated in 64-bit fixed point (masses are at most 1, at most 2^21 of them; 40 fraction
// bits, each mass rounded to nearest): integer atomics add in any order to the same bits, so the selection is the
// same in every run, which floating-point atomics would not give.  The 2^-41 rounding per term moves a bucket's
// mass by a few 1e-10 of the row's mass at most, inside the margin within which a top-p decision counts as open.
template <bool BF16, bool BY_MASS, typename Each>
__device__ __forceinline__ uint32_t radix_select(Each &&each, double mx_over_t, double inv_temp, uint32_t floor_key,
                                                 int k, double target, uint32_t *cnt, double *mass,
                                                 uint32_t *s_pick, double *s_above) {
  constexpr int kRounds = BF16 ? 2 : 4;
  constexpr double kFix = 1099511627776.0;   // 2^40
  unsigned long long *imass = (unsigned long long *)mass;
  const int tid = threadIdx.x;
  uint32_t prefix = 0;          // the bits chosen so far (high bits of the key)
  double above = 0.0;           // BY_MASS: mass of the keys above the chosen prefix range
  int k_rem = k;
#pragma unroll 1
  for (int round = 0; round < kRounds; ++round) {
    const int shift = 24 - 8 * round;
    // kRep copies of the histogram, chosen by lane: the logits of a row crowd into a few of the 256 buckets of the
    // leading byte, and LDS serialises atomics of one instruction that hit the same address
    for (int i = tid; i < kHist * kRep; i += kWarpThreads) {
      if constexpr (BY_MASS)
        imass[i] = 0;
      else
        cnt[i] = 0;
    }
    __syncthreads();
    const int rep = (tid & (kRep - 1)) * kHist;
    each([&](float x) {
      const uint32_t key = order_key(x);
      const bool in_range = round == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8));
      if (!in_range || key < floor_key) return;
      if constexpr (BY_MASS)
        atomicAdd(&imass[rep + ((key >> shift) & 255)],
                  (unsigned long long)__builtin_llrint(mass64(x, mx_over_t, inv_temp) * kFix));
      else
        atomicAdd(&cnt[rep + ((key >> shift) & 255)], 1u);
    });
    __syncthreads();
    if (tid < 256) {   // fold the copies, in order
      if constexpr (BY_MASS) {
        unsigned long long t = 0;
        for (int r = 0; r < kRep; ++r) t += imass[r * kHist + tid];
        imass[tid] = t;
      } else {
        uint32_t t = 0;
        for (int r = 0; r < kRep; ++r) t += cnt[r * kHist + tid];
        cnt[tid] = t;
      }
    }
    __syncthreads();
    if (tid == 0) {
      int pick = -1;
      if constexpr (BY_MASS) {
        double m = above;
        int lowest = -1;
        double low_mass = 0.0;
        for (int b = 255; b >= 0; --b) {
          if (imass[b] == 0) continue;
          const double mb = (double)imass[b] * (1.0 / kFix);
          if (m + mb >= target) {
            pick = b;
            break;
          }
          lowest = b, low_mass = mb;
          m += mb;
        }
        // below the first round the parent bucket did cross; if the running sum misses that by a rounding of its
        // additions, the crossing is in the lowest bucket with mass
        if (pick < 0 && round > 0) pick = lowest, m -= low_mass;
        *s_above = m;
      } else {
        int c = 0;
        for (int b = 255; b >= 0; --b) {
          if (c + (int)cnt[b] >= k_rem) {
            pick = b;
            k_rem -= c;
            break;
          }
          c += (int)cnt[b];
        }
        *s_above = (double)k_rem;
      }
      *s_pick = (uint32_t)pick;
    }
    __syncthreads();
    const uint32_t pick = *s_pick;
    if (pick == 0xFFFFFFFFu) return floor_key;   // BY_MASS only: the target lies beyond the whole mass
    prefix |= pick << shift;
    if constexpr (BY_MASS)
      above = *s_above;
    else
      k_rem = (int)*s_above;
    __syncthreads();
  }
  // a bf16 logit widened to fp32 has 16 zero low bits, which the key turns into 0xFFFF for negative values
  return BF16 ? (prefix | ((prefix >> 31) ? 0u : 0xFFFFu)) : prefix;
}

// Sum over the row of exp((x - max)/T) for keys >= floor_key, fp64, in a fixed order (per lane in token order, then
// a shuffle tree, then the wavefronts in order): the same value in every lane.
template <bool BF16>
__device__ __forceinline__ double kept_mass(const void *row, int V, double mx_over_t, double inv_temp,
                                            uint32_t floor_key, double *red, double *slot) {
  const int tid = threadIdx.x;
  double acc = 0.0;
  row_foreach<BF16>(row, V, [&](float x) {
    if (order_key(x) >= floor_key) acc += mass64(x, mx_over_t, inv_temp);
  });
  acc = wave_sum(acc);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < kWarpThreads / 64; ++w) t += red[w];
    *slot = t;
  }
  __syncthreads();
  const double out = *slot;
  __syncthreads();
  return out;
}

// The logit an order-preserving key came from.
__device__ __forceinline__ float key_value(uint32_t key) {
  return __builtin_bit_cast(float, (key >> 31) ? key ^ 0x80000000u : ~key);
}

constexpr int kSmallK = 128;   // largest top_k the candidate-list path takes
constexpr int kCand = 2048;    // its candidate list (LDS)

// The k-th largest of the workgroup's per-lane keys mk (k <= number of lanes), found bit by bit with ballot counts:
// the largest value lo such that at least k lanes have mk >= lo.  The same value in every lane.  One barrier per
// bit; s_cnt is scratch of 2 x (wavefronts) ints.
template <bool BF16>
__device__ __forceinline__ uint32_t kth_largest_lane_key(uint32_t mk, int k, int (*s_cnt)[kWarpThreads / 64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t lo = 0;
  // (a bf16 logit's key has sixteen equal low bits, so its sixteen high bits decide)
  for (int bit = 31; bit >= (BF16 ? 16 : 0); --bit) {
    const uint32_t c = lo | (1u << bit);
    const int n_w = __popcll(__ballot(mk >= c));
    if (lane == 0) s_cnt[bit & 1][wave] = n_w;
    __syncthreads();
    int tot = 0;
#pragma unroll
    for (int w = 0; w < kWarpThreads / 64; ++w) tot += s_cnt[bit & 1][w];
    if (tot >= k) lo = c;
  }
  if (BF16 && !(lo >> 31)) lo |= 0xFFFFu;   // the low bits of a negative bf16 value's key: lo is that key itself
  return lo;
}

// Append `key` to list[] (capacity cap, length *n in LDS) for the lanes with take set: one LDS atomic per wavefront
// and call instead of one per lane.  *n counts every qualifying token, also past the capacity.
__device__ __forceinline__ void list_append(bool take, uint32_t key, uint32_t *list, int cap, int *n) {
  const uint64_t who = __ballot(take);
  if (!who) return;
  const int lane = threadIdx.x & 63, leader = __ffsll((unsigned long long)who) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(n, __popcll(who));
  base = __shfl(base, leader);
  if (take) {
    const int i = base + __popcll(who & ((1ull << lane) - 1));
    if (i < cap) list[i] = key;
  }
}

// The tokens of a row with value >= lo_val appended to list[] as keys (see list_append), for bounds that about one
// token in a hundred reaches, so that nearly every wavefront-wide step of a plain scan would find one.  On 16-byte
// aligned rows a lane first marks the qualifying ones among the up to 64 tokens of its eight loads in a bit mask (one
// compare and one bit operation per token); then the marked tokens are appended in rounds, one per lane and round,
// their values read again (few, and just loaded).
template <bool BF16>
__device__ __forceinline__ void row_collect(const void *row, int V, float lo_val, uint32_t *list, int cap, int *n) {
  constexpr int kPerVec = BF16 ? 8 : 4;
  constexpr int kInFlight = 8;
  const int tid = threadIdx.x;
  if (V % kPerVec != 0) {
    row_foreach<BF16>(row, V, [&](float x) { list_append(x >= lo_val, order_key(x), list, cap, n); });
    return;
  }
  const int n_vec = V / kPerVec;
  for (int i0 = tid; i0 < n_vec; i0 += kInFlight * kWarpThreads) {
    u32x4 w[kInFlight];
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const int i = i0 + j * kWarpThreads;
      w[j] = *(const u32x4 *)((const uint8_t *)row + (size_t)(i < n_vec ? i : i0) * 16);
    }
    uint64_t marks = 0;   // bit j*kPerVec + e: element e of load j qualifies
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const bool in = i0 + j * kWarpThreads < n_vec;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t word = w[j][k];
        if constexpr (BF16) {
          if (in && bf16_lo(word) >= lo_val) marks |= 1ull << (j * 8 + 2 * k);
          if (in && bf16_hi(word) >= lo_val) marks |= 1ull << (j * 8 + 2 * k + 1);
        } else {
          if (in && as_f32(word) >= lo_val) marks |= 1ull << (j * 4 + k);
        }
      }
    }
    while (__ballot(marks != 0)) {
      const bool take = marks != 0;
      const int bit = take ? __ffsll((unsigned long long)marks) - 1 : 0;
      marks &= marks - 1;
      const int j = bit / kPerVec, e = bit - j * kPerVec;
      const size_t v = (size_t)(i0 + j * kWarpThreads) * kPerVec + e;
      const float x = take ? load_logit<BF16>(row, v) : 0.f;
      list_append(take, order_key(x), list, cap, n);
    }
  }
}

// The same for bounds that only a few dozen tokens of the row reach: a lane first takes the largest of the tokens of
// one 16-byte load; only when some lane of the wavefront has one at or above the bound are that load's tokens tested
// and appended one by one.
template <bool BF16>
__device__ __forceinline__ void row_collect_sparse(const void *row, int V, float lo_val, uint32_t *list, int cap,
                                                   int *n) {
  constexpr int kPerVec = BF16 ? 8 : 4;
  constexpr int kInFlight = 8;
  const int tid = threadIdx.x;
  if (V % kPerVec != 0) {
    row_foreach<BF16>(row, V, [&](float x) { list_append(x >= lo_val, order_key(x), list, cap, n); });
    return;
  }
  const int n_vec = V / kPerVec;
  for (int i0 = tid; i0 < n_vec; i0 += kInFlight * kWarpThreads) {
    u32x4 w[kInFlight];
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const int i = i0 + j * kWarpThreads;
      w[j] = *(const u32x4 *)((const uint8_t *)row + (size_t)(i < n_vec ? i : i0) * 16);
    }
#pragma unroll
    for (int j = 0; j < kInFlight; ++j) {
      const bool in = i0 + j * kWarpThreads < n_vec;
      float x[kPerVec];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t word = w[j][k];
        if constexpr (BF16) {
          x[2 * k] = bf16_lo(word);
          x[2 * k + 1] = bf16_hi(word);
        } else {
          x[k] = as_f32(word);
        }
      }
      float top = x[0];
#pragma unroll
      for (int e = 1; e < kPerVec; ++e) top = fmaxf(top, x[e]);
      if (__ballot(in && top >= lo_val)) {
#pragma unroll
        for (int e = 0; e < kPerVec; ++e) list_append(in && x[e] >= lo_val, order_key(x[e]), list, cap, n);
      }
    }
  }
}

// Bitonic sort of list[0..n) in descending order, in place, by the whole workgroup; n <= kCand.  Entries n..N-1 (N
// the next power of two, at least 128) are filled with 0, which is below every key.  Compare-exchange steps whose
// partners are at least 128 apart involve the whole workgroup and end in a barrier; the steps below that stay inside
// 128-entry blocks, one block per wavefront and one comparator per lane, and need no barrier between them (a
// wavefront's LDS accesses are carried out in order).
__device__ __forceinline__ void sort_desc(uint32_t *list, int n) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int N = 128;
  while (N < n) N <<= 1;
  for (int i = n + threadIdx.x; i < N; i += kWarpThreads) list[i] = 0u;
  __syncthreads();
  auto exchange = [&](int i, int o, int k) {
    const uint32_t a = list[i], b = list[o];
    const bool desc = (i & k) == 0;
    if (desc ? a < b : a > b) list[i] = b, list[o] = a;
  };
  for (int k = 2; k <= N; k <<= 1) {
    int j = k >> 1;
    for (; j >= 128; j >>= 1) {
      for (int c = threadIdx.x; c < N / 2; c += kWarpThreads) {   // comparator c: a zero bit inserted at j
        const int i = ((c & ~(j - 1)) << 1) | (c & (j - 1));
        exchange(i, i | j, k);
      }
      __syncthreads();
    }
    if (wave * 128 < N) {
      for (; j > 0; j >>= 1) {
        const int i = wave * 128 + (((lane & ~(j - 1)) << 1) | (lane & (j - 1)));
        exchange(i, i | j, k);
        __builtin_amdgcn_wave_barrier();
      }
    }
    __syncthreads();
  }
}

// Sort the n <= kCand keys of cand[] into sorted[] in descending order by rank counting (equal keys are the same
// value, so their mutual order does not matter) and put the exact fp64 mass of sorted[i] into cmass[i].
__device__ __forceinline__ void sort_list_with_masses(const uint32_t *cand, int n, uint32_t *sorted, double *cmass,
                                                      double mx_over_t, double inv_temp) {
  for (int i = threadIdx.x; i < n; i += kWarpThreads) {
    const uint32_t ki = cand[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const uint32_t kj = cand[j];
      rank += (kj > ki || (kj == ki && j < i)) ? 1 : 0;
    }
    sorted[rank] = ki;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kWarpThreads) cmass[i] = mass64(key_value(sorted[i]), mx_over_t, inv_temp);
  __syncthreads();
}

// top-k with a small k, then top-p, in two passes over the row and without a histogram.  Pass 1: every lane keeps
// the largest key among its tokens; the k-th largest of these lane maxima (found bit by bit with ballot counts) is a
// lower bound of the row's k-th largest key, because at least k tokens reach it.  Pass 2: the keys at or above that
// bound go to a list in LDS (a few dozen for random logits; when more than kCand qualify, e.g. a row of equal
// logits, the caller takes the histogram path instead: returns false, the same decision in every lane).  The list is
// sorted by rank counting (the order of equal keys does not matter: they are the same value), and one lane walks it
// in descending order exactly as the definition reads: the tokens down to the k-th largest value stay, Z_k is their
// mass, then value groups are taken while the mass above them is below top_p * Z_k.
template <bool BF16>
__device__ __forceinline__ bool warp_small_k(const AcceptParams &p, const void *row, uint32_t *cand, uint32_t *sorted,
                                             double *cmass, float *row_max_out, uint32_t *key_min_out,
                                             double *z_out) {
  __shared__ int s_cnt[2][kWarpThreads / 64];
  __shared__ float s_wmax[kWarpThreads / 64];
  __shared__ int s_n;
  __shared__ uint32_t s_key;
  __shared__ double s_z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int k = p.top_k;
  float mx = -INFINITY;   // a lane without tokens counts as holding -inf
  row_foreach<BF16>(row, p.V, [&](float x) { mx = fmaxf(mx, x); });
  const uint32_t mk = order_key(mx);
  {   // the row maximum falls out of the same pass (made visible by the first barrier of the search below)
    const float wm = wave_max(mx);
    if (lane == 0) s_wmax[wave] = wm;
  }
  const uint32_t lo = kth_largest_lane_key<BF16>(mk, k, s_cnt);   // k <= kSmallK < the number of lanes
  float row_max = s_wmax[0];
#pragma unroll
  for (int w = 1; w < kWarpThreads / 64; ++w) row_max = fmaxf(row_max, s_wmax[w]);
  *row_max_out = row_max;
  const double mx_over_t = (double)row_max * p.inv_temp;
  const float lo_val = key_value(lo);        // the k-th largest lane maximum (-inf when fewer than k lanes own a token)
  if (tid == 0) s_n = 0;
  __syncthreads();
  // comparing the values is comparing the keys (no NaNs; -0 == +0 on both sides)
  row_collect_sparse<BF16>(row, p.V, lo_val, cand, kCand, &s_n);
  __syncthreads();
  const int n_c = s_n;   // >= k
  if (n_c > kCand) return false;
  sort_list_with_masses(cand, n_c, sorted, cmass, mx_over_t, p.inv_temp);
  const uint32_t kth = sorted[k - 1];
  if (n_c <= 64) {
    // the usual case: the whole list fits one wavefront, lane j holding the j-th largest key and its mass
    if (wave == 0) {
      const bool in = lane < n_c;
      const uint32_t key = in ? sorted[lane] : 0u;
      const bool by_k = in && key >= kth;                 // kept by top-k: a leading part of the lanes
      const double mj = by_k ? cmass[lane] : 0.0;
      const uint64_t kmask = __ballot(by_k);
      int kept = __popcll(kmask);
      if (p.top_p < 1.0f) {
        const double zk = wave_sum(mj);
        const double target = (double)p.top_p * zk;
        double incl = mj;                                   // inclusive running mass in descending order
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const double up = __shfl_up(incl, off);
          if (lane >= off) incl += up;
        }
        const double before = __shfl_up(incl, 1);
        const double excl = lane ? before : 0.0;
        // mass above a token = running mass before the first lane of its value group
        const uint32_t prev_key = __shfl_up(key, 1);
        const uint64_t starts = __ballot(lane == 0 || key != prev_key);
        const uint64_t upto = starts & (lane == 63 ? ~0ull : ((2ull << lane) - 1));
        const int g = 63 - __clzll((long long)upto);
        const double above = __shfl(excl, g);
        kept = __popcll(__ballot(by_k && above < target));   // a leading part as well: `above` never falls
      }
      const double z = wave_sum(lane < kept ? mj : 0.0);
      const uint32_t key_last = __shfl(key, kept - 1);
      if (lane == 0) s_key = key_last, s_z = z;
    }
  } else if (tid == 0) {
    int n_k = k;
    while (n_k < n_c && sorted[n_k] == kth) ++n_k;   // ties with the k-th largest stay
    int kept = n_k;
    if (p.top_p < 1.0f) {
      double zk = 0.0;
      for (int j = 0; j < n_k; ++j) zk += cmass[j];
      const double target = (double)p.top_p * zk;
      double above = 0.0;
      int j = 0;
      while (j < n_k && above < target) {   // the tokens of one value stay or go together
        int e = j;
        double group = 0.0;
        while (e < n_k && sorted[e] == sorted[j]) group += cmass[e++];
        above += group;
        j = e;
      }
      kept = j;
    }
    double z = 0.0;
    for (int j = 0; j < kept; ++j) z += cmass[j];
    s_key = sorted[kept - 1];
    s_z = z;
  }
  __syncthreads();
  *key_min_out = s_key;
  *z_out = s_z;
  return true;
}

// top-p without top-k through a candidate list.  zk, the exact fp64 mass of the whole row, is the fold of the row's
// fine-slice sums (accept_rowz_kernel).  One pass gives every lane's largest logit.  The kListRank-th largest of the
// lane maxima is a value that a bounded number of tokens reach (a rank statistic: about 1400 of a long row whatever
// the logits' law, when tokens of all sizes are spread evenly over the lanes); the tokens at or above it are listed
// in a second pass, sorted, given their exact masses, and the kept set is read off the list as the definition says:
// value groups in descending order while the mass above them is below top_p * zk.  The list is checked exactly: it
// must hold at least top_p * zk (then every token outside it has at least that much mass above it and is dropped).
// When it does not, or when more than kCand tokens qualify, the caller takes the histogram path (returns false, the
// same in every lane); zk is returned in either case.
constexpr int kListRank = 768;

template <bool BF16>
__device__ __forceinline__ bool warp_top_p_list(const AcceptParams &p, const void *row, const double *zs,
                                                double mx_over_t, double unit, double *red, uint32_t *list, double *cmass,
                                                double *zk_out, uint32_t *key_min_out, double *z_out) {
  __shared__ int s_cnt[2][kWarpThreads / 64];
  __shared__ int s_n, s_ok;
  __shared__ uint32_t s_key;
  __shared__ double s_z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float mx = -INFINITY;
  row_foreach<BF16>(row, p.V, [&](float x) { mx = fmaxf(mx, x); });
  // zk from the row's fine-slice sums (accept_rowz_kernel), in a fixed order: slice t in lane t, a butterfly per
  // wavefront, the wavefronts in order
  double acc = 0.0;
  for (int t = tid; t < p.n_fine; t += kWarpThreads) acc += zs[t];
  acc = wave_sum(acc);
  if (lane == 0) red[wave] = acc;
  const uint32_t lo = kth_largest_lane_key<BF16>(order_key(mx), kListRank, s_cnt);   // (its barriers publish red[])
  double zk = 0.0;
#pragma unroll
  for (int w = 0; w < kWarpThreads / 64; ++w) zk += red[w];
  zk *= unit;   // in units of e^(max/T), as all masses below
  *zk_out = zk;
  const float lo_val = key_value(lo);   // -inf when fewer than kListRank lanes own a token: the whole row is listed
  if (tid == 0) s_n = 0;
  __syncthreads();
  row_collect<BF16>(row, p.V, lo_val, list, kCand, &s_n);
  __syncthreads();
  const int n_c = s_n;
  if (n_c > kCand || n_c < 1) return false;
  sort_desc(list, n_c);
  for (int i = tid; i < n_c; i += kWarpThreads) cmass[i] = mass64(key_value(list[i]), mx_over_t, p.inv_temp);
  __syncthreads();
  if (wave == 0) {
    // lane l owns the list entries [l*per, (l+1)*per); running masses in descending order of the keys
    const double target = (double)p.top_p * zk;
    const int per = (n_c + 63) / 64;
    const int i0 = min(n_c, lane * per), i1 = min(n_c, i0 + per);
    double own = 0.0;
    for (int i = i0; i < i1; ++i) own += cmass[i];
    double incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    const double total = __shfl(incl, 63);
    const double before = __shfl_up(incl, 1);
    // first entry with at least `target` of mass before it (n_c if none): the entries before it stay whatever
    // their value groups; if it lies inside a value group, that group stays as a whole
    double run = lane ? before : 0.0;
    int cross = INT_MAX;
    for (int i = i0; i < i1; ++i) {
      if (cross == INT_MAX && !(run < target)) cross = i;
      run += cmass[i];
    }
    const uint64_t hits = __ballot(cross != INT_MAX);
    int first = n_c;
    if (hits) first = __shfl(cross, __ffsll((unsigned long long)hits) - 1);
    const uint32_t kref = list[first - 1];   // first >= 1: nothing lies before entry 0
    int end = INT_MAX;
    for (int i = max(i0, first); i < i1; ++i)
      if (end == INT_MAX && list[i] != kref) end = i;
    const uint64_t ends = __ballot(end != INT_MAX);
    int kept = n_c;
    if (ends) kept = __shfl(end, __ffsll((unsigned long long)ends) - 1);
    double zl = 0.0;
    for (int i = i0; i < min(i1, kept); ++i) zl += cmass[i];
    const double z = wave_sum(zl);
    if (lane == 0) {
      s_ok = total >= target ? 1 : 0;   // otherwise the kept set continues below the listed tokens
      s_key = list[kept - 1];
      s_z = z;
    }
  }
  __syncthreads();
  if (!s_ok) return false;
  *key_min_out = s_key;
  *z_out = s_z;
  return true;
}

// rowz: grid (groups of RowzShape::kGroup fine slices, NB*(K+1)).  fp64 sum of exp((x - max)/T) over each 2048-token fine
// slice of one target row, for top-p without top-k, whose threshold is a share of the row's whole mass: the row's
// exponentials are spread over the chip here instead of being one workgroup's pass in the warp kernel.  A workgroup
// takes several slices so that its start-up (the row maximum from the slice statistics) is shared and all its loads
// are in flight together.  With a table six: of four, six and eight, six is the fastest at rows of 75 slices (30 to 256 rows:
// four 1.02, eight 1.01 of its time, whole call); eight is where it divides the row better (32 slices, 256 rows: 41.7 against
// 47.2 us; 128 slices: 93.9 against 99.3).
template <bool TAB>
struct RowzShape {
  static constexpr int kHalves = TAB ? 2 : 1;
  static constexpr int kT = kHalves * kThreads;
  static constexpr int kPer = TAB ? 3 : 4;
  static constexpr int kGroup = kHalves * kPer;   // fine slices of a workgroup
};
__host__ __device__ inline int rowz_group(const AcceptParams &p) {
  return p.exp_tab ? RowzShape<true>::kGroup : RowzShape<false>::kGroup;
}
//
// It also lists the tokens top-p can keep.  With Z the row's mass, tokens whose own mass is below (1 - top_p) Z / V
// weigh less than (1 - top_p) Z together, so none of them is kept, and of a row that is peaked enough for a short list
// the same holds for eight times that mass (normal logits, V = 152064, 31 to 8600 tokens kept: from 24 times on).  The
// bound taken is that of eight times the mass, from the fp32 statistics; whether the listed tokens hold top_p Z is
// checked exactly by the warp kernel.  (Normal logits of deviation 3, T = 0.6, top_p = 0.95: 2900 listed, 350 kept.)
// A workgroup writes its tokens' keys in token order to a segment of p.cand, whose space the lists of the resampling
// path use later; the warp kernel finds the threshold among them without reading the row.  A segment that
// does not fit says so by its count, and the row takes the long way.
struct CandHeader {
  uint32_t n, pad[3];   // tokens at or above the bound (more than fit: the segment is not complete)
};
// A row's space is shared out by slices, so that a last group of few of them does not take a whole group's part.
__device__ __forceinline__ uint8_t *cand_segment(const AcceptParams &p, int rw, int group) {
  return p.cand + (size_t)rw * p.cand_row + (size_t)((uint32_t)group * (uint32_t)p.cand_seg);
}
// Most keys of a segment in the workgroup's LDS: 1792 of bf16 logits (with a table, four workgroups' tables and lists fit a CU's
// LDS), 1024 of fp32 ones.  Of bf16 logits of deviation 3 at T 1.0 and top_p 0.95 one in eight is listed, at 0.98 one in five.
// Rows whose lists are complete but fall short (deviation 2, top_p 0.9: one in five as well) pay the counting before the long
// way (V = 8192: 79 -> 82 us).
template <bool BF16>
constexpr int kCandLds = BF16 ? 1792 : 1024;
__device__ __forceinline__ int cand_capacity(const AcceptParams &p, int group) {
  return group + 1 < p.cand_groups ? p.cand_cap : p.cand_cap_last;
}

template <bool BF16, bool TAB>
__global__ __launch_bounds__(RowzShape<TAB>::kT, (TAB ? 6 : 1)) void accept_rowz_kernel(const AcceptParams p) {
  using Sh = RowzShape<TAB>;
  typedef typename std::conditional<BF16, uint16_t, uint32_t>::type key_t;
  __shared__ double red[Sh::kPer][Sh::kT / 64];
  __shared__ int s_cnt[Sh::kT / 64];
  __shared__ alignas(4) key_t s_list[kCandLds<BF16> + 2];   // (bf16: the second half of the last word)
  __shared__ alignas(16) double s_tab[TAB ? kTab : 2];
  const int rw = blockIdx.y, tid = threadIdx.x;
  // slices c0 .. c0 + kPer - 1 of this half of the workgroup
  const int ht = tid % kThreads, c0 = blockIdx.x * Sh::kGroup + tid / kThreads * Sh::kPer;
  const int lane = tid & 63, wave = tid >> 6;
  const bool vec = ((size_t)p.V * (BF16 ? 2 : 4)) % 16 == 0;
  // the row maximum from the slice statistics (exact, so the same value in every workgroup and in the warp kernel) and
  // its fp32 mass; requested before the logits, so that the fold runs while those are on their way
  const bool one_round = p.n_chunks <= 64;
  f32x2 st = {-INFINITY, 0.f};
  if (one_round && lane < p.n_chunks) st = *(const f32x2 *)(p.stats + ((size_t)rw * p.n_chunks + lane) * 2);
  TableCopy<Sh::kT> copy;
  if constexpr (TAB) copy.load(p.exp_tab);
  FineWords<BF16> w[Sh::kPer];
#pragma unroll
  for (int g = 0; g < Sh::kPer; ++g)   // (slices past the row read as -inf)
    w[g].load(p.target, (size_t)rw * p.V, (c0 + g) * kFine + ht * kFinePer, p.V, vec);
  if constexpr (TAB) {
    copy.store(s_tab);
    __syncthreads();
  }
  float m, z32;
  if (one_round) {
    m = wave_max_dpp(st.x);
    z32 = wave_sum_dpp(lane < p.n_chunks ? st.y * __builtin_amdgcn_exp2f((st.x - m) * p.inv_temp_log2) : 0.f);
  } else {
    wave_fold_row(p, rw, lane, m, z32);
  }
  const double o_t = mass_unit(p, m);
  // (a token without mass -- a masked one, or a place past V -- is never listed)
  const float bound =
      fmaxf(m + __builtin_amdgcn_logf(8.0f * (1.0f - p.top_p) * z32 / (float)p.V) / p.inv_temp_log2, -3.402823466e38f);
  uint32_t marks = 0;   // bit g*8 + e: token e of slice g is listed
#pragma unroll
  for (int g = 0; g < Sh::kPer; ++g) {
    float x[kFinePer];
    double mass[kFinePer], acc = 0.0;
    w[g].get(x);
    masses<BF16, TAB>(w[g], s_tab, o_t, p, mass);   // (past V: -inf, mass 0)
#pragma unroll
    for (int e = 0; e < kFinePer; ++e) {
      acc += mass[e];
      if (x[e] >= bound) marks |= 1u << (g * kFinePer + e);
    }
    acc = wave_sum(acc);
    if (lane == 0) red[g][wave] = acc;
  }
  const int own = __popc(marks);
  int incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) s_cnt[wave] = incl;
  __syncthreads();
  if (ht < Sh::kPer && c0 + ht < p.n_fine) {
    const double *r = red[ht] + tid / kThreads * (kThreads / 64);
    p.warp_zs[(size_t)rw * p.n_fine + c0 + ht] = (r[0] + r[1]) + (r[2] + r[3]);
  }
  if (p.cand_row) {   // (uniform)
    // in rounds, one listed token per lane and round, its logit read once more (few, and just loaded: a test per token in
    // straight code took 4 us of the kernel's 18); through LDS, then in whole words to the segment
    uint8_t *seg = cand_segment(p, rw, blockIdx.x);
    int total = 0;
#pragma unroll
    for (int i = 0; i < Sh::kT / 64; ++i) total += s_cnt[i];
    if (tid == 0) ((CandHeader *)seg)->n = (uint32_t)total;
    if (total > cand_capacity(p, blockIdx.x)) return;   // (uniform)
    int at = incl - own;
    for (int i = 0; i < wave; ++i) at += s_cnt[i];
    for (; marks; marks &= marks - 1, ++at) {
      const int bit = __ffs((int)marks) - 1;
      const int v = (c0 + bit / kFinePer) * kFine + ht * kFinePer + bit % kFinePer;
      const uint32_t key = order_key(load_logit<BF16>(p.target, (size_t)rw * p.V + v));
      s_list[at] = (key_t)(BF16 ? key >> 16 : key);
    }
    __syncthreads();
    uint32_t *to = (uint32_t *)(seg + sizeof(CandHeader));   // (room for a multiple of 16 bytes)
    const int words = BF16 ? (total + 1) / 2 : total;
    for (int i = tid; i < words; i += Sh::kT) to[i] = ((const uint32_t *)s_list)[i];
  }
}

// top-p without top-k from the segments accept_rowz_kernel wrote.  The threshold is the largest c with
// mass{key >= c} >= top_p * zk: the tokens at or above it stay -- the mass above each of them is below the target --
// and no other does.
// bf16 rows have few distinct values between the listed tokens' smallest and the row maximum (128 an octave): the tokens
// are counted per value, and the threshold is read off the running mass over the values in descending order
// (warp_top_p_bins: 14.7 -> 7.8 us at 54 rows of 152064, T 0.6, top_p 0.95; and the list may be of any length: a call with
// 15 rows at T 1.0, whose lists were too long for the form below, takes 36 instead of 214 us).  Where the list spans more
// values, and for fp32 rows, it is found from the top bits down, two bits per round, the fp64 masses of a lane's keys in
// registers and three sums per round; every sum runs in a fixed order.  Bound by its chain of loads, barriers and
// rounds, 54 workgroups on the chip: 44.3 -> 14.6 us at 54 rows of 152064 (T 0.6, top_p 0.95) against two passes of a
// workgroup over its row and a sort; with the sums through LDS shuffles it was 21.4 us.  false: a segment is incomplete, the list is
// longer than the workgroup holds, or it falls short of the target (the same decision in every lane).
constexpr int kCandPer = 8;                        // keys per lane
constexpr int kCandMax = kCandPer * kWarpThreads;  // (the LDS list holds as many)

// The form for bf16 rows.  m: the row maximum; zk: the row's mass; keys0: the first 16 bytes a lane reads of its wavefront's
// first segment, requested before the segments' counts were known; s_n: the counts.  BINS_OUTSIDE: the listed tokens span more
// values than there are bins; BINS_SHORT: they fall short of the target (the same decision in every lane).
enum BinsResult { BINS_DONE, BINS_OUTSIDE, BINS_SHORT };
constexpr int kBinPer = 4;                       // values per lane
constexpr int kBins = kBinPer * kWarpThreads;    // 32 octaves; the counts share the list's storage

__device__ __forceinline__ BinsResult warp_top_p_bins(const AcceptParams &p, int rw, float m, double zk, u32x4 keys0, const int *s_n,
                                                int n_g, uint32_t *bins, uint32_t *key_min_out, double *z_out) {
  constexpr int kW = kWarpThreads / 64;
  __shared__ int s_outside, s_at[kW];
  __shared__ double s_mass[kW], s_at_mass[kW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t top = order_key(m) >> 16;
  if (tid == 0) s_outside = 0;
  *(u32x4 *)(bins + tid * kBinPer) = (u32x4){0, 0, 0, 0};
  __syncthreads();
  for (int g = wave; g < n_g; g += kW) {
    const u32x4 *keys = (const u32x4 *)(cand_segment(p, rw, g) + sizeof(CandHeader));
    const int cnt = s_n[g];
    for (int i = lane; i * 8 < cnt; i += 64) {   // eight keys to a load (a segment holds a multiple of 16 bytes)
      const u32x4 w = g == wave && i == lane ? keys0 : keys[i];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t word = w[k];
        const uint32_t b0 = top - (word & 0xFFFFu), b1 = top - (word >> 16);
        const bool in0 = i * 8 + 2 * k < cnt, in1 = i * 8 + 2 * k + 1 < cnt;
        if (in0 && b0 < kBins) atomicAdd(&bins[b0], 1u);
        if (in1 && b1 < kBins) atomicAdd(&bins[b1], 1u);
        if ((in0 && b0 >= kBins) || (in1 && b1 >= kBins)) s_outside = 1;
      }
    }
  }
  __syncthreads();
  if (s_outside) return BINS_OUTSIDE;
  const double o_t = mass_unit(p, m);
  const u32x4 n_of = *(const u32x4 *)(bins + tid * kBinPer);
  auto key_of = [&](int bin) {   // (the sixteen low bits of a widened bf16 value's key)
    const uint32_t k = (top - (uint32_t)bin) << 16;
    return k | ((k >> 31) ? 0u : 0xFFFFu);
  };
  double mass[kBinPer], own = 0.0;
#pragma unroll
  for (int j = 0; j < kBinPer; ++j) {
    const uint32_t n = n_of[j];
    mass[j] = 0.0;
    if (__ballot(n != 0))
      mass[j] = n ? (double)n * mass64(key_value(key_of(tid * kBinPer + j)), o_t, p.inv_temp) : 0.0;
    own += mass[j];
  }
  // running mass in descending order of the values: lanes, then wavefronts, in order
  double incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) s_mass[wave] = incl;
  __syncthreads();
  double before = 0.0;
  for (int w = 0; w < wave; ++w) before += s_mass[w];
  const double target = (double)p.top_p * zk;
  double run = before + (incl - own), at_mass = 0.0;
  int at = INT_MAX;   // this lane's first value at which the running mass reaches the target
#pragma unroll
  for (int j = 0; j < kBinPer; ++j) {
    run += mass[j];
    if (at == INT_MAX && mass[j] > 0.0 && run >= target) at = tid * kBinPer + j, at_mass = run;
  }
  const uint64_t hits = __ballot(at != INT_MAX);
  const int src = hits ? __ffsll((unsigned long long)hits) - 1 : 0;
  const int first = __shfl(at, src);
  const double first_mass = __shfl(at_mass, src);
  if (lane == 0) s_at[wave] = first, s_at_mass[wave] = first_mass;
  __syncthreads();
  int bin = INT_MAX;
  double z = 0.0;
#pragma unroll
  for (int w = 0; w < kW; ++w)
    if (bin == INT_MAX && s_at[w] != INT_MAX) bin = s_at[w], z = s_at_mass[w];
  if (bin == INT_MAX) return BINS_SHORT;
  *key_min_out = key_of(bin);
  *z_out = z * unit_over_max(p, m);
  return BINS_DONE;
}

template <bool BF16>
__device__ __forceinline__ bool warp_top_p_segments(const AcceptParams &p, int rw, double *red, uint32_t *list, float *row_max_out,
                                                    uint32_t *key_min_out, double *z_out) {
  constexpr int kW = kWarpThreads / 64;
  constexpr int kMaxGroups = kMaxFine / RowzShape<false>::kGroup;
  __shared__ int s_off[kMaxGroups + 1], s_n[kMaxGroups], s_wave[kW], s_bad;
  __shared__ uint32_t s_low[kW];
  __shared__ double s_sum[2][3][kW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_g = p.cand_groups;
  // zk from the row's fine-slice sums, in a fixed order: slice t in lane t, a butterfly per wavefront, the wavefronts
  // in order
  u32x4 keys0 = {0, 0, 0, 0};
  if (BF16 && wave < n_g && lane * 8 < cand_capacity(p, wave))
    keys0 = ((const u32x4 *)(cand_segment(p, rw, wave) + sizeof(CandHeader)))[lane];
  double acc = 0.0;
  for (int t = tid; t < p.n_fine; t += kWarpThreads) acc += p.warp_zs[(size_t)rw * p.n_fine + t];
  // where each segment's keys go in the list (n_g <= kMaxGroups <= the workgroup)
  const int own = tid < n_g ? (int)((const CandHeader *)cand_segment(p, rw, tid))->n : 0;
  float m = -INFINITY;   // the row maximum
  for (int c = lane; c < p.n_chunks; c += 64) m = fmaxf(m, p.stats[((size_t)rw * p.n_chunks + c) * 2]);
  acc = wave_sum(acc);
  if (lane == 0) red[wave] = acc;
  m = wave_max_dpp(m);
  *row_max_out = m;
  const double o_t = mass_unit(p, m);   // the masses here are in the unit of the slice sums
  const bool bad = tid < n_g && own > cand_capacity(p, tid);
  int incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) s_wave[wave] = incl;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  if (bad) s_bad = 1;
  int base = 0, n = 0;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    base += w < wave ? s_wave[w] : 0;
    n += s_wave[w];
  }
  if (tid < n_g) s_off[tid] = base + incl - own, s_n[tid] = own;
  if (tid == n_g) s_off[n_g] = n;
  double zk = 0.0;
#pragma unroll
  for (int w = 0; w < kW; ++w) zk += red[w];
  __syncthreads();
  if (s_bad || n < 1) return false;
  if constexpr (BF16) {
    const BinsResult r = warp_top_p_bins(p, rw, m, zk, keys0, s_n, n_g, list, key_min_out, z_out);
    if (r != BINS_OUTSIDE) return r == BINS_DONE;
    __syncthreads();
  }
  if (n > kCandMax) return false;
  for (int g = wave; g < n_g; g += kW) {
    const uint8_t *keys = cand_segment(p, rw, g) + sizeof(CandHeader);
    const int off = s_off[g], cnt = s_off[g + 1] - off;
    for (int i = lane; i < cnt; i += 64) {
      if constexpr (BF16) {   // (the sixteen low bits of a widened bf16 value's key)
        const uint32_t k = (uint32_t)((const uint16_t *)keys)[i] << 16;
        list[off + i] = k | ((k >> 31) ? 0u : 0xFFFFu);
      } else {
        list[off + i] = ((const uint32_t *)keys)[i];
      }
    }
  }
  __syncthreads();
  uint32_t key[kCandPer], low = 0xFFFFFFFFu;
  double mass[kCandPer], total = 0.0;
#pragma unroll
  for (int j = 0; j < kCandPer; ++j) {
    const int i = tid + j * kWarpThreads;
    key[j] = 0u, mass[j] = 0.0;
    if (j * kWarpThreads < n) {   // (uniform)
      if (i < n) {
        key[j] = list[i];
        low = min(low, key[j]);
        mass[j] = mass64(key_value(key[j]), o_t, p.inv_temp);
      }
      total += mass[j];
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) low = min(low, (uint32_t)__shfl_xor((int)low, off));
  total = wave_sum(total);
  if (lane == 0) s_low[wave] = low, red[wave] = total;
  __syncthreads();
  total = 0.0;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    total += red[w];
    low = min(low, s_low[w]);
  }
  const double target = (double)p.top_p * zk;
  if (!(total >= target)) return false;
  // the bits all listed keys share stay as they are
  const uint32_t top = order_key(m), diff = top ^ low;
  int bit = diff ? 31 - __clz((int)diff) : -1;   // the highest bit that differs
  const int last = BF16 ? 16 : 0;
  uint32_t lo = bit < 31 ? low & ~((2u << bit) - 1) : 0u;
  if (bit < 0) lo = low;
  double z = total;
  for (int round = 0; bit >= last; ++round) {
    const int sh = max(last, bit - 1);             // this round decides bits bit .. sh (two, or the last one alone)
    const int ways = bit == sh ? 1 : 3;
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < kCandPer; ++j)
      if (j * kWarpThreads < n) {
#pragma unroll
        for (int w = 0; w < 3; ++w) s[w] += key[j] >= (lo | ((uint32_t)(w + 1) << sh)) ? mass[j] : 0.0;
      }
#pragma unroll
    for (int w = 0; w < 3; ++w) s[w] = wave_sum(s[w]);
    if (lane == 0) {
#pragma unroll
      for (int w = 0; w < 3; ++w) s_sum[round & 1][w][wave] = s[w];
    }
    __syncthreads();   // (one barrier per round: the next round writes the other half)
    // row w of a wavefront adds up the wavefronts' shares of sum w
    static_assert(kW == 16, "a DPP row holds one share per wavefront");
    const double share = row_sum(lane < 3 * kW ? s_sum[round & 1][lane >> 4][lane & 15] : 0.0);
    int take = 0;
#pragma unroll
    for (int w = 0; w < 3; ++w) {
      const double t = lane_value(share, 16 * w);
      if (w < ways && t >= target) take = w + 1, z = t;   // (falls with w)
    }
    lo |= (uint32_t)take << sh;
    bit = sh - 1;
  }
  *key_min_out = lo;
  *z_out = z * unit_over_max(p, m);
  return true;
}

template <bool BF16>
__global__ __launch_bounds__(kWarpThreads) void accept_warp_kernel(const AcceptParams p) {
  __shared__ alignas(16) double mass[kHist * kRep];   // the count histogram and the lists share this storage (16-byte accesses)
  uint32_t *cnt = (uint32_t *)mass;
  __shared__ uint32_t s_pick;
  __shared__ double s_above, s_slot;
  __shared__ double red[kWarpThreads / 64];
  __shared__ float s_m;
  const int rw = blockIdx.x;   // target row nb*(K+1) + i
  const int tid = threadIdx.x;
  const uint8_t *row = (const uint8_t *)p.target + (size_t)rw * p.V * (BF16 ? 2 : 4);
  auto each_of_row = [&](auto &&f) { row_foreach<BF16>(row, p.V, f); };
  uint32_t key_min = 0;
  double zw = 0.0;
  float m = 0.f;
  bool done = false;
  if (p.top_k > 0 && p.top_k < p.V && p.top_k <= kSmallK)   // the candidate list lives in the histogram's storage
    done = warp_small_k<BF16>(p, row, cnt, cnt + kCand, mass + kCand, &m, &key_min, &zw);
  const bool use_k = p.top_k > 0 && p.top_k < p.V;
  if (!done && !use_k && p.top_p < 1.0f && p.cand_row) {   // (the candidate lists live in the histogram's storage)
    done = warp_top_p_segments<BF16>(p, rw, red, cnt, &m, &key_min, &zw);
    __syncthreads();
  }
  if (!done) {
    if (tid < 64) {
      float z;
      wave_fold_row(p, rw, tid, m, z);
      if (tid == 0) s_m = m;
    }
    __syncthreads();
    m = s_m;
    const double mx_over_t = (double)m * p.inv_temp;
    key_min = 0;
    if (use_k)
      key_min = radix_select<BF16, false>(each_of_row, 0.0, 0.0, 0u, p.top_k, 0.0, cnt, mass, &s_pick, &s_above);
    bool listed = false;
    if (p.top_p < 1.0f) {
      double zk = 0.0;
      if (!use_k)
        listed = warp_top_p_list<BF16>(p, row, p.warp_zs + (size_t)rw * p.n_fine, mx_over_t, unit_over_max(p, m), red, cnt, mass + kCand,
                                       &zk, &key_min, &zw);
      else
        zk = kept_mass<BF16>(row, p.V, mx_over_t, p.inv_temp, key_min, red, &s_slot);
      if (!listed)
        key_min = radix_select<BF16, true>(each_of_row, mx_over_t, p.inv_temp, key_min, 0, (double)p.top_p * zk, cnt,
                                           mass, &s_pick, &s_above);
    }
    if (!listed) zw = kept_mass<BF16>(row, p.V, mx_over_t, p.inv_temp, key_min, red, &s_slot);
  }
  if (tid == 0) {
    // a row that keeps everything (the histogram's floor, 0) has the key of -inf: the keys below it decode to NaNs, which no
    // logit compares above, and the kernels behind this one compare values
    p.warp_key[rw] = max(key_min, order_key(-INFINITY));
    p.warp_z[rw] = zw;
  }
}

// ---------------------------------------------------------------------------------------------
// sample: grid (n_fine slices, one or two to a workgroup; NB).  Accepted length of the branch (every workgroup derives
// it; slice 0 publishes it), then what this slice contributes to the normalisers of the resampling rows and to the
// residual.
//
// The residual max(0, a/Zt - b/Zq) of a token (a, b its unnormalised masses in the target and the draft row) needs both
// normalisers, which all workgroups of the branch contribute to, but its sign nearly never does: Zt/Zq is known from the
// fp32 statistics to a part in 10^5 or better.  So one pass over the two rows gives, per slice, the sums of a and b, and
// the sums of a and of b over the tokens whose residual is positive beyond doubt; the few tokens in doubt go to a list.
// The pick kernel, with the exact normalisers, adds the listed ones that turn out positive -- and checks that the fp32
// quotient was within the margin allowed for it.  With two passes (normalisers, then residuals) and a launch between
// them the exponentials were evaluated twice: 16.5 + 17.7 us at 32 branches of 152064.
// ---------------------------------------------------------------------------------------------
constexpr int kAmb = 48;   // tokens in doubt a wavefront can list of its 512 tokens of a slice
constexpr uint32_t kAmbOver = 255;
struct Doubt {
  double a, b;
};
__device__ __forceinline__ Doubt *doubt_list(const AcceptParams &p, int nb, int c, int wave) {
  return (Doubt *)p.amb + (((size_t)nb * p.n_fine + c) * (kThreads / 64) + wave) * kAmb;
}

// More tokens in doubt than a list holds: one entry per value of x - y among them (target and draft logits).  Tokens of one
// value have one quotient a / b and so residuals of one sign, and their sums can stand for them.  bf16 logits have few such
// values (a draft close to its target: mostly equal logits).  Returns the number of entries, or kAmbOver where there are too
// many or a difference is not exact in fp32: pick evaluates such a slice again, 2 us each at up to 75 slices of V = 152064 (fp32
// rows that agree to 1e-5 of a logit everywhere, which reject one draft in 10^5).  Measured, V = 152064, rows with one normaliser
// that agree in 12 % of the logits: 32 branches 214 -> 57 us (51 without a token in doubt), four 173 -> 24 us.
template <bool BF16>
__device__ __forceinline__ uint32_t list_doubt_groups(const AcceptParams &p, size_t t_at, size_t d_at, uint32_t doubt,
                                                      const double (&a)[kFinePer], const double (&b)[kFinePer], Doubt *to) {
  float d[kFinePer];
  bool exact = true;
#pragma unroll
  for (int e = 0; e < kFinePer; ++e) {   // (the logits once more: no registers for them on the common path)
    d[e] = 0.f;
    if (doubt & (1u << e)) {
      const float x = load_logit<BF16>(p.target, t_at + e), y = load_logit<BF16>(p.draft, d_at + e);
      d[e] = x - y;
      const float back = d[e] - x, front = d[e] - back;   // (the error of the difference, in fp32 without one itself)
      exact = exact && (x - front) - (y + back) == 0.f;
    }
  }
  if (__ballot(!exact)) return kAmbOver;
  uint32_t n = 0;
  for (uint64_t left; (left = __ballot(doubt != 0)) != 0; ++n) {
    if (n == kAmb) return kAmbOver;
    float first = 0.f;   // of the lane's tokens
#pragma unroll
    for (int e = kFinePer - 1; e >= 0; --e) first = doubt & (1u << e) ? d[e] : first;
    const float value = lane_value(first, __ffsll((unsigned long long)left) - 1);
    double ga = 0.0, gb = 0.0;
#pragma unroll
    for (int e = 0; e < kFinePer; ++e)
      if ((doubt & (1u << e)) && d[e] == value) ga += a[e], gb += b[e], doubt &= ~(1u << e);
    ga = wave_sum(ga);
    gb = wave_sum(gb);
    if ((threadIdx.x & 63) == 0) to[n] = {ga, gb};
  }
  return n;
}

// What the resampling of a branch needs besides its slices' sums: maxima of its two rows and their fp32 masses.
struct alignas(16) BranchHead {
  float mt, mq, zt, zq;
  // The residual of a token with logits x, y is positive iff (x - y) / T > ln(e^(mt/T) zt / (e^(mq/T) zq)), here in fp32
  // and log2 units: x - y in doubt if it is within `margin` of that.  One half of the margin is for the fp32 masses (sums
  // of at most 2^21 terms in blocks, a few 1e-6; the exponents' rounding grows with their size), which pick checks, the
  // other for the three roundings of the comparison (each 2^-24 of at most 2 max|m| log2(e)/T + 21).
  __device__ __forceinline__ float margin(const AcceptParams &p) const {
    return 2e-5f + 1e-6f * (fmaxf(fabsf(mt), fabsf(mq)) * p.inv_temp_log2);
  }
};

// Slices of a workgroup, 256 lanes each: two share a table (four workgroups' tables fit a CU's LDS).  Measured: four slices
// per workgroup, in two rounds, leave some CUs three workgroups and others two (15.0 against 14.6 us at 32 branches of
// 152064); 64 registers instead of 70, for a fourth workgroup per CU, spill.
template <bool TAB>
constexpr int kSampleSlices = TAB ? 2 : 1;

template <bool BF16, bool TAB>
__global__ __launch_bounds__(kSampleSlices<TAB> * kThreads, (TAB ? 6 : 1)) void accept_sample_kernel(const AcceptParams p) {
  constexpr int kHalves = kSampleSlices<TAB>, kT = kHalves * kThreads;
  constexpr int kPass = 64;                       // drafted positions examined per pass
  constexpr int kRow = 16;                        // lanes that fold one row's slice statistics (a DPP row)
  __shared__ float sm[2][kPass], sz[2][kPass];    // [target|draft][position in pass]: folded row statistics
  __shared__ BranchHead s_head;                   // of the resampling rows
  __shared__ float s_bonus;                       // maximum of target row K
  __shared__ int s_first;
  __shared__ double red[4][kT / 64];
  __shared__ uint32_t s_amb[kT / 64];
  __shared__ alignas(16) double s_tab[TAB ? kTab : 2];
  const int nb = blockIdx.y, tid = threadIdx.x;
  const int ht = tid % kThreads, c = blockIdx.x * kHalves + tid / kThreads;   // lane of the slice, slice
  const bool first_wg = blockIdx.x == 0;
  const int lane = tid & 63, wave = tid >> 6;
  const int n_t = p.NB * (p.K + 1);
  const int n_which = p.draft ? 2 : 1;   // point-mass draft: there are no draft rows
  if (tid == 0) s_first = p.K;
  TableCopy<kT> copy;
  if constexpr (TAB) {
    copy.load(p.exp_tab);   // (stored once the loads of the first pass have been requested)
  }
  bool have_top = false;
  for (int i0 = 0; i0 < p.K; i0 += kPass) {   // a later pass cannot lower the first rejection found in an earlier one
    const int cnt = min(kPass, p.K - i0);
    // what a position's test needs from global memory besides the row statistics; issued first so that the two
    // dependent round trips (token, then its two logits) overlap the fold below
    int x = 0;
    float tx = 0.f, dx = 0.f, u = 0.f;
    if (tid < cnt) {
      const int i = i0 + tid;
      x = p.tokens[(size_t)nb * p.K + i];
      u = p.u_accept[(size_t)nb * p.K + i];
      tx = load_logit<BF16>(p.target, ((size_t)nb * (p.K + 1) + i) * p.V + x);
      if (p.draft) dx = load_logit<BF16>(p.draft, ((size_t)nb * p.K + i) * p.V + x);
    }
    // rows folded in this pass: cnt target rows, cnt draft rows and, in the last pass, target row K (the bonus row);
    // sixteen lanes per row
    const int bonus = i0 + cnt == p.K ? 1 : 0;
    const int n_rows = n_which * cnt + bonus;
    for (int slot = tid / kRow; slot < n_rows; slot += kT / kRow) {
      const int which = slot >= cnt, j = slot - which * cnt;
      const bool is_bonus = slot == n_which * cnt;
      const int rw = is_bonus ? nb * (p.K + 1) + p.K : which ? n_t + nb * p.K + i0 + j : nb * (p.K + 1) + i0 + j;
      const f32x2 *st = (const f32x2 *)(p.stats + (size_t)rw * p.n_chunks * 2);
      const int l = tid % kRow;
      f32x2 own = {-INFINITY, 0.f};
      if (l < p.n_chunks) own = st[l];
      float m = own.x;
      for (int ch = l + kRow; ch < p.n_chunks; ch += kRow) m = fmaxf(m, st[ch].x);
      m = row_max(m);
      float z = own.y * __builtin_amdgcn_exp2f((own.x - m) * p.inv_temp_log2);
      for (int ch = l + kRow; ch < p.n_chunks; ch += kRow)
        z += st[ch].y * __builtin_amdgcn_exp2f((st[ch].x - m) * p.inv_temp_log2);
      z = row_sum(z);
      if (l == 0) {
        if (is_bonus)
          s_bonus = m;
        else
          sm[which][j] = m, sz[which][j] = z;
      }
    }
    if (TAB && i0 == 0) copy.store(s_tab);
    __syncthreads();
    if (tid < cnt) {
      const int i = i0 + tid;
      float px = __builtin_amdgcn_exp2f((tx - sm[0][tid]) * p.inv_temp_log2) / sz[0][tid];
      if (p.warp_key) {  // warped target: x has mass only if its row keeps it, normalised by the kept mass
        const int wr = nb * (p.K + 1) + i;
        px = order_key(tx) >= p.warp_key[wr]
                 ? __builtin_amdgcn_exp2f((tx - sm[0][tid]) * p.inv_temp_log2) / (float)p.warp_z[wr]
                 : 0.f;
      }
      float qx = 1.0f;   // point-mass draft at x
      if (p.draft) qx = __builtin_amdgcn_exp2f((dx - sm[1][tid]) * p.inv_temp_log2) / sz[1][tid];
      if (!(u * qx < px)) atomicMin(&s_first, i);
      if (first_wg && p.ratio) p.ratio[(size_t)nb * p.K + i] = px / qx;
    }
    __syncthreads();
    if (s_first < p.K) {  // uniform: the first rejection lies in this pass
      // statistics of the resampling rows: target row n and draft row n, both folded in this pass
      if (!have_top && tid == 0) {
        const int j = s_first - i0;
        s_head = {sm[0][j], p.draft ? sm[1][j] : 0.f, sz[0][j], p.draft ? sz[1][j] : 1.f};
      }
      have_top = true;
      // the workgroup that reports the ratios goes on through the remaining passes (every position gets its ratio,
      // also those behind the rejection); s_first cannot change any more, atomicMin only lowers it to values < i
      if (!(first_wg && p.ratio)) break;
    }
    __syncthreads();  // sm / sz free for the next pass
  }
  const int n = s_first;
  // everything accepted: target row K alone (folded in the last pass), which no draft row is compared with
  if (n == p.K && tid == 0) s_head = {s_bonus, 0.f, 1.f, 1.f};
  __syncthreads();
  BranchHead head = s_head;
  const bool with_draft = n < p.K && p.draft;
  float x_min = 0.f;
  if (p.warp_key) {   // the kept mass replaces the row's full normaliser
    x_min = key_value(p.warp_key[nb * (p.K + 1) + n]);
    head.zt = (float)p.warp_z[nb * (p.K + 1) + n];
  }
  // point-mass draft after a rejection: the drafted token has no residual mass
  const int removed = (n < p.K && !p.draft) ? p.tokens[(size_t)nb * p.K + n] : -1;
  const size_t trow = ((size_t)nb * (p.K + 1) + n) * p.V;
  const size_t drow = ((size_t)nb * p.K + (n < p.K ? n : 0)) * p.V;
  const bool vec = ((size_t)p.V * (BF16 ? 2 : 4)) % 16 == 0;
  const int vb = c * kFine + ht * kFinePer;
  FineWords<BF16> wt, wd;   // (a slice past the row reads as -inf)
  wt.load(p.target, trow, vb, p.V, vec);
  if (with_draft) wd.load(p.draft, drow, vb, p.V, vec);
  if (first_wg && tid == 0) {
    p.accepted_len[nb] = n;
    p.n_acc[nb] = n;
    ((BranchHead *)p.heads)[nb] = head;
  }
  const double ot = mass_unit(p, head.mt), oq = mass_unit(p, head.mq);
  // (log2 units; x - y above the threshold: the residual is positive)
  const float margin = head.margin(p);
  const float threshold = (float)(((double)head.mt - (double)head.mq) * (double)p.inv_temp_log2 +
                                  (double)__builtin_amdgcn_logf(head.zt / head.zq));
  // no bounds test per token: places past V read as -inf, whose mass is exactly 0, and the eight masses of a lane can
  // then be evaluated side by side instead of one dependent chain after the other
  if (p.warp_key) wt.keep(x_min);   // (comparing values is comparing keys)
  double a[kFinePer], b[kFinePer];
  masses<BF16, TAB>(wt, s_tab, ot, p, a);
  double sa = 0.0, sb = 0.0, pa = 0.0, pb = 0.0;
  uint32_t doubt = 0;   // bit e: token e is in doubt
  if (with_draft) {
    masses<BF16, TAB>(wd, s_tab, oq, p, b);
    float tx[kFinePer], dx[kFinePer], closest = INFINITY;
    wt.get(tx);
    wd.get(dx);
#pragma unroll
    for (int e = 0; e < kFinePer; ++e) {
      sa += a[e];
      sb += b[e];
      // (where neither row has mass this is a NaN, and both terms are zero)
      const float d = __builtin_fmaf(tx[e] - dx[e], p.inv_temp_log2, -threshold);
      const bool pos = d > margin;
      pa += pos ? a[e] : 0.0;
      pb += pos ? b[e] : 0.0;
      closest = fminf(closest, fabsf(d));
      tx[e] = d;
    }
    if (__ballot(closest <= margin)) {
#pragma unroll
      for (int e = 0; e < kFinePer; ++e)   // (a token without mass in the target row has no residual)
        if (fabsf(tx[e]) <= margin && a[e] > 0.0) doubt |= 1u << e;
    }
  } else {
#pragma unroll
    for (int e = 0; e < kFinePer; ++e) {
      sa += a[e];
      pa += vb + e == removed ? 0.0 : a[e];
    }
  }
  sa = wave_sum(sa);
  pa = wave_sum(pa);
  if (with_draft) sb = wave_sum(sb), pb = wave_sum(pb);
  if (lane == 0) red[0][wave] = sa, red[1][wave] = sb, red[2][wave] = pa, red[3][wave] = pb;
  uint32_t n_amb = 0;
  if (with_draft && __ballot(doubt != 0)) {   // the wavefront's tokens in doubt, in token order
    const int own = __popc(doubt);
    int incl = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    n_amb = (uint32_t)__shfl(incl, 63);
    Doubt *to = doubt_list(p, nb, c, wave % (kThreads / 64));   // (a slice past the row lists none)
    if (n_amb > kAmb) {
      n_amb = list_doubt_groups<BF16>(p, trow + vb, drow + vb, doubt, a, b, to);
    } else {
      to += incl - own;
#pragma unroll
      for (int e = 0; e < kFinePer; ++e)
        if (doubt & (1u << e)) *to++ = {a[e], b[e]};
    }
  }
  if (lane == 0) s_amb[wave] = n_amb;
  __syncthreads();
  if (ht < 4 && c < p.n_fine) {   // lane k of a slice: sum k
    const double *r = red[ht] + tid / kThreads * (kThreads / 64);
    double *to = ht < 2 ? p.zsum : p.rsum;
    to[((size_t)nb * 2 + (ht & 1)) * p.n_fine + c] = (r[0] + r[1]) + (r[2] + r[3]);
    if (ht == 0) {
      const uint32_t *n_of = s_amb + tid / kThreads * (kThreads / 64);
      p.amb_n[(size_t)nb * p.n_fine + c] = n_of[0] | n_of[1] << 8 | n_of[2] << 16 | n_of[3] << 24;
    }
  }
}

// One double per wavefront from LDS, added up: the same value in every lane.
template <int kW>
__device__ __forceinline__ double sum_of_waves(const double *v) {
  static_assert(kW <= 16, "a DPP row holds one value per wavefront");
  const int i = threadIdx.x % 16;
  return row_sum(i < kW ? v[i] : 0.0);
}

// Where a running sum over the workgroup's values crosses thr = u * total: v is a lane's (non-negative) value, lanes in
// order.  Every lane gets the total, its own exclusive prefix, the first lane whose running sum exceeds thr (the last lane
// with a value if rounding hides it; -1 without any).  Two barriers inside, one expected before the next call.
template <int kW>
struct Crossing {
  double total, excl, thr;
  int lane;
  __device__ __forceinline__ void find(double v, double u, double base, bool have_total, double total_in, double *s_tot) {
    const int l = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double up = __shfl_up(incl, off);
      if (l >= off) incl += up;
    }
    const uint64_t some = __ballot(v > 0.0);
    if (l == 63) s_tot[wave] = incl;
    __shared__ int s_last[kW], s_hit[kW];
    if (l == 0) s_last[wave] = some ? (int)threadIdx.x + 63 - __clzll((long long)some) : -1;
    __syncthreads();
    total = have_total ? total_in : sum_of_waves<kW>(s_tot);
    const int i = threadIdx.x % 16;
    excl = base + row_sum(i < wave ? s_tot[i] : 0.0) + (incl - v);
    thr = u * total;
    const uint64_t hit = __ballot(v > 0.0 && excl + v > thr);
    if (l == 0) s_hit[wave] = hit ? (int)threadIdx.x + __ffsll((unsigned long long)hit) - 1 : INT_MAX;
    __syncthreads();
    const uint64_t waves = __ballot(l < kW && s_hit[l < kW ? l : 0] != INT_MAX);
    if (waves) {
      lane = s_hit[__ffsll((unsigned long long)waves) - 1];
    } else {
      lane = -1;
      for (int w = 0; w < kW; ++w) lane = max(lane, s_last[w]);
    }
  }
};

// ---------------------------------------------------------------------------------------------
// pick: grid NB.  Bound by its chain of loads, barriers and scans, one workgroup per branch.  T lanes: 512, four tokens of the
// chosen slice each (32 branches of 152064: 9.3 us; 256 lanes, of eight tokens, 11.8, 1024 lanes 10.7; 8 branches of one
// slice, whole call: 15.6 against 16.1 us).  Where the branches are more than two to a CU, wavefronts are what it waits for:
// 256 lanes and room for 256 slices' sums (1024 branches of one slice, whole call: 32 against 36 us; 4096: 91 against 103; 256:
// 19.9 against 19.3; of 16 slices, 256 branches 34.3 against 33.5, 1024 88.7 against 93.0).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ double residual(double pm, double qm) {
#pragma clang fp contract(off)
  return pm - qm;
}

constexpr int kPickMany = 512;   // branches up to which it runs 512 lanes
template <bool BF16, int T, int kMost>
__global__ __launch_bounds__(T) void accept_pick_kernel(const AcceptParams p) {
  constexpr int kW = T / 64, kOwn = kFine / T, kTerms = kMost / T;   // (a lane's slices: tid * kTerms + j)
  constexpr int kLists = kThreads / 64;         // lists of a slice
  __shared__ double buf0[kMost], buf1[kMost];   // slice sums of the residual and of p
  __shared__ uint32_t s_amb[kMost];             // tokens in doubt per slice, a byte per list
  __shared__ double s_sum[2][kW], s_tot[kW], s_before;
  __shared__ int s_flags[kW], s_slice;
  const int nb = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // everything that does not depend on the accepted length is requested in one round trip
  double ta[kTerms], tb[kTerms], pa[kTerms], pb[kTerms];
  uint32_t amb[kTerms];
  const size_t at0 = ((size_t)nb * 2 + 0) * p.n_fine, at1 = ((size_t)nb * 2 + 1) * p.n_fine;
#pragma unroll
  for (int j = 0; j < kTerms; ++j) {
    const int c = tid * kTerms + j;
    const bool in = c < p.n_fine;
    ta[j] = in ? p.zsum[at0 + c] : 0.0;
    tb[j] = in ? p.zsum[at1 + c] : 0.0;
    pa[j] = in ? p.rsum[at0 + c] : 0.0;
    pb[j] = in ? p.rsum[at1 + c] : 0.0;
    amb[j] = in ? p.amb_n[(size_t)nb * p.n_fine + c] : 0u;
  }
  const BranchHead head = ((const BranchHead *)p.heads)[nb];
  const int n = p.n_acc[nb];
  const double u = (double)p.u_sample[nb];
  const bool with_draft = n < p.K && p.draft;
  const int removed = (n < p.K && !p.draft) ? p.tokens[(size_t)nb * p.K + n] : -1;
  const size_t trow = ((size_t)nb * (p.K + 1) + n) * p.V;
  const size_t drow = ((size_t)nb * p.K + (n < p.K ? n : 0)) * p.V;
  float x_min = -INFINITY;
  double zw = 0.0;
  if (p.warp_key) {   // (comparing values is comparing keys)
    x_min = key_value(p.warp_key[nb * (p.K + 1) + n]);
    zw = p.warp_z[nb * (p.K + 1) + n];
  }
  double zt = 0.0, zq = 0.0;
#pragma unroll
  for (int j = 0; j < kTerms; ++j) zt += ta[j], zq += tb[j];
  zt = wave_sum(zt);
  zq = wave_sum(zq);
  if (lane == 0) s_sum[0][wave] = zt, s_sum[1][wave] = zq;
  __syncthreads();
  zt = sum_of_waves<kW>(s_sum[0]);
  zq = sum_of_waves<kW>(s_sum[1]);
  // the kept mass of a warped row replaces its full normaliser; it and the heads' are in units of e^(max/T)
  if (p.warp_key) zt = zw / unit_over_max(p, head.mt);
  if (!with_draft) zq = 1.0;
  const double inv_zt = 1.0 / zt, inv_zq = 1.0 / zq;
  const double mt_t = mass_unit(p, head.mt), mq_t = mass_unit(p, head.mq);
  // the residual and p of the tokens of slice c that this lane owns: all loads first, then the masses side by side
  // (tokens past V read as -inf and have no mass)
  auto eval = [&](int c, double (&r)[kOwn], double (&pm)[kOwn]) {
    const int v0 = c * kFine + tid * kOwn;
    const bool vec = ((size_t)p.V * (BF16 ? 2 : 4)) % 16 == 0;
    float tx[kOwn], dx[kOwn];
    load_own<BF16, kOwn>(p.target, trow, v0, p.V, vec, tx);
    if (with_draft) load_own<BF16, kOwn>(p.draft, drow, v0, p.V, vec, dx);
#pragma unroll
    for (int e = 0; e < kOwn; ++e) {
      // (no fused multiply-add over the difference: a token's residual is then the same here as from its listed masses)
      pm[e] = tx[e] >= x_min ? mass_again<BF16>(tx[e], mt_t, p) * inv_zt : 0.0;
      r[e] = v0 + e == removed ? 0.0 : pm[e];
      if (with_draft) r[e] = fmax(residual(pm[e], mass_again<BF16>(dx[e], mq_t, p) * inv_zq), 0.0);
    }
  };
  // the tokens counted as positive or negative by the fp32 quotient are so if the exact one lies within half the margin
  // of it; else every slice is evaluated again
  const bool trusted =
      !with_draft || fabs((double)head.zt / (double)head.zq * (zq * unit_over_max(p, head.mq)) /
                              (zt * unit_over_max(p, head.mt)) - 1.0) <= 0.5 * 0.69 * (double)head.margin(p);   // (log2)
  auto overflowed = [](uint32_t w) {
    return (w & 255u) == kAmbOver || (w >> 8 & 255u) == kAmbOver || (w >> 16 & 255u) == kAmbOver || w >> 24 == kAmbOver;
  };
  bool any = false, over = false;
#pragma unroll
  for (int j = 0; j < kTerms; ++j) {
    const int c = tid * kTerms + j;
    if (c < p.n_fine) {
      buf0[c] = residual(pa[j] * inv_zt, pb[j] * inv_zq);
      buf1[c] = ta[j] * inv_zt;
      if (!trusted) amb[j] = kAmbOver;
      s_amb[c] = amb[j];
      any = any || amb[j];
      over = over || overflowed(amb[j]);
    }
  }
  {
    const int flags = (__ballot(any) ? 1 : 0) | (__ballot(over) ? 2 : 0);
    if (lane == 0) s_flags[wave] = flags;
  }
  __syncthreads();
  const int flags = lane < kW ? s_flags[lane] : 0;
  if (__ballot(flags & 1)) {   // (uniform)
    // sixteen lanes per slice, the loads of its four lists in one round trip
    for (int c = tid / 16; c < p.n_fine; c += T / 16) {
      const uint32_t w = s_amb[c];
      if (w == 0 || overflowed(w)) continue;
      Doubt t[kLists][kAmb / 16];
#pragma unroll
      for (int k = 0; k < kLists; ++k)
#pragma unroll
        for (int i = 0; i < kAmb / 16; ++i) {
          t[k][i] = {0.0, 0.0};
          if (i * 16 + tid % 16 < (int)(w >> (8 * k) & 255u)) t[k][i] = doubt_list(p, nb, c, k)[i * 16 + tid % 16];
        }
      double add = 0.0;
#pragma unroll
      for (int k = 0; k < kLists; ++k)
#pragma unroll
        for (int i = 0; i < kAmb / 16; ++i) {
          add += fmax(residual(t[k][i].a * inv_zt, t[k][i].b * inv_zq), 0.0);
        }
      add = row_sum(add);
      if (tid % 16 == 0) buf0[c] += add;
    }
    __syncthreads();
    if (__ballot(flags & 2)) {   // lists that did not hold them: the whole slice again, by the workgroup
      for (int c = 0; c < p.n_fine; ++c) {
        if (!overflowed(s_amb[c])) continue;   // (uniform)
        double r[kOwn], pm[kOwn], sr = 0.0;
        eval(c, r, pm);
#pragma unroll
        for (int e = 0; e < kOwn; ++e) sr += r[e];
        sr = wave_sum(sr);
        if (lane == 0) s_sum[0][wave] = sr;
        __syncthreads();
        sr = sum_of_waves<kW>(s_sum[0]);
        if (tid == 0) buf0[c] = sr;
        __syncthreads();
      }
    }
  }
  // The slice in which the running sum first exceeds u times the total residual mass (the last slice with mass if rounding
  // hides the crossing), the lane of that slice whose tokens contain the crossing, the token.  Without mass (rounding only:
  // in the sums, or in the chosen slice's tokens) the draw is from p_n itself.
  for (int mode = 0; mode < 2; ++mode) {
    const double *buf = mode ? buf1 : buf0;
    double own[kTerms], sum = 0.0;
#pragma unroll
    for (int j = 0; j < kTerms; ++j) {
      const int c = tid * kTerms + j;
      own[j] = c < p.n_fine ? buf[c] : 0.0;
      sum += own[j];
    }
    Crossing<kW> slices;
    slices.find(sum, u, 0.0, false, 0.0, s_tot);
    if (!(slices.total > 0.0) && mode == 0) {   // (uniform)
      __syncthreads();
      continue;
    }
    if (tid == (slices.lane < 0 ? 0 : slices.lane)) {
      double acc = slices.excl, before = acc;
      int cs = tid * kTerms;
      bool found = false;
#pragma unroll
      for (int j = 0; j < kTerms; ++j) {
        if (!found && own[j] > 0.0) cs = tid * kTerms + j, before = acc, found = acc + own[j] > slices.thr;
        acc += own[j];
      }
      s_slice = cs;
      s_before = before;
    }
    __syncthreads();
    const int cs = s_slice;
    double mass[kOwn], mine = 0.0;
    {
      double r[kOwn], pm[kOwn];
      eval(cs, r, pm);
#pragma unroll
      for (int e = 0; e < kOwn; ++e) {
        mass[e] = mode ? pm[e] : r[e];
        mine += mass[e];
      }
    }
    Crossing<kW> lanes;
    lanes.find(mine, u, s_before, true, slices.total, s_tot);
    if (lanes.lane < 0) {   // (uniform)
      __syncthreads();
      continue;
    }
    if (tid == lanes.lane) {
      const int v0 = cs * kFine + tid * kOwn;
      double run = lanes.excl;
      int tok = -1, last = -1;
#pragma unroll
      for (int e = 0; e < kOwn; ++e) {
        run += mass[e];
        if (mass[e] > 0.0) {
          last = v0 + e;
          if (tok < 0 && run > lanes.thr) tok = v0 + e;
        }
      }
      p.next_token[nb] = tok >= 0 ? tok : last;
    }
    return;
  }
  if (tid == 0) p.next_token[nb] = 0;   // (a target row without a finite logit: any token, but an index all the same)
}

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// The part of the workspace that holds lists: 4 KiB per fine slice and branch.  top-p alone: the candidate segments, all
// of it, until the warp kernel has read them; then the lists of tokens in doubt (3 KiB per slice), their counts and the
// branches' heads.
inline size_t lists_bytes(int NB, int n_fine) { return align_up((size_t)NB * n_fine * kThreads * 2 * sizeof(double)); }
static_assert(kThreads / 64 * kAmb * sizeof(Doubt) + sizeof(uint32_t) + sizeof(BranchHead) <=
                  kThreads * 2 * sizeof(double),
              "a slice's share of the lists, its count and (one slice per branch) the branch's head");

template <bool BF16>
hipError_t launch_typed(const AcceptParams &p, hipStream_t stream) {
  const bool vec = ((size_t)p.V * (BF16 ? 2 : 4)) % 16 == 0;
  {
    ProfileScope scope(SLOT_ACCEPT_STATS, stream);
    const dim3 grid(p.n_chunks, p.draft ? p.NB * (2 * p.K + 1) : p.NB * (p.K + 1));
    if (vec)
      hipLaunchKernelGGL((accept_stats_kernel<BF16, true>), grid, dim3(kThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((accept_stats_kernel<BF16, false>), grid, dim3(kThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (p.warp_key) {
    ProfileScope scope(SLOT_ACCEPT_WARP, stream);
    if (p.top_p < 1.0f && !(p.top_k > 0 && p.top_k < p.V)) {   // top-p alone needs every target row's whole mass
      const dim3 grid(p.cand_groups, p.NB * (p.K + 1));
      if (BF16 && p.exp_tab)
        hipLaunchKernelGGL((accept_rowz_kernel<BF16, BF16>), grid, dim3(RowzShape<true>::kT), 0, stream, p);
      else
        hipLaunchKernelGGL((accept_rowz_kernel<BF16, false>), grid, dim3(kThreads), 0, stream, p);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(accept_warp_kernel<BF16>, dim3(p.NB * (p.K + 1)), dim3(kWarpThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  {
    ProfileScope scope(SLOT_ACCEPT_SAMPLE, stream);
    if (BF16 && p.exp_tab)
      hipLaunchKernelGGL((accept_sample_kernel<BF16, BF16>), dim3((p.n_fine + 1) / 2, p.NB), dim3(2 * kThreads), 0, stream, p);
    else
      hipLaunchKernelGGL((accept_sample_kernel<BF16, false>), dim3(p.n_fine, p.NB), dim3(kThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  {
    ProfileScope scope(SLOT_ACCEPT_PICK, stream);
    if (p.NB <= kPickMany || p.n_fine > 256)
      hipLaunchKernelGGL((accept_pick_kernel<BF16, 512, kMaxFine>), dim3(p.NB), dim3(512), 0, stream, p);
    else
      hipLaunchKernelGGL((accept_pick_kernel<BF16, 256, 256>), dim3(p.NB), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
}

}  // namespace

size_t accept_workspace_bytes(int NB, int K, int V, bool bf16, int *n_chunks_out, int *n_fine_out) {
  const int slice = bf16 ? StatsShape<true>::kSlice : StatsShape<false>::kSlice;
  const int n_chunks = (V + slice - 1) / slice;
  const int n_fine = (V + kFine - 1) / kFine;
  if (n_chunks_out) *n_chunks_out = n_chunks;
  if (n_fine_out) *n_fine_out = n_fine;
  size_t b = 0;
  b += align_up((size_t)NB * (2 * K + 1) * n_chunks * 2 * sizeof(float));  // stats
  b += align_up((size_t)NB * sizeof(int32_t));                             // n_acc
  b += align_up((size_t)NB * 2 * n_fine * sizeof(double));                 // zsum
  b += align_up((size_t)NB * 2 * n_fine * sizeof(double));                 // rsum
  b += lists_bytes(NB, n_fine);                                            // lists (tokens in doubt / candidates)
  b += align_up((size_t)NB * (K + 1) * sizeof(uint32_t));                  // warp_key
  b += align_up((size_t)NB * (K + 1) * sizeof(double));                    // warp_z
  b += align_up((size_t)NB * (K + 1) * n_fine * sizeof(double));           // warp_zs
  return b;
}

// Is a table worth its copy to every workgroup's LDS?  With top-p alone, whose rowz kernel takes all target rows, six slices to
// a workgroup: from 2048 slices in all on, rows of at least six (V = 152064, whole call, with and without: 600 slices 31.8 and
// 29.7 us, 1200 32.7 and 33.0, 2400 35.2 and 36.5, 9450 50.8 and 55.8; V = 12000: 2400 slices 38.1 and 41.3; V = 6000, half of
// every workgroup empty: 2400 56.5 and 53.2, 9600 141 and 135).  In calls just large enough to hold one it would also take a
// seventh of the candidates' space, and rows whose candidates do not fit take the long way (V = 65536, two branches, K 8, T 1.0,
// top_p 0.9: 128 against 32 us).  Otherwise the sample kernel alone, two slices to a workgroup: with draft rows from 1200 slices
// on, of long rows (V = 152064: 600 slices 19.2 and 18.6 us, 1200 22.6 and 23.0, 4800 43.3 and 44.9; V = 32000: 2400 31.7 and 31.3;
// V = 512, 4096 branches 89.4 and 75.6).  Without draft rows it is even at best.
static bool worth_a_table(const AcceptParams &p) {
  const size_t slices = (size_t)p.NB * p.n_fine;
  if (p.top_p < 1.0f && !(p.top_k > 0 && p.top_k < p.V)) return slices * (p.K + 1) >= 2048 && p.n_fine >= 6;
  return p.draft && slices >= 1200 && p.n_fine >= 32;
}

void accept_carve_workspace(AcceptParams &p, void *ws) {
  uint8_t *at = (uint8_t *)ws;
  p.stats = (float *)at;
  at += align_up((size_t)p.NB * (2 * p.K + 1) * p.n_chunks * 2 * sizeof(float));
  p.n_acc = (int32_t *)at;
  at += align_up((size_t)p.NB * sizeof(int32_t));
  p.zsum = (double *)at;
  at += align_up((size_t)p.NB * 2 * p.n_fine * sizeof(double));
  p.rsum = (double *)at;
  at += align_up((size_t)p.NB * 2 * p.n_fine * sizeof(double));
  {
    const size_t slices = (size_t)p.NB * p.n_fine;
    p.amb = at;
    p.heads = at + slices * (kThreads / 64) * kAmb * sizeof(Doubt);
    p.amb_n = (uint32_t *)(p.heads + (size_t)p.NB * sizeof(BranchHead));
    // the table ends the space, out of the way of both kinds of lists (64 slices leave 64 KiB behind the lists in doubt)
    const bool room = p.bf16 && slices >= 64 && p.inv_temp <= 1.0 / (double)kTabMinTemperature;
    const bool tab = room && (worth_a_table(p) || (selftest_force_table && selftest_force_table()));
    p.exp_tab = tab ? (double *)(at + lists_bytes(p.NB, p.n_fine) - kTab * sizeof(double)) : nullptr;
    // the candidate segments of a call with top-p alone share the space: rows equally, a row's by its slices; none if they are
    // too small (or one of a single slice could not hold its header)
    const size_t space = slices * kThreads * 2 * sizeof(double) - (tab ? kTab * sizeof(double) : 0);
    p.cand = at;
    p.cand_row = (int)((space / ((size_t)p.NB * (p.K + 1))) & ~(size_t)15);
    const int groups = p.cand_groups = (p.n_fine + rowz_group(p) - 1) / rowz_group(p);
    p.cand_seg = groups > 1 ? (int)((int64_t)p.cand_row * rowz_group(p) / p.n_fine) & ~15 : p.cand_row;
    const int last = p.cand_row - (groups - 1) * p.cand_seg, lds = p.bf16 ? kCandLds<true> : kCandLds<false>;
    auto keys = [&](int bytes) {
      const int fit = (bytes - (int)sizeof(CandHeader)) / (p.bf16 ? 2 : 4);
      return fit < lds ? fit : lds;
    };
    p.cand_cap = keys(p.cand_seg), p.cand_cap_last = keys(last);
    if (p.cand_row / p.n_fine < 16 || p.cand_seg < 64) p.cand_row = 0;
  }
  at += lists_bytes(p.NB, p.n_fine);
  const bool warp = (p.top_k > 0 && p.top_k < p.V) || p.top_p < 1.0f;
  p.warp_key = warp ? (uint32_t *)at : nullptr;
  at += align_up((size_t)p.NB * (p.K + 1) * sizeof(uint32_t));
  p.warp_z = warp ? (double *)at : nullptr;
  at += align_up((size_t)p.NB * (p.K + 1) * sizeof(double));
  p.warp_zs = warp ? (double *)at : nullptr;
}

namespace {
__global__ __launch_bounds__(kThreads) void exp64_probe_kernel(const double *y, double *out, size_t n) {
  const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < n) out[i] = exp64(y[i]);
}
}  // namespace

hipError_t launch_exp64_probe(const double *y, double *out, size_t n, hipStream_t stream) {
  hipLaunchKernelGGL(exp64_probe_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, stream, y, out,
                     n);
  return hipGetLastError();
}

int accept_row_candidates(const AcceptParams &p) {
  return p.cand_row ? (p.cand_groups - 1) * p.cand_cap + p.cand_cap_last : 0;
}

hipError_t launch_accept(const AcceptParams &p, hipStream_t stream) {
  return p.bf16 ? launch_typed<true>(p, stream) : launch_typed<false>(p, stream);
}

}  // namespace la
