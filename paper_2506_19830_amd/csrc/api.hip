// Host side of libla_verify: argument validation, launch planning, the extern "C" entry points
// declared in la_verify.h and the optional per-kernel event timing.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include "la_internal.hpp"
#include <cstdio>

namespace la {
namespace {

// Compute units of the current device, asked once (256 on MI355X, also the fallback when no device answers, e.g. a
// workspace query on a machine without a GPU).
int num_cus() {
  static std::once_flag once;
  static int cus = 256;
  std::call_once(once, [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      cus = n;
  });
  return cus;
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

enum AttnPath { PATH_NONE = 0, PATH_F32, PATH_MFMA };

// Kernel shapes of the MFMA path, numbered as la_attn_desc.kernel_shape - 1 numbers them: the row-tile shapes of
// attn_mfma_kernel first, then the streaming shapes of attn_stream_kernel.
struct ShapeInfo {
  bool stream;
  bool fp8;        // streaming shapes: storage type of cache and branch K/V the shape is built for
  int local;       // index inside its kernel's own shape table
  int tile_m;      // query rows per workgroup
  int per_cu;      // workgroups that share a CU
  int step_keys;   // keys a workgroup advances per pipeline step
  double t_step;   // microseconds per step of one workgroup with the CU shared by per_cu (fitted)
  double t_step_shared;  // the same when several row tiles stream the same keys (streaming shapes: arithmetic-bound
                         // steps; with one row tile a step is bound by its share of the HBM stream)
  double t_fixed;  // microseconds of start-up and write-out per workgroup (fitted)
};
int num_shapes() { return attn_mfma_num_shapes() + attn_stream_num_shapes(); }
ShapeInfo shape_info(int shape) {
  ShapeInfo s{};
  if (shape < attn_mfma_num_shapes()) {
    s.stream = false, s.local = shape;
    s.tile_m = attn_mfma_tile_m(shape), s.per_cu = attn_mfma_wgs_per_cu(shape), s.step_keys = 64;
    s.t_step = s.t_step_shared = s.per_cu > 1 ? 2.25 : 1.87;
    s.t_fixed = s.per_cu > 1 ? 8.0 : 9.0;
  } else {
    s.stream = true, s.local = shape - attn_mfma_num_shapes();
    s.tile_m = attn_stream_tile_m(s.local), s.per_cu = 1;
    s.step_keys = attn_stream_step_keys(s.local);
    // every wavefront reduces one 64-key tile for its 32 rows per step, whatever the shape: the time of a step is
    // the time of two such units on one SIMD
    s.fp8 = attn_stream_shape_is_fp8(s.local);
    if (s.fp8) {
      s.t_step = s.tile_m == 64 ? 3.1 : s.tile_m == 128 ? 2.3 : 3.0;
      s.t_step_shared = s.tile_m == 64 ? 2.15 : s.tile_m == 128 ? 2.05 : 2.2;
    } else {
      // (1.8: fitted to a tile with branches; the present one is 4 to 5 % faster)
      s.t_step = s.t_step_shared = s.tile_m == 256 ? 1.8 : 2.45;
    }
    // (the 256-row bf16 shape: eight row blocks' Q into registers and a branch-private tile per wavefront at the end)
    s.t_fixed = (!s.fp8 && s.tile_m == 256) ? 12.0 : 5.0;
  }
  return s;
}

struct AttnPlan {
  AttnPath path;
  bool kv_fp8, br_fp8;
  int shape, tile_m, n_row_tiles, chunk_len, last_short, s_max, total_units;
  // (general path: shape = row blocks of 16 per workgroup, 0 = a wavefront per row; the workspace is optional there)
  size_t part_o_bytes, part_ml_bytes;
};

la_status validate_desc(const la_attn_desc *d) {
  if (!d) return LA_ERR_INVALID_ARG;
  if (d->num_requests < 1 || d->num_q_heads < 1 || d->num_kv_heads < 1 || d->head_dim < 1 || d->gamma < 1 ||
      d->branch_len < 1)
    return LA_ERR_INVALID_ARG;
  if (d->num_q_heads % d->num_kv_heads) return LA_ERR_INVALID_ARG;
  if (d->block_size < 16 || (d->block_size & (d->block_size - 1))) return LA_ERR_INVALID_ARG;  // power of two
  if (d->max_blocks_per_request < 0) return LA_ERR_INVALID_ARG;
  if (!(d->softmax_scale > 0.f) || !isfinite(d->softmax_scale)) return LA_ERR_INVALID_ARG;
  if (d->kv_split_tokens < 0 || d->kv_split_tokens % 64) return LA_ERR_INVALID_ARG;
  if (d->kernel_shape < 0 || d->kernel_shape > num_shapes()) return LA_ERR_INVALID_ARG;
  const int32_t dts[4] = {d->q_dtype, d->kv_dtype, d->branch_kv_dtype, d->out_dtype};
  for (int i = 0; i < 4; ++i)
    if (dts[i] < LA_F32 || dts[i] > LA_FP8_E4M3) return LA_ERR_INVALID_ARG;
  // rows and prefix tokens are indexed with 32-bit integers on the device
  const int64_t n_rows = (int64_t)d->gamma * d->branch_len * d->num_q_heads;
  if (n_rows * d->num_requests > (int64_t)1 << 30) return LA_ERR_UNSUPPORTED;
  if ((int64_t)d->max_blocks_per_request * d->block_size > (int64_t)1 << 30) return LA_ERR_UNSUPPORTED;
  return LA_OK;
}

// Partial slots, workspace sizes and the number of (request, chunk) units, once chunk_len is chosen.
void size_partials(const la_attn_desc *d, const int32_t *prefix_lens_host, AttnPlan *plan) {
  const size_t n_rows = (size_t)d->gamma * d->branch_len * d->num_q_heads;
  int s_max = 1, total = 0;
  for (int b = 0; b < d->num_requests; ++b) {
    const int nc = attn_num_chunks(prefix_lens_host[b], plan->chunk_len);
    s_max = nc > s_max ? nc : s_max;
    total += nc;
  }
  plan->s_max = s_max;
  plan->total_units = total;
  plan->part_o_bytes = align_up((size_t)d->num_requests * s_max * n_rows * d->head_dim * sizeof(float));
  plan->part_ml_bytes = align_up((size_t)d->num_requests * s_max * n_rows * 2 * sizeof(float));
}

constexpr int kWholePrefix = 1 << 30;   // chunk length of an unsplit plan (no prefix is longer)

// The general path: one workgroup per (row block, kv head) and request, and, for bf16 / fp8 storage, chunks of the
// prefix where that leaves the chip idle.  fp32 calls have no workspace (their sizes are small, and the query says so).
void make_general_plan(const la_attn_desc *d, const int32_t *prefix_lens_host, int64_t max_p, bool f32, AttnPlan *plan) {
  const int R = d->gamma * d->branch_len * (d->num_q_heads / d->num_kv_heads);
  plan->path = PATH_F32;
  // two row blocks share every operand of a key where the registers allow it (measured figures: attn_f32.hip)
  plan->shape = !f32 && d->head_dim == 64 && R > 16 ? 2 : 1;
  plan->tile_m = 16 * plan->shape;
  plan->n_row_tiles = (R + plan->tile_m - 1) / plan->tile_m;
  plan->chunk_len = kWholePrefix;
  const int priv = plan->tile_m + d->branch_len < d->gamma * d->branch_len ? plan->tile_m + d->branch_len : d->gamma * d->branch_len;
  plan->last_short = (priv + 63) / 64;
  if (!f32 && d->kv_split_tokens) {
    plan->chunk_len = d->kv_split_tokens;
  } else if (!f32) {
    // microseconds: rounds of workgroups over the slots x (blocks a wavefront walks + start and fold) + the merge; block
    // times fitted to the figures in attn_f32.hip (head dimension 64, two row blocks: 41 us for 32 blocks)
    const double t_block = d->head_dim == 64 ? (plan->shape == 2 ? 1.3 : 0.9) : 3.0, t_fixed = 5.0;
    const int64_t base = (int64_t)d->num_kv_heads * plan->n_row_tiles, slots = (int64_t)num_cus() * (d->head_dim == 64 && plan->shape == 1 ? 2 : 1);
    const size_t n_rows = (size_t)d->gamma * d->branch_len * d->num_q_heads;
    double best = 0.0;
    for (int n = 1; n <= 64; ++n) {
      const int64_t len = ((max_p + n - 1) / n + 63) / 64 * 64;
      if (n > 1 && len < 256) break;   // less than a block per wavefront
      int64_t units = 0;
      for (int b = 0; b < d->num_requests; ++b) units += n == 1 ? 1 : attn_num_chunks(prefix_lens_host[b], (int)len);
      const int64_t rounds = (base * units + slots - 1) / slots;
      const int64_t steps = ((n == 1 ? max_p : len) + 64 * plan->last_short / n + 255) / 256;
      const double cost = (double)rounds * ((double)steps * t_block + t_fixed) +
                          (n == 1 ? 0.0 : 4.0 + (double)units * n_rows * (d->head_dim + 2) * 4.0 / 3.0e6);
      if (n == 1 || cost < best) best = cost, plan->chunk_len = n == 1 ? kWholePrefix : (int)len;
      if (n > 1 && base * units > 2 * slots) break;
    }
  }
  size_partials(d, prefix_lens_host, plan);
  if (plan->s_max == 1) plan->part_o_bytes = plan->part_ml_bytes = 0;   // the kernel writes the output itself
}

// Does a general-path call run one wavefront per query row (attn_rows.hip) instead of matrix tiles?  Both times are
// estimated in microseconds for `units` (request, KV head) pairs of R rows that see at most `keys` keys: the matrix kernel
// takes a time per unit whatever it holds, the other one per key and row, and at least the latency of its walk.
// (Fitted to 512 to 16384 units of 1 to 8 rows and 1 to 63 keys; with 8 rows and one key, 4096 units take 23 against 63 us
// at head dimension 64, fp32; with 16 rows the matrix kernel is the faster one at any length: 88 against 74 us.  What the
// fit gets wrong, over 252 such points, is 13 us at most and more than 6 us at five of them.)
// chain_len: tokens of the drafted chain or pool.
bool general_by_rows(const la_attn_desc *d, const int32_t *prefix_lens_host, int chain_len) {
  const int R = d->gamma * d->branch_len * (d->num_q_heads / d->num_kv_heads);
  if (R > 8 || (int64_t)d->num_requests * d->num_kv_heads * R > attn_rows_max()) return false;
  int64_t longest = 0;
  for (int b = 0; b < d->num_requests; ++b) longest = prefix_lens_host[b] > longest ? prefix_lens_host[b] : longest;
  const int64_t keys = longest + chain_len + d->branch_len;
  if (keys > (d->head_dim == 64 ? 48 : 64)) return false;   // (64: one round of the walk)
  const bool f32 = d->kv_dtype == LA_F32, fp8 = d->kv_dtype == LA_FP8_E4M3;
  // per_unit: matrix kernel; even: the keys of one row at which many units take the same time either way
  const double per_unit = d->head_dim == 64 ? (f32 ? 0.015 : 0.0085) : d->head_dim == 128 ? 0.016 : fp8 ? 0.024 : 0.028;
  const double even = d->head_dim == 64 ? (f32 ? 77.0 : fp8 ? 52.0 : 48.0) : d->head_dim == 128 || fp8 ? 77.0 : 100.0;
  // rows of a unit share their keys through the caches; a workgroup's four rows fall into one unit only if R divides
  const double shared = (0.55 + 0.45 * R) * ((R & (R - 1)) ? 1.25 : 1.0);
  const double matrix_us = 3.0 + per_unit * (double)d->num_requests * d->num_kv_heads;
  const double walk_us = 4.0 + (double)keys * (0.2 + d->head_dim / 400.0), launch_us = 10.0;
  return (double)keys * shared < even && walk_us < matrix_us && launch_us < matrix_us;
}

// The same plan serves the flat, nested and tree forms of a call (count_extra_tiles shifts its chunk ranges for a chain).
la_status make_plan(const la_attn_desc *d, const int32_t *prefix_lens_host, AttnPlan *plan) {
  la_status st = validate_desc(d);
  if (st != LA_OK) return st;
  if (!prefix_lens_host) return LA_ERR_INVALID_ARG;
  int64_t max_p = 0;
  for (int b = 0; b < d->num_requests; ++b) {
    const int64_t P = prefix_lens_host[b];
    if (P < 0 || P > (int64_t)d->max_blocks_per_request * d->block_size) return LA_ERR_INVALID_ARG;
    max_p = P > max_p ? P : max_p;
  }
  memset(plan, 0, sizeof *plan);
  const bool all_f32 =
      d->q_dtype == LA_F32 && d->kv_dtype == LA_F32 && d->branch_kv_dtype == LA_F32 && d->out_dtype == LA_F32;
  if (all_f32) {
    if (d->head_dim != 64 && d->head_dim != 128 && d->head_dim != 256) return LA_ERR_UNSUPPORTED;
    make_general_plan(d, prefix_lens_host, max_p, true, plan);
    return LA_OK;
  }
  const bool out_ok = d->out_dtype == LA_BF16 || d->out_dtype == LA_F32;
  const bool bf16_all = d->q_dtype == LA_BF16 && d->kv_dtype == LA_BF16 && d->branch_kv_dtype == LA_BF16;
  const bool fp8_kv = d->q_dtype == LA_BF16 && d->kv_dtype == LA_FP8_E4M3 &&
                      (d->branch_kv_dtype == LA_FP8_E4M3 || d->branch_kv_dtype == LA_BF16);
  if (!out_ok || !(bf16_all || fp8_kv)) return LA_ERR_UNSUPPORTED;
  if (d->head_dim != 128) {
    // the MFMA and streaming kernels are written for head dimension 128; 64 and 256 run on the general kernel
    // (exactly widened inputs, fp32-accurate)
    if (d->head_dim != 64 && d->head_dim != 256) return LA_ERR_UNSUPPORTED;
    if (d->kernel_shape > 0) return LA_ERR_UNSUPPORTED;
    make_general_plan(d, prefix_lens_host, max_p, false, plan);
    return LA_OK;
  }
  plan->path = PATH_MFMA;
  plan->kv_fp8 = d->kv_dtype == LA_FP8_E4M3;
  plan->br_fp8 = d->branch_kv_dtype == LA_FP8_E4M3;

  const int G = d->num_q_heads / d->num_kv_heads;
  const int R = d->gamma * d->branch_len * G;
  const size_t n_rows = (size_t)d->gamma * d->branch_len * d->num_q_heads;
  // the streaming shapes exist for cache and branch K/V of one storage type
  auto stream_ok = [&](const ShapeInfo &si) {
    return plan->kv_fp8 == si.fp8 && plan->br_fp8 == si.fp8 &&
           (int64_t)d->num_kv_heads * d->block_size * d->head_dim * (si.fp8 ? 1 : 2) < ((int64_t)1 << 32);
  };
  // Tiles of other work that the last chunk's workgroup carries.  (A streaming shape advances whole steps: the private
  // tiles are steps of their own, so the last chunk gets as many prefix steps fewer, or its workgroup would finish a step
  // after all the others.)
  auto last_short_tiles = [&](const ShapeInfo &si) -> int {
    const int priv_tokens = si.tile_m / G + d->branch_len < d->gamma * d->branch_len ? si.tile_m / G + d->branch_len
                                                                                     : d->gamma * d->branch_len;
    const int priv_tiles = (priv_tokens + 63) / 64, step_tiles = si.step_keys / 64;
    return si.stream ? step_tiles * ((priv_tiles + step_tiles - 1) / step_tiles) : 3 * priv_tiles;
  };
  // The longest chunk a shape can take: its block ids live in LDS (-2: a chunk need not start on a block boundary).
  auto max_chunk = [&](const ShapeInfo &si, int last_short) -> int64_t {
    const int blk_cap = si.stream ? attn_stream_max_chunk_blocks() : attn_mfma_max_chunk_blocks();
    return ((int64_t)(blk_cap - 2) * d->block_size - 64 * (last_short + 2)) / 64 * 64;
  };
  auto chunk_fits = [&](int64_t longest) { return longest >= 64 && d->kv_split_tokens <= longest; };
  if (d->kernel_shape > 0) {
    const ShapeInfo forced = shape_info(d->kernel_shape - 1);
    if (forced.stream && !stream_ok(forced)) return LA_ERR_UNSUPPORTED;
  }

  // Choose the kernel shape and the number of chunks that minimise a simple cost model (microseconds, constants
  // fitted to measurements on MI355X):
  //   rounds of workgroups over the CU slots  x  (steps per chunk x time per step + fixed start-up)
  //   + the merge of the partials (rows x (D+2) floats per chunk, written once and read once).
  // Few long chunks keep the partial traffic small, many short ones fill the chip when there are few rows.
  // A request's key tiles are dealt out evenly over its chunks (attn_chunk_range); the workgroup of the last chunk
  // also runs the branch-private tiles (masked, general form: about three prefix tiles each in the row-tile
  // shapes, whole pipeline steps in the streaming shapes), which count as `last_short` tiles of its share.
  // With a bf16 cache the row-tile shapes are left to calls that force them (and to block strides the streaming shapes
  // cannot address): over 48 calls of all forms, 15 to 3248 rows and 295 to 32450 keys, the better of the two bf16
  // streaming shapes took 0.7 to 1.0 of the better row-tile shape's time, 0.85 in the mean (29697 + 21770 + 18197 keys,
  // 112 rows: 65 against 95 us; 25402 keys, 3248 rows: 180 against 200 us).  A chunk length asked for (kv_split_tokens)
  // that only the row tiles can hold, with twice the streaming shapes' table of block ids, leaves the call to them as
  // well.
  bool skip_row_tiles = false;
  if (d->kernel_shape == 0 && !plan->kv_fp8)
    for (int shape = attn_mfma_num_shapes(); shape < num_shapes(); ++shape) {
      const ShapeInfo si = shape_info(shape);
      skip_row_tiles |= stream_ok(si) && chunk_fits(max_chunk(si, last_short_tiles(si)));
    }
  // fp8, at most 64 rows per KV head: of the streaming shapes only the one of 64 rows.  The others have wavefronts whose
  // rows do not exist, and fewer key slices.  Their shorter step tempts the model to chunks of one tile, but over 40 flat
  // calls of 8 to 64 rows and 305 to 29507 keys the 128-row shape took 1.0 to 1.38 of the time, 1.15 in the mean (28431 +
  // 307 keys, 64 rows, two heads: 23.3 against 19.0 us), and no less at any chunk length asked for.  bf16 has no such line:
  // there each of its two shapes is ahead in part of the range.
  bool narrow = false;
  if (d->kernel_shape == 0 && R <= 64)
    for (int shape = attn_mfma_num_shapes(); shape < num_shapes(); ++shape) {
      const ShapeInfo si = shape_info(shape);
      narrow |= si.fp8 && si.tile_m == 64 && stream_ok(si) && chunk_fits(max_chunk(si, last_short_tiles(si)));
    }
  double best_cost = 0.0;
  int best_len = 0, best_shape = -1, best_short = 0;
  const int64_t T = (max_p + 63) / 64;
  const bool exhaustive = selftest_exhaustive_plans && selftest_exhaustive_plans();   // (a test's search without shortcuts)
  for (int shape = 0; shape < num_shapes(); ++shape) {
    if (d->kernel_shape > 0 && shape != d->kernel_shape - 1) continue;
    const ShapeInfo si = shape_info(shape);
    if (si.stream ? !stream_ok(si) || (narrow && si.tile_m > 64) : skip_row_tiles) continue;
    const int64_t base_wgs = (int64_t)d->num_kv_heads * ((R + si.tile_m - 1) / si.tile_m);
    const int last_short = last_short_tiles(si);
    const int64_t slots = (int64_t)num_cus() * si.per_cu;
    const int64_t longest = max_chunk(si, last_short);
    if (!chunk_fits(longest)) continue;
    const double t_step = R > si.tile_m ? si.t_step_shared : si.t_step;
    const double shared_us = (double)base_wgs * (double)(T + last_short) * 64.0 / si.step_keys / (double)slots * t_step;
    double prev_cost = 0.0;
    // Many numbers of chunks round to the same chunk length, ceil(T / n) tiles: only the first of them is looked at (and
    // n = 9, from where several requests are no longer dealt out).  Every call plans, and a call of few keys is no longer than
    // a plan was: three requests of 3553, 1018 and 7148 keys, 25 rows, 14 -> 2 us; one of 5120, 16 rows, 7 -> 1 us.
    for (int n = 1, n_next; n <= 512; n = n_next) {
      const int64_t tiles = T > 0 ? (T + n - 1) / n : 1;
      n_next = tiles > 1 ? (int)((T + tiles - 2) / (tiles - 1)) : n + 1;
      if (d->num_requests > 1 && n < 9 && n_next > 9) n_next = 9;
      if (exhaustive) n_next = n + 1;
      int64_t len = 64 * tiles;
      if (len > longest) len = longest;
      if (d->kv_split_tokens) len = d->kv_split_tokens;
      int64_t units = 0;
      for (int b = 0; b < d->num_requests; ++b) units += attn_num_chunks(prefix_lens_host[b], (int)len);
      const int64_t rounds = (base_wgs * units + slots - 1) / slots;
      const double merge_us = 3.0 + (double)units * n_rows * (d->head_dim + 2) * 4.0 / 3.0e6;  // read at ~3 TB/s
      const double margin = si.stream && si.fp8 && rounds > 1 ? 1.06 : 1.0;
      // Whatever the chunks, the slots share all steps of the longest request (and of the others), every round (of several
      // requests, dealt out: every workgroup) starts workgroups and the merge reads more partials the more chunks there
      // are.  Once that alone costs the best plan so far, no later count can win.
      const double starts = d->num_requests == 1 ? (double)rounds : (double)(base_wgs * units) / (double)slots;
      if (!exhaustive && best_shape >= 0 &&
          (merge_us + margin * (starts * si.t_fixed + shared_us)) * (1.0 - 1e-9) >= best_cost)
        break;
      const int64_t n_max = attn_num_chunks((int)max_p, (int)len);
      const int64_t wg_tiles = (T + last_short + n_max - 1) / n_max;  // of the longest request
      const int64_t wg_steps = (wg_tiles * 64 + si.step_keys - 1) / si.step_keys;
      double busy_us = (double)rounds * ((double)wg_steps * t_step + si.t_fixed);
      bool model = d->num_requests > 1 && rounds > 1 && n <= 8 && units <= 64;
      if (!exhaustive && model && best_shape >= 0 && base_wgs * units <= 2 * slots) {
        // Dealing the workgroups out costs microseconds of host time per candidate, and every call plans: not where even
        // a bound of the result from below (the mean over the slots; `rounds` of the shortest workgroups on one slot; the
        // longest one) leaves the best plan so far in place.  (Below twice the slots, where neither this candidate's cost
        // nor the next one's ends the search.  Eight requests of 1500 keys, one row per KV head: 50 -> 15 us per plan.)
        double total = 0.0, shortest = 0.0, longest_wg = 0.0;
        for (int b = 0; b < d->num_requests; ++b) {
          const int64_t nc = attn_num_chunks(prefix_lens_host[b], (int)len);
          const int64_t tiles_b = (prefix_lens_host[b] + 63) / 64 + last_short;
          const int64_t lo_tiles = tiles_b / nc, n_hi = tiles_b % nc;
          const double lo = (double)((lo_tiles * 64 + si.step_keys - 1) / si.step_keys) * t_step + si.t_fixed;
          const double hi = (double)(((lo_tiles + 1) * 64 + si.step_keys - 1) / si.step_keys) * t_step + si.t_fixed;
          total += (double)base_wgs * (lo * (double)(nc - n_hi) + hi * (double)n_hi);
          shortest = b == 0 || lo < shortest ? lo : shortest;
          longest_wg = (n_hi ? hi : lo) > longest_wg ? (n_hi ? hi : lo) : longest_wg;
        }
        double bound = total / (double)slots;
        bound = bound > (double)rounds * shortest ? bound : (double)rounds * shortest;
        bound = bound > longest_wg ? bound : longest_wg;
        if (bound * margin * (1.0 - 1e-9) + merge_us >= best_cost) {
          busy_us = bound;
          model = false;
        }
      }
      if (model) {
        // Several requests of different lengths in several rounds, few chunks each: rounds x the longest chunk is
        // what the dispatch of equal workgroups gives; with unequal ones the workgroups are dealt out here as the
        // hardware deals them, in launch order (all workgroups of a chunk, chunk after chunk, request after request),
        // each to the slot that is free first.  (Measured at configuration 4's ragged batch: one chunk per request,
        // 1.17 ms; chunks of 8192 keys, 1.04 ms, where rounds x longest saw the two as equal.)  With many chunks per
        // request they are nearly equal and the simple form holds; every call plans, so this stays small (fixed
        // arrays, at most 64 chunks).
        constexpr int kCap = 256;
        struct Free { double t; int64_t n; };
        Free cur[kCap], nxt[kCap], mrg[kCap];
        int n_cur = 1;
        cur[0] = {0.0, slots};
        bool fits = true;
        for (int b = 0; b < d->num_requests && fits; ++b) {
          const int64_t nc = attn_num_chunks(prefix_lens_host[b], (int)len);
          const int64_t tiles_b = (prefix_lens_host[b] + 63) / 64 + last_short;
          for (int64_t c = 0; c < nc && fits; ++c) {
            const int64_t tiles = tiles_b / nc + (c < tiles_b % nc ? 1 : 0);
            const double dur = (double)((tiles * 64 + si.step_keys - 1) / si.step_keys) * t_step + si.t_fixed;
            for (int64_t left = base_wgs; left > 0 && fits;) {
              int64_t need = left < slots ? left : slots;  // (the entries always add up to `slots`)
              left -= need;
              int i = 0, n_nxt = 0;
              for (; need > 0 && i < n_cur; ++i) {
                const int64_t k = need < cur[i].n ? need : cur[i].n;
                nxt[n_nxt++] = {cur[i].t + dur, k};
                cur[i].n -= k, need -= k;
                if (cur[i].n > 0) break;
              }
              // what was not taken keeps its place; the slots just filled come free later, in the order taken
              int a2 = i, b2 = 0, n_mrg = 0;
              while (a2 < n_cur || b2 < n_nxt) {
                if (n_mrg >= kCap) {
                  fits = false;
                  break;
                }
                if (b2 >= n_nxt || (a2 < n_cur && cur[a2].t <= nxt[b2].t)) {
                  if (cur[a2].n > 0) mrg[n_mrg++] = cur[a2];
                  ++a2;
                } else {
                  mrg[n_mrg++] = nxt[b2++];
                }
              }
              if (n_mrg + 2 >= kCap) fits = false;
              for (int j = 0; j < n_mrg; ++j) cur[j] = mrg[j];
              n_cur = n_mrg;
            }
          }
        }
        if (fits && n_cur > 0) busy_us = cur[n_cur - 1].t;
      }
      // (an fp8 streaming plan of several rounds has measured at its model cost, the row-tile shapes it competes with there
      // -- partly filled row tiles of 256 rows -- below theirs: the margin keeps those cases with the row tiles)
      const double cost = busy_us * margin + merge_us;
      if (best_shape < 0 || cost < best_cost)
        best_cost = cost, best_len = (int)len, best_shape = shape, best_short = last_short;
      if (len <= 64 || d->kv_split_tokens) break;
      // once every slot is used and the cost has started to rise, more chunks only add partials
      if (n > 1 && rounds > 1 && cost > prev_cost && base_wgs * units > 4 * slots) break;
      prev_cost = cost;
    }
  }
  if (best_shape < 0) return LA_ERR_UNSUPPORTED;
  const ShapeInfo si = shape_info(best_shape);
  plan->shape = best_shape;
  plan->tile_m = si.tile_m;
  plan->n_row_tiles = (R + plan->tile_m - 1) / plan->tile_m;
  plan->chunk_len = best_len;
  plan->last_short = best_short;
  size_partials(d, prefix_lens_host, plan);
  return LA_OK;
}

// A chain or pool of drafted tokens is reduced by the last chunk's workgroups too: deal them that many tiles less of
// the prefix.  The number of chunks, and with it the workspace, does not depend on this (the workspace query does not
// know the chain's length).  tokens: the longest part any branch sees.  A forced shape keeps the flat call's chunk
// ranges, so that forms compared under it sum in the same order.
void count_extra_tiles(const la_attn_desc *d, int64_t tokens, AttnPlan *plan) {
  if (plan->path != PATH_MFMA || tokens <= 0 || d->kernel_shape > 0) return;
  const ShapeInfo si = shape_info(plan->shape);
  const int64_t tiles = (tokens + 63) / 64, step_tiles = si.step_keys / 64;
  // the block ids of the longest chunk have to fit the kernel's table (make_plan's bound, with the tiles added here)
  const int64_t cap = si.stream ? attn_stream_max_chunk_blocks() : attn_mfma_max_chunk_blocks();
  const int64_t most = ((cap - 2) * d->block_size - plan->chunk_len) / 64 - 2;
  int64_t ls = plan->last_short + (si.stream ? step_tiles * ((tiles + step_tiles - 1) / step_tiles) : 3 * tiles);
  ls = ls < most ? ls : most;
  if (ls > plan->last_short) plan->last_short = (int)ls;
}

}  // namespace

}  // namespace la

using namespace la;

extern "C" {

const char *la_status_string(int32_t status) {
  switch (status) {
    case LA_OK: return "ok";
    case LA_ERR_INVALID_ARG: return "invalid argument";
    case LA_ERR_UNSUPPORTED: return "unsupported shape or dtype combination";
    case LA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case LA_ERR_LAUNCH: return "kernel launch failed";
  }
  return "unknown status";
}

la_status la_verify_attention_workspace(const la_attn_desc *desc, const int32_t *prefix_lens_host,
                                        size_t *bytes_out) {
  if (!bytes_out) return LA_ERR_INVALID_ARG;
  AttnPlan plan;
  la_status st = make_plan(desc, prefix_lens_host, &plan);
  if (st != LA_OK) return st;
  *bytes_out = plan.part_o_bytes + plan.part_ml_bytes;
  return LA_OK;
}

la_status la_verify_attention_plan(const la_attn_desc *desc, const int32_t *prefix_lens_host, int32_t chain_len,
                                   la_attn_plan *out) {
  if (!out || chain_len < 0) return LA_ERR_INVALID_ARG;
  AttnPlan plan;
  la_status st = make_plan(desc, prefix_lens_host, &plan);
  if (st != LA_OK) return st;
  memset(out, 0, sizeof *out);
  out->path = (int32_t)plan.path;
  if (plan.path == PATH_F32 && general_by_rows(desc, prefix_lens_host, chain_len)) {
    out->rows_per_workgroup = 4;
    out->chunks_total = desc->num_requests;
    out->workgroups = (int32_t)(((int64_t)desc->num_requests * desc->gamma * desc->branch_len * desc->num_q_heads + 3) / 4);
    return LA_OK;
  }
  if (plan.path == PATH_MFMA) out->kernel_shape = plan.shape + 1;
  out->rows_per_workgroup = plan.tile_m;
  out->row_tiles = plan.n_row_tiles;
  out->chunk_tokens = plan.s_max > 1 || plan.path == PATH_MFMA ? plan.chunk_len : 0;
  out->chunks_total = plan.total_units;
  const int64_t workgroups = (int64_t)desc->num_kv_heads * plan.n_row_tiles * plan.total_units;
  out->workgroups = workgroups < INT32_MAX ? (int32_t)workgroups : INT32_MAX;
  return LA_OK;
}

// Shared by the three attention entry points.  chain_len tokens of extra K/V per request: a chain with a visible
// leading part per branch (chain_vis), or a pool with segment labels and a segment mask per branch (pool_seg).
static la_status verify_attention(const la_attn_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                                  const int32_t *block_tables, const int32_t *prefix_lens,
                                  const int32_t *prefix_lens_host, const void *k_branch, const void *v_branch,
                                  const void *k_chain, const void *v_chain, int32_t chain_len,
                                  const int32_t *chain_vis, const int32_t *chain_vis_host, const int32_t *pool_seg,
                                  const int32_t *pool_seg_host, const uint64_t *seg_mask, const float *k_scale,
                                  const float *v_scale, void *out, float *lse, void *workspace,
                                  size_t workspace_bytes, void *hip_stream) {
  AttnPlan plan;
  la_status st = make_plan(desc, prefix_lens_host, &plan);
  if (st != LA_OK) return st;
  if (!q || !prefix_lens || !k_branch || !v_branch || !out) return LA_ERR_INVALID_ARG;
  bool any_prefix = false;
  for (int b = 0; b < desc->num_requests; ++b) any_prefix |= prefix_lens_host[b] > 0;
  if (any_prefix && (!k_cache || !v_cache)) return LA_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(k_branch) || !aligned16(v_branch) ||
      !aligned16(out) || !aligned16(workspace))
    return LA_ERR_INVALID_ARG;
  if (chain_len < 0) return LA_ERR_INVALID_ARG;
  const bool tree = pool_seg != nullptr || pool_seg_host != nullptr || seg_mask != nullptr;
  if (chain_len > 0) {
    if (!k_chain || !v_chain || !aligned16(k_chain) || !aligned16(v_chain)) return LA_ERR_INVALID_ARG;
    if (tree) {
      if (!pool_seg || !pool_seg_host || !seg_mask || ((uintptr_t)seg_mask & 7)) return LA_ERR_INVALID_ARG;
      for (int64_t t = 0; t < (int64_t)desc->num_requests * chain_len; ++t)
        if (pool_seg_host[t] < 0 || pool_seg_host[t] > 63) return LA_ERR_INVALID_ARG;
    } else {
      if (!chain_vis || !chain_vis_host) return LA_ERR_INVALID_ARG;
      for (int64_t t = 0; t < (int64_t)desc->num_requests * desc->gamma; ++t)
        if (chain_vis_host[t] < 0 || chain_vis_host[t] > chain_len) return LA_ERR_INVALID_ARG;
    }
  }
  int64_t seen = tree ? chain_len : 0;
  if (chain_len > 0 && !tree)
    for (int64_t t = 0; t < (int64_t)desc->num_requests * desc->gamma; ++t)
      seen = chain_vis_host[t] > seen ? chain_vis_host[t] : seen;
  if (plan.path == PATH_F32 && general_by_rows(desc, prefix_lens_host, chain_len)) plan.shape = 0;
  count_extra_tiles(desc, seen, &plan);
  const size_t need = plan.part_o_bytes + plan.part_ml_bytes;
  bool partials = need > 0;
  if (need > 0 && (!workspace || workspace_bytes < need)) {
    if (plan.path == PATH_MFMA) return LA_ERR_WORKSPACE_TOO_SMALL;
    partials = false;   // the general path does without, unsplit
    plan.chunk_len = kWholePrefix;
    size_partials(desc, prefix_lens_host, &plan);
  }

  AttnParams p;
  memset(&p, 0, sizeof p);
  p.q = q, p.k_cache = k_cache, p.v_cache = v_cache, p.k_branch = k_branch, p.v_branch = v_branch;
  p.k_chain = k_chain, p.v_chain = v_chain, p.chain_vis = chain_vis, p.C = chain_len;
  if (chain_len > 0 && tree) p.pool_seg = pool_seg, p.seg_mask = seg_mask;
  p.block_tables = block_tables, p.prefix_lens = prefix_lens;
  p.k_scale = k_scale, p.v_scale = v_scale;
  p.out = out, p.lse = lse;
  p.B = desc->num_requests, p.Hq = desc->num_q_heads, p.Hkv = desc->num_kv_heads;
  p.G = p.Hq / p.Hkv, p.D = desc->head_dim, p.gamma = desc->gamma, p.L = desc->branch_len;
  p.block_size = desc->block_size, p.max_blocks = desc->max_blocks_per_request;
  p.block_shift = __builtin_ctz((unsigned)desc->block_size);
  p.R = p.gamma * p.L * p.G;
  p.n_rows = p.gamma * p.L * p.Hq;
  p.out_f32 = desc->out_dtype == LA_F32;
  p.q_type = desc->q_dtype, p.kv_type = desc->kv_dtype, p.br_type = desc->branch_kv_dtype;
  p.scale_log2 = desc->softmax_scale * 1.44269504088896340736f;
  hipStream_t stream = (hipStream_t)hip_stream;

  p.n_row_tiles = plan.n_row_tiles, p.chunk_len = plan.chunk_len, p.s_max = plan.s_max;
  p.last_short = plan.last_short;
  p.total_units = plan.total_units;
  if (partials) {
    p.part_o = (float *)workspace;
    p.part_ml = (float *)((uint8_t *)workspace + plan.part_o_bytes);
  }
  if (p.B <= kMaxInlineLens) {
    p.n_inline = p.B;
    for (int b = 0; b < p.B; ++b) {
      AttnParams::Req &rq = p.req[b];
      rq.P = prefix_lens_host[b];
      rq.n = attn_num_chunks(rq.P, p.chunk_len);
      const int64_t tv = ((int64_t)rq.P + 63) / 64 + p.last_short;
      rq.q = (int)(tv / rq.n), rq.r = (int)(tv % rq.n);
      // n == 1: r == 0, the quotient is never needed.  The multiply-shift is exact for x < 2^32 / n; the kernel
      // applies it to x <= n * r < n^2, so very many chunks take the kernel's general path instead.
      rq.inv = rq.n > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)rq.n) + 1u : 0u;
      if (rq.n > 1024) p.n_inline = 0;
    }
  }
  if (plan.path == PATH_F32) {
    if (plan.shape == 0) return launch_attn_rows(p, stream) == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
    if (launch_attn_f32(p, plan.shape, stream) != hipSuccess) return LA_ERR_LAUNCH;
    return !partials || launch_attn_merge(p, stream) == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
  }
  const ShapeInfo si = shape_info(plan.shape);
  const hipError_t e =
      si.stream ? launch_attn_stream(p, si.local, stream) : launch_attn_mfma(p, si.local, plan.kv_fp8, plan.br_fp8, stream);
  if (e != hipSuccess) return LA_ERR_LAUNCH;
  if (launch_attn_merge(p, stream) != hipSuccess) return LA_ERR_LAUNCH;
  return LA_OK;
}

la_status la_verify_attention(const la_attn_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                              const int32_t *block_tables, const int32_t *prefix_lens,
                              const int32_t *prefix_lens_host, const void *k_branch, const void *v_branch,
                              const float *k_scale, const float *v_scale, void *out, float *lse, void *workspace,
                              size_t workspace_bytes, void *hip_stream) {
  return verify_attention(desc, q, k_cache, v_cache, block_tables, prefix_lens, prefix_lens_host, k_branch, v_branch,
                          nullptr, nullptr, 0, nullptr, nullptr, nullptr, nullptr, nullptr, k_scale, v_scale, out, lse,
                          workspace, workspace_bytes, hip_stream);
}

la_status la_verify_attention_nested(const la_attn_desc *desc, const void *q, const void *k_cache,
                                     const void *v_cache, const int32_t *block_tables, const int32_t *prefix_lens,
                                     const int32_t *prefix_lens_host, const void *k_branch, const void *v_branch,
                                     const void *k_chain, const void *v_chain, int32_t chain_len,
                                     const int32_t *chain_vis, const int32_t *chain_vis_host, const float *k_scale,
                                     const float *v_scale, void *out, float *lse, void *workspace,
                                     size_t workspace_bytes, void *hip_stream) {
  return verify_attention(desc, q, k_cache, v_cache, block_tables, prefix_lens, prefix_lens_host, k_branch, v_branch,
                          k_chain, v_chain, chain_len, chain_vis, chain_vis_host, nullptr, nullptr, nullptr, k_scale,
                          v_scale, out, lse, workspace, workspace_bytes, hip_stream);
}

la_status la_verify_attention_tree(const la_attn_desc *desc, const void *q, const void *k_cache, const void *v_cache,
                                   const int32_t *block_tables, const int32_t *prefix_lens,
                                   const int32_t *prefix_lens_host, const void *k_branch, const void *v_branch,
                                   const void *k_pool, const void *v_pool, int32_t pool_len, const int32_t *pool_seg,
                                   const int32_t *pool_seg_host, const uint64_t *seg_mask, const float *k_scale,
                                   const float *v_scale, void *out, float *lse, void *workspace,
                                   size_t workspace_bytes, void *hip_stream) {
  if (pool_len > 0 && (!pool_seg || !pool_seg_host || !seg_mask)) return LA_ERR_INVALID_ARG;
  return verify_attention(desc, q, k_cache, v_cache, block_tables, prefix_lens, prefix_lens_host, k_branch, v_branch,
                          k_pool, v_pool, pool_len, nullptr, nullptr, pool_len > 0 ? pool_seg : nullptr,
                          pool_len > 0 ? pool_seg_host : nullptr, pool_len > 0 ? seg_mask : nullptr, k_scale, v_scale,
                          out, lse, workspace, workspace_bytes, hip_stream);
}

// Shared by la_kv_commit (pool_seg == nullptr: the first n_chain tokens of the chain are kept) and
// la_kv_commit_tree (the pool tokens whose node has its bit in commit_mask are kept; n_chain == nullptr).
static la_status kv_commit(const la_attn_desc *desc, void *k_cache, void *v_cache, const int32_t *block_tables,
                           const int32_t *prefix_lens, const int32_t *prefix_lens_host, const void *k_branch,
                           const void *v_branch, const void *k_chain, const void *v_chain, int32_t chain_len,
                           const int32_t *pool_seg, const uint64_t *commit_mask, const int32_t *src_branch,
                           const int32_t *n_chain, const int32_t *n_own, const float *k_scale, const float *v_scale,
                           int32_t *new_prefix_lens, const la_layer_strides *layers, void *hip_stream) {
  const bool tree = commit_mask != nullptr;
  la_status st = validate_desc(desc);
  if (st != LA_OK) return st;
  if (!k_cache || !v_cache || !prefix_lens || !prefix_lens_host || !k_branch || !v_branch || !src_branch ||
      (!tree && !n_chain) || !n_own || !new_prefix_lens)
    return LA_ERR_INVALID_ARG;
  if (new_prefix_lens == prefix_lens) return LA_ERR_INVALID_ARG;  // read by every workgroup while one writes
  if (chain_len < 0 || (chain_len > 0 && (!k_chain || !v_chain))) return LA_ERR_INVALID_ARG;
  if (tree && ((chain_len > 0 && !pool_seg) || ((uintptr_t)commit_mask & 7))) return LA_ERR_INVALID_ARG;
  if (!aligned16(k_cache) || !aligned16(v_cache) || !aligned16(k_branch) || !aligned16(v_branch) ||
      !aligned16(k_chain) || !aligned16(v_chain))
    return LA_ERR_INVALID_ARG;
  const int kv = desc->kv_dtype, br = desc->branch_kv_dtype;
  const bool quantise = kv == LA_FP8_E4M3 && br == LA_BF16;
  if (kv != br && !quantise) return LA_ERR_UNSUPPORTED;
  if (desc->head_dim % 16) return LA_ERR_UNSUPPORTED;
  const int64_t capacity = (int64_t)desc->max_blocks_per_request * desc->block_size;
  // what is appended is decided on the device; the block table must have room for the most it can be
  for (int b = 0; b < desc->num_requests; ++b)
    if (prefix_lens_host[b] < 0 || (int64_t)prefix_lens_host[b] + chain_len + desc->branch_len > capacity)
      return LA_ERR_INVALID_ARG;
  const int n_layers = layers ? layers->num_layers : 1;
  if (n_layers < 1 || n_layers > 65535 || desc->num_requests > 65535) return LA_ERR_INVALID_ARG;
  const int elem_bytes[3] = {4, 2, 1};  // LA_F32, LA_BF16, LA_FP8_E4M3
  if (layers) {
    if (layers->cache_stride < 0 || layers->branch_stride < 0 || layers->chain_stride < 0 ||
        layers->scale_stride < 0)
      return LA_ERR_INVALID_ARG;
    // every layer's tensors must start on a 16-byte boundary
    if ((layers->cache_stride * elem_bytes[kv]) % 16 || (layers->branch_stride * elem_bytes[br]) % 16 ||
        (layers->chain_stride * elem_bytes[br]) % 16)
      return LA_ERR_INVALID_ARG;
  }

  CommitParams p;
  memset(&p, 0, sizeof p);
  p.k_cache = k_cache, p.v_cache = v_cache;
  p.k_branch = k_branch, p.v_branch = v_branch, p.k_chain = k_chain, p.v_chain = v_chain;
  p.block_tables = block_tables, p.prefix_lens = prefix_lens;
  p.src_branch = src_branch, p.n_chain = n_chain, p.n_own = n_own;
  p.pool_seg = tree && chain_len > 0 ? pool_seg : nullptr;  // an empty pool is the chain form with nothing kept
  p.commit_mask = commit_mask;
  p.k_scale = k_scale, p.v_scale = v_scale;
  p.new_prefix_lens = new_prefix_lens;
  p.B = desc->num_requests, p.Hkv = desc->num_kv_heads, p.D = desc->head_dim, p.gamma = desc->gamma;
  p.L = desc->branch_len, p.C = chain_len;
  p.block_size = desc->block_size, p.block_shift = __builtin_ctz((unsigned)desc->block_size);
  p.max_blocks = desc->max_blocks_per_request;
  p.capacity = (int)capacity;
  p.num_layers = n_layers;
  if (layers) {
    p.cache_stride = layers->cache_stride, p.branch_stride = layers->branch_stride;
    p.chain_stride = layers->chain_stride, p.scale_stride = layers->scale_stride;
  }
  return launch_kv_commit(p, elem_bytes[br], quantise, (hipStream_t)hip_stream) == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

la_status la_kv_commit(const la_attn_desc *desc, void *k_cache, void *v_cache, const int32_t *block_tables,
                       const int32_t *prefix_lens, const int32_t *prefix_lens_host, const void *k_branch,
                       const void *v_branch, const void *k_chain, const void *v_chain, int32_t chain_len,
                       const int32_t *src_branch, const int32_t *n_chain, const int32_t *n_own, const float *k_scale,
                       const float *v_scale, int32_t *new_prefix_lens, const la_layer_strides *layers,
                       void *hip_stream) {
  if (!n_chain) return LA_ERR_INVALID_ARG;
  return kv_commit(desc, k_cache, v_cache, block_tables, prefix_lens, prefix_lens_host, k_branch, v_branch, k_chain,
                   v_chain, chain_len, nullptr, nullptr, src_branch, n_chain, n_own, k_scale, v_scale,
                   new_prefix_lens, layers, hip_stream);
}

la_status la_kv_commit_tree(const la_attn_desc *desc, void *k_cache, void *v_cache, const int32_t *block_tables,
                            const int32_t *prefix_lens, const int32_t *prefix_lens_host, const void *k_branch,
                            const void *v_branch, const void *k_pool, const void *v_pool, int32_t pool_len,
                            const int32_t *pool_seg, const uint64_t *commit_mask, const int32_t *src_branch,
                            const int32_t *n_own, const float *k_scale, const float *v_scale,
                            int32_t *new_prefix_lens, const la_layer_strides *layers, void *hip_stream) {
  if (!commit_mask) return LA_ERR_INVALID_ARG;
  return kv_commit(desc, k_cache, v_cache, block_tables, prefix_lens, prefix_lens_host, k_branch, v_branch, k_pool,
                   v_pool, pool_len, pool_seg, commit_mask, src_branch, nullptr, n_own, k_scale, v_scale,
                   new_prefix_lens, layers, hip_stream);
}

static la_status validate_accept(const la_accept_desc *d) {
  if (!d) return LA_ERR_INVALID_ARG;
  if (d->num_branches < 1 || d->num_draft < 1 || d->vocab < 1) return LA_ERR_INVALID_ARG;
  if (d->top_k < 0 || !(d->top_p > 0.0f) || d->top_p > 1.0f) return LA_ERR_INVALID_ARG;
  if (d->logits_dtype != LA_F32 && d->logits_dtype != LA_BF16)
    return d->logits_dtype == LA_FP8_E4M3 ? LA_ERR_UNSUPPORTED : LA_ERR_INVALID_ARG;
  if (!(d->temperature > 0.f) || !isfinite(d->temperature)) return LA_ERR_INVALID_ARG;
  if ((int64_t)d->num_branches * (2 * (int64_t)d->num_draft + 1) > 65535) return LA_ERR_UNSUPPORTED;  // grid.y
  if (d->vocab > (1 << 21)) return LA_ERR_UNSUPPORTED;  // fine slices of one row are staged in LDS
  return LA_OK;
}

la_status la_spec_accept_workspace(const la_accept_desc *desc, size_t *bytes_out) {
  la_status st = validate_accept(desc);
  if (st != LA_OK) return st;
  if (!bytes_out) return LA_ERR_INVALID_ARG;
  *bytes_out = accept_workspace_bytes(desc->num_branches, desc->num_draft, desc->vocab,
                                      desc->logits_dtype == LA_BF16, nullptr, nullptr);
  return LA_OK;
}

la_status la_spec_accept(const la_accept_desc *desc, const void *target_logits, const void *draft_logits,
                         const int32_t *draft_tokens, const float *u_accept, const float *u_sample,
                         int32_t *accepted_len, int32_t *next_token, float *accept_ratio, void *workspace,
                         size_t workspace_bytes, void *hip_stream) {
  la_status st = validate_accept(desc);
  if (st != LA_OK) return st;
  if (!target_logits || !draft_tokens || !u_accept || !u_sample || !accepted_len || !next_token)
    return LA_ERR_INVALID_ARG;
  if (!aligned16(target_logits) || (draft_logits && !aligned16(draft_logits)) || !aligned16(workspace))
    return LA_ERR_INVALID_ARG;
  AcceptParams p;
  memset(&p, 0, sizeof p);
  const size_t need = accept_workspace_bytes(desc->num_branches, desc->num_draft, desc->vocab,
                                             desc->logits_dtype == LA_BF16, &p.n_chunks, &p.n_fine);
  if (!workspace || workspace_bytes < need) return LA_ERR_WORKSPACE_TOO_SMALL;
  p.target = target_logits, p.draft = draft_logits, p.tokens = draft_tokens;
  p.u_accept = u_accept, p.u_sample = u_sample;
  p.accepted_len = accepted_len, p.next_token = next_token, p.ratio = accept_ratio;
  p.NB = desc->num_branches, p.K = desc->num_draft, p.V = desc->vocab;
  p.bf16 = desc->logits_dtype == LA_BF16;
  p.inv_temp_log2 = 1.44269504088896340736f / desc->temperature;
  p.inv_temp = 1.0 / (double)desc->temperature;
  p.top_k = desc->top_k, p.top_p = desc->top_p;
  accept_carve_workspace(p, workspace);
  return launch_accept(p, (hipStream_t)hip_stream) == hipSuccess ? LA_OK : LA_ERR_LAUNCH;
}

}  // extern "C"
