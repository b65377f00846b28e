// Small kernels around the scoring kernels: merging the per-range softmax statistics, chunk sums for chunk sizes too large to fit one key tile, and the row
// reduction of the single-pass scoring.
#include "internal.h"

namespace ckv {

int launch_score_bf16(int pass, int head_dim, const ScoreGeom &g, const ScoreArgs &a, dim3 grid, hipStream_t s);
int launch_score_f16(int pass, int head_dim, const ScoreGeom &g, const ScoreArgs &a, dim3 grid, hipStream_t s);
int launch_score_f32(int pass, int head_dim, const ScoreGeom &g, const ScoreArgs &a, dim3 grid, hipStream_t s);
int launch_score_single_bf16(const ScoreArgs &a, dim3 grid, hipStream_t s);
int launch_score_single_f16(const ScoreArgs &a, dim3 grid, hipStream_t s);

bool score_geometry(int dtype, int head_dim, int rows, ScoreGeom *g) {
  if (dtype != CHUNKKV_F32 && dtype != CHUNKKV_BF16 && dtype != CHUNKKV_F16) return false;
  if (head_dim != 64 && head_dim != 128) return false;
  if (rows < 1 || rows > kMaxRows) return false;
  g->row_bytes = head_dim * elem_bytes(dtype);
  g->tile_keys = kTileBytes / g->row_bytes;
  g->nq_blocks = (rows + 31) / 32;
  if (g->nq_blocks == 1) { g->nqw = 1; g->wq = 1; }
  else if (g->nq_blocks == 2) { g->nqw = 1; g->wq = 2; }
  else if (g->nq_blocks <= 4) { g->nqw = 1; g->wq = 4; }
  else if (g->nq_blocks <= 8) { g->nqw = 2; g->wq = 4; }
  else { g->nqw = 4; g->wq = 4; }
  if (g->nqw == 4 && dtype == CHUNKKV_F32 && head_dim == 128) return false;  // operand registers exceed the file
  return true;
}

int launch_score_pass(int pass, int dtype, int head_dim, const ScoreGeom &g, const ScoreArgs &a, dim3 grid,
                      hipStream_t s) {
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return CHUNKKV_OK;
  if (dtype == CHUNKKV_BF16) return launch_score_bf16(pass, head_dim, g, a, grid, s);
  if (dtype == CHUNKKV_F16) return launch_score_f16(pass, head_dim, g, a, grid, s);
  return launch_score_f32(pass, head_dim, g, a, grid, s);
}

// Does the single-pass kernel take this problem?  16-bit caches of head_dim 128, 65 to 256 window rows per
// kv-head, chunk sizes that cut a lane half's 80 keys into a multiple of four chunks.
bool single_pass_ok(int dtype, int head_dim, int rows, int chunk) {
  return (dtype == CHUNKKV_BF16 || dtype == CHUNKKV_F16) && head_dim == 128 && rows > 64 && rows <= 256 &&
         (chunk == 5 || chunk == 10 || chunk == 20);
}

int launch_score_single(int dtype, const ScoreArgs &a, dim3 grid, hipStream_t s) {
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return CHUNKKV_OK;
  if (dtype == CHUNKKV_BF16) return launch_score_single_bf16(a, grid, s);
  if (dtype == CHUNKKV_F16) return launch_score_single_f16(a, grid, s);
  return CHUNKKV_ERR_UNSUPPORTED;
}

// ref_r = max_r + log2(sum_r) over all key ranges of a problem.  Up to kMaxRanges ranges as the second pass does it where it merges the
// pairs itself, in launches of fewer rounds of workgroups: the same bits.  More of them: four lanes share a row, each merges a
// quarter of the ranges in one pass ((m, l) pairs merge associatively), then the four partial pairs are
// merged with two shuffles, always in the same order, kCombineAhead pairs of a lane in flight.
// grid: x = (sequence, kv-head), y = leader, z = block of 64 rows; 256 threads.
constexpr int kCombineAhead = 8;
__global__ __launch_bounds__(256) void stats_combine_kernel(ScoreArgs a, int tile_keys) {
  const int bl = blockIdx.x / a.n_kv_heads, h = blockIdx.x % a.n_kv_heads, z = blockIdx.y;
  const int64_t problem = ((int64_t)CKV_ARG(ScoreArgs, leader, z) * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const int L = CKV_ARG(ScoreArgs, seq.seqlen, bl);
  const int ntiles = (L + tile_keys - 1) / tile_keys;
  const int nsplit = (ntiles + a.range_tiles - 1) / a.range_tiles;
  const int part = threadIdx.x & 3;
  const int row = blockIdx.z * 64 + (threadIdx.x >> 2);  // rows_pad is a multiple of 32; rows past it are skipped below
  const bool live = row < a.rows_pad;
  const float2 *ps = a.part_stats + (((int64_t)z * a.batch_slice + bl) * a.n_kv_heads + h) * a.max_split * a.rows_pad + (live ? row : 0);
  if (nsplit <= kMaxRanges) {
    if (live && part == 0) a.refs[problem * a.rows_pad + row] = merge_pairs(ps, nsplit, a.rows_pad);
    return;
  }
  float m = -1.0e30f, l = 0.f;
  for (int s0 = part; s0 < nsplit; s0 += 4 * kCombineAhead) {
    float2 x[kCombineAhead];
#pragma unroll
    for (int i = 0; i < kCombineAhead; ++i) x[i] = ps[(int64_t)(s0 + 4 * i < nsplit ? s0 + 4 * i : s0) * a.rows_pad];
#pragma unroll
    for (int i = 0; i < kCombineAhead; ++i) {
      if (s0 - part + 4 * i >= nsplit) break;   // the same for all lanes
      if (s0 + 4 * i < nsplit) {
        const float mm = fmaxf(m, x[i].x);
        l = l * __builtin_amdgcn_exp2f(m - mm) + x[i].y * __builtin_amdgcn_exp2f(x[i].x - mm);
        m = mm;
      }
    }
  }
#pragma unroll
  for (int o = 1; o < 4; o <<= 1) {
    const float mo = __shfl_xor(m, o), lo = __shfl_xor(l, o);
    const float mm = fmaxf(m, mo);
    // both partners compute the same sum in the same order: lower lane's term first
    const bool low = (part & o) == 0;
    const float a0 = (low ? l : lo) * __builtin_amdgcn_exp2f((low ? m : mo) - mm), a1 = (low ? lo : l) * __builtin_amdgcn_exp2f((low ? mo : m) - mm);
    l = a0 + a1;
    m = mm;
  }
  if (live && part == 0) a.refs[problem * a.rows_pad + row] = m + log2f(l);
}

int launch_stats_combine(const ScoreArgs &a, int n_leaders_slice, int batch_slice, int tile_keys, hipStream_t s) {
  if (n_leaders_slice <= 0 || batch_slice <= 0) return CHUNKKV_OK;
  dim3 grid(batch_slice * a.n_kv_heads, n_leaders_slice, (a.rows_pad + 63) / 64);
  hipLaunchKernelGGL(stats_combine_kernel, grid, dim3(256), 0, s, a, tile_keys);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

// Chunk sums from per-token importance, one wavefront per chunk, fixed summation order.
// grid: x = chunk group of 4, y = (sequence, kv-head), z = leader.
__global__ void chunk_sums_kernel(ScoreArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int bl = blockIdx.y / a.n_kv_heads, h = blockIdx.y % a.n_kv_heads, z = blockIdx.z;
  const int64_t problem = ((int64_t)CKV_ARG(ScoreArgs, leader, z) * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const int P = pick(a.seq.seqlen, bl) - a.window, c = a.chunk;
  const int C = (P + c - 1) / c;
  const int ci = blockIdx.x * 4 + wave;
  if (ci >= C) return;
  const float *imp = a.token_imp + problem * a.imp_pitch;
  const int64_t j0 = (int64_t)ci * c, j1 = j0 + c < P ? j0 + c : P;
  float sum = 0.f;
  for (int64_t j = j0 + lane; j < j1; j += 64) sum += imp[j];
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if (lane == 0) a.chunk_scores[problem * a.score_cap + ci] = sum;
}

int launch_chunk_sums(const ScoreArgs &a, int n_leaders_slice, int batch_slice, hipStream_t s) {
  int maxC = 0;
  for (int b = 0; b < batch_slice; ++b) {
    const int P = a.seq.seqlen[b] - a.window;
    const int C = (P + a.chunk - 1) / a.chunk;
    maxC = C > maxC ? C : maxC;
  }
  if (maxC == 0 || n_leaders_slice <= 0) return CHUNKKV_OK;
  dim3 grid((maxC + 3) / 4, batch_slice * a.n_kv_heads, n_leaders_slice);
  hipLaunchKernelGGL(chunk_sums_kernel, grid, dim3(256), 0, s, a);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

// Single-pass path, second kernel: the row references and the chunk scores.
//   ref_r = m_r + log2(sum_r), merged from the (reference, sum) pairs the key ranges left for row r
//           (pairs merge associatively; always in the same order: range by range);
//   score[chunk] = sum over rows of E[chunk][row] * exp2(m[chunk][row] - ref[row]).
// A workgroup of 256 threads merges the statistics of its problem (one row per thread, sixteen ranges' pairs in flight)
// and then takes `periods_per_wg` consecutive periods.  Per period the scoring kernel left, for each lane half h and
// each group of eight consecutive chunks of that half, rows_pad pieces of 16 + 4 bytes (eight sums as 20-bit floats:
// 8 exponent and 12 mantissa bits; chunk size 20 has four chunks per half: pieces of 12 bytes, four 24-bit floats), and
// rows_pad references (one per row).  A wavefront takes one (period, half, group) at a time: its lanes walk the rows
// (consecutive lanes read consecutive pieces, all pieces of a task in flight), weigh, and the sums are reduced over
// the lanes in a fixed order, halving the values a lane holds with every step (10 shuffles for eight sums instead of
// 48).  The chunk of (half h, position s) is 2 s + h of the period's 2 S chunks.  Rows past the real ones are skipped:
// nothing was written for them.
// Bound by HBM over a stack; over a single layer by how many workgroups share it: one layer of 20011 tokens, c = 5, took
// 98 us with 32 periods per workgroup (32 workgroups); the launcher now cuts it finer.  The pieces of a task are read while
// the references are merged and while the lanes of the task before are added up, from a base that is wavefront-uniform:
// 32 layers of 32768 tokens 93 -> 75 us, a ragged batch at c = 20 130 -> 90, one layer of 8192 tokens 8.8 -> 7.5 (16 layers
// of 131072, at the memory's rate before and after: 222 -> 217).  Two groups of sums per task, which share the weights,
// took 84 us on the first and 24 instead of 13 on one layer at c = 5; reads that are not streaming, 81.
// grid: x = period group of any sequence, y = kv-head, z = leader.
constexpr int kSinglePeriod = 160, kSingleHalf = 80;   // as in the single-pass scoring kernel
constexpr int kScoresTargetWgs = 2048, kScoresMaxPeriods = 32;

// Sum over the 64 lanes of N (4 or 8) values per lane; lane l returns the total of value (l >> (6 - log2 N)).
template <int N>
__device__ __forceinline__ float wave_sum_scatter(float (&v)[N]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int n = N / 2, o = 32; n >= 1; n /= 2, o /= 2) {
    const bool upper = (lane & o) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const float keep = upper ? v[n + i] : v[i], send = upper ? v[i] : v[n + i];
      v[i] = keep + __shfl_xor(send, o);
    }
  }
  float x = v[0];
#pragma unroll
  for (int o = 32 / N; o >= 1; o /= 2) x += __shfl_xor(x, o);
  return x;
}

template <int S, int RB>   // chunks per lane half and period; 64-row blocks of rows_pad; a: the kernel's argument
__device__ __forceinline__ void single_scores(const ScoreArgs &a, int periods_per_wg, float *s_ref) {
  typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform, and known to be
  int group = blockIdx.x;
  const int bl = find_sequence(a, group), h = blockIdx.y, z = blockIdx.z;
  const int64_t problem = ((int64_t)CKV_ARG(ScoreArgs, leader, z) * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const int L = CKV_ARG(ScoreArgs, seq.seqlen, bl), P = L - a.window, c = kSingleHalf / S;
  const int C = (P + c - 1) / c;
  const int np = (P + kSinglePeriod - 1) / kSinglePeriod;   // periods that hold prefix keys
  const int p0 = group * periods_per_wg;
  const int p1 = p0 + periods_per_wg < np ? p0 + periods_per_wg : np;
  const int nrows = (a.n_q_heads / a.n_kv_heads) * a.window;

  constexpr int G8 = S / 8, NV = S == 4 ? 4 : 8, combos = S == 4 ? 2 : 2 * G8;   // values and tasks per period
  constexpr int kRowBytes = S == 4 ? 24 : combos * 20;                           // E bytes per period and row
  const int64_t prow = (int64_t)a.rows_pad;
  const float *m_problem = a.m_period + problem * a.n_periods * prow;
  const char *e_problem = (const char *)a.e_buf + problem * a.n_periods * prow * a.e_row_bytes;
  float *scores = a.chunk_scores + problem * a.score_cap;
  const int n_tasks = (p1 - p0) * combos;

  float mr[RB];
  u32x4 w[RB];
  uint32_t w4[RB];
  auto load = [&](int task) __attribute__((always_inline)) {
    const int period = p0 + task / combos, combo = task % combos;   // combo = half * G8 + group
    const char *pbase = e_problem + (int64_t)period * prow * kRowBytes;
    const float *mp = m_problem + (int64_t)period * prow;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const uint32_t row = 64 * i + lane < nrows ? 64 * i + lane : 0;
      mr[i] = mp[row];
      if constexpr (S == 4) {
        const u32x3 d = __builtin_nontemporal_load((const u32x3 *)((pbase + (int64_t)combo * prow * 12) + row * 12));
        w[i] = u32x4{d.x, d.y, d.z, 0u};
      } else {
        w[i] = __builtin_nontemporal_load((const u32x4 *)((pbase + (int64_t)combo * prow * 16) + row * 16));
        w4[i] = __builtin_nontemporal_load((const uint32_t *)((pbase + (int64_t)combos * prow * 16 + (int64_t)combo * prow * 4) + row * 4));
      }
    }
  };
  if (wave < n_tasks) load(wave);   // in flight while the references are merged

  // ---- references
  {
    const int np_total = (L + kSinglePeriod - 1) / kSinglePeriod, ppr = single_periods_per_range(np_total);
    const int nsplit = (np_total + ppr - 1) / ppr;
    s_ref[tid] = tid < nrows ? merge_row_stats(a.row_stats + problem * a.max_split * a.rows_pad + tid, m_problem + tid, a.refs + problem * nrows + tid,
                                               nsplit, ppr, np, a.rows_pad) : 3.0e38f;
  }
  __syncthreads();
  float ref[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) ref[i] = s_ref[64 * i + lane];   // 3e38 past the real rows: weight 0

  // ---- chunk scores
  for (int task = wave; task < n_tasks; task += 4) {
    const int period = p0 + task / combos, combo = task % combos;
    const int hh = S == 4 ? combo : combo / G8, g8 = S == 4 ? 0 : combo % G8;
    float v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = 0.f;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const float wgt = exp2f(mr[i] - ref[i]);
      if constexpr (S == 4) {
        v[0] += __uint_as_float(w[i].x << 8) * wgt;
        v[1] += __uint_as_float(__builtin_amdgcn_alignbit(w[i].y, w[i].x, 24) << 8) * wgt;
        v[2] += __uint_as_float(__builtin_amdgcn_alignbit(w[i].z, w[i].y, 16) << 8) * wgt;
        v[3] += __uint_as_float(w[i].z & 0xFFFFFF00u) * wgt;
      } else {
        uint32_t q[8];
        q[0] = w[i].x & 0xFFFFFu;
        q[1] = (w[i].x >> 20) | ((w[i].y & 0xFFu) << 12);
        q[2] = (w[i].y >> 8) & 0xFFFFFu;
        q[3] = (w[i].y >> 28) | ((w[i].z & 0xFFFFu) << 4);
        q[4] = (w[i].z >> 16) | ((w[i].w & 0xFu) << 16);
        q[5] = (w[i].w >> 4) & 0xFFFFFu;
        q[6] = (w[i].w >> 24) | ((w4[i] & 0xFFFu) << 8);
        q[7] = w4[i] >> 12;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] += __uint_as_float(q[j] << 11) * wgt;
      }
    }
    if (task + 4 < n_tasks) load(task + 4);
    const float val = wave_sum_scatter<NV>(v);
    constexpr int kLanes = 64 / NV;   // lanes that hold the same total
    if (lane % kLanes == 0) {
      const int chunk = period * 2 * S + 2 * (8 * g8 + lane / kLanes) + hh;
      if (chunk < C) scores[chunk] = val;
    }
  }
}

template <int S, int RB>
__global__ __launch_bounds__(256) void single_scores_kernel(ScoreArgs a, int periods_per_wg) {
  __shared__ float s_ref[256];
  single_scores<S, RB>(a, periods_per_wg, s_ref);
}

// Layers of different chunk sizes in one launch.
template <int RB>
__global__ __launch_bounds__(256) void single_scores_mixed_kernel(ScoreArgs a, int periods_per_wg) {
  __shared__ float s_ref[256];
  const int c = CKV_ARG(ScoreArgs, chunk_of, blockIdx.z);
  if (c == 5) single_scores<16, RB>(a, periods_per_wg, s_ref);
  else if (c == 10) single_scores<8, RB>(a, periods_per_wg, s_ref);
  else single_scores<4, RB>(a, periods_per_wg, s_ref);
}

int launch_single_scores(ScoreArgs &a, int n_leaders_slice, int batch_slice, hipStream_t s) {
  auto periods_of = [&](int b) { return (a.seq.seqlen[b] - a.window + kSinglePeriod - 1) / kSinglePeriod; };
  int64_t periods = 0;
  for (int b = 0; b < batch_slice; ++b) periods += periods_of(b);
  if (periods == 0 || n_leaders_slice <= 0) return CHUNKKV_OK;
  if (a.rows_pad != 128 && a.rows_pad != 256) return CHUNKKV_ERR_UNSUPPORTED;
  // at most about kScoresTargetWgs workgroups (eight per CU, one generation), with at least one task for each of their four
  // wavefronts; with 256 rows at least two periods, as 32 ranges of them are 64 KB of statistics for a period's 20 (32 calls
  // on 20011 tokens, 16 of them scored, c = 5: 927 us, with one period 968)
  const bool wide = a.rows_pad == 256;
  const int sums = kSingleHalf / a.chunk, least = sums == 16 && !wide && !a.mixed_chunks ? 1 : 2;
  int64_t ppw = (periods * a.n_kv_heads * n_leaders_slice + kScoresTargetWgs - 1) / kScoresTargetWgs;
  ppw = ppw < least ? least : (ppw > kScoresMaxPeriods ? kScoresMaxPeriods : ppw);
  int groups = 0;
  for (int b = 0; b < batch_slice; ++b) {
    a.first_range[b] = groups;
    groups += (periods_of(b) + (int)ppw - 1) / (int)ppw;
  }
  dim3 grid(groups, a.n_kv_heads, n_leaders_slice);
  if (a.mixed_chunks) hipLaunchKernelGGL((wide ? single_scores_mixed_kernel<4> : single_scores_mixed_kernel<2>), grid, dim3(256), 0, s, a, (int)ppw);
  else switch (sums) {
    case 4: hipLaunchKernelGGL((wide ? single_scores_kernel<4, 4> : single_scores_kernel<4, 2>), grid, dim3(256), 0, s, a, (int)ppw); break;
    case 8: hipLaunchKernelGGL((wide ? single_scores_kernel<8, 4> : single_scores_kernel<8, 2>), grid, dim3(256), 0, s, a, (int)ppw); break;
    case 16: hipLaunchKernelGGL((wide ? single_scores_kernel<16, 4> : single_scores_kernel<16, 2>), grid, dim3(256), 0, s, a, (int)ppw); break;
    default: return CHUNKKV_ERR_UNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

}  // namespace ckv
