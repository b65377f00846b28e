// Internal declarations shared by the translation units of libchunkkv (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "chunkkv.h"
#include "decode_plan.h"
#include "score_plan.h"

namespace ckv {

constexpr int kMaxLayersPerLaunch = 32;  // pointer tables travel as kernel arguments
constexpr int kTileBytes = 16384;        // one K tile staged in LDS (ring slot)
constexpr int kSuperKeys = 256;        // most keys per importance / chunk-sum step of pass 1 (several tiles)
constexpr int kThreads = 256;            // 4 wavefronts of 64
constexpr int kMaxRows = 512;            // g * w limit
constexpr int kMaxRanges = 64;           // two passes: most key ranges of a sequence whose statistics pass 1 merges
constexpr int kCompactEntries = 64;      // most selection entries per compaction workgroup

// Per-sequence metadata of one launch slice (<= kMaxBatchPerLaunch sequences).
struct SeqTable {
  int32_t seqlen[kMaxBatchPerLaunch];
  int32_t n_keep[kMaxBatchPerLaunch];
  int64_t kv_base[kMaxBatchPerLaunch];
  int64_t out_base[kMaxBatchPerLaunch];
};

// Arguments of the two scoring passes.  "problem" = (leader layer, sequence, kv-head).
// Arrays indexed by problem use the FULL batch (batch_total) so slices address the same buffers.
struct ScoreArgs {
  const void *q[kMaxLayersPerLaunch];
  const void *k[kMaxLayersPerLaunch];
  SeqTable seq;
  int32_t leader[kMaxLayersPerLaunch];    // leader index of every slice layer: whose problems of the workspace are its own
  int32_t chunk_of[kMaxLayersPerLaunch];  // chunk size of every slice layer
  int32_t batch0;          // index of this slice's first sequence
  int32_t batch_total;
  int32_t n_q_heads, n_kv_heads, window, chunk;   // chunk: of all slice layers, unless theirs may differ (importance pass, mixed_chunks)
  int64_t kv_stride_head, kv_stride_tok;
  float scale_log2e;       // softmax scale * log2(e)
  int32_t tiles_per_wg;    // pass 1: super-tiles each workgroup walks
  int32_t range_tiles;     // two passes: key tiles of a key range of pass 0
  int32_t ranges_per_wg;   // pass 0: key ranges each workgroup walks
  int32_t batch_slice;     // sequences of this slice
  // Number of the first key range (the reduction: group of periods) of every sequence, INT32_MAX past the last one; two passes
  // without heads_first: of its first workgroup.  The grids count the ranges of all sequences, so there are no empty workgroups:
  // these go to the XCDs, and there to the shader engines, in turn, and with a row of the grid as long as the longest sequence
  // has ranges some CUs got two of them and others none.  us of a call, so and with empty ones: two passes, five sequences of 3246 to
  // 14215 tokens in fp32 159 / 191, six of 1000 to 40000 with 224 rows 60 / 84; single pass, one of 20400 and eleven of 300 40 / 116
  // (16 ranges for the long one instead of 32: 108), eight of up to 20300 at c = 20 49 / 61 (59).
  int32_t first_range[kMaxBatchPerLaunch + 1];   // two passes: and the end of the last one
  int32_t heads_first;     // two passes: neighbouring workgroups are 1: heads of one range, 0: ranges of one head
  int32_t max_split;       // pitch of part_stats and row_stats in ranges
  int32_t rows_pad;        // g*w rounded up to 32
  float2 *part_stats;      // [slice layer][slice sequence][Hkv][max_split][rows_pad]  (running max, sum) in log2 units
  float *refs;             // [problem][rows_pad]  max + log2(sum), where pass 1 does not merge; single pass: [problem][g * window]
                           // reference of the last key range's sum
  float *chunk_scores;     // [leader][batch_total][Hkv][score_cap]
  int32_t score_cap;
  float *token_imp;        // [leader][batch_total][Hkv][imp_pitch] or null
  int64_t imp_pitch;
  const float *lse[kMaxLayersPerLaunch];  // pass 1 with use_lse: per leader layer [batch_total][Hq][w], natural log
  int32_t use_lse;
  int32_t merge_stats;     // pass 1: 1 = merge the pairs of pass 0 here
  int32_t super_keys;      // pass 1: super-tiles of at most this many keys, or of one chunk
  int32_t fuse_chunks;     // pass 1: 1 = super-tiles hold whole chunks and chunk sums are written
  // single-pass path (score_single.h): key ranges are single_periods_per_range() whole periods of 160 keys
  int32_t n_periods;       // pitch of e_buf / m_period: max over sequences of ceil(L / 160)
  void *e_buf;             // [problem][n_periods][rows_pad][2 lane halves][80 / c] x 3 bytes: per-(chunk, row) sums of e
  float *m_period;         // [problem][n_periods][rows_pad]  reference those sums are relative to
  float *row_stats;        // [problem][max_split][rows_pad]  a row's sum over a key range, see merge_row_stats
  int32_t row_groups;      // workgroups that share the rows of a key range (1 or 2)
  int32_t e_row_bytes;     // of e_buf, per period and row of a problem: the most of any layer
  int32_t mixed_chunks;    // 1: the layers' chunk sizes differ
  int32_t stream_k;        // 1: K is read with streaming (non-temporal) loads
};

struct TopkArgs {
  SeqTable seq;
  int32_t group0;             // first selection group of this launch
  int32_t chunk_of[kMaxLayersPerLaunch];   // chunk size of every group of the launch
  int32_t batch0, batch_total, n_kv_heads, window;
  const float *chunk_scores;  // [group][batch_total][Hkv][score_cap]
  int32_t score_cap, sel_cap;
  int32_t *sel_chunk, *sel_len, *sel_count;
  int32_t *sel_off;           // [group][batch_total][Hkv][sel_cap] exclusive token offsets, or null
  int32_t whole_chunks;       // 1: Algorithm 3 as printed: floor(n_keep / c) whole chunks, nothing is cut
};

// Which accesses to K, V, K' and V' are streaming (non-temporal): none, the loads, the gather's stores too.
enum class Stream : int32_t { kNone, kLoads, kAll };

struct CompactArgs {
  const void *k[kMaxLayersPerLaunch];
  const void *v[kMaxLayersPerLaunch];
  void *k_out[kMaxLayersPerLaunch];
  void *v_out[kMaxLayersPerLaunch];
  SeqTable seq;
  int32_t layer0, reuse;      // selection group of slice layer z is (layer0 + z) / reuse
  int32_t chunk_of[kMaxLayersPerLaunch];   // chunk size of every slice layer
  int32_t batch0, batch_total, n_kv_heads, window;
  int32_t elem_bytes;
  int64_t kv_stride_head, kv_stride_tok, out_stride_head, out_stride_tok;
  const int32_t *sel_chunk, *sel_len, *sel_count, *sel_off;  // sel_off may be null
  int32_t sel_cap;
  int32_t rows_per_wg;        // chosen by the launcher: rows a workgroup copies, in whole entries
  int32_t whole_chunks;       // 1: the window follows the kept tokens directly (their count varies per head)
  Stream stream;
};

// Decode attention over one layer's cache (decode.hip).  Per-head partial results use the FULL batch index.
struct DecodeArgs {
  const void *q, *k, *v;
  float *out, *lse;           // [batch_total][Hq][d], [batch_total][Hq] or null
  float2 *part_ml;            // (max in log2 units, sum) of every range: cut.first_split[i] * Hq entries of the sequences before, then [Hq][cut.splits[i]]
  float *part_o;              // [d] each, in the same order
  const int32_t *kv_len;      // [batch_total][Hkv] tokens to attend to, or null (= n_tok)
  int32_t n_tok[kMaxBatchPerLaunch];  // tokens the cache of a sequence holds per head
  int64_t base[kMaxBatchPerLaunch];   // element offset of the sequence in k / v
  int64_t stride_head, stride_tok;
  int32_t batch0, n_q_heads, n_kv_heads, group;   // group: query heads per kv-head
  float scale_log2e;
  DecodeCut cut;
};

// Absolute mass of one layer's cache (quality.hip): sum of |K| + |V| over blocks of rows of every (sequence, kv-head).
struct AbsSumArgs {
  const void *k, *v;
  float *partial;             // [batch_total][Hkv][n_blocks]; blocks past a head's rows hold 0
  const int32_t *kv_len;      // as in DecodeArgs
  int32_t n_tok[kMaxBatchPerLaunch];
  int64_t base[kMaxBatchPerLaunch];
  int64_t stride_head, stride_tok;
  int32_t batch0, n_kv_heads, head_dim, n_blocks;
};

struct QualityFinishArgs {
  const float *partial_full, *partial_kept;   // [B][Hkv][blocks_full], [B][Hkv][blocks_kept]
  const float *lse_full, *lse_kept;           // [B][Hq]: decode log-sum-exps at twice the softmax scale
  float *l1_loss, *attn_cos;                  // [B], [B][Hq]
  int32_t n_q_heads, n_kv_heads, blocks_full, blocks_kept;
};

// Reads element i of a small table that travels as a kernel argument.  A chain of selects on the
// (wavefront-uniform) index keeps the table in scalar registers; a dynamic subscript would make the
// compiler copy the whole argument struct to scratch memory first.
template <typename T, int N>
__device__ __forceinline__ T pick(const T (&arr)[N], int i) {
  T r = arr[0];
#pragma unroll
  for (int j = 1; j < N; ++j) r = (i == j) ? arr[j] : r;
  return r;
}

// Element i of a table inside a kernel's argument struct (the kernel's first parameter): one scalar load from the
// argument segment, where a chain of selects would load the whole table first.
template <typename T>
__device__ __forceinline__ T kernarg_at(size_t offset, int i) {
  typedef __attribute__((address_space(4))) const char *arg_ptr;
  return *(__attribute__((address_space(4))) const T *)((arg_ptr)__builtin_amdgcn_kernarg_segment_ptr() + offset + (size_t)i * sizeof(T));
}
#define CKV_ARG(STRUCT, FIELD, I) kernarg_at<std::remove_cv_t<std::remove_extent_t<decltype(STRUCT::FIELD)>>>(offsetof(STRUCT, FIELD), (I))

// Single-pass scoring: periods (160 keys) one workgroup walks, for a sequence of n_periods periods.  A function
// of the sequence alone (at most 32 ranges per sequence and kv-head, at least 4 periods each), so the key ranges,
// and with them every rounding of a score, do not depend on how many layers or sequences share a launch.
constexpr int kSingleMaxRanges = 32, kSingleLeastPeriods = 4;
__host__ __device__ inline int single_periods_per_range(int n_periods) {
  const int p = (n_periods + kSingleMaxRanges - 1) / kSingleMaxRanges;
  return p < kSingleLeastPeriods ? kSingleLeastPeriods : p + (p & 1);
}

// reference + log2(sum) of a row over its n key ranges of ppr periods each (np periods with prefix keys in all), in range
// order, with the loads of kRowStatsAhead ranges in flight (32 calls on 20011 tokens, 32 ranges: 927 us, 12 in flight 934).
// sums[s]: sum of range s, relative to the reference of its last period with prefix keys (periods[]), that of the last range
// to *last.  No range but the last has window keys alone: a window has at most 256, a range at least four periods.
constexpr int kRowStatsAhead = 16;
__device__ __forceinline__ float merge_row_stats(const float *sums, const float *periods, const float *last, int n, int ppr, int np, int pitch) {
  float m = -1.0e30f, l = 0.f;
  for (int s0 = 0; s0 < n; s0 += kRowStatsAhead) {
    float x[kRowStatsAhead], y[kRowStatsAhead], mm = m;
#pragma unroll
    for (int i = 0; i < kRowStatsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      const int s = s0 + i < n ? s0 + i : n - 1, end = (s + 1) * ppr < np ? (s + 1) * ppr : np;
      y[i] = sums[(int64_t)s * pitch];
      x[i] = *(s < n - 1 ? periods + (int64_t)(end - 1) * pitch : last);
    }
#pragma unroll
    for (int i = 0; i < kRowStatsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      mm = fmaxf(mm, x[i]);
    }
    l *= __builtin_amdgcn_exp2f(m - mm);
#pragma unroll
    for (int i = 0; i < kRowStatsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      l += s0 + i < n ? y[i] * __builtin_amdgcn_exp2f(x[i] - mm) : 0.f;
    }
    m = mm;
  }
  return m + __builtin_log2f(l);
}

// max + log2(sum) of a row's (max, sum) pairs, in range order, kPairsAhead loads in flight (16000 tokens, d = 64, 32 ranges 26.5 us a
// call, with eight 27.6)
constexpr int kPairsAhead = 16;
__device__ __forceinline__ float merge_pairs(const float2 *ps, int n, int pitch) {
  float m = -1.0e30f, l = 0.f;
  for (int s0 = 0; s0 < n; s0 += kPairsAhead) {
    float2 x[kPairsAhead];
#pragma unroll
    for (int i = 0; i < kPairsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      x[i] = ps[(int64_t)(s0 + i < n ? s0 + i : n - 1) * pitch];
    }
    float mm = m;
#pragma unroll
    for (int i = 0; i < kPairsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      mm = fmaxf(mm, x[i].x);
    }
    l *= __builtin_amdgcn_exp2f(m - mm);
#pragma unroll
    for (int i = 0; i < kPairsAhead; ++i) {
      if (i % 4 == 0 && s0 + i >= n) break;
      l += s0 + i < n ? x[i].y * __builtin_amdgcn_exp2f(x[i].x - mm) : 0.f;
    }
    m = mm;
  }
  return m + __builtin_log2f(l);
}

// Sequence of the x-th range (or group of periods) of a launch; x becomes its number within the sequence.
__device__ __forceinline__ int find_sequence(const ScoreArgs &a, int &x) {
  int seq = 0, first = 0;
#pragma unroll
  for (int i = 1; i < kMaxBatchPerLaunch; ++i)
    if (x >= a.first_range[i]) { seq = i; first = a.first_range[i]; }
  x -= first;
  return seq;
}

// Geometry of the scoring kernels for one (dtype, head_dim, row count).
struct ScoreGeom {
  int row_bytes;   // head_dim * sizeof(element)
  int tile_keys;   // keys per LDS tile
  int nq_blocks;   // 32-row blocks of window rows (padded)
  int nqw;         // blocks held by one wavefront
  int wq;          // wavefronts splitting the rows (the other 4/wq split keys)
};
bool score_geometry(int dtype, int head_dim, int rows, ScoreGeom *g);
// Workgroups of a pass (0 or 1) of the two that a CU holds: what the kernels are compiled for, and what their launches are cut for.  Two
// (73 KB of LDS each), except where half the register file does not do: four row blocks per wavefront, and fp32 operands at head_dim
// 128 with two of them or, in pass 0, with up to 64 rows (60 bytes of scratch).
constexpr int score_workgroups_per_cu(int dtype, int head_dim, int nqw, int wq, int pass) {
  if (dtype == CHUNKKV_F32 && head_dim == 128) return nqw == 1 && (pass == 1 || wq == 4) ? 2 : 1;
  return nqw >= 4 ? 1 : 2;
}

// Launchers (each checks hipGetLastError and returns a chunkkv_status).
int launch_score_pass(int pass, int dtype, int head_dim, const ScoreGeom &g, const ScoreArgs &a,
                      dim3 grid, hipStream_t s);
int launch_stats_combine(const ScoreArgs &a, int n_leaders_slice, int batch_slice, int tile_keys,
                         hipStream_t s);
int launch_chunk_sums(const ScoreArgs &a, int n_leaders_slice, int batch_slice, hipStream_t s);
int launch_score_single(int dtype, const ScoreArgs &a, dim3 grid, hipStream_t s);
int launch_jaccard(const int32_t *sel_chunk, const int32_t *sel_len, const int32_t *sel_count, int sel_cap, int chunk,
                   int rows_per_group, int n_pairs, float *out, hipStream_t s);
int launch_single_scores(ScoreArgs &a, int n_leaders_slice, int batch_slice, hipStream_t s);
bool single_pass_ok(int dtype, int head_dim, int rows, int chunk);
// bytes of e_buf per period and row: 20-bit floats in groups of eight, four per lane half as 24-bit ones
inline int single_e_row_bytes(int chunk) { return 80 / chunk == 4 ? 24 : 5 * (80 / chunk); }
int launch_topk(const TopkArgs &a, int n_groups, int batch_slice, hipStream_t s);
int launch_decode_mfma(int dtype, int head_dim, const DecodeArgs &a, int batch_slice, hipStream_t s);
int launch_decode(int dtype, int head_dim, bool matrix_cores, const DecodeArgs &a, int batch_slice, hipStream_t s);
int abs_sum_blocks(int n_tok_max);
int launch_abs_sum(int dtype, const AbsSumArgs &a, int batch_slice, hipStream_t s);
int launch_quality_finish(const QualityFinishArgs &a, int batch, hipStream_t s);
int launch_compact(int row_bytes, CompactArgs &a, int n_layers_slice, int batch_slice, hipStream_t s);
// Does the gather select as well, and how: decided before anything is launched.
struct SelectInGather {
  bool yes, wide;    // wide: 1024 threads
  int chunks, groups, rows_per_wg;   // chunks of the longest head, workgroups of a head
};
SelectInGather select_in_gather(CompactArgs &a, int n_layers_slice, int batch_slice);
int launch_select_compact(int row_bytes, CompactArgs &a, int n_layers_slice, int batch_slice, const float *chunk_scores, int score_cap,
                          const SelectInGather &how, hipStream_t s);

}  // namespace ckv
