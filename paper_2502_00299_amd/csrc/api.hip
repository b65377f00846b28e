// Host side of libchunkkv: argument checks, workspace plans and launch sequences of the C-ABI calls.
#include <math.h>
#include <string.h>

#include <mutex>

#include "decode_plan.h"
#include "internal.h"

namespace ckv {
namespace {

constexpr int kTargetWorkgroups = 4096;  // eight rounds of 2 workgroups on each of 256 CUs
// Two-pass scoring of up to this many key tiles: pass 1 merges the row statistics of the ranges itself, every workgroup for
// itself while its first tiles travel.  A kernel in between took 5 us, and 9 to 49 for one layer of a hundred ranges or more:
// 16000 tokens 34.3 -> 28.9 us a call, 19000 with 64 rows 66 -> 42, 120602 in fp32 288 -> 234.  Above it that kernel is a
// percent or two and merging everywhere more (10 layers of 109334 tokens, 224 rows 906 us, 947 merged).  A layer of up to so many
// tiles has at most kMaxRanges ranges.
constexpr int64_t kMergeTiles = 16384;
// How the two passes are cut into workgroups (units_per_workgroup in score_plan.h): whole rounds, as far as a launch has few.  What
// a workgroup costs, in microseconds: a 32-key block against 32 rows with two workgroups on the CU; beside its tiles start, queries,
// first tiles and end; in pass 1 the merge of eight ranges' statistics.  us of a call (ranges of pass 0 chosen per launch, too), and with about
// 32 ranges of eight tiles or more and up to 1536 workgroups in pass 1 whatever the rounds are: 12345 tokens, three of eight groups in two passes 198 / 210;
// 32 layers of 4270 tokens, 64 rows 112 / 133; 59567 tokens in fp32, 256 rows 328 / 358; 32 layers of five sequences of 1379 to 3768
// tokens, d = 64 85 / 107.  In a long launch that memory bounds few long walks lose (eight sequences of 7138 to 47085 tokens, 32 rows
// 248, in one round 266): there only those of up to kFewRounds rounds are cut anew.
constexpr double kBlockUs[2] = {0.6, 1.9}, kStartUs = 2.4, kMergeUs = 0.7, kHalfRound[2] = {0.7, 0.75};   // [0]: 16-bit types, [1]: fp32
constexpr int kFewRounds = 4, kCUs = 256;
// Single-pass scoring with 256 rows: up to this many workgroups leave half the CUs empty, so two of them, with 128 rows each,
// share a key range; K is read twice.  us of a call on one layer, split / not: 104 workgroups 26.9 / 30.0, 128 of them at 65536
// tokens 59.6 / 69.8; 200 36.1 / 35.9, 256 at 20011 tokens 42.6 / 41.8, 256 at 131072 155 / 140.
constexpr int64_t kRowSplitWorkgroups = 128;
constexpr int kSinglePeriodKeys = 160;   // granule of the single-pass kernel's key ranges
// Key tiles (16 KB) one scoring launch set should hold.  Sets would let the gather of one run beside the scoring of the next on a
// second stream, which takes longer (the 131072-token stack 2.17 ms in one set, 2.23 in two, 2.45 in eight), so one set it is.
constexpr int64_t kTilesPerLaunch = 1 << 30;

// Streaming (non-temporal) loads leave the memory-side cache (256 MB) to others.  They are for calls whose K and V fill most of
// it: nothing a pass reads is still there for the next, while smaller ones lose what they find there.  us of a call, streaming and
// plain: 32 layers of 32768 tokens 679 / 696, 28 of 17734 97 / 101; 16 layers of 1477 tokens 24.8 / 23.2, 7 of 47180 (170 MB, d = 64)
// 57.1 / 55.5.  A per-layer call is one of many, so a third of that: 16 calls one after the other on layers of 67 MB 360 / 375, 101 MB 424 / 441,
// 201 MB 677 / 703, 268 MB 828 / 863, but a call right behind a kernel that wrote its K and V 67 MB 26.2 / 25.7, 101 MB 30.7 / 29.8, 201 MB 45.8 / 46.2,
// 268 MB 55.6 / 57.5, and behind one that read them the same within 3 %.  Below the line the same call again on the same layer of 34 MB takes
// 25.4 / 24.1, calls on one layer after the other 259 / 269.
constexpr int64_t kStreamBytes = 192 << 20, kStreamLayerBytes = 64 << 20;
// Stores of the gather, and then the loads too, where K' and V' are more than half of that cache (a per-layer call, one of many: a
// thirty-second of that).  Smaller ones are still there for the decoding step that reads them next.  us of compressing and of one such step
// over 32 layers, streaming and plain: 31 MB written 284 / 254, 57 MB 373 / 318, 111 MB 443 / 422, two passes 29 MB 288 / 262, 111 MB 505 / 486.
// Above, what is still there and what the next call has to write back for it even out: 218 MB 564 / 528, 163 MB in eight chunk sizes 334 / 340, 433 MB
// 770 / 763, 1291 MB 1165 / 1201, and compressing alone, call after call, 4 to 8 % slower with plain stores (48 / 47, 83 / 82, 136 / 130 below the
// line, two passes 52 / 56, 179 / 190; above 242 / 253, 168 / 179, 434 / 451, 733 / 777).  Layer by layer 3 MB each 874 / 851 (4096 tokens at 20 %, two passes 778 / 770), 7 MB 1009 / 1004,
// 10 MB 917 / 922, 14 MB 547 / 556, 30 MB 1393 / 1422.
constexpr int64_t kStreamOutBytes = 128 << 20, kStreamOutLayerBytes = 4 << 20;

struct Plan {
  ScoreGeom geom;
  int n_leaders, rows_pad;
  int batch_leaders;  // leader layers scored per launch set
  int fuse_chunks;
  // single-pass path: usable for this problem?  geometry and workspace
  int single_ok, n_periods_fit, rows_pad_s, n_periods, max_split_s;
  size_t part_bytes;      // of the region at off_part
  size_t off_part, off_refs, off_scores, off_seloff, off_imp, off_ebuf, off_mper, total;
};

// ---- optional per-kernel timing (chunkkv_timing_begin / chunkkv_timing_end) -----------------------
enum Kind { kStats = 0, kCombine, kColsum, kChunkSums, kTopk, kCompact, kDecode, kKinds };
static_assert(kKinds == CHUNKKV_TIMING_KINDS, "timing kinds of the header");
struct Timing {
  bool on = false;
  int cap = 0, used = 0;
  hipEvent_t *ev = nullptr;  // 2 per record
  int *kind = nullptr;
} g_timing;

struct Timed {  // records an event pair around one launch when timing is on
  hipStream_t s;
  int slot = -1;
  Timed(int kind, hipStream_t stream) : s(stream) {
    if (g_timing.on && g_timing.used < g_timing.cap) {
      slot = g_timing.used++;
      g_timing.kind[slot] = kind;
      (void)hipEventRecord(g_timing.ev[2 * slot], s);
    }
  }
  ~Timed() {
    if (slot >= 0) (void)hipEventRecord(g_timing.ev[2 * slot + 1], s);
  }
};

// ---- device-resident scratch for chunkkv_decode_attention_static ---------------------------------
// One array per GPU the library runs on, held until the process ends.  Its name is only a host-side
// stand-in: the device address is looked up once per device and kept; host code uses that pointer.
constexpr size_t kStaticScratchBytes = CHUNKKV_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
}  // namespace
}  // namespace ckv
static __device__ __align__(256) unsigned char scratch[ckv::kStaticScratchBytes];
namespace ckv {
namespace {
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};
// device address of `scratch` on the current device (looked up on the first call per device)
int static_scratch(void **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CHUNKKV_ERR_LAUNCH;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return CHUNKKV_ERR_LAUNCH;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CHUNKKV_OK;
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

int check_problem(const chunkkv_problem *p, bool need_out) {
  if (!p) return CHUNKKV_ERR_NULL;
  if (!p->seqlen || !p->n_keep || !p->kv_base) return CHUNKKV_ERR_NULL;
  if (need_out && !p->out_base) return CHUNKKV_ERR_NULL;
  if (p->batch < 1 || p->n_q_heads < 1 || p->n_kv_heads < 1 || p->window < 1 || p->chunk < 1)
    return CHUNKKV_ERR_SHAPE;
  if (p->n_q_heads % p->n_kv_heads != 0) return CHUNKKV_ERR_SHAPE;
  if (!(p->softmax_scale >= 0.f) || isinf(p->softmax_scale)) return CHUNKKV_ERR_SHAPE;
  if (p->dtype != CHUNKKV_F32 && p->dtype != CHUNKKV_BF16 && p->dtype != CHUNKKV_F16) return CHUNKKV_ERR_UNSUPPORTED;
  if (p->flags & ~(uint32_t)(CHUNKKV_FLAG_WHOLE_CHUNKS | CHUNKKV_FLAG_TWO_PASS)) return CHUNKKV_ERR_UNSUPPORTED;
  if (p->head_dim != 64 && p->head_dim != 128) return CHUNKKV_ERR_UNSUPPORTED;
  const int64_t rows = (int64_t)(p->n_q_heads / p->n_kv_heads) * p->window;
  ScoreGeom g;
  if (rows > kMaxRows || !score_geometry(p->dtype, p->head_dim, (int)rows, &g)) return CHUNKKV_ERR_UNSUPPORTED;
  const int esz = elem_bytes(p->dtype);
  if (p->kv_stride_tok < p->head_dim || p->kv_stride_head < 0) return CHUNKKV_ERR_SHAPE;
  if ((p->kv_stride_tok * esz) % 16 || (p->kv_stride_head * esz) % 16) return CHUNKKV_ERR_SHAPE;
  if (p->kv_stride_tok * esz > (1 << 22)) return CHUNKKV_ERR_UNSUPPORTED;  // tile offsets are 32-bit
  if (need_out) {
    if (p->out_stride_tok < p->head_dim || p->out_stride_head < 0) return CHUNKKV_ERR_SHAPE;
    if ((p->out_stride_tok * esz) % 16 || (p->out_stride_head * esz) % 16) return CHUNKKV_ERR_SHAPE;
  }
  if (p->sel_cap < 1 || p->score_cap < 0) return CHUNKKV_ERR_SHAPE;
  for (int b = 0; b < p->batch; ++b) {
    const int64_t L = p->seqlen[b], nk = p->n_keep[b];
    if (L < p->window || nk < 0 || nk > L - p->window) return CHUNKKV_ERR_SHAPE;
    if (p->kv_base[b] < 0 || (p->kv_base[b] * esz) % 16) return CHUNKKV_ERR_SHAPE;
    // the scoring kernels address the K rows of one (sequence, kv-head) through a buffer descriptor with
    // 32-bit byte offsets (one tile of slack past the end)
    if (((int64_t)L + 256) * p->kv_stride_tok * esz >= (int64_t)1 << 31) return CHUNKKV_ERR_UNSUPPORTED;
    if (need_out && (p->out_base[b] < 0 || (p->out_base[b] * esz) % 16)) return CHUNKKV_ERR_SHAPE;
    if (p->sel_cap < (nk + p->chunk - 1) / p->chunk + 1) return CHUNKKV_ERR_SHAPE;
    if (p->score_cap < (L - p->window + p->chunk - 1) / p->chunk) return CHUNKKV_ERR_SHAPE;
  }
  return CHUNKKV_OK;
}

bool misaligned(const void *p) { return ((uintptr_t)p & 15) != 0; }

// Do the single-pass kernels score a group with this chunk size (no log-sum-exps, no token importance asked for)?
bool takes_one_pass(const chunkkv_problem *p, const Plan &pl, int chunk) {
  return !(p->flags & CHUNKKV_FLAG_TWO_PASS) && pl.n_periods_fit && single_pass_ok(p->dtype, p->head_dim, (p->n_q_heads / p->n_kv_heads) * p->window, chunk);
}

// Which accesses of a call over `layers` layers are streaming, by the bytes of K and V, and of K' and V'.
Stream streams(const chunkkv_problem *p, int64_t layers, int64_t most, int64_t most_out) {
  int64_t tokens = 0, kept = 0;
  for (int b = 0; b < p->batch; ++b) {
    tokens += p->seqlen[b];
    kept += p->n_keep[b] + p->window;
  }
  const int64_t token_bytes = 2 * layers * p->n_kv_heads * p->head_dim * elem_bytes(p->dtype);
  return kept * token_bytes > most_out ? Stream::kAll : tokens * token_bytes > most ? Stream::kLoads : Stream::kNone;
}

// How a pass of the two is cut into workgroups.
struct PassCut {
  int slots;            // workgroups on the chip at once
  int rounds, least_rounds;
  double half, tile_us;   // of units_per_workgroup; what a workgroup's tile costs
};
PassCut pass_cut(const chunkkv_problem *p, const ScoreGeom &g, int pass, bool short_launch) {
  const int f32 = p->dtype == CHUNKKV_F32 ? 1 : 0, blocks = g.tile_keys / 32, key_waves = 4 / g.wq < blocks ? 4 / g.wq : blocks;
  PassCut c;
  c.slots = score_workgroups_per_cu(p->dtype, p->head_dim, g.nqw, g.wq, pass) * kCUs;
  // Long launches: two rounds or more, and where memory is not what bounds them (65536 tokens, 8 layers, 256 rows with log-sum-exps in 3 whole
  // rounds 482 us a call, in 6.6 499).
  c.rounds = short_launch || g.wq * g.nqw >= 4 ? kTargetWorkgroups / c.slots : kFewRounds;
  c.least_rounds = short_launch ? -3 : 2;
  c.half = c.slots == kCUs ? 1.0 : kHalfRound[f32];
  c.tile_us = (double)(blocks / key_waves) * g.nqw * kBlockUs[f32];
  return c;
}

// Key tiles of a range of pass 0 for the sequences b0 .. b0 + nb - 1: what cuts ONE layer of them best.  A function of the sequences and
// the geometry, as the ranges of the single-pass kernel are, so that the row references, and with them every rounding of a score, do not
// depend on how many layers share a launch: the stack call and the per-layer calls agree bit for bit.  In a launch of many layers a
// workgroup walks several ranges, in whole rounds.  us of a call, so and with ranges chosen per launch, which saves statistics, their
// merge and sets of layers: 32 layers of 20873 tokens, 4 heads 358 / 338; 3 of 40842 193 / 180; 6 of 6343 63.6 / 60.4; one layer the same.
int stats_range_tiles(const chunkkv_problem *p, const ScoreGeom &g, int b0, int nb) {
  int64_t all = 0, tiles = 0;
  int most = 1;
  for (int b = 0; b < p->batch; ++b) all += ceil_div(p->seqlen[b], g.tile_keys);
  for (int b = b0; b < b0 + nb; ++b) {
    const int t = ceil_div(p->seqlen[b], g.tile_keys);
    tiles += t;
    most = t > most ? t : most;
  }
  int least = (int)((all * p->n_kv_heads + kTargetWorkgroups - 1) / kTargetWorkgroups);
  const bool merge = tiles * p->n_kv_heads <= kMergeTiles;
  if (merge && least < ceil_div(most, kMaxRanges)) least = ceil_div(most, kMaxRanges);
  const PassCut c = pass_cut(p, g, 0, merge);
  return units_per_workgroup(least, most, c.slots, c.least_rounds, c.rounds, c.half, kStartUs / c.tile_us, [&](int t) {
    int64_t n = 0;
    for (int b = b0; b < b0 + nb; ++b) n += ceil_div(ceil_div(p->seqlen[b], g.tile_keys), t);
    return n * p->n_kv_heads;
  }, [&](int t) { return merge ? kMergeUs / c.tile_us * ceil_div(ceil_div(most, t), 8) : 0.0; });
}

// Workspace layout; a pure function of (problem, n_layers, reuse).
int make_plan(const chunkkv_problem *p, int n_layers, int reuse, Plan *pl) {
  if (n_layers < 1 || reuse < 1) return CHUNKKV_ERR_SHAPE;
  const int rows = (p->n_q_heads / p->n_kv_heads) * p->window;
  if (!score_geometry(p->dtype, p->head_dim, rows, &pl->geom)) return CHUNKKV_ERR_UNSUPPORTED;
  pl->n_leaders = ceil_div(n_layers, reuse);
  pl->rows_pad = pl->geom.nqw * pl->geom.wq * 32;
  const int TK = pl->geom.tile_keys;
  pl->fuse_chunks = p->chunk <= kSuperKeys;
  int64_t tiles0 = 0;
  for (int b = 0; b < p->batch; ++b) {
    tiles0 += ceil_div(p->seqlen[b], TK);
  }
  // leader layers per launch set: about kTilesPerLaunch key tiles and what the pointer tables hold; sets are balanced in size
  int64_t per_leader = tiles0 * p->n_kv_heads;
  int gb = (int)((kTilesPerLaunch + per_leader - 1) / (per_leader > 0 ? per_leader : 1));
  if (gb < 1) gb = 1;
  if (gb > pl->n_leaders) gb = pl->n_leaders;
  if (gb > kMaxLayersPerLaunch) gb = kMaxLayersPerLaunch;
  const int nsets = ceil_div(pl->n_leaders, gb);
  pl->batch_leaders = ceil_div(pl->n_leaders, nsets);
  const int64_t heads = (int64_t)pl->batch_leaders * p->n_kv_heads;
  // Room for the pairs of pass 0: about kTargetWorkgroups ranges of every set of layers, the longest sequence's number of them for every
  // sequence.  That is room for the ranges of one layer at least (n times ceil(t / ceil(n x)) is no less than ceil(t / ceil(x)), and
  // a layer's ranges have ceil(x) tiles or more), and pass 0 is launched over as many layers at a time as fit.
  const int tiles_even = (int)((tiles0 * heads + kTargetWorkgroups - 1) / kTargetWorkgroups);
  int max_split0 = 1;
  for (int b = 0; b < p->batch; ++b) {
    const int s = ceil_div(ceil_div(p->seqlen[b], TK), tiles_even);
    if (s > max_split0) max_split0 = s;
  }
  // single-pass path
  pl->rows_pad_s = rows > 128 ? 256 : 128;
  pl->n_periods = 0;
  pl->max_split_s = 1;
  int room = 1;   // pairs of floats per row the workspace holds for the ranges' statistics (one float each, at most twice as many)
  for (int b = 0; b < p->batch; ++b) {
    const int np = ceil_div(p->seqlen[b], kSinglePeriodKeys);
    if (np > pl->n_periods) pl->n_periods = np;
  }
  // the kernels address E of one problem with 32-bit byte offsets
  pl->n_periods_fit = (int64_t)pl->n_periods * pl->rows_pad_s * 80 < (int64_t)1 << 32;
  pl->single_ok = pl->n_periods_fit && single_pass_ok(p->dtype, p->head_dim, rows, p->chunk);
  if (pl->single_ok) {
    // key ranges: single_periods_per_range() periods each, a function of the sequence alone
    for (int b = 0; b < p->batch; ++b) {
      const int np = ceil_div(p->seqlen[b], kSinglePeriodKeys);
      const int sp = ceil_div(np, single_periods_per_range(np)), per = ceil_div(np, 32) < 8 ? 8 : ceil_div(np, 32);
      if (sp > pl->max_split_s) pl->max_split_s = sp;
      if (ceil_div(np, per) > room) room = ceil_div(np, per);
    }
  }
  const size_t problems = (size_t)pl->n_leaders * p->batch * p->n_kv_heads;
  pl->part_bytes = problems * max_split0 * pl->rows_pad * sizeof(float2);
  if (pl->single_ok) {
    const size_t pb = problems * room * pl->rows_pad_s * sizeof(float2);
    pl->part_bytes = pb > pl->part_bytes ? pb : pl->part_bytes;
  }
  size_t off = 0;
  pl->off_part = off;   off += align256(pl->part_bytes);
  pl->off_refs = off;   off += align256(problems * pl->rows_pad * sizeof(float));
  pl->off_scores = off; off += align256(problems * (size_t)p->score_cap * sizeof(float));
  pl->off_seloff = off; off += align256(problems * (size_t)p->sel_cap * sizeof(int32_t));
  pl->off_imp = off;
  if (!pl->fuse_chunks) off += align256(problems * (size_t)p->score_cap * p->chunk * sizeof(float));
  pl->off_ebuf = pl->off_mper = off;
  if (pl->single_ok) {
    const size_t cells = problems * (size_t)pl->n_periods * pl->rows_pad_s;   // (period, row)
    pl->off_ebuf = off; off += align256(cells * (size_t)single_e_row_bytes(p->chunk));
    pl->off_mper = off; off += align256(cells * sizeof(float));
  }
  pl->total = off < 256 ? 256 : off;
  return CHUNKKV_OK;
}

void fill_seq(SeqTable *t, const chunkkv_problem *p, int b0, int nb) {
  memset(t, 0, sizeof(*t));
  for (int i = 0; i < nb; ++i) {
    t->seqlen[i] = p->seqlen[b0 + i];
    t->n_keep[i] = p->n_keep[b0 + i];
    t->kv_base[i] = p->kv_base[b0 + i];
    t->out_base[i] = p->out_base ? p->out_base[b0 + i] : 0;
  }
}

// Scores ng leader layers (pointer tables already gathered) for all sequences; leaders[i] is the index of the i-th, whose
// problems of the workspace and scores are its own, chunks[i] its chunk size.  Where they differ, pl and p are those of any of them,
// pl with the workspace of the one that needs most, and either all of them or none take one pass.
// lse == nullptr: the row normalisation is computed here; otherwise lse[i] is leader i's caller-supplied
// [B][Hq][w] array and only the importance pass runs.
int run_score(const chunkkv_problem *p, const Plan &pl, const void *const *q, const void *const *k,
              const float *const *lse, int ng, const int32_t *leaders, const int32_t *chunks, float *chunk_scores, float *token_imp,
              int64_t imp_pitch, Stream stream, char *ws, hipStream_t s) {
  const int TK = pl.geom.tile_keys;
  for (int b0 = 0; b0 < p->batch; b0 += kMaxBatchPerLaunch) {
    const int nb = p->batch - b0 < kMaxBatchPerLaunch ? p->batch - b0 : kMaxBatchPerLaunch;
    ScoreArgs a;
    memset(&a, 0, sizeof(a));
    for (int i = 0; i < ng; ++i) { a.q[i] = q[i]; a.k[i] = k[i]; }
    fill_seq(&a.seq, p, b0, nb);
    for (int i = 0; i < ng; ++i) { a.leader[i] = leaders[i]; a.chunk_of[i] = chunks[i]; }
    a.batch0 = b0; a.batch_total = p->batch;
    a.n_q_heads = p->n_q_heads; a.n_kv_heads = p->n_kv_heads; a.window = p->window; a.chunk = p->chunk;
    a.kv_stride_head = p->kv_stride_head; a.kv_stride_tok = p->kv_stride_tok;
    const float scale = p->softmax_scale > 0.f ? p->softmax_scale : 1.0f / sqrtf((float)p->head_dim);
    a.scale_log2e = scale * 1.4426950408889634f;
    a.rows_pad = pl.rows_pad;
    a.part_stats = (float2 *)(ws + pl.off_part);
    a.refs = (float *)(ws + pl.off_refs);
    a.chunk_scores = chunk_scores; a.score_cap = p->score_cap;
    a.token_imp = token_imp; a.imp_pitch = imp_pitch;
    a.fuse_chunks = pl.fuse_chunks;
    if (!pl.fuse_chunks && !token_imp) { a.token_imp = (float *)(ws + pl.off_imp); a.imp_pitch = (int64_t)p->score_cap * p->chunk; }
    for (int i = 1; i <= kMaxBatchPerLaunch; ++i) a.first_range[i] = INT32_MAX;
    // Super-tiles: smaller ones where a launch would leave CUs without a workgroup (512 tokens in fp32, 4 workgroups 12 us,
    // 16 of them 8); the sums of a chunk are the same bits whatever super-tile it lies in.
    a.super_keys = kSuperKeys;
    auto super_tiles = [&](int i, int z) { return ceil_div(a.seq.seqlen[i] - p->window, pl.fuse_chunks ? super_stride(a.super_keys, chunks[z]) : kSuperKeys); };
    int64_t units1 = 0;   // super-tiles of all sequences and layers
    for (;; a.super_keys /= 2) {
      units1 = 0;
      for (int z = 0; z < ng; ++z)
        for (int i = 0; i < nb; ++i) units1 += super_tiles(i, z);
      if (!pl.fuse_chunks || units1 * p->n_kv_heads >= 256 || a.super_keys / 2 < TK || a.super_keys <= 64) break;
    }
    int rc;
    if (lse) {
      a.use_lse = 1;
      for (int i = 0; i < ng; ++i) a.lse[i] = lse[i];
    } else if (takes_one_pass(p, pl, chunks[0]) && !token_imp) {
      // one pass over K: per-(chunk, row) sums and the references they are relative to; then the merge of the
      // range statistics and the weighted row sum in one small kernel
      a.n_periods = pl.n_periods;
      a.stream_k = stream != Stream::kNone;
      a.e_buf = ws + pl.off_ebuf;
      a.m_period = (float *)(ws + pl.off_mper);
      a.row_stats = (float *)(ws + pl.off_part);
      a.max_split = pl.max_split_s;
      for (int i = 0; i < ng; ++i) {
        const int bytes = single_e_row_bytes(chunks[i]);
        a.e_row_bytes = bytes > a.e_row_bytes ? bytes : a.e_row_bytes;
        a.mixed_chunks |= chunks[i] != chunks[0];
      }
      a.rows_pad = pl.rows_pad_s;
      int ranges = 0;
      for (int i = 0; i < nb; ++i) {
        const int np = ceil_div(a.seq.seqlen[i], kSinglePeriodKeys);
        a.first_range[i] = ranges;
        ranges += ceil_div(np, single_periods_per_range(np));
      }
      a.row_groups = pl.rows_pad_s == 256 && (int64_t)ranges * p->n_kv_heads * ng <= kRowSplitWorkgroups ? 2 : 1;
      { Timed t(kStats, s); rc = launch_score_single(p->dtype, a, dim3(ranges, p->n_kv_heads, ng * a.row_groups), s); }
      if (rc) return rc;
      if (units1 > 0) { Timed t(kColsum, s); rc = launch_single_scores(a, ng, nb, s); }
      if (rc) return rc;
      continue;
    }
    int64_t tiles = 0;
    int most = 1;   // tiles of the longest sequence
    for (int i = 0; i < nb; ++i) {
      const int t = ceil_div(a.seq.seqlen[i], TK);
      tiles += t;
      most = t > most ? t : most;
    }
    const bool short_launch = tiles * p->n_kv_heads * ng <= kMergeTiles;
    const PassCut cut0 = pass_cut(p, pl.geom, 0, short_launch), cut1 = pass_cut(p, pl.geom, 1, short_launch);
    double start1 = kStartUs / cut1.tile_us;
    // Neighbours are the heads of one range in short launches (one layer of 23344 tokens, 32 rows 37.9 us, the ranges of one head
    // 43.0), the ranges of one head in longer ones (packed, 32 layers of 3812 and 12202 tokens, 8 heads of 16 rows 332, heads 359).
    a.heads_first = short_launch;
    const int per_range = short_launch ? 1 : p->n_kv_heads;   // entries of the grid's x or y for one range
    auto grid = [&](int64_t n, int layers) { return short_launch ? dim3(p->n_kv_heads, (uint32_t)n, layers) : dim3((uint32_t)(n * p->n_kv_heads), 1, layers); };
    if (!lse) {
      a.range_tiles = stats_range_tiles(p, pl.geom, b0, nb);
      a.max_split = ceil_div(most, a.range_tiles);
      a.batch_slice = nb;
      // layers whose pairs fit the workspace
      const int64_t fit = (int64_t)(pl.part_bytes / sizeof(float2)) / ((int64_t)nb * p->n_kv_heads * a.max_split * a.rows_pad);
      if (fit < 1) return CHUNKKV_ERR_WORKSPACE;
      const int sets = (int)((ng + fit - 1) / fit), per_set = ceil_div(ng, sets);
      a.merge_stats = short_launch && sets == 1;   // else a kernel between the passes does, set by set
      for (int z0 = 0; z0 < ng; z0 += per_set) {
        const int nz = ng - z0 < per_set ? ng - z0 : per_set;
        ScoreArgs set = a;
        for (int i = 0; i < nz; ++i) { set.q[i] = a.q[z0 + i]; set.k[i] = a.k[z0 + i]; set.leader[i] = a.leader[z0 + i]; }
        auto wgs = [&](int n) {   // of n ranges
          int64_t all = 0;
          for (int i = 0; i < nb; ++i) all += ceil_div(ceil_div(ceil_div(a.seq.seqlen[i], TK), a.range_tiles), n);
          return all;
        };
        const int least = (int)((tiles * p->n_kv_heads * nz + kTargetWorkgroups - 1) / kTargetWorkgroups);
        set.ranges_per_wg = units_per_workgroup(ceil_div(least, a.range_tiles), a.max_split, cut0.slots, cut0.least_rounds, cut0.rounds, cut0.half,
                                                kStartUs / cut0.tile_us / a.range_tiles, [&](int n) { return wgs(n) * p->n_kv_heads * nz; }, [](int) { return 0.0; });
        for (int i = 0, n = 0; i < nb; ++i) {
          n += ceil_div(ceil_div(ceil_div(a.seq.seqlen[i], TK), a.range_tiles), set.ranges_per_wg);
          set.first_range[i + 1] = n * per_range;
        }
        { Timed t(kStats, s); rc = launch_score_pass(0, p->dtype, p->head_dim, pl.geom, set, grid(wgs(set.ranges_per_wg), nz), s); }
        if (rc) return rc;
        if (!a.merge_stats) {
          { Timed t(kCombine, s); rc = launch_stats_combine(set, nz, nb, TK, s); }
          if (rc) return rc;
        }
      }
      if (a.merge_stats) start1 += kMergeUs / cut1.tile_us * ceil_div(a.max_split, 8);
    }
    if (units1 == 0) continue;   // no prefix: nothing to sum
    // super-tiles of a sequence: those of the layer with most, which differ where chunk sizes do
    int most1 = 1, seq_units[kMaxBatchPerLaunch];
    for (int i = 0; i < nb; ++i) {
      seq_units[i] = 0;
      for (int z = 0; z < ng; ++z) seq_units[i] = super_tiles(i, z) > seq_units[i] ? super_tiles(i, z) : seq_units[i];
      most1 = seq_units[i] > most1 ? seq_units[i] : most1;
    }
    const int64_t all1 = units1 * p->n_kv_heads;
    auto ranges1 = [&](int t) {
      int64_t n = 0;
      for (int i = 0; i < nb; ++i) n += ceil_div(seq_units[i], t);
      return n;
    };
    a.tiles_per_wg = units_per_workgroup((int)((all1 + kTargetWorkgroups - 1) / kTargetWorkgroups), most1, cut1.slots, cut1.least_rounds, cut1.rounds, cut1.half, start1 * TK / a.super_keys,
                                         [&](int t) { return ranges1(t) * p->n_kv_heads * ng; }, [](int) { return 0.0; });
    for (int i = 0, n = 0; i < nb; ++i) {
      n += ceil_div(seq_units[i], a.tiles_per_wg);
      a.first_range[i + 1] = n * per_range;
    }
    { Timed t(kColsum, s); rc = launch_score_pass(1, p->dtype, p->head_dim, pl.geom, a, grid(ranges1(a.tiles_per_wg), ng), s); }
    if (rc) return rc;
    if (!pl.fuse_chunks) {
      { Timed t(kChunkSums, s); rc = launch_chunk_sums(a, ng, nb, s); }
      if (rc) return rc;
    }
  }
  return CHUNKKV_OK;
}

int run_topk(const chunkkv_problem *p, const int32_t *chunks, const float *chunk_scores, int group0, int n_groups, int32_t *sel_chunk,
             int32_t *sel_len, int32_t *sel_count, int32_t *sel_off, hipStream_t s) {
  for (int b0 = 0; b0 < p->batch; b0 += kMaxBatchPerLaunch) {
    const int nb = p->batch - b0 < kMaxBatchPerLaunch ? p->batch - b0 : kMaxBatchPerLaunch;
    TopkArgs a;
    memset(&a, 0, sizeof(a));
    fill_seq(&a.seq, p, b0, nb);
    a.group0 = group0;
    for (int i = 0; i < n_groups; ++i) a.chunk_of[i] = chunks[i];
    a.batch0 = b0; a.batch_total = p->batch; a.n_kv_heads = p->n_kv_heads; a.window = p->window;
    a.chunk_scores = chunk_scores; a.score_cap = p->score_cap; a.sel_cap = p->sel_cap;
    a.sel_chunk = sel_chunk; a.sel_len = sel_len; a.sel_count = sel_count; a.sel_off = sel_off;
    a.whole_chunks = (p->flags & CHUNKKV_FLAG_WHOLE_CHUNKS) ? 1 : 0;
    int rc;
    { Timed t(kTopk, s); rc = launch_topk(a, n_groups, nb, s); }
    if (rc) return rc;
  }
  return CHUNKKV_OK;
}

// Arguments of a gather: layers [l0, l0 + nl) and sequences [b0, b0 + nb), of the pointers' first layer on.  chunks[i]: chunk
// size of the i-th reuse group from that of layer l_begin on.
void fill_compact(CompactArgs *a, const chunkkv_problem *p, const int32_t *chunks, int l_begin, int l0, int nl, int b0, int nb, int reuse, Stream stream,
                  const void *const *k, const void *const *v, void *const *k_out, void *const *v_out, const int32_t *sel_chunk,
                  const int32_t *sel_len, const int32_t *sel_count, const int32_t *sel_off) {
  memset(a, 0, sizeof(*a));
  for (int i = 0; i < nl; ++i) {
    a->k[i] = k[l0 + i]; a->v[i] = v[l0 + i]; a->k_out[i] = k_out[l0 + i]; a->v_out[i] = v_out[l0 + i];
    a->chunk_of[i] = chunks[(l0 + i) / reuse - l_begin / reuse];
  }
  fill_seq(&a->seq, p, b0, nb);
  a->layer0 = l0; a->reuse = reuse; a->batch0 = b0; a->batch_total = p->batch;
  a->n_kv_heads = p->n_kv_heads; a->window = p->window; a->elem_bytes = elem_bytes(p->dtype);
  a->kv_stride_head = p->kv_stride_head; a->kv_stride_tok = p->kv_stride_tok;
  a->out_stride_head = p->out_stride_head; a->out_stride_tok = p->out_stride_tok;
  a->sel_chunk = sel_chunk; a->sel_len = sel_len; a->sel_count = sel_count; a->sel_off = sel_off;
  a->sel_cap = p->sel_cap;
  a->whole_chunks = (p->flags & CHUNKKV_FLAG_WHOLE_CHUNKS) ? 1 : 0;
  a->stream = stream;
}

int run_compact(const chunkkv_problem *p, const int32_t *chunks, int l_begin, int n_layers, int reuse, Stream stream, const void *const *k, const void *const *v,
                void *const *k_out, void *const *v_out, const int32_t *sel_chunk, const int32_t *sel_len,
                const int32_t *sel_count, const int32_t *sel_off, hipStream_t s) {
  const int row_bytes = p->head_dim * elem_bytes(p->dtype);
  for (int l0 = l_begin; l0 < n_layers; l0 += kMaxLayersPerLaunch) {
    const int nl = n_layers - l0 < kMaxLayersPerLaunch ? n_layers - l0 : kMaxLayersPerLaunch;
    for (int b0 = 0; b0 < p->batch; b0 += kMaxBatchPerLaunch) {
      const int nb = p->batch - b0 < kMaxBatchPerLaunch ? p->batch - b0 : kMaxBatchPerLaunch;
      CompactArgs a;
      fill_compact(&a, p, chunks, l_begin, l0, nl, b0, nb, reuse, stream, k, v, k_out, v_out, sel_chunk, sel_len, sel_count, sel_off);
      int rc;
      { Timed t(kCompact, s); rc = launch_compact(row_bytes, a, nl, nb, s); }
      if (rc) return rc;
    }
  }
  return CHUNKKV_OK;
}

// Selection of the reuse groups from that of layer l_begin on and gather of layers [l_begin, l_end) with it: in one launch
// where one can carry them and that suits the problem.
int run_selection(const chunkkv_problem *p, const int32_t *chunks, const float *chunk_scores, int group0, int n_groups, int l_begin, int l_end,
                  int reuse, Stream stream, const void *const *k, const void *const *v, void *const *k_out, void *const *v_out, int32_t *sel_chunk,
                  int32_t *sel_len, int32_t *sel_count, int32_t *sel_off, hipStream_t s) {
  const int row_bytes = p->head_dim * elem_bytes(p->dtype), nl = l_end - l_begin;
  int rc;
  if (nl <= kMaxLayersPerLaunch && p->batch <= kMaxBatchPerLaunch) {
    CompactArgs a;
    fill_compact(&a, p, chunks, l_begin, l_begin, nl, 0, p->batch, reuse, stream, k, v, k_out, v_out, sel_chunk, sel_len, sel_count, sel_off);
    const SelectInGather how = select_in_gather(a, nl, p->batch);
    if (how.yes) {
      Timed t(kCompact, s);
      return launch_select_compact(row_bytes, a, nl, p->batch, chunk_scores, p->score_cap, how, s);
    }
    rc = run_topk(p, chunks, chunk_scores, group0, n_groups, sel_chunk, sel_len, sel_count, sel_off, s);
    if (rc) return rc;
    Timed t(kCompact, s);
    return launch_compact(row_bytes, a, nl, p->batch, s);
  }
  rc = run_topk(p, chunks, chunk_scores, group0, n_groups, sel_chunk, sel_len, sel_count, sel_off, s);
  if (rc) return rc;
  return run_compact(p, chunks, l_begin, l_end, reuse, stream, k, v, k_out, v_out, sel_chunk, sel_len, sel_count, sel_off, s);
}

}  // namespace
}  // namespace ckv

using namespace ckv;

// Runs of consecutive reuse groups with one chunk size; fn(problem with that chunk, first group, end group).
template <typename F>
static int for_chunk_runs(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse, const int32_t *chunk_per_group,
                          F fn) {
  if (!prob) return CHUNKKV_ERR_NULL;
  if (!chunk_per_group) return CHUNKKV_ERR_NULL;
  if (n_layers < 1 || reuse < 1) return CHUNKKV_ERR_SHAPE;
  const int n_groups = ceil_div(n_layers, reuse);
  for (int g0 = 0; g0 < n_groups;) {
    int g1 = g0 + 1;
    while (g1 < n_groups && chunk_per_group[g1] == chunk_per_group[g0]) ++g1;
    chunkkv_problem run = *prob;
    run.chunk = chunk_per_group[g0];
    int rc = check_problem(&run, true);
    if (rc) return rc;
    rc = fn(run, g0, g1);
    if (rc) return rc;
    g0 = g1;
  }
  return CHUNKKV_OK;
}

extern "C" {

const char *chunkkv_status_string(int status) {
  switch (status) {
    case CHUNKKV_OK: return "ok";
    case CHUNKKV_ERR_NULL: return "a required pointer is NULL";
    case CHUNKKV_ERR_SHAPE: return "inconsistent shape, stride, alignment, budget or capacity";
    case CHUNKKV_ERR_UNSUPPORTED: return "unsupported dtype, head_dim or window rows per kv-head";
    case CHUNKKV_ERR_WORKSPACE: return "workspace too small or NULL";
    case CHUNKKV_ERR_LAUNCH: return "HIP launch failed";
    default: return "unknown status";
  }
}

size_t chunkkv_workspace_bytes(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse) {
  if (check_problem(prob, false) != CHUNKKV_OK) return 0;
  Plan pl;
  if (make_plan(prob, n_layers, reuse, &pl) != CHUNKKV_OK) return 0;
  return pl.total;
}

static int score_entry(const chunkkv_problem *prob, const void *q_obs, const void *k, const float *lse, bool with_lse,
                       float *chunk_scores, float *token_importance, void *workspace, size_t workspace_bytes,
                       void *stream) {
  int rc = check_problem(prob, false);
  if (rc) return rc;
  if (!q_obs || !k || !chunk_scores || (with_lse && !lse)) return CHUNKKV_ERR_NULL;
  if (misaligned(q_obs) || misaligned(k)) return CHUNKKV_ERR_SHAPE;
  Plan pl;
  rc = make_plan(prob, 1, 1, &pl);
  if (rc) return rc;
  if (!workspace || workspace_bytes < pl.total) return CHUNKKV_ERR_WORKSPACE;
  const int32_t leader = 0;
  return run_score(prob, pl, &q_obs, &k, with_lse ? &lse : nullptr, 1, &leader, &prob->chunk, chunk_scores, token_importance,
                   (int64_t)prob->score_cap * prob->chunk, streams(prob, 1, kStreamBytes, kStreamOutBytes), (char *)workspace, (hipStream_t)stream);
}

int chunkkv_score(const chunkkv_problem *prob, const void *q_obs, const void *k, float *chunk_scores,
                  float *token_importance, void *workspace, size_t workspace_bytes, void *stream) {
  return score_entry(prob, q_obs, k, nullptr, false, chunk_scores, token_importance, workspace, workspace_bytes, stream);
}

int chunkkv_score_lse(const chunkkv_problem *prob, const void *q_obs, const void *k, const float *lse,
                      float *chunk_scores, float *token_importance, void *workspace, size_t workspace_bytes,
                      void *stream) {
  return score_entry(prob, q_obs, k, lse, true, chunk_scores, token_importance, workspace, workspace_bytes, stream);
}

int chunkkv_chunk_topk(const chunkkv_problem *prob, const float *chunk_scores, int32_t *sel_chunk,
                       int32_t *sel_len, int32_t *sel_count, void *workspace, size_t workspace_bytes,
                       void *stream) {
  (void)workspace; (void)workspace_bytes;  // the selection kernel keeps its state in LDS
  int rc = check_problem(prob, false);
  if (rc) return rc;
  if (!chunk_scores || !sel_chunk || !sel_len || !sel_count) return CHUNKKV_ERR_NULL;
  return run_topk(prob, &prob->chunk, chunk_scores, 0, 1, sel_chunk, sel_len, sel_count, nullptr, (hipStream_t)stream);
}

int chunkkv_compact(const chunkkv_problem *prob, const void *k, const void *v, const int32_t *sel_chunk,
                    const int32_t *sel_len, const int32_t *sel_count, void *k_out, void *v_out, void *stream) {
  int rc = check_problem(prob, true);
  if (rc) return rc;
  if (!k || !v || !sel_chunk || !sel_len || !sel_count || !k_out || !v_out) return CHUNKKV_ERR_NULL;
  if (misaligned(k) || misaligned(v) || misaligned(k_out) || misaligned(v_out)) return CHUNKKV_ERR_SHAPE;
  return run_compact(prob, &prob->chunk, 0, 1, 1, streams(prob, 1, kStreamBytes, kStreamOutBytes), &k, &v, &k_out, &v_out, sel_chunk, sel_len, sel_count, nullptr,
                     (hipStream_t)stream);
}

static int check_stack_pointers(int32_t n_layers, int32_t reuse, const void *const *q_obs, const void *const *k,
                                const void *const *v, const float *const *lse, bool with_lse, void *const *k_out,
                                void *const *v_out, const int32_t *sel_chunk, const int32_t *sel_len,
                                const int32_t *sel_count) {
  if (n_layers < 1 || reuse < 1) return CHUNKKV_ERR_SHAPE;
  if (!q_obs || !k || !v || !k_out || !v_out || !sel_chunk || !sel_len || !sel_count) return CHUNKKV_ERR_NULL;
  if (with_lse && !lse) return CHUNKKV_ERR_NULL;
  for (int l = 0; l < n_layers; ++l) {
    if (!k[l] || !v[l] || !k_out[l] || !v_out[l]) return CHUNKKV_ERR_NULL;
    if (l % reuse == 0 && !q_obs[l]) return CHUNKKV_ERR_NULL;
    if (with_lse && l % reuse == 0 && !lse[l]) return CHUNKKV_ERR_NULL;
    if (misaligned(k[l]) || misaligned(v[l]) || misaligned(k_out[l]) || misaligned(v_out[l])) return CHUNKKV_ERR_SHAPE;
    if (l % reuse == 0 && misaligned(q_obs[l])) return CHUNKKV_ERR_SHAPE;
  }
  return CHUNKKV_OK;
}

// Algorithm 2 over the reuse groups [g_begin, g_end) of a stack of n_layers layers: leader layers (l % reuse == 0)
// are scored and selected, then every layer of these groups is gathered with the selection of its group.
// `pl` is the plan of the whole stack for prob->chunk.  Everything is enqueued on `s`.
static int stack_groups(const chunkkv_problem *prob, const Plan &pl, int g_begin, int g_end, int32_t n_layers,
                        int32_t reuse, const void *const *q_obs, const void *const *k, const void *const *v,
                        const float *const *lse, bool with_lse, void *const *k_out, void *const *v_out,
                        int32_t *sel_chunk, int32_t *sel_len, int32_t *sel_count, char *ws, hipStream_t s) {
  float *scores = (float *)(ws + pl.off_scores);
  int32_t *sel_off = (int32_t *)(ws + pl.off_seloff);
  const Stream stream = streams(prob, n_layers, kStreamBytes, kStreamOutBytes);
  for (int g0 = g_begin; g0 < g_end; g0 += pl.batch_leaders) {
    const int ng = g_end - g0 < pl.batch_leaders ? g_end - g0 : pl.batch_leaders;
    const void *qs[kMaxLayersPerLaunch], *ks[kMaxLayersPerLaunch];
    const float *ls[kMaxLayersPerLaunch];
    int32_t leaders[kMaxLayersPerLaunch], chunks[kMaxLayersPerLaunch];
    for (int i = 0; i < ng; ++i) {
      qs[i] = q_obs[(g0 + i) * reuse]; ks[i] = k[(g0 + i) * reuse];
      ls[i] = with_lse ? lse[(g0 + i) * reuse] : nullptr;
      leaders[i] = g0 + i; chunks[i] = prob->chunk;
    }
    int rc = run_score(prob, pl, qs, ks, with_lse ? ls : nullptr, ng, leaders, chunks, scores, nullptr, 0, stream, ws, s);
    if (rc) return rc;
    const int l_begin = g0 * reuse, l_end = (g0 + ng) * reuse < n_layers ? (g0 + ng) * reuse : n_layers;
    rc = run_selection(prob, chunks, scores, g0, ng, l_begin, l_end, reuse, stream, k, v, k_out, v_out, sel_chunk, sel_len, sel_count, sel_off, s);
    if (rc) return rc;
  }
  return CHUNKKV_OK;
}

static int stack_entry(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse, const void *const *q_obs,
                       const void *const *k, const void *const *v, const float *const *lse, bool with_lse,
                       void *const *k_out, void *const *v_out, int32_t *sel_chunk, int32_t *sel_len,
                       int32_t *sel_count, void *workspace, size_t workspace_bytes, void *stream) {
  int rc = check_problem(prob, true);
  if (rc) return rc;
  rc = check_stack_pointers(n_layers, reuse, q_obs, k, v, lse, with_lse, k_out, v_out, sel_chunk, sel_len, sel_count);
  if (rc) return rc;
  Plan pl;
  rc = make_plan(prob, n_layers, reuse, &pl);
  if (rc) return rc;
  if (!workspace || workspace_bytes < pl.total) return CHUNKKV_ERR_WORKSPACE;
  return stack_groups(prob, pl, 0, pl.n_leaders, n_layers, reuse, q_obs, k, v, lse, with_lse, k_out, v_out, sel_chunk,
                      sel_len, sel_count, (char *)workspace, (hipStream_t)stream);
}

}  // extern "C"

// A stack whose groups' chunk sizes differ, each kernel launched over all groups it can take at once: the single-pass
// kernels once for the chunk sizes they are compiled for, pass 0 and pass 1 once for all other groups, selection and gather once
// for all.  One run of groups after the other is a chain of four or five launches that do not fill the chip, per run: eight
// sizes over 16 layers of 12345 tokens 171 us, with a single-pass launch and a reduction per size 199; 32 groups of seven sizes and
// 400 tokens 37, 67.  `pl` is the plan of the chunk size that needs the most
// workspace; the others fit its regions.
static int stack_mixed(const chunkkv_problem *prob, const Plan &pl, int32_t n_layers, int32_t reuse, const int32_t *chunks,
                       const void *const *q_obs, const void *const *k, const void *const *v, const float *const *lse,
                       void *const *k_out, void *const *v_out, int32_t *sel_chunk, int32_t *sel_len, int32_t *sel_count,
                       char *ws, hipStream_t s) {
  const int n_groups = pl.n_leaders;
  float *scores = (float *)(ws + pl.off_scores);
  int32_t *sel_off = (int32_t *)(ws + pl.off_seloff);
  const Stream stream = streams(prob, n_layers, kStreamBytes, kStreamOutBytes);
  bool done[kMaxLayersPerLaunch] = {};
  for (int first = 0; first < n_groups; ++first) {
    if (done[first]) continue;
    chunkkv_problem run = *prob;
    run.chunk = chunks[first];
    Plan rp;
    int rc = make_plan(&run, n_layers, reuse, &rp);
    if (rc) return rc;
    rp.part_bytes = pl.part_bytes; rp.off_part = pl.off_part; rp.off_refs = pl.off_refs; rp.off_scores = pl.off_scores; rp.off_seloff = pl.off_seloff;
    rp.off_imp = pl.off_imp; rp.off_ebuf = pl.off_ebuf; rp.off_mper = pl.off_mper;
    auto one_pass = [&](int c) { return !lse && takes_one_pass(prob, pl, c); };
    const void *qs[kMaxLayersPerLaunch], *ks[kMaxLayersPerLaunch];
    const float *ls[kMaxLayersPerLaunch];
    int32_t leaders[kMaxLayersPerLaunch], cs[kMaxLayersPerLaunch];
    int ng = 0;
    for (int g = first; g < n_groups; ++g) {
      if (done[g] || one_pass(chunks[first]) != one_pass(chunks[g])) continue;
      done[g] = true;
      qs[ng] = q_obs[g * reuse]; ks[ng] = k[g * reuse]; ls[ng] = lse ? lse[g * reuse] : nullptr;
      leaders[ng] = g; cs[ng] = chunks[g];
      ++ng;
    }
    rc = run_score(&run, rp, qs, ks, lse ? ls : nullptr, ng, leaders, cs, scores, nullptr, 0, stream, ws, s);
    if (rc) return rc;
  }
  return run_selection(prob, chunks, scores, 0, n_groups, 0, n_layers, reuse, stream, k, v, k_out, v_out, sel_chunk, sel_len, sel_count, sel_off, s);
}

extern "C" {

size_t chunkkv_workspace_bytes_hybrid(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse,
                                      const int32_t *chunk_per_group) {
  size_t need = 0;
  const int rc = for_chunk_runs(prob, n_layers, reuse, chunk_per_group, [&](const chunkkv_problem &run, int, int) {
    Plan pl;
    const int r = make_plan(&run, n_layers, reuse, &pl);
    if (r) return r;
    need = pl.total > need ? pl.total : need;
    return (int)CHUNKKV_OK;
  });
  return rc ? 0 : need;
}

int chunkkv_compress_stack_hybrid(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse,
                                  const int32_t *chunk_per_group, const void *const *q_obs, const void *const *k,
                                  const void *const *v, const float *const *lse, void *const *k_out,
                                  void *const *v_out, int32_t *sel_chunk, int32_t *sel_len, int32_t *sel_count,
                                  void *workspace, size_t workspace_bytes, void *stream) {
  // everything is checked for every run before the first launch
  const size_t need = chunkkv_workspace_bytes_hybrid(prob, n_layers, reuse, chunk_per_group);
  if (need == 0) {
    const int rc = for_chunk_runs(prob, n_layers, reuse, chunk_per_group, [&](const chunkkv_problem &run, int, int) {
      Plan pl;
      return make_plan(&run, n_layers, reuse, &pl);
    });
    return rc ? rc : CHUNKKV_ERR_SHAPE;
  }
  const bool with_lse = lse != nullptr;
  int rc = check_stack_pointers(n_layers, reuse, q_obs, k, v, lse, with_lse, k_out, v_out, sel_chunk, sel_len, sel_count);
  if (rc) return rc;
  if (!workspace || workspace_bytes < need) return CHUNKKV_ERR_WORKSPACE;
  // Groups of different sizes together, if a launch can carry them all and every size is formed in the importance pass; one
  // size (one run) is the plain stack call.
  const int n_groups = ceil_div(n_layers, reuse);
  bool together = n_groups <= kMaxLayersPerLaunch, differ = false;
  Plan most;
  most.total = 0;
  for (int g = 0; together && g < n_groups; ++g) {
    together = chunk_per_group[g] <= kSuperKeys;
    differ |= chunk_per_group[g] != chunk_per_group[0];
    chunkkv_problem run = *prob;
    run.chunk = chunk_per_group[g];
    Plan pl;
    if ((rc = make_plan(&run, n_layers, reuse, &pl))) return rc;
    if (pl.total > most.total) most = pl;
  }
  if (together && differ)
    return stack_mixed(prob, most, n_layers, reuse, chunk_per_group, q_obs, k, v, lse, k_out, v_out, sel_chunk, sel_len,
                       sel_count, (char *)workspace, (hipStream_t)stream);
  return for_chunk_runs(prob, n_layers, reuse, chunk_per_group, [&](const chunkkv_problem &run, int g0, int g1) {
    Plan pl;
    const int r = make_plan(&run, n_layers, reuse, &pl);
    if (r) return r;
    return stack_groups(&run, pl, g0, g1, n_layers, reuse, q_obs, k, v, lse, with_lse, k_out, v_out, sel_chunk, sel_len,
                        sel_count, (char *)workspace, (hipStream_t)stream);
  });
}

int chunkkv_compress_stack(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse, const void *const *q_obs,
                           const void *const *k, const void *const *v, void *const *k_out, void *const *v_out,
                           int32_t *sel_chunk, int32_t *sel_len, int32_t *sel_count, void *workspace,
                           size_t workspace_bytes, void *stream) {
  return stack_entry(prob, n_layers, reuse, q_obs, k, v, nullptr, false, k_out, v_out, sel_chunk, sel_len, sel_count,
                     workspace, workspace_bytes, stream);
}

int chunkkv_compress_stack_lse(const chunkkv_problem *prob, int32_t n_layers, int32_t reuse, const void *const *q_obs,
                               const void *const *k, const void *const *v, const float *const *lse,
                               void *const *k_out, void *const *v_out, int32_t *sel_chunk, int32_t *sel_len,
                               int32_t *sel_count, void *workspace, size_t workspace_bytes, void *stream) {
  return stack_entry(prob, n_layers, reuse, q_obs, k, v, lse, true, k_out, v_out, sel_chunk, sel_len, sel_count,
                     workspace, workspace_bytes, stream);
}

int chunkkv_compress_layer(const chunkkv_problem *prob, int32_t layer, int32_t reuse, const void *q_obs,
                           const float *lse, const void *k, const void *v, void *k_out, void *v_out,
                           int32_t *sel_chunk, int32_t *sel_len, int32_t *sel_count, void *workspace,
                           size_t workspace_bytes, void *stream) {
  int rc = check_problem(prob, true);
  if (rc) return rc;
  if (layer < 0 || reuse < 1) return CHUNKKV_ERR_SHAPE;
  const bool leader = layer % reuse == 0;
  if (!k || !v || !k_out || !v_out || !sel_chunk || !sel_len || !sel_count || (leader && !q_obs)) return CHUNKKV_ERR_NULL;
  if (misaligned(k) || misaligned(v) || misaligned(k_out) || misaligned(v_out) || (leader && misaligned(q_obs)))
    return CHUNKKV_ERR_SHAPE;
  Plan pl;
  rc = make_plan(prob, 1, 1, &pl);
  if (rc) return rc;
  if (!workspace || workspace_bytes < pl.total) return CHUNKKV_ERR_WORKSPACE;
  char *ws = (char *)workspace;
  hipStream_t s = (hipStream_t)stream;
  // the kernels see this layer's group as group 0 of arrays that start at the group's rows
  const int64_t row0 = (int64_t)(layer / reuse) * prob->batch * prob->n_kv_heads;
  const Stream how = streams(prob, 1, kStreamLayerBytes, kStreamOutLayerBytes);
  int32_t *sc = sel_chunk + row0 * prob->sel_cap, *sl = sel_len + row0 * prob->sel_cap, *cnt = sel_count + row0;
  if (leader) {
    float *scores = (float *)(ws + pl.off_scores);
    const int32_t leader0 = 0;
    rc = run_score(prob, pl, &q_obs, &k, lse ? &lse : nullptr, 1, &leader0, &prob->chunk, scores, nullptr, 0, how, ws, s);
    if (rc) return rc;
    return run_selection(prob, &prob->chunk, scores, 0, 1, 0, 1, 1, how, &k, &v, &k_out, &v_out, sc, sl, cnt, nullptr, s);
  }
  return run_compact(prob, &prob->chunk, 0, 1, 1, how, &k, &v, &k_out, &v_out, sc, sl, cnt, nullptr, s);
}

int chunkkv_jaccard(const chunkkv_problem *prob, int32_t n_groups, const int32_t *sel_chunk, const int32_t *sel_len,
                    const int32_t *sel_count, float *jaccard, void *stream) {
  int rc = check_problem(prob, false);
  if (rc) return rc;
  if (n_groups < 2) return CHUNKKV_ERR_SHAPE;
  if (!sel_chunk || !sel_len || !sel_count || !jaccard) return CHUNKKV_ERR_NULL;
  return launch_jaccard(sel_chunk, sel_len, sel_count, prob->sel_cap, prob->chunk, prob->batch * prob->n_kv_heads,
                        n_groups - 1, jaccard, (hipStream_t)stream);
}

size_t chunkkv_decode_workspace_bytes(const chunkkv_problem *prob, int32_t compacted) {
  DecodePlan pl;
  if (check_problem(prob, compacted != 0)) return 0;
  decode_plan(prob, compacted != 0, &pl);
  return pl.total;
}

int chunkkv_decode_attention(const chunkkv_problem *prob, int32_t compacted, const int32_t *kv_len, const void *q,
                             const void *k, const void *v, float *out, float *lse, void *workspace,
                             size_t workspace_bytes, void *stream) {
  int rc = check_problem(prob, compacted != 0);
  if (rc) return rc;
  if (!q || !k || !v || !out) return CHUNKKV_ERR_NULL;
  if (misaligned(q) || misaligned(k) || misaligned(v)) return CHUNKKV_ERR_SHAPE;
  DecodePlan pl;
  decode_plan(prob, compacted != 0, &pl);
  if (!workspace || workspace_bytes < pl.total) return CHUNKKV_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const float scale = prob->softmax_scale > 0.f ? prob->softmax_scale : 1.0f / sqrtf((float)prob->head_dim);
  for (int b0 = 0; b0 < prob->batch; b0 += kMaxBatchPerLaunch) {
    const int nb = prob->batch - b0 < kMaxBatchPerLaunch ? prob->batch - b0 : kMaxBatchPerLaunch;
    DecodeArgs a{};
    a.q = q; a.k = k; a.v = v; a.out = out; a.lse = lse; a.kv_len = kv_len;
    a.part_ml = (float2 *)((char *)workspace + pl.off_ml);
    a.part_o = (float *)((char *)workspace + pl.off_o);
    for (int i = 0; i < nb; ++i) {
      a.n_tok[i] = compacted ? prob->n_keep[b0 + i] + prob->window : prob->seqlen[b0 + i];
      a.base[i] = compacted ? prob->out_base[b0 + i] : prob->kv_base[b0 + i];
    }
    a.stride_head = compacted ? prob->out_stride_head : prob->kv_stride_head;
    a.stride_tok = compacted ? prob->out_stride_tok : prob->kv_stride_tok;
    a.batch0 = b0; a.n_q_heads = prob->n_q_heads; a.n_kv_heads = prob->n_kv_heads; a.group = prob->n_q_heads / prob->n_kv_heads;
    a.scale_log2e = scale * 1.4426950408889634f;
    decode_cut(prob, compacted != 0, b0, nb, &a.cut);
    const bool mfma = decode_on_matrix_cores(prob, compacted != 0);
    { Timed t(kDecode, s); rc = launch_decode(prob->dtype, prob->head_dim, mfma, a, nb, s); }
    if (rc) return rc;
  }
  return CHUNKKV_OK;
}

int chunkkv_decode_attention_static(const chunkkv_problem *prob, int32_t compacted, const int32_t *kv_len,
                                    const void *q, const void *k, const void *v, float *out, float *lse,
                                    void *stream) {
  // the size check comes first: a problem that does not fit is refused before anything else happens
  int rc = check_problem(prob, compacted != 0);
  if (rc) return rc;
  DecodePlan pl;
  decode_plan(prob, compacted != 0, &pl);
  if (pl.total > kStaticScratchBytes) return CHUNKKV_ERR_WORKSPACE;
  void *ws = nullptr;
  if ((rc = static_scratch(&ws))) return rc;
  // every partial result the merge kernel reads is written by the range kernel of the same call, so nothing
  // in the array has to be cleared between calls
  return chunkkv_decode_attention(prob, compacted, kv_len, q, k, v, out, lse, ws, pl.total, stream);
}

// Workspace of chunkkv_quality_metrics: the decode workspace (the larger of the two caches' needs), one decode
// output, two log-sum-exp arrays and the block partials of the two absolute masses.
namespace {
struct QualityPlan {
  int blocks_full, blocks_kept;
  size_t off_decode, off_out, off_lse_full, off_lse_kept, off_part_full, off_part_kept, total, decode_bytes;
};
int quality_plan(const chunkkv_problem *p, QualityPlan *q) {
  DecodePlan df, dk;
  decode_plan(p, false, &df);
  decode_plan(p, true, &dk);
  int full_max = 0, kept_max = 0;
  for (int b = 0; b < p->batch; ++b) {
    full_max = p->seqlen[b] > full_max ? p->seqlen[b] : full_max;
    kept_max = p->n_keep[b] + p->window > kept_max ? p->n_keep[b] + p->window : kept_max;
  }
  q->blocks_full = abs_sum_blocks(full_max);
  q->blocks_kept = abs_sum_blocks(kept_max);
  const size_t heads = (size_t)p->batch * p->n_q_heads, kvh = (size_t)p->batch * p->n_kv_heads;
  q->decode_bytes = df.total > dk.total ? df.total : dk.total;
  size_t off = 0;
  q->off_decode = off;    off += align256(q->decode_bytes);
  q->off_out = off;       off += align256(heads * p->head_dim * sizeof(float));
  q->off_lse_full = off;  off += align256(heads * sizeof(float));
  q->off_lse_kept = off;  off += align256(heads * sizeof(float));
  q->off_part_full = off; off += align256(kvh * q->blocks_full * sizeof(float));
  q->off_part_kept = off; off += align256(kvh * q->blocks_kept * sizeof(float));
  q->total = off;
  return CHUNKKV_OK;
}
}  // namespace

size_t chunkkv_quality_workspace_bytes(const chunkkv_problem *prob) {
  QualityPlan q;
  if (check_problem(prob, true) || quality_plan(prob, &q)) return 0;
  return q.total;
}

int chunkkv_quality_metrics(const chunkkv_problem *prob, const int32_t *kv_len, const void *q, const void *k,
                            const void *v, const void *k_out, const void *v_out, float *l1_loss, float *attn_cos,
                            void *workspace, size_t workspace_bytes, void *stream) {
  int rc = check_problem(prob, true);
  if (rc) return rc;
  if (!q || !k || !v || !k_out || !v_out || !l1_loss || !attn_cos) return CHUNKKV_ERR_NULL;
  if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(k_out) || misaligned(v_out)) return CHUNKKV_ERR_SHAPE;
  QualityPlan pl;
  if ((rc = quality_plan(prob, &pl))) return rc;
  if (!workspace || workspace_bytes < pl.total) return CHUNKKV_ERR_WORKSPACE;
  char *ws = (char *)workspace;
  hipStream_t s = (hipStream_t)stream;
  // attention statistics at twice the softmax scale: exp(lse) = sum_t exp(2 scale q . k_t)
  chunkkv_problem twice = *prob;
  twice.softmax_scale = 2.f * (prob->softmax_scale > 0.f ? prob->softmax_scale : 1.0f / sqrtf((float)prob->head_dim));
  float *out = (float *)(ws + pl.off_out);
  float *lse_full = (float *)(ws + pl.off_lse_full), *lse_kept = (float *)(ws + pl.off_lse_kept);
  rc = chunkkv_decode_attention(&twice, 0, nullptr, q, k, v, out, lse_full, ws + pl.off_decode, pl.decode_bytes, stream);
  if (rc) return rc;
  rc = chunkkv_decode_attention(&twice, 1, kv_len, q, k_out, v_out, out, lse_kept, ws + pl.off_decode, pl.decode_bytes, stream);
  if (rc) return rc;
  for (int which = 0; which < 2; ++which) {
    for (int b0 = 0; b0 < prob->batch; b0 += kMaxBatchPerLaunch) {
      const int nb = prob->batch - b0 < kMaxBatchPerLaunch ? prob->batch - b0 : kMaxBatchPerLaunch;
      AbsSumArgs a{};
      a.k = which ? k_out : k; a.v = which ? v_out : v;
      a.partial = (float *)(ws + (which ? pl.off_part_kept : pl.off_part_full));
      a.kv_len = which ? kv_len : nullptr;
      for (int i = 0; i < nb; ++i) {
        a.n_tok[i] = which ? prob->n_keep[b0 + i] + prob->window : prob->seqlen[b0 + i];
        a.base[i] = which ? prob->out_base[b0 + i] : prob->kv_base[b0 + i];
      }
      a.stride_head = which ? prob->out_stride_head : prob->kv_stride_head;
      a.stride_tok = which ? prob->out_stride_tok : prob->kv_stride_tok;
      a.batch0 = b0; a.n_kv_heads = prob->n_kv_heads; a.head_dim = prob->head_dim;
      a.n_blocks = which ? pl.blocks_kept : pl.blocks_full;
      if ((rc = launch_abs_sum(prob->dtype, a, nb, s))) return rc;
    }
  }
  QualityFinishArgs f{};
  f.partial_full = (const float *)(ws + pl.off_part_full); f.partial_kept = (const float *)(ws + pl.off_part_kept);
  f.lse_full = lse_full; f.lse_kept = lse_kept; f.l1_loss = l1_loss; f.attn_cos = attn_cos;
  f.n_q_heads = prob->n_q_heads; f.n_kv_heads = prob->n_kv_heads;
  f.blocks_full = pl.blocks_full; f.blocks_kept = pl.blocks_kept;
  return launch_quality_finish(f, prob->batch, s);
}

int chunkkv_timing_begin(int32_t max_records) {
  if (g_timing.on || max_records < 1) return CHUNKKV_ERR_SHAPE;
  hipEvent_t *ev = new hipEvent_t[2 * (size_t)max_records];
  int *kind = new int[max_records];
  for (int i = 0; i < 2 * max_records; ++i) {
    if (hipEventCreate(&ev[i]) != hipSuccess) {
      for (int j = 0; j < i; ++j) (void)hipEventDestroy(ev[j]);
      delete[] ev;
      delete[] kind;
      return CHUNKKV_ERR_LAUNCH;
    }
  }
  g_timing.ev = ev;
  g_timing.kind = kind;
  g_timing.cap = max_records;
  g_timing.used = 0;
  g_timing.on = true;
  return CHUNKKV_OK;
}

int chunkkv_timing_end(double *total_ms, int64_t *launches) {
  if (!g_timing.on) return CHUNKKV_ERR_SHAPE;
  if (!total_ms || !launches) return CHUNKKV_ERR_NULL;
  g_timing.on = false;
  for (int k = 0; k < kKinds; ++k) { total_ms[k] = 0; launches[k] = 0; }
  int rc = CHUNKKV_OK;
  for (int i = 0; i < g_timing.used; ++i) {
    float ms = 0.f;
    if (hipEventSynchronize(g_timing.ev[2 * i + 1]) != hipSuccess ||
        hipEventElapsedTime(&ms, g_timing.ev[2 * i], g_timing.ev[2 * i + 1]) != hipSuccess) {
      rc = CHUNKKV_ERR_LAUNCH;
      continue;
    }
    total_ms[g_timing.kind[i]] += ms;
    launches[g_timing.kind[i]] += 1;
  }
  for (int i = 0; i < 2 * g_timing.cap; ++i) (void)hipEventDestroy(g_timing.ev[i]);
  delete[] g_timing.ev;
  delete[] g_timing.kind;
  g_timing.ev = nullptr; g_timing.kind = nullptr; g_timing.cap = g_timing.used = 0;
  return rc;
}

}  // extern "C"
