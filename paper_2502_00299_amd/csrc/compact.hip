// Compaction (Algorithm 1: index_select of the kept chunks + concatenation of the window).
//
// Pure data movement: every kept row of K and V is read once and written once.  A workgroup takes `rows_per_wg` rows' worth of
// consecutive selection entries (a kept chunk is a run of `len` consecutive rows; the window is handled as extra
// entries of up to `c` rows) and copies their rows as one flat list of 16-byte segments, K rows first, then V rows:
// consecutive lanes copy consecutive segments whatever the chunk size is, five segments in flight per lane.  The
// entries' chunk, length and offset are loaded once, by one wavefront, into LDS.
// Streaming (non-temporal) loads where the call's caches fill most of the memory-side one, streaming stores where what is written is more than half
// of it (the lines, with both sides measured, are in api.hip): smaller ones are found there by the next call.  An instance per kind, as a branch
// around the accesses parts them from their addresses: 32 layers of 131072 tokens 1978 us, as a branch 2045, the ragged batch at c = 20 1965 and 2075.
// Over a stack the kernel is bound by HBM (copy speed) and a workgroup takes about 80 rows, over a single layer by
// the latency of entry -> rows -> stores, and 40 rows (one round of loads) give four times the workgroups:
// one layer of 20011 tokens, c = 5, keep 20 %, 13.8 -> 9.6 us; two layers of 12345 tokens, c = 1, 23.7 -> 11.3 us, c = 20,
// 17.5 -> 10.2 us.  A 32-layer stack of 131072 tokens (3.45 GB) takes 599 us = 5.8 TB/s, with plain stores 626; a plain
// device copy of 1 to 4 GiB reaches 4.9 to 5.1.
// Grid: x = group of entries, y = (sequence, kv-head), z = layer; all layers of the stack are one launch.
#include "select.h"

namespace ckv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Selection and gather in one launch, by chunks of the longest head and workgroups.  Every workgroup selects for itself, which
// costs little as long as all of them run at once, or with one chunk per thread.  us of a call, together and apart:
//   up to 256 chunks: 64, 1024 workgroups 24.2 / 27.9; 200, 2816 32.8 / 33.7; 256, 3584 34.8 / 36.6; 200, 5376 49.4 / 49.1
//   up to 1024: 300, 1024 workgroups 20.4 / 21.7; 400, 1344 24.5 / 25.0; 1024, 1408 23.3 / 26.6; 300, 1536 25.8 / 25.7;
//     800, 1968 33.2 / 30.7; 300, 2048 33.6 / 29.6; 512, 3456 43.6 / 39.7; 300, 4096 50.7 / 42.1
//   more chunks take 1024 threads, and as long as every workgroup has a CU: 3000, 152 workgroups 30.5 / 32.7; 4000, 208
//     35.8 / 38.5; 3000, 304 43.5 / 36.3
constexpr int kSelectCompactFewChunks = kThreads, kSelectCompactFewWorkgroups = 4096;
constexpr int kSelectCompactChunks = 1024, kSelectCompactWorkgroups = 1408;
constexpr int kSelectCompactWideChunks = 4096, kSelectCompactWideWorkgroups = 256;

// selection entries of a workgroup
__host__ __device__ inline int compact_entries(int rows, int chunk) {
  const int n = rows / chunk;
  return n < 1 ? 1 : (n > kCompactEntries ? kCompactEntries : n);
}

// Copies the rows of entries [0, n) of the lists (source token, destination token, length) of one layer, sequence and
// kv-head; ne: entries a workgroup can have.
template <int NSEG, int T, Stream STREAM>  // 16-byte segments per row, threads
__device__ __forceinline__ void copy_entries(const CompactArgs &a, int layer, int bl, int h, int c, int ne, int n, const int *s_src, const int *s_dst, const int *s_len) {
  const int64_t esz = a.elem_bytes;
  const int64_t base = CKV_ARG(CompactArgs, seq.kv_base, bl), obase = CKV_ARG(CompactArgs, seq.out_base, bl);
  const int64_t in_head = (base + (int64_t)h * a.kv_stride_head) * esz, out_head = (obase + (int64_t)h * a.out_stride_head) * esz;
  const char *kin = (const char *)CKV_ARG(CompactArgs, k, layer) + in_head;
  const char *vin = (const char *)CKV_ARG(CompactArgs, v, layer) + in_head;
  char *kout = (char *)CKV_ARG(CompactArgs, k_out, layer) + out_head;
  char *vout = (char *)CKV_ARG(CompactArgs, v_out, layer) + out_head;
  const int64_t in_tok = a.kv_stride_tok * esz, out_tok = a.out_stride_tok * esz;

  // rows of this workgroup's list: c per entry, or one entry's own length; rows past an entry's length copy nothing
  const int half = (ne > 1 ? n * c : s_len[0]) * NSEG, total = 2 * half;
  const float inv_c = 1.0f / (float)c;
  for (int u0 = threadIdx.x; u0 < total; u0 += 5 * T) {
    u32x4 r[5];
    char *to[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      // lanes without a segment re-read one of theirs and store nothing
      const int u = u0 + j * T < total ? u0 + j * T : u0;
      const bool is_v = u >= half;
      const int uu = is_v ? u - half : u, row = uu / NSEG, seg = uu % NSEG;
      int en = 0, i = row;
      if (ne > 1) {   // row < 160: the rounded quotient is off by at most one
        en = (int)((float)row * inv_c);
        i = row - en * c;
        if (i < 0) { --en; i += c; }
        if (i >= c) { ++en; i -= c; }
      }
      const int len = s_len[en];
      const bool live = i < len && u0 + j * T < total;
      i = i < len ? i : 0;
      const u32x4 *from = (const u32x4 *)((is_v ? vin : kin) + (int64_t)(s_src[en] + i) * in_tok + seg * 16);
      if constexpr (STREAM != Stream::kNone) r[j] = __builtin_nontemporal_load(from);
      else r[j] = *from;
      to[j] = live ? (is_v ? vout : kout) + (int64_t)(s_dst[en] + i) * out_tok + seg * 16 : nullptr;
    }
#pragma unroll
    for (int j = 0; j < 5; ++j)
      if (to[j] != nullptr) {
        if constexpr (STREAM == Stream::kAll) __builtin_nontemporal_store(r[j], (u32x4 *)to[j]);
        else *(u32x4 *)to[j] = r[j];
      }
  }
}

template <int NSEG, Stream STREAM>  // 16-byte segments per row
__global__ __launch_bounds__(kThreads) void compact_kernel(CompactArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int bl = blockIdx.y / a.n_kv_heads, h = blockIdx.y % a.n_kv_heads;
  const int layer = blockIdx.z;
  const int L = CKV_ARG(CompactArgs, seq.seqlen, bl), n_keep = CKV_ARG(CompactArgs, seq.n_keep, bl);
  const int w = a.window, c = CKV_ARG(CompactArgs, chunk_of, layer), P = L - w, ne = compact_entries(a.rows_per_wg, c);
  const int group = (a.layer0 + layer) / a.reuse;
  const int64_t selrow = ((int64_t)group * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const int32_t *sel_chunk = a.sel_chunk + selrow * a.sel_cap;
  const int32_t *sel_len = a.sel_len + selrow * a.sel_cap;
  const int n_win = (w + c - 1) / c;
  const int e0 = blockIdx.x * ne;
  // The number of entries, this workgroup's own and the lengths of those before them are read together: the arrays have room for
  // sel_cap entries, and what lies past the last one is not used.
  const int e = e0 + lane, own = e < a.sel_cap ? e : 0;
  int count = n_keep > 0 ? a.sel_count[selrow] : 0;
  int ch = 0, len = 0, dst = 0;
  if (wave == 0) {
    ch = sel_chunk[own];
    len = sel_len[own];
    if (a.sel_off != nullptr) dst = a.sel_off[selrow * a.sel_cap + own];
  }
  int before[4] = {0, 0, 0, 0};   // this thread's share of the first 4 * kThreads of them, if offsets are not at hand
  const int most_before = e0 < a.sel_cap ? e0 : a.sel_cap;
  if (a.sel_off == nullptr) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = j * kThreads + threadIdx.x;
      before[j] = i < most_before ? sel_len[i] : 0;
    }
  }
  count = count < 0 ? 0 : (count > a.sel_cap ? a.sel_cap : count);
  if (e0 >= count + n_win) return;

  __shared__ int s_src[kCompactEntries], s_dst[kCompactEntries], s_len[kCompactEntries];
  __shared__ int s_red[kThreads / 64];
  // Token offset of each entry inside the output: the stack call passes the offsets the selection kernel already
  // produced, otherwise the lengths are summed here.
  int kept_before = 0;   // kept tokens before entry min(e0, count)
  if (a.sel_off == nullptr) {
    const int lim = e0 < count ? e0 : count;
#pragma unroll
    for (int j = 0; j < 4; ++j) kept_before += (int)(j * kThreads + threadIdx.x) < lim ? before[j] : 0;
    for (int i0 = 4 * kThreads; i0 < lim; i0 += 4 * kThreads) {
      int x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + j * kThreads + threadIdx.x;
        x[j] = i < lim ? sel_len[i] : 0;
      }
      kept_before += (x[0] + x[1]) + (x[2] + x[3]);
    }
    for (int o = 32; o > 0; o >>= 1) kept_before += __shfl_xor(kept_before, o);
    if (lane == 0) s_red[wave] = kept_before;
    __syncthreads();
    kept_before = s_red[0] + s_red[1] + s_red[2] + s_red[3];
  }
  if (wave == 0) {
    const bool mine = lane < ne && e < count + n_win, chosen = mine && e < count;
    if (!chosen) ch = len = dst = 0;
    int kept = n_keep;   // where the window starts
    if (a.sel_off != nullptr) {
      if (a.whole_chunks) kept = count > 0 ? a.sel_off[selrow * a.sel_cap + count - 1] + sel_len[count - 1] : 0;
    } else {
      int inc = len;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
      }
      dst = kept_before + inc - len;
      // a group that holds window entries has seen every selection entry by its last lane
      if (a.whole_chunks) kept = kept_before + __shfl(inc, 63);
    }
    kept = kept < 0 ? 0 : (kept > n_keep ? n_keep : kept);
    int src = ch * c;
    if (chosen) {
      // a malformed selection is skipped, never followed out of bounds
      if (ch < 0 || len < 1 || len > c || (int64_t)ch * c + len > P || dst < 0 || dst > n_keep - len) len = src = 0;
    } else if (mine) {
      const int wi = e - count;
      src = P + wi * c;
      len = w - wi * c < c ? w - wi * c : c;
      dst = kept + wi * c;
    }
    if (lane < ne) { s_src[lane] = src; s_dst[lane] = dst; s_len[lane] = mine ? len : 0; }
  }
  __syncthreads();
  copy_entries<NSEG, kThreads, STREAM>(a, layer, bl, h, c, ne, count + n_win - e0 < ne ? count + n_win - e0 : ne, s_src, s_dst, s_len);
}

// Selection and gather in one launch: every workgroup selects the chunks of its head for itself and keeps the places that
// are its own; one workgroup per head and reuse group writes the selection out.  For short launches over few chunks, where a
// dependent launch costs more than the selection's 2 to 5 us.
template <int NSEG, int T, int KR, Stream STREAM>
__global__ __launch_bounds__(T) void select_compact_kernel(CompactArgs a, const float *chunk_scores, int score_cap) {
  const int bl = blockIdx.y / a.n_kv_heads, h = blockIdx.y % a.n_kv_heads, layer = blockIdx.z;
  const int n_keep = CKV_ARG(CompactArgs, seq.n_keep, bl), w = a.window, c = CKV_ARG(CompactArgs, chunk_of, layer);
  const int P = CKV_ARG(CompactArgs, seq.seqlen, bl) - w, ne = compact_entries(a.rows_per_wg, c), n_win = (w + c - 1) / c;
  const int e0 = blockIdx.x * ne;
  if (e0 >= (n_keep > 0 ? (n_keep + c - 1) / c + 1 : 0) + n_win) return;   // more entries there cannot be
  const int group = (a.layer0 + layer) / a.reuse;
  const int64_t selrow = ((int64_t)group * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const bool writer = blockIdx.x == 0 && (layer == 0 || (a.layer0 + layer) % a.reuse == 0);
  int32_t *sel_chunk = const_cast<int32_t *>(a.sel_chunk) + selrow * a.sel_cap, *sel_len = const_cast<int32_t *>(a.sel_len) + selrow * a.sel_cap;
  __shared__ int s_src[kCompactEntries], s_dst[kCompactEntries], s_len[kCompactEntries];
  const Selected sel = select_chunks<T, KR, true>(chunk_scores + selrow * score_cap, P, c, n_keep, a.whole_chunks != 0, [&](int i, int pos, int len, int off) {
    if (pos >= e0 && pos < e0 + ne) { s_src[pos - e0] = i * c; s_dst[pos - e0] = off; s_len[pos - e0] = len; }
    if (writer && pos < a.sel_cap) { sel_chunk[pos] = i; sel_len[pos] = len; }
  });
  if (writer && threadIdx.x == 0) const_cast<int32_t *>(a.sel_count)[selrow] = sel.count;
  const int wi = e0 + (int)threadIdx.x - sel.count;   // window entry of this thread, if it is one
  if ((int)threadIdx.x < ne && wi >= 0 && wi < n_win) {
    s_src[threadIdx.x] = P + wi * c;
    s_dst[threadIdx.x] = sel.kept + wi * c;
    s_len[threadIdx.x] = w - wi * c < c ? w - wi * c : c;
  }
  __syncthreads();
  const int n = sel.count + n_win - e0;
  if (n > 0) copy_entries<NSEG, T, STREAM>(a, layer, bl, h, c, ne, n < ne ? n : ne, s_src, s_dst, s_len);
}

// Workgroups of a launch with `rows` rows each.
struct GatherGroups {
  int most;        // of a head
  int64_t total;   // with entries, of all heads
};
static GatherGroups gather_groups(const CompactArgs &a, int n_layers_slice, int batch_slice, int rows) {
  GatherGroups g = {0, 0};
  for (int z = 0; z < n_layers_slice; ++z) {
    const int c = a.chunk_of[z], ne = compact_entries(rows, c), n_win = (a.window + c - 1) / c;
    int entries = 0;
    for (int i = 0; i < batch_slice; ++i) {
      const int nk = a.seq.n_keep[i];
      int e = nk > 0 ? (nk + c - 1) / c + 1 : 0;
      e = (e > a.sel_cap ? a.sel_cap : e) + n_win;
      entries = e > entries ? e : entries;
    }
    const int n = (entries + ne - 1) / ne;
    g.most = n > g.most ? n : g.most;
    g.total += (int64_t)n * batch_slice * a.n_kv_heads;
  }
  return g;
}
// Sets the rows of a workgroup: fewer in a launch that would leave CUs without one.
static GatherGroups choose_rows(CompactArgs &a, int n_layers_slice, int batch_slice) {
  a.rows_per_wg = 80;
  GatherGroups g = gather_groups(a, n_layers_slice, batch_slice, a.rows_per_wg);
  if (g.total >= 8192) return g;
  a.rows_per_wg = 40;
  return gather_groups(a, n_layers_slice, batch_slice, a.rows_per_wg);
}

int launch_select_compact(int row_bytes, CompactArgs &a, int n_layers_slice, int batch_slice, const float *chunk_scores, int score_cap,
                          const SelectInGather &how, hipStream_t s) {
  a.rows_per_wg = how.rows_per_wg;
  const dim3 grid(how.groups, batch_slice * a.n_kv_heads, n_layers_slice), block(how.wide ? 1024 : kThreads);
#define CKV_SELECT_AS(NSEG, STREAM) \
  hipLaunchKernelGGL((how.wide ? select_compact_kernel<NSEG, 1024, 4, STREAM> : how.chunks <= kSelectCompactFewChunks ? select_compact_kernel<NSEG, kThreads, 1, STREAM> : select_compact_kernel<NSEG, kThreads, 4, STREAM>), \
                     grid, block, 0, s, a, chunk_scores, score_cap)
#define CKV_SELECT(NSEG) \
  do { \
    if (a.stream == Stream::kAll) CKV_SELECT_AS(NSEG, Stream::kAll); \
    else if (a.stream == Stream::kLoads) CKV_SELECT_AS(NSEG, Stream::kLoads); \
    else CKV_SELECT_AS(NSEG, Stream::kNone); \
  } while (0)
  switch (row_bytes / 16) {
    case 8: CKV_SELECT(8); break;
    case 16: CKV_SELECT(16); break;
    case 32: CKV_SELECT(32); break;
    default: return CHUNKKV_ERR_UNSUPPORTED;
  }
#undef CKV_SELECT
#undef CKV_SELECT_AS
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

SelectInGather select_in_gather(CompactArgs &a, int n_layers_slice, int batch_slice) {
  SelectInGather how = {};
  for (int z = 0; z < n_layers_slice; ++z)
    for (int i = 0; i < batch_slice; ++i) {
      const int C = (a.seq.seqlen[i] - a.window + a.chunk_of[z] - 1) / a.chunk_of[z];
      how.chunks = C > how.chunks ? C : how.chunks;
    }
  if (how.chunks > kSelectCompactWideChunks) return how;
  how.wide = how.chunks > kSelectCompactChunks;
  GatherGroups g = choose_rows(a, n_layers_slice, batch_slice);
  how.rows_per_wg = how.wide ? 160 : a.rows_per_wg;   // few workgroups, each wide and long
  if (how.wide) g = gather_groups(a, n_layers_slice, batch_slice, how.rows_per_wg);
  how.groups = g.most;
  how.yes = g.total <= (how.wide ? kSelectCompactWideWorkgroups : how.chunks > kSelectCompactFewChunks ? kSelectCompactWorkgroups : kSelectCompactFewWorkgroups);
  return how;
}

int launch_compact(int row_bytes, CompactArgs &a, int n_layers_slice, int batch_slice, hipStream_t s) {
  const dim3 grid(choose_rows(a, n_layers_slice, batch_slice).most, batch_slice * a.n_kv_heads, n_layers_slice);
#define CKV_COMPACT(NSEG) \
  hipLaunchKernelGGL((a.stream == Stream::kAll ? compact_kernel<NSEG, Stream::kAll> : a.stream == Stream::kLoads ? compact_kernel<NSEG, Stream::kLoads> : compact_kernel<NSEG, Stream::kNone>), \
                     grid, dim3(kThreads), 0, s, a)
  switch (row_bytes / 16) {
    case 8: CKV_COMPACT(8); break;
    case 16: CKV_COMPACT(16); break;
    case 32: CKV_COMPACT(32); break;
    default: return CHUNKKV_ERR_UNSUPPORTED;
  }
#undef CKV_COMPACT
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

}  // namespace ckv
