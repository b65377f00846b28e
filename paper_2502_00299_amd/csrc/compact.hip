// Compaction (Algorithm 1: index_select of the kept chunks + concatenation of the window).
//
// Pure data movement: every kept row of K and V is read once and written once.  A workgroup takes `entries_per_wg`
// consecutive selection entries (a kept chunk is a run of `len` consecutive rows; the window is handled as extra
// entries of up to `c` rows) and copies their rows as one flat list of 16-byte segments, K rows first, then V rows:
// consecutive lanes copy consecutive segments whatever the chunk size is, five segments in flight per lane.  The
// entries' chunk, length and offset are loaded once, by one wavefront, into LDS.
// Over a stack the kernel is bound by HBM (copy speed) and a workgroup takes about 160 rows, over a single layer by
// the latency of entry -> rows -> stores, and 40 rows (one round of loads) give four times the workgroups:
// one layer of 20011 tokens, c = 5, keep 20 %, 13.8 -> 9.6 us; two layers of 12345 tokens, c = 1, 23.7 -> 11.3 us, c = 20,
// 17.5 -> 10.2 us.  A 32-layer stack of 131072 tokens (3.45 GB) takes 626 us = 5.5 TB/s; a plain device
// copy of 1 to 4 GiB reaches 4.9 to 5.1.
// Grid: x = group of entries, y = (sequence, kv-head), z = layer; all layers of the stack are one launch.
#include "internal.h"

namespace ckv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// selection entries of a workgroup
__host__ __device__ inline int compact_entries(int rows, int chunk) {
  const int n = rows / chunk;
  return n < 1 ? 1 : (n > kCompactEntries ? kCompactEntries : n);
}

template <int NSEG>  // 16-byte segments per row
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
  int count = n_keep > 0 ? a.sel_count[selrow] : 0;
  count = count < 0 ? 0 : (count > a.sel_cap ? a.sel_cap : count);
  const int n_win = (w + c - 1) / c;
  const int e0 = blockIdx.x * ne;
  if (e0 >= count + n_win) return;

  __shared__ int s_src[kCompactEntries], s_dst[kCompactEntries], s_len[kCompactEntries];
  __shared__ int s_red[kThreads / 64];
  // Token offset of each entry inside the output: the stack call passes the offsets the selection kernel already
  // produced, otherwise the lengths are summed here.
  int before = 0;   // kept tokens before entry min(e0, count)
  if (a.sel_off == nullptr) {
    const int lim = e0 < count ? e0 : count;
    for (int i0 = 0; i0 < lim; i0 += 4 * kThreads) {
      int x[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + j * kThreads + threadIdx.x;
        x[j] = i < lim ? sel_len[i] : 0;
      }
      before += (x[0] + x[1]) + (x[2] + x[3]);
    }
    for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
    if (lane == 0) s_red[wave] = before;
    __syncthreads();
    before = s_red[0] + s_red[1] + s_red[2] + s_red[3];
  }
  if (wave == 0) {
    const int e = e0 + lane;
    const bool mine = lane < ne && e < count + n_win, chosen = mine && e < count;
    int ch = 0, len = 0, dst = 0;
    if (chosen) {
      ch = sel_chunk[e];
      len = sel_len[e];
    }
    int kept = n_keep;   // where the window starts
    if (a.sel_off != nullptr) {
      if (chosen) dst = a.sel_off[selrow * a.sel_cap + e];
      if (a.whole_chunks) kept = count > 0 ? a.sel_off[selrow * a.sel_cap + count - 1] + sel_len[count - 1] : 0;
    } else {
      int inc = len;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
      }
      dst = before + inc - len;
      // a group that holds window entries has seen every selection entry by its last lane
      if (a.whole_chunks) kept = before + __shfl(inc, 63);
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

  const int64_t esz = a.elem_bytes;
  const int64_t base = CKV_ARG(CompactArgs, seq.kv_base, bl), obase = CKV_ARG(CompactArgs, seq.out_base, bl);
  const int64_t in_head = (base + (int64_t)h * a.kv_stride_head) * esz, out_head = (obase + (int64_t)h * a.out_stride_head) * esz;
  const char *kin = (const char *)CKV_ARG(CompactArgs, k, layer) + in_head;
  const char *vin = (const char *)CKV_ARG(CompactArgs, v, layer) + in_head;
  char *kout = (char *)CKV_ARG(CompactArgs, k_out, layer) + out_head;
  char *vout = (char *)CKV_ARG(CompactArgs, v_out, layer) + out_head;
  const int64_t in_tok = a.kv_stride_tok * esz, out_tok = a.out_stride_tok * esz;

  // rows of this workgroup's list: c per entry, or one entry's own length; rows past an entry's length copy nothing
  const int last = count + n_win - e0 < ne ? count + n_win - e0 : ne;
  const int half = (ne > 1 ? last * c : s_len[0]) * NSEG, total = 2 * half;
  const float inv_c = 1.0f / (float)c;
  for (int u0 = threadIdx.x; u0 < total; u0 += 5 * kThreads) {
    u32x4 r[5];
    char *to[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      // lanes without a segment re-read one of theirs and store nothing
      const int u = u0 + j * kThreads < total ? u0 + j * kThreads : u0;
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
      const bool live = i < len && u0 + j * kThreads < total;
      i = i < len ? i : 0;
      // every byte is read once: streaming (non-temporal) loads (measured 2.6 % faster; the same hint on the
      // stores is 2 % slower)
      r[j] = __builtin_nontemporal_load((const u32x4 *)((is_v ? vin : kin) + (int64_t)(s_src[en] + i) * in_tok + seg * 16));
      to[j] = live ? (is_v ? vout : kout) + (int64_t)(s_dst[en] + i) * out_tok + seg * 16 : nullptr;
    }
#pragma unroll
    for (int j = 0; j < 5; ++j)
      if (to[j] != nullptr) *(u32x4 *)to[j] = r[j];
  }
}

int launch_compact(int row_bytes, CompactArgs &a, int n_layers_slice, int batch_slice, hipStream_t s) {
  if (n_layers_slice <= 0 || batch_slice <= 0) return CHUNKKV_OK;
  int64_t total = 0;   // workgroups with entries, of one kv-head per sequence
  auto groups = [&](int rows) {   // most workgroups of a head
    a.rows_per_wg = rows;
    int most = 0;
    total = 0;
    for (int z = 0; z < n_layers_slice; ++z) {
      const int c = a.chunk_of[z], ne = compact_entries(rows, c);
      int entries = 0;
      for (int i = 0; i < batch_slice; ++i) {
        const int nk = a.seq.n_keep[i], n_win = (a.window + c - 1) / c;
        int e = nk > 0 ? (nk + c - 1) / c + 1 : 0;
        e = (e > a.sel_cap ? a.sel_cap : e) + n_win;
        entries = e > entries ? e : entries;
      }
      const int n = (entries + ne - 1) / ne;
      most = n > most ? n : most;
      total += n;
    }
    return most;
  };
  int nx = groups(160);
  if (total * batch_slice * a.n_kv_heads < 4096) nx = groups(40);
  if (nx <= 0) return CHUNKKV_OK;
  dim3 grid(nx, batch_slice * a.n_kv_heads, n_layers_slice);
  switch (row_bytes / 16) {
    case 8: hipLaunchKernelGGL(compact_kernel<8>, grid, dim3(kThreads), 0, s, a); break;
    case 16: hipLaunchKernelGGL(compact_kernel<16>, grid, dim3(kThreads), 0, s, a); break;
    case 32: hipLaunchKernelGGL(compact_kernel<32>, grid, dim3(kThreads), 0, s, a); break;
    default: return CHUNKKV_ERR_UNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

}  // namespace ckv
