// Chunk selection (Algorithm 1, top-k step, with the exact-budget rule).
//
// One workgroup per (selection group, sequence, kv-head).  Chunks are ranked by (score descending, index ascending).
// The m-th ranked chunk, the threshold, is found on the order-preserving integer image of the fp32 scores: a
// histogram over ten bits of the keys' distance from the head's lowest narrows the candidates to one bin (one digit
// deeper as long as it holds more than kTopkList of them), then they are listed in LDS and ranked against each other,
// index included, so ties need no further step.  Only more equal keys than that go through the histograms to the last
// bit and a prefix count in index order.
// m = ceil(n_keep / c); if the ragged last chunk is among those m and leaves the budget short, one more chunk is
// taken.  The lowest-ranked selected chunk is cut to the tokens still missing.
// Thread t owns chunks t, t + T, ...: loads are coalesced, and a ballot per wavefront and stripe plus one scan over the
// stripes' counts give every selected chunk its place in ascending order; its token offset follows from the place
// and from which side of the threshold chunk it lies on.
//
// Bound by latency: one workgroup per head, a chain of block-wide steps, code that every workgroup runs through once.
// Hence few barriers (about 11), and variants whose unrolled loops are no longer than the head needs.  Measured against
// the three-pass radix select over consecutive chunks that this replaced, us per launch back to back:
//   chunks per head   62: 11.8 -> 4.3   816: 12.4 -> 5.5   2000: 13.2 -> 8.1   4000: 14.7 -> 7.3   13101: 20.7 -> 14.5
//   (128 heads: 21.4 -> 14.7)   20000: 54 -> 26   131072: 479 -> 133
#include "internal.h"

namespace ckv {

constexpr int kTopkBins = 1024, kTopkBits = 10;
constexpr int kTopkList = 512;   // candidates ranked by comparing all pairs

__device__ __forceinline__ uint32_t order_key(float x) {
  uint32_t u = __float_as_uint(x);
  if (u == 0x80000000u) u = 0;  // -0 ranks as +0
  if (u == 0xFFFFFFFFu) u = 0xFFFFFFFEu;   // key 0 is no chunk's: the lowest NaN shares the next one's
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// T: threads, KR: chunks a thread takes at a time, REG: all keys of the head stay in registers (C <= KR T), otherwise
// every step re-reads the scores
template <int T, int KR, bool REG>
__global__ __launch_bounds__(T) void topk_kernel(TopkArgs a) {
  constexpr int NW = T / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bl = blockIdx.x / a.n_kv_heads, h = blockIdx.x % a.n_kv_heads, group = a.group0 + blockIdx.y;
  const int64_t row = ((int64_t)group * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;
  const float *scores = a.chunk_scores + row * a.score_cap;
  int32_t *sel_chunk = a.sel_chunk + row * a.sel_cap;
  int32_t *sel_len = a.sel_len + row * a.sel_cap;
  int32_t *sel_off = a.sel_off ? a.sel_off + row * a.sel_cap : nullptr;
  const int c = CKV_ARG(TopkArgs, chunk_of, blockIdx.y), P = CKV_ARG(TopkArgs, seq.seqlen, bl) - a.window, n_keep = CKV_ARG(TopkArgs, seq.n_keep, bl);
  const int C = (P + c - 1) / c;
  // exact budget: ceil(n_keep / c) chunks, the lowest-ranked one cut; whole-chunk mode: floor(n_keep / c)
  // chunks (at most C), none cut
  const int m0 = n_keep <= 0 || C <= 0 ? 0 : (a.whole_chunks ? (n_keep / c < C ? n_keep / c : C) : (n_keep + c - 1) / c);
  if (m0 <= 0) {
    if (tid == 0) a.sel_count[row] = 0;
    return;
  }
  const int tail_size = P - (C - 1) * c;  // == c when there is no ragged tail

  __shared__ int s_hist[kTopkBins];
  __shared__ uint64_t s_list[kTopkList];
  __shared__ uint32_t s_mn[NW], s_mx[NW];
  __shared__ int s_wave[NW], s_cnt[KR * NW];
  __shared__ int s_bin, s_rem, s_ncand, s_nlist, s_idx, s_total;
  __shared__ uint32_t s_key;

  uint32_t low = 0;   // subtracted from every key, see below
  uint32_t kreg[REG ? KR : 1];
  if constexpr (REG) {
#pragma unroll
    for (int j = 0; j < KR; ++j)
      kreg[j] = __float_as_uint(scores[j * T + tid < C ? j * T + tid : C - 1]);
#pragma unroll
    for (int j = 0; j < KR; ++j) kreg[j] = j * T + tid < C ? order_key(__uint_as_float(kreg[j])) : 0u;
  }
  // f(chunk index, key) for every own chunk, in index order.  Places past the last chunk carry key 0, which ranks below
  // every chunk: they may be counted and listed but are never the threshold or above it.
  auto each = [&](auto f) __attribute__((always_inline)) {
    if constexpr (REG) {
#pragma unroll
      for (int j = 0; j < KR; ++j)
        if (KR <= 4 || j * T < C) f(j * T + tid, kreg[j]);
    } else {
      for (int i = tid; i < C; i += T) f(i, order_key(scores[i]) - low);
    }
  };
  // f(chunk index, rank) for every own chunk with pred(index, key), rank = how many such chunks lie before it
  auto ranked = [&](auto pred, auto f) __attribute__((always_inline)) {
    int base = 0;
    for (int i0 = 0; i0 < C; i0 += KR * T) {
      uint32_t own = 0;   // bit j: the chunk of stripe j satisfies pred
#pragma unroll
      for (int j = 0; j < KR; ++j) {
        int n = 0;
        if (KR <= 4 || i0 + j * T < C) {
          const int i = i0 + j * T + tid;
          const bool p = REG ? pred(i, kreg[REG ? j : 0]) : i < C && pred(i, order_key(scores[i < C ? i : C - 1]) - low);
          own |= p ? 1u << j : 0u;
          n = (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(p));
        }
        if (lane == 0) s_cnt[j * NW + wave] = n;
      }
      __syncthreads();
      if (wave == 0) {   // exclusive prefix of the 16 NW counts, 16 NW / 64 per lane
        constexpr int N = (KR * NW + 63) / 64;
        int x[N], sum = 0;
#pragma unroll
        for (int k = 0; k < N; ++k) { x[k] = lane * N + k < KR * NW ? s_cnt[lane * N + k] : 0; sum += x[k]; }
        int inc = sum;
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(inc, o);
          if (lane >= o) inc += y;
        }
        int run = inc - sum;
#pragma unroll
        for (int k = 0; k < N; ++k) { if (lane * N + k < KR * NW) s_cnt[lane * N + k] = run; run += x[k]; }
        if (lane == 63) s_total = run;
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < KR; ++j) {
        if (KR > 4 && i0 + j * T >= C) break;
        const bool p = (own >> j) & 1;
        const uint64_t below = __builtin_amdgcn_ballot_w64(p) & ((1ull << lane) - 1);
        if (p) f(i0 + j * T + tid, base + s_cnt[j * NW + wave] + (int)__builtin_popcountll(below));
      }
      base += s_total;
      if (i0 + KR * T < C) __syncthreads();
    }
  };

  for (int i = tid; i < kTopkBins; i += T) s_hist[i] = 0;
  uint32_t kmn = 0xFFFFFFFFu, kmx = 0u;
  each([&](int, uint32_t key) { kmn = key - 1 < kmn - 1 ? key : kmn; kmx = key > kmx ? key : kmx; });   // 0 - 1 is no minimum
  for (int o = 32; o > 0; o >>= 1) {
    const uint32_t x = __shfl_xor(kmn, o), y = __shfl_xor(kmx, o);
    kmn = x < kmn ? x : kmn; kmx = y > kmx ? y : kmx;
  }
  if (lane == 0) { s_mn[wave] = kmn; s_mx[wave] = kmx; }
  if (tid == 0) s_nlist = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) { kmn = s_mn[i] < kmn ? s_mn[i] : kmn; kmx = s_mx[i] > kmx ? s_mx[i] : kmx; }
  // From here on keys are counted from the head's lowest (1): the first digit then spreads them over the bins however
  // the scores lie around a power of two, which flips high bits of the image.
  low = kmn - 1;
  if constexpr (REG) {
#pragma unroll
    for (int j = 0; j < KR; ++j) kreg[j] = kreg[j] != 0 ? kreg[j] - low : 0u;
  }
  const uint32_t tail_key = order_key(scores[C - 1]) - low;
  const int hi = 32 - __builtin_clz(kmx - low);   // bits [0, hi) may be set

  uint32_t thr = 0;    // key and index of the m-th ranked chunk
  int thr_idx = 0;
  int m = m0, total = 0;
  bool tail_sel = false;
  for (int attempt = 0; attempt < 2; ++attempt) {
    uint32_t prefix = 0;
    int rem = m, top = hi;   // the threshold is the rem-th largest among the keys that share `prefix` above bit `top`
    for (;;) {
      if (top == 0) {   // every candidate has this key: the rem-th in index order
        ranked([&](int, uint32_t key) { return key == prefix; }, [&](int i, int rank) { if (rank == rem - 1) { s_idx = i; s_key = prefix; } });
        __syncthreads();
        break;
      }
      const int shift = top > kTopkBits ? top - kTopkBits : 0;
      const uint32_t mask = top >= 32 ? 0u : (0xFFFFFFFFu << top);   // bits settled so far; prefix is zero below
      each([&](int, uint32_t key) { if ((key & mask) == prefix) atomicAdd(&s_hist[(key >> shift) & (kTopkBins - 1)], 1); });
      __syncthreads();
      {
        // thread t owns NB digits in descending order from kTopkBins - 1 - NB t on; one scan over the threads
        constexpr int NB = kTopkBins / T;
        int v[NB], sum = 0;
#pragma unroll
        for (int j = 0; j < NB; ++j) { v[j] = s_hist[kTopkBins - 1 - NB * tid - j]; sum += v[j]; }
        int inc = sum;
        for (int o = 1; o < 64; o <<= 1) {
          const int y = __shfl_up(inc, o);
          if (lane >= o) inc += y;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        int before = inc - sum;
#pragma unroll
        for (int i = 0; i < NW; ++i) before += i < wave ? s_wave[i] : 0;
        if (before < rem && before + sum >= rem) {
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (before < rem && before + v[j] >= rem) { s_bin = kTopkBins - 1 - NB * tid - j; s_rem = rem - before; s_ncand = v[j]; }
            before += v[j];
          }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) s_hist[kTopkBins - 1 - NB * tid - j] = 0;   // for the next pass
        __syncthreads();
      }
      prefix |= (uint32_t)s_bin << shift;   // fewer varying bits than a digit: its upper bits repeat the prefix
      rem = s_rem;
      const int ncand = s_ncand;
      top = shift;
      if (ncand <= kTopkList) {
        const uint32_t settled = shift >= 32 ? 0u : (0xFFFFFFFFu << shift);
        each([&](int i, uint32_t key) {
          if ((key & settled) == prefix) s_list[atomicAdd(&s_nlist, 1)] = ((uint64_t)key << 32) | (uint32_t)~i;   // larger ranks first
        });
        __syncthreads();
        for (int t = tid; t < ncand; t += T) {
          const uint64_t mine = s_list[t];
          int rank = 1;
          for (int j = 0; j < ncand; ++j) rank += s_list[j] > mine;
          if (rank == rem) { s_key = (uint32_t)(mine >> 32); s_idx = (int)~(uint32_t)mine; }
        }
        __syncthreads();
        break;
      }
    }
    thr = s_key;
    thr_idx = s_idx;
    tail_sel = tail_key > thr || (tail_key == thr && thr_idx == C - 1);
    total = m * c - (tail_sel ? c - tail_size : 0);
    if (total >= n_keep || a.whole_chunks) break;
    m = m0 + 1;  // tail selected and budget short by < c tokens: exactly one more chunk is needed
    __syncthreads();
    if (tid == 0) s_nlist = 0;
  }
  const int size_trunc = thr_idx == C - 1 ? tail_size : c;
  const int len_trunc = a.whole_chunks ? size_trunc : n_keep - (total - size_trunc);

  ranked([&](int i, uint32_t key) { return key > thr || (key == thr && i <= thr_idx); },
         [&](int i, int pos) {
           if (pos >= a.sel_cap) return;
           sel_chunk[pos] = i;
           sel_len[pos] = i == thr_idx ? len_trunc : (i == C - 1 ? tail_size : c);
           if (sel_off) sel_off[pos] = pos * c - (i > thr_idx ? size_trunc - len_trunc : 0);
         });
  if (tid == 0) a.sel_count[row] = m;
}

int launch_topk(const TopkArgs &a, int n_groups, int batch_slice, hipStream_t s) {
  if (n_groups <= 0 || batch_slice <= 0) return CHUNKKV_OK;
  dim3 grid(batch_slice * a.n_kv_heads, n_groups);
  int c_max = 0;
  for (int j = 0; j < n_groups; ++j)
    for (int i = 0; i < batch_slice; ++i) {
      const int C = (a.seq.seqlen[i] - a.window + a.chunk_of[j] - 1) / a.chunk_of[j];
      c_max = C > c_max ? C : c_max;
    }
  // few chunks: 256 threads (cheaper barriers); a thread's chunks are unrolled, so no more of them than needed (a
  // workgroup runs through the code once, and bringing it in costs)
  if (c_max <= 256) hipLaunchKernelGGL((topk_kernel<256, 1, true>), grid, dim3(256), 0, s, a);
  else if (c_max <= 1024) hipLaunchKernelGGL((topk_kernel<256, 4, true>), grid, dim3(256), 0, s, a);
  else if (c_max <= 4096) hipLaunchKernelGGL((topk_kernel<1024, 4, true>), grid, dim3(1024), 0, s, a);
  else if (c_max <= 16384) hipLaunchKernelGGL((topk_kernel<1024, 16, true>), grid, dim3(1024), 0, s, a);
  else hipLaunchKernelGGL((topk_kernel<1024, 16, false>), grid, dim3(1024), 0, s, a);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

// Adjacent-group Jaccard similarity of two selections of one (sequence, kv-head).  Both are ascending lists
// of (chunk, leading tokens kept); a chunk present in both shares min(len) tokens.  One workgroup per
// (pair of groups, sequence, kv-head): every thread takes entries of the first list and finds their chunk
// in the second by binary search; sums are reduced in a fixed order.
__global__ __launch_bounds__(256) void jaccard_kernel(const int32_t *sel_chunk, const int32_t *sel_len,
                                                      const int32_t *sel_count, int sel_cap, int rows_per_group,
                                                      float *out) {
  const int64_t ra = (int64_t)blockIdx.y * rows_per_group + blockIdx.x, rb = ra + rows_per_group;
  int na = sel_count[ra], nb = sel_count[rb];
  na = na < 0 ? 0 : (na > sel_cap ? sel_cap : na);
  nb = nb < 0 ? 0 : (nb > sel_cap ? sel_cap : nb);
  const int32_t *ca = sel_chunk + ra * sel_cap, *la = sel_len + ra * sel_cap;
  const int32_t *cb = sel_chunk + rb * sel_cap, *lb = sel_len + rb * sel_cap;
  int inter = 0, size_a = 0, size_b = 0;
  for (int i = threadIdx.x; i < na; i += 256) {
    const int ch = ca[i], ln = la[i];
    size_a += ln;
    int lo = 0, hi = nb;  // first entry of b with chunk >= ch
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (cb[mid] < ch) lo = mid + 1; else hi = mid;
    }
    if (lo < nb && cb[lo] == ch) inter += ln < lb[lo] ? ln : lb[lo];
  }
  for (int i = threadIdx.x; i < nb; i += 256) size_b += lb[i];
  __shared__ int s_red[3][4];
  for (int o = 32; o > 0; o >>= 1) {
    inter += __shfl_xor(inter, o); size_a += __shfl_xor(size_a, o); size_b += __shfl_xor(size_b, o);
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[0][threadIdx.x >> 6] = inter; s_red[1][threadIdx.x >> 6] = size_a; s_red[2][threadIdx.x >> 6] = size_b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int it = s_red[0][0] + s_red[0][1] + s_red[0][2] + s_red[0][3];
    const int un = s_red[1][0] + s_red[1][1] + s_red[1][2] + s_red[1][3] +
                   s_red[2][0] + s_red[2][1] + s_red[2][2] + s_red[2][3] - it;
    out[ra] = un > 0 ? (float)it / (float)un : 1.0f;
  }
}

int launch_jaccard(const int32_t *sel_chunk, const int32_t *sel_len, const int32_t *sel_count, int sel_cap, int chunk,
                   int rows_per_group, int n_pairs, float *out, hipStream_t s) {
  (void)chunk;
  if (rows_per_group <= 0 || n_pairs <= 0) return CHUNKKV_OK;
  hipLaunchKernelGGL(jaccard_kernel, dim3(rows_per_group, n_pairs), dim3(256), 0, s, sel_chunk, sel_len, sel_count,
                     sel_cap, rows_per_group, out);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

}  // namespace ckv
