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
// Past 16384 chunks the scores are re-read, eight loads in flight per thread (one before): 40201: 70 -> 61.5, 131000: 149 -> 127.
// 32 or 64 keys per thread in registers there do not fit into 128 registers: 26200: 34 -> 101.
#pragma once
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

struct Selected {
  int count, kept;   // chunks and tokens
};

// T: threads of the workgroup, KR: chunks a thread takes at a time, REG: all keys of the head stay in registers (C <= KR T),
// otherwise every step re-reads the scores.  P candidate tokens, chunk size c; emit(chunk, place, length, token offset) is
// called once for every selected chunk, by the thread that owns it.
template <int T, int KR, bool REG, typename Emit>
__device__ __forceinline__ Selected select_chunks(const float *scores, int P, int c, int n_keep, bool whole_chunks, Emit emit) {
  constexpr int NW = T / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int C = (P + c - 1) / c;
  // exact budget: ceil(n_keep / c) chunks, the lowest-ranked one cut; whole-chunk mode: floor(n_keep / c)
  // chunks (at most C), none cut
  const int m0 = n_keep <= 0 || C <= 0 ? 0 : (whole_chunks ? (n_keep / c < C ? n_keep / c : C) : (n_keep + c - 1) / c);
  if (m0 <= 0) return {0, 0};
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
      for (int i0 = tid; i0 < C; i0 += 8 * T) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = scores[i0 + j * T < C ? i0 + j * T : C - 1];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (i0 + j * T < C) f(i0 + j * T, order_key(x[j]) - low);
      }
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
    if (total >= n_keep || whole_chunks) break;
    m = m0 + 1;  // tail selected and budget short by < c tokens: exactly one more chunk is needed
    __syncthreads();
    if (tid == 0) s_nlist = 0;
  }
  const int size_trunc = thr_idx == C - 1 ? tail_size : c;
  const int len_trunc = whole_chunks ? size_trunc : n_keep - (total - size_trunc);

  ranked([&](int i, uint32_t key) { return key > thr || (key == thr && i <= thr_idx); },
         [&](int i, int pos) {
           emit(i, pos, i == thr_idx ? len_trunc : (i == C - 1 ? tail_size : c), pos * c - (i > thr_idx ? size_trunc - len_trunc : 0));
         });
  return {m, whole_chunks ? total : n_keep};
}

}  // namespace ckv
