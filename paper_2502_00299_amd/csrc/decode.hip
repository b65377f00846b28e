// Decoding over the (compressed) cache: one new query token per head attends to every token of K', V'
// (the stage whose cache Eq. 1 sizes and whose latency Section 4.4 tabulates; Algorithm 1's output is its
// input).  out_i = sum_t softmax_t(scale * q_i . k_t) v_t, query head i reading kv-head i / g.
//
// This file holds the vector-ALU kernel and the merge of the key ranges.  16-bit caches go to the matrix-core kernel of
// decode_mfma.hip; here remain fp32 caches, and 16-bit ones whose rows are more than 64 MB apart, one head at a time.
//
// Bound by HBM bandwidth: every K and V row is read once, and the g dot products and g axpys of an fp32 row are within the
// vector ALU's rate.  A row (d elements) is spread over LPR = d * element size / 16 lanes, 16 bytes each, so one load
// instruction of a wavefront reads 64 / LPR consecutive rows as one contiguous piece.  The lanes of a row reduce their
// partial dot products with DPP adds (no LDS).  Each group of LPR lanes runs its own online softmax over the
// rows it meets; the groups of a wavefront, the wavefronts of a workgroup and the key ranges of a head are
// merged afterwards by the usual (max, sum, weighted output) rule, always in the same order.
// With 16 lanes per row and 4 heads per workgroup (fp32, d = 64) the 4 x 4 partial dot products of a step are not
// all-reduced but reduce-scattered: the lanes hold them in an order permuted by their own index (the rows
// they load and the heads they keep in registers are XOR-swizzled), so each of the four halving steps is
// one DPP add per kept value and lane (4u + j) of a row group ends with the complete score of row u for
// head j.  That lane alone does the softmax arithmetic of that score; the weights reach the 16 lanes again as DPP
// row broadcasts feeding the value accumulation.
// Grid: x = key range, y = (sequence, kv-head), z = batch of G query heads of the kv-head.
#include <type_traits>
#include <utility>

#include "internal.h"

namespace ckv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kDecodeUnroll = 4;        // row loads of K (and of V) in flight per lane
constexpr float kDecodeNegBig = -1.0e30f;

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_amdgcn_update_dpp(0.f, x, CTRL, 0xf, 0xf, false);
}
// Sum over the LPR lanes that share a row; every lane of the group ends with the same bits.
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0xB1>(x);                          // quad_perm [1,0,3,2]
  x = dpp_add<0x4E>(x);                          // quad_perm [2,3,0,1]
  if constexpr (LPR >= 8) x = dpp_add<0x141>(x);   // row_half_mirror: the other quad of 8 lanes
  if constexpr (LPR >= 16) x = dpp_add<0x140>(x);  // row_mirror: the other half of 16 lanes
  if constexpr (LPR >= 32) x += __shfl_xor(x, 16);
  return x;
}

template <int CTRL>
__device__ __forceinline__ float dpp_get(float x) {
  return __builtin_amdgcn_update_dpp(0.f, x, CTRL, 0xf, 0xf, false);
}
// value of lane N of every row of 16 lanes
template <int N>
__device__ __forceinline__ float row_bcast(float x) {
  return dpp_get<0x150 + N>(x);  // row_newbcast:N
}
template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F f) {
  (f(std::integral_constant<int, I>{}), ...);
}

// 16 bytes of a row as fp32 values (8 for the 16-bit types, 4 for fp32)
template <int DT>
__device__ __forceinline__ void widen16(const u32x4 &r, float (&f)[16 / (DT == CHUNKKV_F32 ? 4 : 2)]) {
  if constexpr (DT == CHUNKKV_F32) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  } else if constexpr (DT == CHUNKKV_BF16) {
    const uint32_t d[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { f[2 * i] = __uint_as_float(d[i] << 16); f[2 * i + 1] = __uint_as_float(d[i] & 0xFFFF0000u); }
  } else {
    const uint32_t d[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f16x2 h = __builtin_bit_cast(f16x2, d[i]);
      f[2 * i] = (float)h[0]; f[2 * i + 1] = (float)h[1];
    }
  }
}

// partial dot product of a lane's 16 bytes of a K row with its 16 bytes of a query row
template <int DT>
__device__ __forceinline__ float dot16(const u32x4 &k, const u32x4 &q) {
  if constexpr (DT == CHUNKKV_F32) {
    float s = __uint_as_float(k.x) * __uint_as_float(q.x);
    s = __builtin_fmaf(__uint_as_float(k.y), __uint_as_float(q.y), s);
    s = __builtin_fmaf(__uint_as_float(k.z), __uint_as_float(q.z), s);
    return __builtin_fmaf(__uint_as_float(k.w), __uint_as_float(q.w), s);
  } else if constexpr (DT == CHUNKKV_BF16) {
    // the pairs are taken from whole-vector casts: a bit cast of a single vector element reads element 0
    const bf16x8 kk = __builtin_bit_cast(bf16x8, k), qq = __builtin_bit_cast(bf16x8, q);
    float s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kk, kk, 0, 1), __builtin_shufflevector(qq, qq, 0, 1), 0.f, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kk, kk, 2, 3), __builtin_shufflevector(qq, qq, 2, 3), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kk, kk, 4, 5), __builtin_shufflevector(qq, qq, 4, 5), s, false);
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(kk, kk, 6, 7), __builtin_shufflevector(qq, qq, 6, 7), s, false);
  } else {
    const f16x8 kk = __builtin_bit_cast(f16x8, k), qq = __builtin_bit_cast(f16x8, q);
    float s = __builtin_amdgcn_fdot2(__builtin_shufflevector(kk, kk, 0, 1), __builtin_shufflevector(qq, qq, 0, 1), 0.f, false);
    s = __builtin_amdgcn_fdot2(__builtin_shufflevector(kk, kk, 2, 3), __builtin_shufflevector(qq, qq, 2, 3), s, false);
    s = __builtin_amdgcn_fdot2(__builtin_shufflevector(kk, kk, 4, 5), __builtin_shufflevector(qq, qq, 4, 5), s, false);
    return __builtin_amdgcn_fdot2(__builtin_shufflevector(kk, kk, 6, 7), __builtin_shufflevector(qq, qq, 6, 7), s, false);
  }
}

// DT: chunkkv_dtype, HD: head dim, G: query heads of the kv-head handled by one workgroup, NW: its wavefronts
template <int DT, int HD, int G, int NW>
__global__ __launch_bounds__(NW * 64) void decode_kernel(DecodeArgs a) {
  constexpr int ESZ = DT == CHUNKKV_F32 ? 4 : 2;
  constexpr int ROWB = HD * ESZ;
  constexpr int LPR = ROWB / 16;   // lanes per row
  constexpr int RPW = 64 / LPR;    // rows per wavefront load
  constexpr int EPL = 16 / ESZ;    // elements per lane
  constexpr int U = kDecodeUnroll;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int grp = lane / LPR, seg = lane % LPR;
  const int h = blockIdx.y;
  int bl = 0, split = blockIdx.x;   // range of any sequence: no workgroups beyond the ranges of a short one
  while (bl + 1 < kMaxBatchPerLaunch && (int)blockIdx.x >= CKV_ARG(DecodeArgs, cut.first_split, bl + 1)) ++bl;
  if (bl > 0) split -= CKV_ARG(DecodeArgs, cut.first_split, bl);
  const int g = a.n_q_heads / a.n_kv_heads;
  const int j0 = blockIdx.z * G;  // first query head (within the kv-head's group) of this workgroup
  const int b = a.batch0 + bl;

  // tokens of this (sequence, kv-head): the capacity of the cache, or the caller's count clamped to it
  const int cap = CKV_ARG(DecodeArgs, n_tok, bl);
  int n = cap;
  if (a.kv_len != nullptr) {
    n = a.kv_len[(int64_t)b * a.n_kv_heads + h];
    n = n < 0 ? 0 : (n > cap ? cap : n);
  }
  const int rps = CKV_ARG(DecodeArgs, cut.rows_per_split, bl);
  const int r0 = split * rps;
  const int r1 = r0 + rps < n ? r0 + rps : n;
  if (r0 >= n && split > 0) return;   // the merge knows how many ranges hold rows

  const int64_t head_off = (CKV_ARG(DecodeArgs, base, bl) + (int64_t)h * a.stride_head) * ESZ;
  const char *kbase = (const char *)a.k + head_off + seg * 16;
  const char *vbase = (const char *)a.v + head_off + seg * 16;
  const int64_t tok = a.stride_tok * ESZ;

  // reduce-scatter variant (see the file header): lane (4 * ub + jb) of a row group owns row ub, head jb
  constexpr bool kScatter = LPR == 16 && U == 4 && G == 4;
  const int ub = kScatter ? (lane & 15) >> 2 : 0, jb = kScatter ? lane & 3 : 0;

  u32x4 qreg[G];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int jh = j ^ jb;   // register j holds head j ^ jb
    qreg[j] = u32x4{0, 0, 0, 0};
    if (j0 + jh < g)
      qreg[j] = *(const u32x4 *)((const char *)a.q + ((int64_t)b * a.n_q_heads + (int64_t)h * g + j0 + jh) * ROWB + seg * 16);
  }
  float m_own = kDecodeNegBig, l_own = 0.f;   // scatter variant: statistics of the head this lane owns
  float m[G], l[G], o[G][EPL];
#pragma unroll
  for (int j = 0; j < G; ++j) {
    m[j] = kDecodeNegBig;
    l[j] = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[j][e] = 0.f;
  }
  const float c1 = a.scale_log2e;

  // rows r0 .. r1-1; a step of the workgroup covers NW * U * RPW consecutive rows
  constexpr bool kAhead = NW > 4;   // the rows of the next step are on their way while those of this one are worked on
  u32x4 kr[U], vr[U], kn[U], vn[U];
  auto load = [&](int base, u32x4 (&k)[U], u32x4 (&v)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int rowv = base + u * RPW + grp;           // V: register u holds row u
      const int rowk = base + (u ^ ub) * RPW + grp;    // K: register u holds row u ^ ub (ub = 0 without the swizzle)
      // every row is read once: streaming (non-temporal) loads
      k[u] = __builtin_nontemporal_load((const u32x4 *)(kbase + (int64_t)(rowk < r1 ? rowk : r1 - 1) * tok));  // r1 >= 1: there are rows
      v[u] = __builtin_nontemporal_load((const u32x4 *)(vbase + (int64_t)(rowv < r1 ? rowv : r1 - 1) * tok));
    }
  };
  const int base0 = r0 + wave * (U * RPW);
  if (kAhead && base0 < r1) load(base0, kn, vn);
  for (int base = base0; base < r1; base += NW * U * RPW) {
    if constexpr (kAhead) {
#pragma unroll
      for (int u = 0; u < U; ++u) { kr[u] = kn[u]; vr[u] = vn[u]; }
      if (base + NW * U * RPW < r1) load(base + NW * U * RPW, kn, vn);
    } else {
      load(base, kr, vr);
    }
    if constexpr (kScatter) {
      float x[U][G];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int jj = 0; jj < G; ++jj) x[u][jj] = dot16<DT>(kr[u], qreg[jj]);
      // four halving steps; the partner lane differs in bit 3 / bits 0-2 / bit 1 / bit 0 of the lane index
      float y[2][G], z[G], t[2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int jj = 0; jj < G; ++jj) y[u][jj] = x[u][jj] + dpp_get<0x128>(x[u ^ 2][jj]);   // row_ror:8
#pragma unroll
      for (int jj = 0; jj < G; ++jj) z[jj] = y[0][jj] + dpp_get<0x141>(y[1][jj ^ 3]);         // row_half_mirror
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) t[jj] = z[jj] + dpp_get<0x4E>(z[jj ^ 2]);                // quad_perm [2,3,0,1]
      const float r = t[0] + dpp_get<0xB1>(t[1]);                                             // quad_perm [1,0,3,2]
      // r: row ub of the step, head jb.  Softmax statistics per head: maximum over the four rows, which sit in the
      // lanes 4, 8 and 12 further on.
      const float sc = base + ub * RPW + grp < r1 ? r * c1 : -3.0e38f;
      float smax = fmaxf(sc, dpp_get<0x128>(sc));
      smax = fmaxf(smax, dpp_get<0x124>(smax));   // row_ror:4; the value is already the same 8 lanes apart
      if (__builtin_amdgcn_ballot_w64(smax > m_own) != 0) {
        const float m_new = fmaxf(m_own, smax);
        const float f = __builtin_amdgcn_exp2f(m_own - m_new);
        l_own *= f;
        m_own = m_new;
        // the outputs of a head live in all 16 lanes: its factor comes from the lane that owns it
        static_for(std::make_integer_sequence<int, G>{}, [&](auto j_c) __attribute__((always_inline)) {
          constexpr int JJ = decltype(j_c)::value;
          const float fb = row_bcast<JJ>(f);
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[JJ][e] *= fb;
        });
      }
      const float p = __builtin_amdgcn_exp2f(sc - m_own);
      l_own += p;
      static_for(std::make_integer_sequence<int, U>{}, [&](auto u_c) __attribute__((always_inline)) {
        constexpr int UU = decltype(u_c)::value;
        float vf[EPL];
        widen16<DT>(vr[UU], vf);
        static_for(std::make_integer_sequence<int, G>{}, [&](auto j_c) __attribute__((always_inline)) {
          constexpr int JJ = decltype(j_c)::value;
          const float pb = row_bcast<4 * UU + JJ>(p);   // weight of (row UU, head JJ)
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[JJ][e] = __builtin_fmaf(pb, vf[e], o[JJ][e]);
        });
      });
    } else {
      float s[U][G];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool valid = base + u * RPW + grp < r1;
#pragma unroll
        for (int jj = 0; jj < G; ++jj) {
          const float d = row_sum<LPR>(dot16<DT>(kr[u], qreg[jj]));
          s[u][jj] = valid ? d * c1 : -3.0e38f;
        }
      }
#pragma unroll
      for (int jj = 0; jj < G; ++jj) {
        float smax = s[0][jj];
#pragma unroll
        for (int u = 1; u < U; ++u) smax = fmaxf(smax, s[u][jj]);
        if (__builtin_amdgcn_ballot_w64(smax > m[jj]) != 0) {
          const float m_new = fmaxf(m[jj], smax);
          const float f = __builtin_amdgcn_exp2f(m[jj] - m_new);
          l[jj] *= f;
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[jj][e] *= f;
          m[jj] = m_new;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) s[u][jj] = __builtin_amdgcn_exp2f(s[u][jj] - m[jj]);  // now the weight p
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float vf[EPL];
        widen16<DT>(vr[u], vf);
#pragma unroll
        for (int jj = 0; jj < G; ++jj) {
          l[jj] += s[u][jj];
#pragma unroll
          for (int e = 0; e < EPL; ++e) o[jj][e] = __builtin_fmaf(s[u][jj], vf[e], o[jj][e]);
        }
      }
    }
  }
  if constexpr (kScatter) {
    // back to the replicated form the merges below expect: every lane learns (m, l) of every head
    float lsum = l_own + dpp_get<0x128>(l_own);
    lsum += dpp_get<0x124>(lsum);
    static_for(std::make_integer_sequence<int, G>{}, [&](auto j_c) __attribute__((always_inline)) {
      constexpr int JJ = decltype(j_c)::value;
      m[JJ] = row_bcast<JJ>(m_own);
      l[JJ] = row_bcast<JJ>(lsum);
    });
  }

  // merge the row groups of the wavefront (lanes that hold the same 16 bytes of the row)
#pragma unroll
  for (int x = LPR; x < 64; x *= 2) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      const float m_o = __shfl_xor(m[j], x), l_o = __shfl_xor(l[j], x);
      const float M = fmaxf(m[j], m_o);
      const float fa = __builtin_amdgcn_exp2f(m[j] - M), fb = __builtin_amdgcn_exp2f(m_o - M);
      l[j] = l[j] * fa + l_o * fb;
#pragma unroll
      for (int e = 0; e < EPL; ++e) o[j][e] = o[j][e] * fa + __shfl_xor(o[j][e], x) * fb;
      m[j] = M;
    }
  }
  // merge the wavefronts through LDS: thread (j, seg) folds the states in wavefront order
  __shared__ float s_m[NW][G][LPR], s_l[NW][G][LPR], s_o[NW][G][LPR][EPL];
  if (grp == 0) {
#pragma unroll
    for (int j = 0; j < G; ++j) {
      s_m[wave][j][seg] = m[j];
      s_l[wave][j][seg] = l[j];
#pragma unroll
      for (int e = 0; e < EPL; ++e) s_o[wave][j][seg][e] = o[j][e];
    }
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < G * LPR) {
    const int j = t / LPR, sg = t % LPR;
    if (j0 + j < g) {
      float M = s_m[0][j][sg];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][j][sg]);
      float Lsum = 0.f, acc[EPL];
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_m[w][j][sg] - M);
        Lsum += s_l[w][j][sg] * f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] += s_o[w][j][sg][e] * f;
      }
      if (a.cut.n_split == 1) {   // one range per head: no merge kernel follows
        const int64_t hd = (int64_t)b * a.n_q_heads + (int64_t)h * g + j0 + j;
        float *out = a.out + hd * HD + sg * EPL;
#pragma unroll
        for (int e = 0; e < EPL; ++e) out[e] = Lsum > 0.f ? acc[e] / Lsum : 0.f;
        if (a.lse != nullptr && sg == 0) a.lse[hd] = Lsum > 0.f ? (M + __builtin_log2f(Lsum)) * 0.6931471805599453f : -__builtin_inff();
        return;
      }
      const int64_t slot = (int64_t)CKV_ARG(DecodeArgs, cut.first_split, bl) * a.n_q_heads + ((int64_t)h * g + j0 + j) * CKV_ARG(DecodeArgs, cut.splits, bl) + split;
      if (sg == 0) a.part_ml[slot] = make_float2(M, Lsum);
      float *po = a.part_o + slot * HD + sg * EPL;
#pragma unroll
      for (int e = 0; e < EPL; ++e) po[e] = acc[e];
    }
  }
}

// out = sum_s o_s 2^(m_s - M) / sum_s l_s 2^(m_s - M) over the key ranges of one query head that hold rows.
// grid: x = query head, y = sequence of the slice; 256 threads: a thread owns four consecutive output elements and
// every NG-th key range.  Bound by latency, so the (m, l) pairs and the partial rows are loaded together (one round
// trip) and merged online; the groups are folded through LDS in group order, so the summation order is fixed.
constexpr int kCombineThreads = 256;
template <int HD>
__global__ __launch_bounds__(kCombineThreads) void decode_combine_kernel(DecodeArgs a) {
  constexpr int TPR = HD / 4;                     // threads per partial row
  constexpr int NG = kCombineThreads / TPR;       // key-range groups
  constexpr int UN = 4;
  const int bl = blockIdx.y, hq = blockIdx.x, b = a.batch0 + bl;
  const int64_t head = (int64_t)b * a.n_q_heads + hq;
  int n = CKV_ARG(DecodeArgs, n_tok, bl);
  if (a.kv_len != nullptr) {
    const int x = a.kv_len[(int64_t)b * a.n_kv_heads + hq / (a.n_q_heads / a.n_kv_heads)];
    n = x < 0 ? 0 : (x > n ? n : x);
  }
  const int rps = CKV_ARG(DecodeArgs, cut.rows_per_split, bl);
  const int used = n > 0 ? (n + rps - 1) / rps : 1;
  const int64_t slot = (int64_t)CKV_ARG(DecodeArgs, cut.first_split, bl) * a.n_q_heads + (int64_t)hq * CKV_ARG(DecodeArgs, cut.splits, bl);
  const float2 *ml = a.part_ml + slot;
  const int t = threadIdx.x, col = t % TPR, grp = t / TPR;
  __shared__ float s_acc[NG][HD + 2];
  const float *po = a.part_o + slot * HD + col * 4;
  float acc[4] = {0.f, 0.f, 0.f, 0.f}, m = kDecodeNegBig, lsum = 0.f;
  for (int s0 = grp; s0 < used; s0 += UN * NG) {
    float2 p[UN];
    float4 o4[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int s = s0 + u * NG < used ? s0 + u * NG : s0;
      p[u] = ml[s];
      o4[u] = *(const float4 *)(po + (int64_t)s * HD);
    }
    float mm = m;
#pragma unroll
    for (int u = 0; u < UN; ++u) mm = fmaxf(mm, p[u].x);
    const float f0 = __builtin_amdgcn_exp2f(m - mm);
    lsum *= f0;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= f0;
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const bool on = s0 + u * NG < used;   // what was read in place of a missing range must not count, be it infinite
      const float f = on ? __builtin_amdgcn_exp2f(p[u].x - mm) : 0.f;
      lsum += p[u].y * f;
      acc[0] += on ? o4[u].x * f : 0.f; acc[1] += on ? o4[u].y * f : 0.f;
      acc[2] += on ? o4[u].z * f : 0.f; acc[3] += on ? o4[u].w * f : 0.f;
    }
    m = mm;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) s_acc[grp][col * 4 + e] = acc[e];
  if (col == 0) { s_acc[grp][HD] = lsum; s_acc[grp][HD + 1] = m; }
  __syncthreads();
  if (t < HD) {
    float M = s_acc[0][HD + 1];
#pragma unroll
    for (int g2 = 1; g2 < NG; ++g2) M = fmaxf(M, s_acc[g2][HD + 1]);
    float v = 0.f, L = 0.f;
#pragma unroll
    for (int g2 = 0; g2 < NG; ++g2) {
      const float f = __builtin_amdgcn_exp2f(s_acc[g2][HD + 1] - M);
      v += s_acc[g2][t] * f;
      L += s_acc[g2][HD] * f;
    }
    a.out[head * HD + t] = L > 0.f ? v / L : 0.f;
    if (a.lse != nullptr && t == 0)
      a.lse[head] = L > 0.f ? (M + __builtin_log2f(L)) * 0.6931471805599453f : -__builtin_inff();
  }
}

// fp32 caches; for 16-bit caches only rows more than 64 MB apart come here, one head at a time
template <int DT, int HD, int NW, bool FOUR = true>   // FOUR: compiled for four heads per workgroup
int launch_decode_valu(const DecodeArgs &a, int batch_slice, int g, hipStream_t s) {
  const int G = DT == CHUNKKV_F32 ? decode_heads_per_wg(DT, g) : 1;
  const dim3 grid(a.cut.first_split[batch_slice - 1] + a.cut.splits[batch_slice - 1], a.n_kv_heads, (g + G - 1) / G);
  if (G == 1) hipLaunchKernelGGL((decode_kernel<DT, HD, 1, NW>), grid, dim3(NW * 64), 0, s, a);
  else if constexpr (DT == CHUNKKV_F32) {
    if (G == 2) hipLaunchKernelGGL((decode_kernel<DT, HD, 2, NW>), grid, dim3(NW * 64), 0, s, a);
    else if constexpr (FOUR) hipLaunchKernelGGL((decode_kernel<DT, HD, 4, NW>), grid, dim3(NW * 64), 0, s, a);
    else return CHUNKKV_ERR_UNSUPPORTED;
  }
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

template <int HD>
int launch_decode_f32(const DecodeArgs &a, int batch_slice, int g, hipStream_t s) {
  const int waves = decode_f32_waves(HD, g, a.n_kv_heads, batch_slice, a.cut);
  if (waves == 16) return launch_decode_valu<CHUNKKV_F32, HD, 16, HD != 128>(a, batch_slice, g, s);
  if constexpr (HD == 128)
    if (waves == 8) return launch_decode_valu<CHUNKKV_F32, HD, 8>(a, batch_slice, g, s);
  return launch_decode_valu<CHUNKKV_F32, HD, 4>(a, batch_slice, g, s);
}

template <int HD>
int launch_decode_hd(int dtype, bool matrix_cores, const DecodeArgs &a, int batch_slice, hipStream_t s) {
  const int g = a.n_q_heads / a.n_kv_heads;
  int rc;
  if (matrix_cores) rc = launch_decode_mfma(dtype, HD, a, batch_slice, s);
  else if (dtype == CHUNKKV_BF16) rc = launch_decode_valu<CHUNKKV_BF16, HD, 4>(a, batch_slice, g, s);
  else if (dtype == CHUNKKV_F16) rc = launch_decode_valu<CHUNKKV_F16, HD, 4>(a, batch_slice, g, s);
  else rc = launch_decode_f32<HD>(a, batch_slice, g, s);
  if (rc) return rc;
  if (a.cut.n_split == 1) return CHUNKKV_OK;   // the range kernel wrote the outputs
  hipLaunchKernelGGL((decode_combine_kernel<HD>), dim3(a.n_q_heads, batch_slice), dim3(kCombineThreads), 0, s, a);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

int launch_decode(int dtype, int head_dim, bool matrix_cores, const DecodeArgs &a, int batch_slice, hipStream_t s) {
  if (a.cut.n_split == 0 || batch_slice * a.n_kv_heads == 0) return CHUNKKV_OK;
  if (head_dim == 128) return launch_decode_hd<128>(dtype, matrix_cores, a, batch_slice, s);
  if (head_dim == 64) return launch_decode_hd<64>(dtype, matrix_cores, a, batch_slice, s);
  return CHUNKKV_ERR_UNSUPPORTED;
}

}  // namespace ckv
