// Single-pass observation-window scoring (Algorithm 1, first two steps) for bf16 and fp16 caches, head_dim 128,
// chunk sizes that divide 80 into a multiple of four chunks (5, 10, 20).
//
// K is streamed ONCE and nothing is rounded below fp32.  For every window row r the kernel keeps a reference
// m_r and forms e = exp2(logit * scale * log2e - m_r) in fp32 for every key; the e of one chunk are added up in
// registers, so after a PERIOD of 160 keys a lane holds the sums E[chunk][r] of the chunks it owns, relative to
// m_r.  These per-(chunk, row) sums and the reference they are relative to go to the workspace; the row's total
// follows from them (plus the window keys, which belong to no chunk).  A second, small kernel
// (single_scores_kernel in score_misc.hip) merges the per-range (reference, sum) pairs of a row into
// ref_r = m_r + log2(sum_r) and forms score[chunk] = sum_r E[chunk][r] * exp2(m[chunk][r] - ref_r).
//
// Who owns which key.  The logits come from v_mfma_f32_32x32x16 with the keys as the M dimension: a lane owns
// one window row (N index) and, of the 32 keys of a block, the 16 whose M index has bit 2 equal to its lane
// half.  Which key sits at which M index is the kernel's choice (the operand fragments are read from LDS row
// by row), and it is chosen so that both lane halves see the SAME chunk pattern in their registers: the chunks
// of a period alternate between the halves (half h owns chunks h, h + 2, ...), and register v of step t of a
// period holds position u = 16 t + v of the lane half's own sequence of 80 keys.  Position u belongs to own
// chunk u / c: a compile-time function of (t, v), so every exponential is added to its chunk's register with
// one plain add, no matrix product and no cross-lane traffic.
//
// The reference is lazy.  fp32 has room for e up to 2^100 before the sums are in danger, so the reference moves
// only when a step's sum reaches that bound (the first step of a range always does, its reference starts at
// -1e30); the step is then redone against the step's own maximum and the lane's sums are rescaled.  On ordinary
// inputs that happens once per range.  Values more than 2^126 below the reference vanish: their probability is
// below what fp32 chunk scores can represent.
//
// K: HBM -> LDS by buffer loads with an LDS destination (16 bytes per lane, rows past the end of the prefix
// read as zero).  The ring holds two periods; a period is 5 slots of 32 key rows, slot t holding the rows of
// step t in M-index order, so the permutation above lives in the global addresses of the loads and the operand
// reads are "lane register + compile-time slot offset".  The 16-byte segments of a row are XOR-swizzled by the
// M index (global-address side), so the reads of 16 consecutive lanes hit distinct banks.  Slots are refilled twice per
// period, as soon as every wavefront has their fragments in registers, so 32 to 56 KB per workgroup are in flight all the
// time; refilled a period at a time, 40 KB were, and none of it while the last of it was awaited: 16 layers of 131072 tokens
// 1327 -> 1240 us, ten layers of a ragged batch at c = 20 964 -> 858.  The waits count the loads and stores behind the awaited one.
//
// A call on one layer is short: launch, queries, a few periods per workgroup, and code that every workgroup fetches and
// runs through once.  Hence one instance of the period for all periods (the ragged last one masked through the operand the
// products are added to), the window keys in a short loop of their own, the queries through LDS, key ranges of as few as
// four periods, and for the shortest launches two workgroups that share the rows of a key range.  One layer, c = 5, 256 rows,
// 20011 tokens: 46 -> 21 us (of that 16: registers no longer spilled in the loop); 128 rows, 8192 tokens, c = 10: 16.5 -> 12.
//
// A wavefront holds NQ blocks of 32 window rows as resident operand fragments and the four wavefronts of a
// workgroup split the rows, so each K fragment read from LDS feeds NQ matrix instructions.  The work advances
// in micro-steps (one 32-key block against one 32-row block).  The instruction stream of a micro-step is laid
// out by hand: eight slots of one matrix instruction of the NEXT micro-step and the vector work of two keys of
// THIS one.  Everything that is not one of the 16 scalings, 16 exponentials and 16 adds of a micro-step and lane has
// been moved out of the steady state.  What bounds a launch that fills the chip is power: a micro-step takes 150 ns on a few
// CUs and about 200 on all of them, where the clock falls to 1.6 to 1.9 GHz of 2.4; with 128 rows, reads of K as well.
#pragma once
#include <mutex>
#include <type_traits>

#include "score_impl.h"

namespace ckv {

constexpr int kSpPeriod = 160;                          // keys per period
constexpr int kSpHalf = 80;                             // keys of a period one lane half owns
constexpr int kSpSteps = 5;                             // 32-key blocks per period
constexpr int kSpStepBytes = 32 * 256;                  // one ring slot: 32 rows of 128 16-bit values
constexpr int kSpPeriodBytes = kSpSteps * kSpStepBytes; // 40 KB
constexpr int kSpRingBytes = 2 * kSpPeriodBytes;        // two periods
constexpr float kSpBig = 1.2676506e30f;                 // 2^100: a step whose sum reaches this is redone
constexpr int kNonTemporal = 2;                         // cache policy of a buffer access: streaming
constexpr int kSpMaxSeg = 5;                            // chunk segments 16 consecutive keys can touch (c >= 5)

typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));

// four non-negative finite fp32 values -> their rounded upper three bytes, packed into three dwords
__device__ __forceinline__ u32x3 pack24(float x, float y, float z, float w) {
  const uint32_t a = __float_as_uint(x) + 0x80u, b = __float_as_uint(y) + 0x80u;
  const uint32_t c = __float_as_uint(z) + 0x80u, d = __float_as_uint(w) + 0x80u;
  return u32x3{__builtin_amdgcn_perm(b, a, 0x05030201u), __builtin_amdgcn_perm(c, b, 0x06050302u),
               __builtin_amdgcn_perm(d, c, 0x07060503u)};
}

// eight non-negative finite fp32 values -> their upper 20 bits below the sign (8 exponent, 12 mantissa bits,
// rounded: relative 2^-13), packed into five dwords
__device__ __forceinline__ void pack20(const float (&v)[8], u32x4 &lo, uint32_t &hi) {
  uint32_t q[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) q[i] = (__float_as_uint(v[i]) + 0x400u) >> 11;
  lo.x = q[0] | (q[1] << 20);
  lo.y = (q[1] >> 12) | (q[2] << 8) | (q[3] << 28);
  lo.z = (q[3] >> 4) | (q[4] << 16);
  lo.w = (q[4] >> 16) | (q[5] << 4) | (q[6] << 24);
  hi = (q[6] >> 8) | (q[7] << 12);
}

// Nothing about x is known behind this: what follows from it is formed from here on.
__device__ __forceinline__ void opaque(int &x) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass knows no vector registers
  asm volatile("" : "+v"(x));
#endif
}

// period-relative key of position u of lane half 0's own sequence (lane half 1: + C)
template <int C>
__host__ __device__ constexpr int sp_key(int u) { return 2 * C * (u / C) + u % C; }

template <int DT>
__device__ __forceinline__ f32x16 mma0(const u32x4 &a, const u32x4 &b, const f32x16 &c) {  // first product of a chain
  if constexpr (DT == CHUNKKV_BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// DT: chunkkv_dtype (16-bit), C: chunk size, NQ: 32-row blocks per wavefront (rows_pad = 128 * NQ), STREAM: streaming loads of K; smem:
// kSpRingBytes of LDS; a: the kernel's argument
template <int DT, int C, int NQ, bool STREAM>
__device__ __forceinline__ void score_single_range(const ScoreArgs &a, char *smem) {
  static_assert(is_16bit(DT), "the single-pass kernel takes bf16 or fp16 caches");
  static_assert(kSpHalf % C == 0 && (kSpHalf / C) % 4 == 0 && kSpHalf / C <= 16, "chunk size");
  static_assert(NQ == 1 || NQ == 2, "row blocks per wavefront");
  constexpr int S = kSpHalf / C;  // chunks per lane half and period
  constexpr int ROWB = 256, NKS = 8, ESZ = 2;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform, and known to be
  const int n = lane & 31, half = lane >> 5;
  int split = blockIdx.x;
  const int bl = find_sequence(a, split), h = blockIdx.y, z = blockIdx.z / a.row_groups;
  const int row0 = (blockIdx.z % a.row_groups) * (128 * NQ);   // first window row of this workgroup
  const int g = a.n_q_heads / a.n_kv_heads, w = a.window;
  const int L = CKV_ARG(ScoreArgs, seq.seqlen, bl), P = L - w, nrows = g * w;
  const int64_t problem = ((int64_t)CKV_ARG(ScoreArgs, leader, z) * a.batch_total + (a.batch0 + bl)) * a.n_kv_heads + h;

  const int np_total = (L + kSpPeriod - 1) / kSpPeriod;
  const int ppr = single_periods_per_range(np_total);
  const int u0 = split * ppr;
  const int u1 = u0 + ppr < np_total ? u0 + ppr : np_total;
  const int np_prefix = (P + kSpPeriod - 1) / kSpPeriod;   // periods with keys before the window
  const int np = (u1 < np_prefix ? u1 : np_prefix) - u0;   // periods of this workgroup: none, if it has window keys alone
  const int range0 = u0 * kSpPeriod;    // its first key

  const char *qbase = (const char *)CKV_ARG(ScoreArgs, q, z) + ((int64_t)(a.batch0 + bl) * a.n_q_heads + (int64_t)h * g) * w * ROWB;
  const char *kbase = (const char *)CKV_ARG(ScoreArgs, k, z) + (CKV_ARG(ScoreArgs, seq.kv_base, bl) + (int64_t)h * a.kv_stride_head) * ESZ;
  const int64_t ktok = a.kv_stride_tok * ESZ;
  const float c1 = a.scale_log2e;

  // ---- K: HBM -> LDS.  Load j of a wavefront fills rows 8 wave + 4 j .. + 3 of a slot; lane l lands at row
  // 8 wave + 4 j + l / 16, 16-byte position l % 16, and fetches the segment that position holds after the
  // swizzle, of the key that M index stands for in step t.  M index 8 wave + 4 j + b is position
  // u = 16 t + 4 wave + b of lane half j, so the two loads of a step differ by a lane constant.
  uint32_t klane[kSpSteps], kdelta;
  {
    const int b = lane / 16, pos = lane % 16;
    const int seg0 = pos ^ (8 * (wave & 1) + b), seg1 = seg0 ^ 4;   // M index & 15 = 8 (wave & 1) + 4 j + b
#pragma unroll
    for (int t = 0; t < kSpSteps; ++t) {
      const int u = 16 * t + 4 * wave + b;
      klane[t] = (uint32_t)((2 * C * (u / C) + u % C) * (int)ktok + seg0 * 16);
    }
    kdelta = (uint32_t)(C * (int)ktok + (seg1 - seg0) * 16);
  }
  // step T of period prel, into its slot of the ring.  Only prefix keys: window rows in the last period read as zero (its
  // masked logits are minus infinity plus a product, which an infinite key would make NaN), and so do periods that are not
  // there, so that the number of loads in flight is a compile-time constant at every wait.
  auto issue_step = [&](int prel, auto t_c) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value;
    const RingRows rows = ring_rows(range0 + prel * kSpPeriod, P, (uint32_t)ktok, ROWB, prel < np);  // wavefront-uniform
    const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void *)kbase, 0, (int)rows.records, 0x00020000);
    char *dst = smem + (prel & 1) * kSpPeriodBytes + wave * 2048 + T * kSpStepBytes;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, (__attribute__((address_space(3))) void *)dst, 16, klane[T], rows.offset, 0, STREAM ? kNonTemporal : 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, (__attribute__((address_space(3))) void *)(dst + 1024), 16, klane[T] + kdelta, rows.offset, 0, STREAM ? kNonTemporal : 0);
  };
  // The window queries come through the ring as well (a row block is 8 KB, like a step): read straight into operand
  // fragments, every load would touch 32 lines, 10 thousand cycles for 64 KB.  The first steps of K share the way.
  constexpr int kQSlot = NQ == 2 ? 2 : 3;   // ring slots of the row blocks start here
  issue_step(0, std::integral_constant<int, 0>{});
  issue_step(0, std::integral_constant<int, 1>{});
  if constexpr (NQ == 1) issue_step(0, std::integral_constant<int, 2>{});
  {
    const __amdgpu_buffer_rsrc_t qrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)qbase, 0, nrows * ROWB, 0x00020000);   // rows past the last read as zero
    char *dst = smem + (kQSlot + wave * NQ) * kSpStepBytes;
    const uint32_t off = (uint32_t)(row0 + wave * NQ * 32) * ROWB;
#pragma unroll
    for (int j = 0; j < 8 * NQ; ++j) {
      const int row = 4 * (j % 8) + lane / 16;
      // (no scalar offset: a wavefront without rows starts behind the last record)
      const uint32_t vo = off + (uint32_t)(j / 8 * kSpStepBytes + row * ROWB + ((lane % 16) ^ (row & 15)) * 16);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(qrsrc, (__attribute__((address_space(3))) void *)(dst + j * 1024), 16, vo, 0, 0, 0);
    }
  }

  // wavefronts whose rows are all padding only move K
  const bool active = row0 + wave * NQ * 32 < nrows;

  float m_run[NQ], l_run[NQ], slot[NQ][S];
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi) {
    m_run[qi] = kNegBig;
    l_run[qi] = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) slot[qi][s] = 0.f;
  }

  // ---- K operand fragments: lane (n, half) reads row n of a slot, segment 2 ks + half, at its swizzled position.
  // kaddr points into the ring half the reads currently go to; it is flipped (all values are below 8 KB, the
  // half offset 0xA000 has no bit in common with them) when the reads cross into the next period.
  uint32_t kaddr[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) kaddr[ks] = (uint32_t)(n * ROWB + (((2 * ks + half) ^ (n & 15)) * 16));
  static_assert(kSpPeriodBytes == 0xA000 && 32 * ROWB <= 0x2000, "ring half flip");
  // window queries: resident operand fragments (lane n: row n of the block, elements 16 ks + 8 half ..)
  u32x4 qf[NQ][NKS];
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
  for (int qi = 0; qi < NQ; ++qi)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[qi][ks] = *(const u32x4 *)(smem + (kaddr[ks] + (uint32_t)((kQSlot + wave * NQ + qi) * kSpStepBytes)));
  lds_barrier();   // every wavefront's rows are in registers and its part of the first steps has landed
  if constexpr (NQ == 2) issue_step(0, std::integral_constant<int, 2>{});
  issue_step(0, std::integral_constant<int, 3>{});
  issue_step(0, std::integral_constant<int, 4>{});
  issue_step(1, std::integral_constant<int, 0>{});
  issue_step(1, std::integral_constant<int, 1>{});
  issue_step(1, std::integral_constant<int, 2>{});
  issue_step(1, std::integral_constant<int, 3>{});
  auto frag = [&](auto t_c, int ks) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value;
    return *(const u32x4 *)(smem + (kaddr[ks] + (uint32_t)(T * kSpStepBytes)));
  };

  // Two accumulator tiles: the matrix instructions of micro-step mu + 1 (one key block against one row block)
  // fill one while the exponentials of micro-step mu read the other.  All eight K fragments of the current
  // block are resident; fragment ks is re-read for the next block right behind its last product.
  f32x16 acc[2];
  u32x4 kf[NKS];
  // E and the references of this problem (byte offsets inside stay below 2^32).  Layout per period, with a
  // group = eight chunk sums of one lane half as 20-bit floats: [lane half][group][rows_pad] x 16 bytes, then
  // [lane half][group][rows_pad] x 4 bytes (c = 20 has four sums per lane half: [lane half][rows_pad] x 12 bytes,
  // 24-bit floats); m [rows_pad] floats.  Consecutive lanes write consecutive pieces.
  constexpr int G8 = S / 8;                                  // groups of eight sums per lane half
  constexpr int kPeriodRowBytes = S == 4 ? 24 : 2 * G8 * 20;  // E bytes per period and row
  constexpr int kPeriodStores = NQ * (S == 4 ? 2 : 2 * G8 + 1);   // store instructions of a wavefront per period
  // Buffer stores: one address register at a time, and the lane half that has no reference to store has its offset out of
  // range, so the period's end is no branch (which would let the compiler move sums across it).  The wide ones keep the
  // scalar offset a constant: with a register there the compiler takes the data registers for free at once, and the
  // vector instruction behind the store overwrote them before they were read.
  const uint32_t rp = (uint32_t)a.rows_pad;
  const __amdgpu_buffer_rsrc_t e_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (char *)a.e_buf + problem * a.n_periods * a.rows_pad * a.e_row_bytes, 0, (int)((uint32_t)a.n_periods * rp * (uint32_t)kPeriodRowBytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t m_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (char *)a.m_period + problem * a.n_periods * a.rows_pad * 4, 0, (int)((uint32_t)a.n_periods * rp * 4u), 0x00020000);
  const uint32_t lane_row = (uint32_t)(row0 + wave * NQ * 32 + n);
  const uint32_t e_lane = (uint32_t)half * (uint32_t)(S == 4 ? 1 : G8) * rp + lane_row, m_lane = half == 0 ? lane_row * 4u : 0x7FFFFFFFu;
  // What the products of a step are added to: zero, but minus infinity for keys that are not before the window, which
  // only the ragged last period has.  It takes the code of the others: a workgroup would run through code of its own once,
  // and fetching that took longer than four periods.
  f32x16 mask = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const int ragged = P % kSpPeriod != 0 ? P / kSpPeriod - u0 : -1;   // period of the range, if it is in it
  auto set_mask = [&](auto t_c) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value;
    int lim = P % kSpPeriod - C * half;   // first position, as a key of lane half 0, that is not before the window
    opaque(lim);                          // the masks are formed here, not kept for all steps
#pragma unroll
    for (int v = 0; v < 16; ++v) mask[v] = sp_key<C>(16 * T + v) < lim ? 0.f : -__builtin_inff();
  };

  // logits of one micro-step; REFILL: the fragments are re-read from slot TR behind their product
  auto chain = [&](f32x16 &dst, auto qi_c, auto refill_c, auto tr_c) __attribute__((always_inline)) {
    constexpr int QI = decltype(qi_c)::value;
    constexpr bool REFILL = decltype(refill_c)::value;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if (ks == 0) dst = mma0<DT>(kf[0], qf[QI][0], mask);
      else mma<DT>(dst, kf[ks], qf[QI][ks]);  // D[key][row]
      if constexpr (REFILL) kf[ks] = frag(tr_c, ks);
    }
  };

  // exponentials of one micro-step against the current reference: sums per chunk segment of the step
  auto exps = [&](const f32x16 &x, auto qi_c, auto t_c, float (&seg)[kSpMaxSeg]) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value, QI = decltype(qi_c)::value;
    const float negm = -m_run[QI];
    constexpr int U0 = 16 * T;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = fast_exp2(__builtin_fmaf(x[v], c1, negm));
      const int u = U0 + v, sg = u / C - U0 / C;
      seg[sg] = v == 0 || u % C == 0 ? e : seg[sg] + e;
    }
  };

  // The micro-step in issue order: eight slots of one matrix instruction of the NEXT micro-step (with
  // its fragment re-read) and the vector work of two keys of THIS one, software-pipelined over the slots (the
  // scaling of slot k + 1, the exponentials of slot k, the adds of slot k - 1), so that nothing in a slot
  // waits for anything in the same slot and the vector work of a slot takes about as long as its matrix
  // instruction.  Fences keep the compiler from regrouping the slots.
  auto fused = [&](f32x16 &dst, const f32x16 &x, auto qnx_c, auto refill_c, auto tr_c, auto qi_c, auto t_c,
                   float (&seg)[kSpMaxSeg]) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value, QI = decltype(qi_c)::value, QNX = decltype(qnx_c)::value;
    constexpr bool REFILL = decltype(refill_c)::value;
    constexpr int U0 = 16 * T;
    const float negm = -m_run[QI];
    float xs[2], es[2];
    xs[0] = __builtin_fmaf(x[0], c1, negm);
    xs[1] = __builtin_fmaf(x[1], c1, negm);
#pragma unroll
    for (int k = 0; k <= NKS; ++k) {
      if (k < NKS) {
        if (k == 0) dst = mma0<DT>(kf[0], qf[QNX][0], mask);
        else mma<DT>(dst, kf[k], qf[QNX][k]);
        if constexpr (REFILL) kf[k] = frag(tr_c, k);
      }
      // adds of slot k - 1
      if (k >= 1) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int v = 2 * (k - 1) + i, u = U0 + v, sg = u / C - U0 / C;
          const bool first = v == 0 || (u % C == 0);
          seg[sg] = first ? es[i] : seg[sg] + es[i];
        }
      }
      // exponentials of slot k
      if (k < NKS) {
        es[0] = fast_exp2(xs[0]);
        es[1] = fast_exp2(xs[1]);
      }
      // scaling of slot k + 1
      if (k + 1 < NKS) {
        xs[0] = __builtin_fmaf(x[2 * k + 2], c1, negm);
        xs[1] = __builtin_fmaf(x[2 * k + 3], c1, negm);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // One micro-step: (ring hand-over at the micro-step whose reads cross into the next period,) the matrix work
  // of the micro-step after it, the exponentials of this one.
  // prel: period relative to the range; T: step within the period; QI: row block; TILE: accumulator tile that
  // holds this micro-step's logits.
  auto micro = [&](int prel, auto t_c, auto qi_c, auto tile_c) __attribute__((always_inline)) {
    constexpr int T = decltype(t_c)::value, QI = decltype(qi_c)::value, TILE = decltype(tile_c)::value;
    constexpr bool STEP_END = QI == NQ - 1;                 // the next micro-step belongs to the next step
    constexpr int TNX = STEP_END ? (T + 1) % kSpSteps : T;  // its step ...
    constexpr int QNX = STEP_END ? 0 : QI + 1;              // ... and row block
    // if it is the last use of its block's fragments they are re-read for the block after (slot TR)
    constexpr bool REFILL = QNX == NQ - 1;
    constexpr int TR = (TNX + 1) % kSpSteps;
    // Ring hand-over, twice per period: where the re-reads come to step 3 or to the next period's first.  The loads of the steps
    // up to the next hand-over are waited for, with those of four later steps (and the sums of one period, which leave behind
    // the awaited loads) in flight; behind the barrier they are there for all, and every wavefront has the fragments of step
    // TR - 1 in registers, so the slots of the steps up to TR - 2 are free.  At every step: 16 layers of 20011 tokens, c = 5,
    // 225 instead of 218 us, and 32 layers of 32768 tokens with 128 rows 579 instead of 518.
    // With two row blocks per wavefront the first period's step 2 is loaded behind the queries: a wait of its own.
    if constexpr (REFILL && NQ == 2 && TR == 2) {
      if (__builtin_expect(prel == 0, 0)) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(6 * 2));
        __builtin_amdgcn_s_barrier();
      }
    }
    if constexpr (REFILL && (TR == 0 || TR == 3)) {
      if (active && prel >= 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * 2 + kPeriodStores));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * 2));
      __builtin_amdgcn_s_barrier();
      if constexpr (TR == 3) {
        issue_step(prel + 1, std::integral_constant<int, 4>{});
        issue_step(prel + 2, std::integral_constant<int, 0>{});
        issue_step(prel + 2, std::integral_constant<int, 1>{});
      } else {
        issue_step(prel + 2, std::integral_constant<int, 2>{});
        issue_step(prel + 2, std::integral_constant<int, 3>{});
      }
    }
    if constexpr (REFILL && TR == 0) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) kaddr[ks] ^= (uint32_t)kSpPeriodBytes;
    }
    if (active) {
      // (at the very end of the range the matrix work multiplies stale rows of the ring: in bounds, never used)
      if constexpr (STEP_END)
        if (__builtin_expect(prel + (T == kSpSteps - 1 ? 1 : 0) == ragged, 0)) set_mask(std::integral_constant<int, TNX>{});
      float seg[kSpMaxSeg];
      constexpr int NSEG = (16 * T + 15) / C - (16 * T) / C + 1;
      static_assert(NSEG <= kSpMaxSeg, "segments per step");
      fused(acc[TILE ^ 1], acc[TILE], std::integral_constant<int, QNX>{}, std::integral_constant<bool, REFILL>{},
            std::integral_constant<int, TR>{}, qi_c, t_c, seg);
      float tot = seg[0];
#pragma unroll
      for (int sg = 1; sg < NSEG; ++sg) tot += seg[sg];
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(tot >= kSpBig) != 0, 0)) {
        // rare: a sum reached 2^100 (always on the first step of a range).  Lanes that did move their
        // reference to the step's own maximum, rescale what they hold and redo the step.
        float bm = acc[TILE][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) bm = fmaxf(bm, acc[TILE][v]);
        // the two lane halves of a row move together, so a row has one reference per period
        bm = fmaxf(bm, __shfl_xor(bm, 32));
        const bool mine = __shfl_xor(tot, 32) >= kSpBig || tot >= kSpBig;
        const float m_new = mine ? bm * c1 : m_run[QI];
        const float f = fast_exp2(m_run[QI] - m_new);
#pragma unroll
        for (int s = 0; s < S; ++s) slot[QI][s] *= f;
        l_run[QI] *= f;
        m_run[QI] = m_new;
        exps(acc[TILE], qi_c, t_c, seg);
      }
      // commit: every segment goes to its chunk's register (the first segment of a chunk in a period starts
      // the register afresh)
#pragma unroll
      for (int sg = 0; sg < NSEG; ++sg) {
        constexpr int SL0 = (16 * T) / C;
        const int sl = SL0 + sg;
        const bool fresh = sl * C >= 16 * T;
        slot[QI][sl] = fresh ? seg[sg] : slot[QI][sl] + seg[sg];
      }
      if constexpr (T == kSpSteps - 1) {
        // end of the period: the sums and the reference they are relative to leave the lane.  Streaming
        // (non-temporal) stores: the 1.2 GB a launch writes is read back by the next kernel only, and a read
        // that follows plain stores of that size runs at 4.5 TB/s instead of 6 (the write-back competes)
        float sum = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s) sum += slot[QI][s];
        l_run[QI] += sum;
        const uint32_t pbase = (uint32_t)(u0 + prel) * rp, ebase = pbase * (uint32_t)kPeriodRowBytes;   // wavefront-uniform
        constexpr uint32_t row = QI * 32;
        if constexpr (S == 4) {
          __builtin_amdgcn_raw_buffer_store_b96(pack24(slot[QI][0], slot[QI][1], slot[QI][2], slot[QI][3]), e_rsrc,
                                                (int)(e_lane * 12u + (ebase + row * 12u)), 0, kNonTemporal);
        } else {
#pragma unroll
          for (int g8 = 0; g8 < G8; ++g8) {
            float v8[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v8[i] = slot[QI][8 * g8 + i];
            u32x4 lo;
            uint32_t hi;
            pack20(v8, lo, hi);
            const uint32_t cell = (uint32_t)g8 * rp + row;
            __builtin_amdgcn_raw_buffer_store_b128(lo, e_rsrc, (int)(e_lane * 16u + (ebase + cell * 16u)), 0, kNonTemporal);
            __builtin_amdgcn_raw_buffer_store_b32(hi, e_rsrc, (int)(e_lane * 4u + (ebase + (uint32_t)(2 * G8) * rp * 16u + cell * 4u)), 0, kNonTemporal);
          }
        }
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m_run[QI]), m_rsrc, (int)m_lane, (int)((pbase + row) * 4u), kNonTemporal);
      }
    }
  };

  // one step (all row blocks of the wavefront); P0: accumulator tile of the step's first micro-step
  auto step = [&](int prel, auto t_c, auto p0_c) __attribute__((always_inline)) {
    constexpr int P0 = decltype(p0_c)::value;
    micro(prel, t_c, std::integral_constant<int, 0>{}, std::integral_constant<int, P0>{});
    if constexpr (NQ == 2)
      micro(prel, t_c, std::integral_constant<int, 1>{}, std::integral_constant<int, P0 ^ 1>{});
  };
  auto period = [&](int prel) __attribute__((always_inline)) {
    constexpr int ALT = NQ == 1 ? 1 : 0;  // the tile alternates from step to step
    step(prel, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    step(prel, std::integral_constant<int, 1>{}, std::integral_constant<int, ALT>{});
    step(prel, std::integral_constant<int, 2>{}, std::integral_constant<int, 0>{});
    step(prel, std::integral_constant<int, 3>{}, std::integral_constant<int, ALT>{});
    step(prel, std::integral_constant<int, 4>{}, std::integral_constant<int, 0>{});
    if constexpr (NQ == 1) acc[0] = acc[1];   // an odd number of micro-steps: the next period starts with the same tile
  };

  // ---- fragments of block 0, logits of micro-step 0
  if (active && np > 0) {
    if (ragged == 0) set_mask(std::integral_constant<int, 0>{});
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) kf[ks] = frag(std::integral_constant<int, 0>{}, ks);
    chain(acc[0], std::integral_constant<int, 0>{}, std::integral_constant<bool, NQ == 1>{}, std::integral_constant<int, 1>{});
  }
  for (int prel = 0; prel < np; ++prel) period(prel);

  // ---- window keys, which count for the row sums only: the last range takes them, 32 at a time in their order, each
  // against its own maximum.  All of them fit the ring (no more than 256 rows of one head).
  if (u1 == np_total) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    lds_barrier();   // the ring is dead
    const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc((void *)kbase, 0, (int)((uint32_t)(L - 1) * (uint32_t)ktok + ROWB), 0x00020000);
    const uint32_t row = (uint32_t)(8 * wave + lane / 16), seg = (uint32_t)((lane % 16) ^ (int)(row & 15));
    for (int key0 = P, sl = 0; key0 < L; key0 += 32, ++sl) {
      char *dst = smem + sl * kSpStepBytes + wave * 2048;
      const uint32_t vo = row * (uint32_t)ktok + seg * 16u, v1 = (row + 4u) * (uint32_t)ktok + (seg ^ 4u) * 16u, off = (uint32_t)key0 * (uint32_t)ktok;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, (__attribute__((address_space(3))) void *)dst, 16, vo, off, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(krsrc, (__attribute__((address_space(3))) void *)(dst + 1024), 16, v1, off, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    lds_barrier();
    if (active) {
      for (int key0 = P, sl = 0; key0 < L; key0 += 32, ++sl) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) kf[ks] = *(const u32x4 *)(smem + ((kaddr[ks] & 0x1FFFu) + (uint32_t)(sl * kSpStepBytes)));
#pragma unroll
        for (int qi = 0; qi < NQ; ++qi) {
          f32x16 x = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks) mma<DT>(x, kf[ks], qf[qi][ks]);
          const int r = row0 + (wave * NQ + qi) * 32 + n;
          const int lim = P + (r < nrows ? r % w : 0) - key0 - 4 * half;   // last key the row may see
          float bm = kNegBig;
#pragma unroll
          for (int v = 0; v < 16; ++v) bm = fmaxf(bm, 8 * (v / 4) + v % 4 <= lim ? x[v] : kNegBig);
          bm = fmaxf(bm, __shfl_xor(bm, 32));   // the lane halves of a row share its reference
          const float m_new = fmaxf(m_run[qi], bm * c1);
          float sum = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) sum += 8 * (v / 4) + v % 4 <= lim ? fast_exp2(__builtin_fmaf(x[v], c1, -m_new)) : 0.f;
          l_run[qi] = __builtin_fmaf(l_run[qi], fast_exp2(m_run[qi] - m_new), sum);
          m_run[qi] = m_new;
        }
      }
    }
  }

  // the range's sum of every row for the merge (the lane halves share the reference): relative to the reference of its last
  // period, which is in the workspace already, and in the last range to one of its own, which the window keys may have moved
  if (active) {
#pragma unroll
    for (int qi = 0; qi < NQ; ++qi) {
      const int row = row0 + (wave * NQ + qi) * 32 + n;
      const float l = l_run[qi] + __shfl_xor(l_run[qi], 32);
      if (half == 0) a.row_stats[(problem * a.max_split + split) * a.rows_pad + row] = l;
      if (half == 0 && u1 == np_total && row < nrows) a.refs[problem * nrows + row] = m_run[qi];
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // the empty loads past the last step still write zeros into the ring
}

template <int DT, int C, int NQ, bool STREAM>
__global__ __launch_bounds__(kThreads, 2) void score_single_kernel(ScoreArgs a) {
  extern __shared__ __align__(16) char smem[];
  score_single_range<DT, C, NQ, STREAM>(a, smem);
}

// Layers of different chunk sizes in one launch: a workgroup runs the code of its layer's.
template <int DT, int NQ, bool STREAM>
__global__ __launch_bounds__(kThreads, 2) void score_single_mixed_kernel(ScoreArgs a) {
  extern __shared__ __align__(16) char smem[];
  const int c = CKV_ARG(ScoreArgs, chunk_of, blockIdx.z / a.row_groups);
  if (c == 5) score_single_range<DT, 5, NQ, STREAM>(a, smem);
  else if (c == 10) score_single_range<DT, 10, NQ, STREAM>(a, smem);
  else score_single_range<DT, 20, NQ, STREAM>(a, smem);
}

template <typename Kernel>
int launch_single(Kernel kern, std::once_flag &once, hipError_t &attr_rc, const ScoreArgs &a, dim3 grid, hipStream_t s) {
  std::call_once(once, [&] {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kSpRingBytes);
  });
  if (attr_rc != hipSuccess) return CHUNKKV_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, grid, dim3(kThreads), kSpRingBytes, s, a);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}
template <int DT, int C, int NQ, bool STREAM>
int launch_single_cfg(const ScoreArgs &a, dim3 grid, hipStream_t s) {
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  return launch_single(score_single_kernel<DT, C, NQ, STREAM>, once, attr_rc, a, grid, s);
}
template <int DT, int NQ, bool STREAM>
int launch_single_mixed(const ScoreArgs &a, dim3 grid, hipStream_t s) {
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  return launch_single(score_single_mixed_kernel<DT, NQ, STREAM>, once, attr_rc, a, grid, s);
}

// every compiled geometry of one storage type: chunk size x row blocks per wavefront x streaming loads
template <int DT, int NQ, bool STREAM>
int launch_single_chunk(const ScoreArgs &a, dim3 grid, hipStream_t s) {
  if (a.mixed_chunks) return launch_single_mixed<DT, NQ, STREAM>(a, grid, s);
  switch (a.chunk) {
    case 5: return launch_single_cfg<DT, 5, NQ, STREAM>(a, grid, s);
    case 10: return launch_single_cfg<DT, 10, NQ, STREAM>(a, grid, s);
    case 20: return launch_single_cfg<DT, 20, NQ, STREAM>(a, grid, s);
    default: return CHUNKKV_ERR_UNSUPPORTED;
  }
}
template <int DT>
int launch_single_dt(const ScoreArgs &a, dim3 grid, hipStream_t s) {
  const int nq = a.rows_pad / (128 * a.row_groups);
  if (nq == 1) return a.stream_k ? launch_single_chunk<DT, 1, true>(a, grid, s) : launch_single_chunk<DT, 1, false>(a, grid, s);
  if (nq == 2) return a.stream_k ? launch_single_chunk<DT, 2, true>(a, grid, s) : launch_single_chunk<DT, 2, false>(a, grid, s);
  return CHUNKKV_ERR_UNSUPPORTED;
}

}  // namespace ckv
