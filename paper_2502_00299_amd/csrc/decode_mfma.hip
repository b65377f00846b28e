// Decode attention over 16-bit caches on the matrix cores (one query token per head over every token of K, V).
//
// Bound by HBM bandwidth: every K and V row is read once.  The vector ALU cannot keep up with that stream once a
// kv-head serves more than four query heads (two dot products' worth of work per loaded value and head), so both
// contractions run on the matrix cores and the vector work per 32 keys is one exponential per key and head.
// Measured against the streaming vector-ALU kernel this replaced for 16-bit caches (d = 128, per layer with the merge):
// eight sequences of 10 to 55 thousand tokens with 7 heads per kv-head 142 -> 97 us (4.0 -> 5.9 TB/s), 13171 tokens with 4
// heads 18.9 -> 15.7 us, 848 tokens 13.4 -> 10.0 us.  Short caches are bound by latency: launch, arguments, first rows,
// merge of the wavefronts.
//
//   scores   S[key][head] = K Q^T   v_mfma_f32_16x16x32: keys are the M dimension (16 per tile, two tiles of a
//            32-key step), query heads the N dimension.  A lane ends with the scores of keys 4q..4q+3 of both
//            tiles (q = lane / 16) for head column lane % 16.
//   output   O^T[dim][head] = V^T P^T: the weights sit exactly where the B operand wants them (eight keys of one
//            head column per lane), V^T comes out of LDS with transposing reads (ds_read_b64_tr_b16).
//
// 16 head columns are more than the G = 4 or 8 heads of a workgroup, and the spare ones carry precision: a weight is
// an fp32 number and the operands are 16 bits wide, so it is cut into parts whose sum it is.  bf16: the upper 8 bits of
// what is left, three times, exact.  fp16: 11 bits of what is left, four times, the parts scaled up by 2^15, 2^26, 2^37
// and 2^48 so that they stay in range: exact for weights down to 2^-49 (34 nats below the reference, which is within a
// factor of 2 of the largest weight so far), and below that what is cut off is less than 2^-72.
// With G = 4 the parts of a head occupy columns h, h + 4, h + 8 and h + 12 of one product; with G = 8 the first two parts
// share one product and the others a second one.  Products of 16-bit numbers are exact in the fp32 accumulators, so
// nothing else is rounded below fp32.
//
// A part may be zero under a weight that is not, and zero times an infinite value is NaN.  So a workgroup whose merged
// output holds something that is not finite goes through its rows a second time with every part at least the type's
// least number, and takes those elements from there: an infinity stays one.  Ordinary caches never do; the check costs
// them one barrier.
//
// The reference of the online softmax is lazy: it moves when a step's weights of a head column reach 16 (bf16: their
// sum; fp16: when one reaches 1.97, the range its scaled parts have room for), a few times per wavefront.  The bound
// is kept this low for accuracy: an exponential of 2^x carries the rounding of x, an ulp of |x|.
//
// Memory: every wavefront streams its own 32-key steps through its own LDS slots (K and V separately) by buffer loads
// with an LDS destination; there is no barrier in the loop.  As soon as the K fragments of a step are in registers
// its K slot is refilled, as soon as the V fragments are read its V slot is.  A workgroup holds 64 KB of slots and two
// fit a CU (measured against one workgroup of 128 KB: the same 6.1 TB/s over one 131072-token sequence, 104 against
// 109 us over eight sequences of 10 to 55 thousand tokens in 1024 ranges: the second workgroup covers the ends of the
// first).  16-byte segments are XOR-swizzled on the global-address side so that both the
// fragment reads and the transposing reads touch all banks evenly.  The buffer descriptor covers exactly the rows of
// a step that are there: rows past the end read as zero.
// Grid: x = key range, y = (batch of G query heads, kv-head), z = sequence.
#include <mutex>
#include <type_traits>

#include "internal.h"

namespace ckv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __fp16 fp16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int kStepKeys = 32;
static constexpr float kNegBig = -1.0e30f;

template <int DT>
__device__ __forceinline__ f32x4 mma16(const u32x4 &a, const u32x4 &b, const f32x4 &c) {
  if constexpr (DT == CHUNKKV_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// lane i of a row of 16 gets the value of lane i + N
template <int N>
__device__ __forceinline__ float row_shl(float x) {
  return __builtin_amdgcn_update_dpp(0.f, x, 0x100 + N, 0xf, 0xf, true);
}

// Transposing reads of four 16-dim pieces of V, keys 4 q .. of both 16-key tiles (the second `OFF` bytes further on).
// One assembly block with its own wait: the compiler takes the builtin for a read of everything that is on its way
// into LDS and would wait for all of it.
template <int OFF>
__device__ __forceinline__ void read_v4(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x4 (&v)[4]) {
  uint64_t x[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:%12\n\t"
      "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
      : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "n"(OFF)
      : "memory");
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = u32x4{(uint32_t)x[2 * i], (uint32_t)(x[2 * i] >> 32), (uint32_t)x[2 * i + 1], (uint32_t)(x[2 * i + 1] >> 32)};
}

constexpr int vm_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0F70; }

// The integer form of isfinite, kept from the optimizer: the build lets it assume that nothing is NaN.
__device__ __forceinline__ bool finite_bits(float x) {
  uint32_t u = __float_as_uint(x);
  asm("" : "+v"(u));
  return (u & 0x7F800000u) != 0x7F800000u;
}

// DT: bf16 or fp16, HD: head dim, G: 4 or 8 query heads per workgroup, NW: wavefronts, NST: K/V slot pairs per wavefront
template <int DT, int HD, int G, int NW, int NST>
__global__ __launch_bounds__(NW * 64, 2) void decode_mfma_kernel(DecodeArgs a) {
  constexpr int ROWB = HD * 2;              // bytes per row
  constexpr int SEGS = ROWB / 16;           // 16-byte segments per row
  constexpr int RPL = 1024 / ROWB;          // rows one 1 KB load fills
  constexpr int NLD = kStepKeys / RPL;      // loads per slot
  constexpr int SLOT = kStepKeys * ROWB;
  constexpr int NKS = HD / 32;              // products of a 16-key score tile
  constexpr int NMT = HD / 16;              // 16-dim output tiles
  constexpr int NSET = G == 4 ? 1 : 2;      // products per output tile
  constexpr bool BF = DT == CHUNKKV_BF16;
  const u16x2 kLeastPart = BF ? u16x2{0x0080, 0x0080} : u16x2{0x0001, 0x0001};

  extern __shared__ __align__(16) char smem[];
  __shared__ int s_again;   // some element of the merged output is not finite

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int bl = blockIdx.z, split = blockIdx.x;
  int h = blockIdx.y, j0 = 0;
  if (gridDim.y != (uint32_t)a.n_kv_heads) {   // more than one batch of heads per kv-head
    h = blockIdx.y % a.n_kv_heads;
    j0 = blockIdx.y / a.n_kv_heads * G;
  }
  const int g = a.group, b = a.batch0 + bl;

  const int cap = CKV_ARG(DecodeArgs, n_tok, bl), rps = CKV_ARG(DecodeArgs, cut.rows_per_split, bl);
  const int splits = CKV_ARG(DecodeArgs, cut.splits, bl);
  const int64_t slot0 = (int64_t)CKV_ARG(DecodeArgs, cut.first_split, bl) * a.n_q_heads + (int64_t)(h * g) * splits + split;   // first partial result
  int nrow = cap;
  if (a.kv_len != nullptr) {
    nrow = a.kv_len[(int64_t)b * a.n_kv_heads + h];
    nrow = nrow < 0 ? 0 : (nrow > cap ? cap : nrow);
  }
  const int r0 = split * rps;
  const int len = r0 + rps < nrow ? rps : nrow - r0;   // rows of this range
  if (len <= 0 && split > 0) return;                   // the merge knows how many ranges hold rows
  const int nstep_all = len > 0 ? (len + kStepKeys - 1) / kStepKeys : 0;
  const int nstep = (nstep_all - wave + NW - 1) / NW;  // steps wave, wave + NW, ... are this wavefront's

  const int64_t tok = a.stride_tok * 2;
  const int64_t off0 = (CKV_ARG(DecodeArgs, base, bl) + (int64_t)h * a.stride_head) * 2 + (int64_t)r0 * tok;
  // query operand (first in the queue of loads): column n holds head n % G (heads the kv-head does not have
  // read as zero)
  const int head = n % G, part = n / G;
  u32x4 qf[NKS];
  {
    const char *qrow = (const char *)a.q + ((int64_t)b * a.n_q_heads + (int64_t)h * g + j0) * ROWB;
    const __amdgpu_buffer_rsrc_t qrs = __builtin_amdgcn_make_buffer_rsrc((void *)qrow, 0, (g - j0) * ROWB, 0x00020000);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, head * ROWB + (4 * ks + q) * 16, 0, 0));
  }

  // Load j of a slot fills rows RPL j ..; lane l lands at row RPL j + l / SEGS, position l % SEGS and fetches segment
  // position ^ swizzle(row).  K: 16 rows of one segment per fragment read; V: 8 rows of two segments per transposing read.
  auto kswz = [](int row) { return SEGS == 16 ? (row & 15) : ((row >> 1) & 7); };
  auto vswz = [](int row) { return SEGS == 16 ? 2 * (row & 7) : 2 * ((row >> 1) & 3); };
  uint32_t koff[NLD], voff[NLD];
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int row = RPL * j + lane / SEGS, pos = lane % SEGS;
    koff[j] = (uint32_t)row * (uint32_t)tok + (uint32_t)((pos ^ kswz(row)) * 16);
    voff[j] = (uint32_t)row * (uint32_t)tok + (uint32_t)((pos ^ vswz(row)) * 16);
  }
  // A descriptor covers the rows of one step, so only 32 rows have to be within reach of 32-bit offsets.  Steps past the
  // last one are issued too, through an empty descriptor (no memory traffic, zeros into the slot), so the number of loads
  // in flight is a compile-time constant at every wait.
  const uint32_t ring = (uint32_t)(wave * (2 * NST * SLOT));
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
  auto issue = [&](const void *base, const uint32_t *off, int step, uint32_t slot) __attribute__((always_inline)) {
    const int first = (wave + step * NW) * kStepKeys, last = (first + kStepKeys < len ? first + kStepKeys : len) - 1;
    const uint32_t span = step < nstep ? (uint32_t)(last - first) * (uint32_t)tok + ROWB : 0u;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)base + off0 + first * tok), 0, (int)span, 0x00020000);
#pragma unroll
    for (int j = 0; j < NLD; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(smem + slot + j * 1024), 16, off[j], 0, 0, 2);
  };
  auto kslot = [&](int s) { return ring + (uint32_t)((s % NST) * (2 * SLOT)); };
  auto vslot = [&](int s) { return ring + (uint32_t)((s % NST) * (2 * SLOT) + SLOT); };

  // LDS addresses: K fragment of row 16 t + n, segment 4 ks + q; V piece of keys 16 t + 4 q + (n / 4), dims 16 mt + 4 (n % 4)
  uint32_t kaddr[NKS], vaddr[NMT];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) kaddr[ks] = (uint32_t)(n * ROWB + (((4 * ks + q) ^ kswz(n)) * 16));
  {
    const int row = 4 * q + n / 4;
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
      vaddr[mt] = lds0 + (uint32_t)(row * ROWB + (((2 * mt + (n % 4) / 2) ^ vswz(row)) * 16) + (n & 1) * 8);
  }
  static_assert(SEGS == 16 || SEGS == 8, "rows 16 apart share the swizzle");

  const float c1 = a.scale_log2e;
  if (tid == 0) s_again = 0;
  uint32_t redo = 0;   // bit i: element tid + 64 NW i of the output was not finite in the first pass
  for (int pass = 0;; ++pass) {
#pragma unroll
    for (int s = 0; s < NST; ++s) { issue(a.k, koff, s, kslot(s)); issue(a.v, voff, s, vslot(s)); }
    float m = kNegBig, l = 0.f;
    f32x4 acc[NSET][NMT];
#pragma unroll
    for (int s = 0; s < NSET; ++s)
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt) acc[s][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int s = 0; s < nstep; ++s) {
      // behind K of step s: its V and the slot pairs of the next NST - 1 steps
      __builtin_amdgcn_s_waitcnt(vm_imm((2 * NST - 1) * NLD));
      const uint32_t ks_ = kslot(s), vs_ = vslot(s);
      u32x4 kf[2][NKS];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) kf[t][ks] = *(const u32x4 *)(smem + (ks_ + kaddr[ks] + (uint32_t)(t * 16 * ROWB)));
      f32x4 sc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        // two chains, added at the end: half the roundings at full magnitude
        f32x4 even = {0.f, 0.f, 0.f, 0.f}, odd = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ks += 2) {
          even = mma16<DT>(kf[t][ks], qf[ks], even);
          odd = mma16<DT>(kf[t][ks + 1], qf[ks + 1], odd);
        }
        sc[t] = even + odd;
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);   // the fragments are in registers: the K slot is free
      issue(a.k, koff, s + NST, ks_);

      const int key0 = (wave + s * NW) * kStepKeys;
      if (key0 + kStepKeys > len) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[t][i] = key0 + 16 * t + 4 * q + i < len ? sc[t][i] : -3.0e38f;
      }
      float p[8];
      auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i / 4][i % 4], c1, -m));
      };
      weights();
      float sum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      float over = sum;
      if constexpr (!BF)
        over = fmaxf(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])), fmaxf(fmaxf(p[4], p[5]), fmaxf(p[6], p[7])));
      constexpr float kOver = BF ? 16.f : 1.96875f;   // fp16: 2^15 times it is the largest 11-bit number below 2^16
      if (__builtin_amdgcn_ballot_w64(over >= kOver) != 0) {
        // move the reference of the head columns that outgrew it (the four lanes of a column together)
        float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])), fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        over = fmaxf(over, __shfl_xor(over, 16));
        over = fmaxf(over, __shfl_xor(over, 32));
        const float m_new = over >= kOver ? mx * c1 : m;
        const float f = __builtin_amdgcn_exp2f(m - m_new);
        m = m_new;
        l *= f;
#pragma unroll
        for (int st = 0; st < NSET; ++st)
#pragma unroll
          for (int mt = 0; mt < NMT; ++mt) acc[st][mt] *= f;
        weights();
        sum = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      }
      l += sum;

      // the weights' parts as B operands: element i = key 4 q + i (i < 4) or 16 + 4 q + i - 4
      u32x4 pf[NSET];
#pragma unroll
      for (int i2 = 0; i2 < 4; ++i2) {
        if constexpr (BF) {
          float x[2][NSET];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float p0 = p[2 * i2 + e];
            const float p1 = p0 - __uint_as_float(__float_as_uint(p0) & 0xFFFF0000u);
            const float p2 = p1 - __uint_as_float(__float_as_uint(p1) & 0xFFFF0000u);
            if constexpr (G == 4) x[e][0] = part == 0 ? p0 : (part == 1 ? p1 : p2);
            else { x[e][0] = part == 0 ? p0 : p1; x[e][1] = p2; }
          }
#pragma unroll
          for (int st = 0; st < NSET; ++st)   // upper halves: the truncation
            pf[st][i2] = __builtin_amdgcn_perm(__float_as_uint(x[1][st]), __float_as_uint(x[0][st]), 0x07060302u);
        } else {
          const float a0 = p[2 * i2] * 32768.f, b0 = p[2 * i2 + 1] * 32768.f;   // exact
          const fp16x2 h0 = __builtin_amdgcn_cvt_pkrtz(a0, b0);
          const float a1 = (a0 - (float)h0[0]) * 2048.f, b1 = (b0 - (float)h0[1]) * 2048.f;   // what is left of a number below 2^16 is below 2^5
          const fp16x2 h1 = __builtin_amdgcn_cvt_pkrtz(a1, b1);
          const float a2 = (a1 - (float)h1[0]) * 2048.f, b2 = (b1 - (float)h1[1]) * 2048.f;
          const fp16x2 h2 = __builtin_amdgcn_cvt_pkrtz(a2, b2);
          const float a3 = (a2 - (float)h2[0]) * 2048.f, b3 = (b2 - (float)h2[1]) * 2048.f;
          const fp16x2 h3 = __builtin_amdgcn_cvt_pkrtz(a3, b3);
          const uint32_t w0 = __builtin_bit_cast(uint32_t, h0), w1 = __builtin_bit_cast(uint32_t, h1), w2 = __builtin_bit_cast(uint32_t, h2), w3 = __builtin_bit_cast(uint32_t, h3);
          if constexpr (G == 4) pf[0][i2] = part < 2 ? (part == 0 ? w0 : w1) : (part == 2 ? w2 : w3);
          else { pf[0][i2] = part == 0 ? w0 : w1; pf[1][i2] = part == 0 ? w2 : w3; }
        }
      }

      // Second pass: no part is zero.  The least one is 2^-126 (bf16) or 2^-24 before its scale (fp16); rows that are not
      // there read as zero values.
      if (pass != 0) {
#pragma unroll
        for (int st = 0; st < NSET; ++st)
#pragma unroll
          for (int i2 = 0; i2 < 4; ++i2) {
            const uint32_t w = pf[st][i2];   // a scalar: a bit cast of a vector's element takes its first one
            pf[st][i2] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, w), kLeastPart));
          }
      }

      // behind V of step s: the next NST - 1 slot pairs and K of step s + NST
      __builtin_amdgcn_s_waitcnt(vm_imm((2 * NST - 1) * NLD));
#pragma unroll
      for (int m4 = 0; m4 < NMT; m4 += 4) {
        u32x4 vf[4];
        read_v4<16 * ROWB>(vs_ + vaddr[m4], vs_ + vaddr[m4 + 1], vs_ + vaddr[m4 + 2], vs_ + vaddr[m4 + 3], vf);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int st = 0; st < NSET; ++st) acc[st][m4 + i] = mma16<DT>(vf[i], pf[st], acc[st][m4 + i]);
      }
      issue(a.v, voff, s + NST, vs_);
    }

    // ---- parts of a head -> its output (lanes n < G), lanes of a column -> its sum
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    constexpr float kS0 = BF ? 1.f : 0x1p-15f, kS1 = BF ? 1.f : 0x1p-26f, kS2 = BF ? 1.f : 0x1p-37f, kS3 = BF ? 0.f : 0x1p-48f;
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = acc[0][mt][i];
        if constexpr (G == 4) {
          const float rest = BF ? row_shl<8>(x) : row_shl<8>(x) * kS2 + row_shl<12>(x) * kS3;
          acc[0][mt][i] = x * kS0 + (row_shl<4>(x) * kS1 + rest);
        } else {
          const float y = acc[1][mt][i], rest = BF ? y : y * kS2 + row_shl<8>(y) * kS3;
          acc[0][mt][i] = x * kS0 + (row_shl<8>(x) * kS1 + rest);
        }
      }
    // ---- merge the wavefronts through LDS, in wavefront order
    // the loads of the empty steps past the last one still write zeros into the slots
    __builtin_amdgcn_s_waitcnt(vm_imm(0));
    __syncthreads();   // the slots are dead
    float *s_m = (float *)smem, *s_l = s_m + NW * G, *s_o = s_l + NW * G;   // [NW][G], [NW][G], [NW][G][HD]
    if (n < G) {
      if (q == 0) { s_m[wave * G + n] = m; s_l[wave * G + n] = l; }
#pragma unroll
      for (int mt = 0; mt < NMT; ++mt) *(f32x4 *)(s_o + (wave * G + n) * HD + 16 * mt + 4 * q) = acc[0][mt];
    }
    __syncthreads();
    uint32_t bad = 0;
    for (int t = tid, i = 0; t < G * HD; t += NW * 64, ++i) {
      const int j = t / HD, e = t % HD;
      if (j0 + j >= g) break;
      if (pass != 0 && (redo >> i & 1) == 0) continue;
      float M = s_m[j];
#pragma unroll
      for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w * G + j]);
      float L = 0.f, o = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_m[w * G + j] - M);
        L += s_l[w * G + j] * f;
        o += s_o[(w * G + j) * HD + e] * f;
      }
      bad |= finite_bits(o) ? 0u : 1u << i;
      const int64_t hd = (int64_t)b * a.n_q_heads + (int64_t)h * g + j0 + j;
      if (a.cut.n_split == 1) {   // one range per head: no merge kernel follows
        a.out[hd * HD + e] = L > 0.f ? o / L : 0.f;
        if (a.lse != nullptr && e == 0) a.lse[hd] = L > 0.f ? (M + __builtin_log2f(L)) * 0.6931471805599453f : -__builtin_inff();
      } else {
        const int64_t slot = slot0 + (j0 + j) * splits;
        if (e == 0) a.part_ml[slot] = make_float2(M, L);
        a.part_o[slot * HD + e] = o;
      }
    }
    if (pass != 0) break;
    if (bad != 0) s_again = 1;
    // a barrier for LDS alone, s_again's address its operand so that it is read again behind it: nothing waits for the stores
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::"v"(&s_again) : "memory");
    if (s_again == 0) break;
    redo = bad;
    __builtin_amdgcn_s_waitcnt(vm_imm(0));   // the stores: the waits of the second pass count loads only
  }
}

template <int DT, int HD, int G, int NW, int NST>
int launch_decode_mfma_cfg(const DecodeArgs &a, dim3 grid, hipStream_t s) {
  constexpr int kLds = NW * NST * 2 * kStepKeys * HD * 2;
  static_assert(kLds >= NW * G * (HD + 2) * 4 && kLds <= 160 * 1024, "LDS");
  static std::once_flag once;
  static hipError_t rc = hipSuccess;
  auto kern = decode_mfma_kernel<DT, HD, G, NW, NST>;
  std::call_once(once, [&] { rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLds); });
  if (rc != hipSuccess) return CHUNKKV_ERR_LAUNCH;
  hipLaunchKernelGGL(kern, grid, dim3(NW * 64), kLds, s, a);
  return hipGetLastError() == hipSuccess ? CHUNKKV_OK : CHUNKKV_ERR_LAUNCH;
}

template <int DT, int HD>
int launch_decode_mfma_hd(const DecodeArgs &a, int batch_slice, int g, hipStream_t s) {
  const int G = g <= 4 ? 4 : 8;
  const dim3 grid(a.cut.n_split, a.n_kv_heads * ((g + G - 1) / G), batch_slice);
  constexpr int NST = HD == 128 ? 1 : 2;
  // one range per head: eight wavefronts share it
  if (a.cut.n_split == 1) return G == 4 ? launch_decode_mfma_cfg<DT, HD, 4, 8, NST>(a, grid, s) : launch_decode_mfma_cfg<DT, HD, 8, 8, NST>(a, grid, s);
  return G == 4 ? launch_decode_mfma_cfg<DT, HD, 4, 4, NST>(a, grid, s) : launch_decode_mfma_cfg<DT, HD, 8, 4, NST>(a, grid, s);
}

int launch_decode_mfma(int dtype, int head_dim, const DecodeArgs &a, int batch_slice, hipStream_t s) {
  const int g = a.n_q_heads / a.n_kv_heads;
  if (dtype == CHUNKKV_BF16) return head_dim == 128 ? launch_decode_mfma_hd<CHUNKKV_BF16, 128>(a, batch_slice, g, s) : launch_decode_mfma_hd<CHUNKKV_BF16, 64>(a, batch_slice, g, s);
  return head_dim == 128 ? launch_decode_mfma_hd<CHUNKKV_F16, 128>(a, batch_slice, g, s) : launch_decode_mfma_hd<CHUNKKV_F16, 64>(a, batch_slice, g, s);
}

}  // namespace ckv
