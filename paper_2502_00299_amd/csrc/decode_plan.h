// How decode attention cuts the sequences of a batch into key ranges, and the room their partial results need.  Host
// arithmetic only: no HIP header, so that it can be checked by itself.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "chunkkv.h"

namespace ckv {

constexpr int kMaxBatchPerLaunch = 16;

inline int elem_bytes(int dtype) { return dtype == CHUNKKV_F32 ? 4 : 2; }  // bf16 and fp16: 2
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Query heads of one kv-head that a decode workgroup serves.  16-bit caches (matrix cores): 4 or 8; 5..7 heads are one
// padded batch of 8, not two passes over K and V.  fp32 caches (vector ALU): 1, 2 or 4 (registers).
inline int decode_heads_per_wg(int dtype, int g) {
  if (dtype != CHUNKKV_F32) return g > 4 ? 8 : 4;
  return g > 2 ? 4 : g;
}

// Key ranges of the sequences of one launch.
struct DecodeCut {
  int32_t rows_per_split[kMaxBatchPerLaunch];  // rows of one key range of the sequence
  int32_t splits[kMaxBatchPerLaunch];          // key ranges of the sequence
  int32_t first_split[kMaxBatchPerLaunch];     // key ranges of the slice's sequences before it, INT32_MAX past the last one
  int32_t n_split;                             // most key ranges of a sequence; 1: every head is one range and no merge follows
};

// Key ranges and workspace of the decode-attention call: a pure function of the problem.
// 16-bit caches (matrix-core kernel): few ranges mean few starts, ends and partial results, many even out unequal
// sequences.  One to four workgroups per CU (a whole number: with one and a half, half the CUs wait), about
// kDecodeRangeRows rows each.  Microseconds with 256 / 512 / 1024 workgroups: 13171 tokens of 8 kv-heads 15.9 / 16.5 /
// 22.0; 30000 tokens 26.5 / 25.6 / 28.9; 131072 tokens 87.2 / 88.3 / 88.3; eight sequences of 10 to 55 thousand tokens,
// 4 kv-heads 124 / 109 / 96 (2048: 98); five of 600 to 30000 57 / 51 / 47.  A sequence is cut into equal ranges.
// Up to kDecodeDirectRows rows a head is one range of eight wavefronts and needs no merge: 300 tokens of 8 kv-heads 7.8 us
// in one launch, 8.7 in ranges and merge; 512 tokens 9.9 and 9.8, sixteen sequences of 500 tokens 11.3 and 12.7; 700 tokens
// 12 and 10.
// fp32 caches (vector-ALU kernel): ranges of one length for the slice, about kDecodeTargetWorkgroups of them, never
// fewer than kDecodeMinRows rows.
constexpr int kDecodeCUs = 256;
constexpr int kDecodeTargetWorkgroups = 1024;
constexpr int kDecodeMinRows = 256;
constexpr int kDecodeRangeRows = 448, kDecodeMaxRounds = 4;
constexpr int kDecodeDirectRows = 512;
constexpr int kDecodeStepRows = 32;    // rows a wavefront of the matrix-core kernel takes in one step
struct DecodePlan {
  size_t off_ml, off_o, total;
};
inline int64_t decode_tokens(const chunkkv_problem *p, bool compacted, int b) {
  return compacted ? (int64_t)p->n_keep[b] + p->window : p->seqlen[b];
}
// The matrix-core kernel reaches the rows of a step by 32-bit byte offsets: rows up to 64 MB apart.
inline bool decode_on_matrix_cores(const chunkkv_problem *p, bool compacted) {
  const int64_t tok = (compacted ? p->out_stride_tok : p->kv_stride_tok) * elem_bytes(p->dtype);
  return p->dtype != CHUNKKV_F32 && tok * kDecodeStepRows < (int64_t)1 << 31;
}
// rows per range that give about kDecodeTargetWorkgroups workgroups
inline int64_t decode_even_rows(int64_t rows_times_wgs) {
  const int64_t r = (rows_times_wgs + kDecodeTargetWorkgroups - 1) / kDecodeTargetWorkgroups;
  return r < kDecodeMinRows ? kDecodeMinRows : (r + 127) / 128 * 128;
}
// The workspace holds the partial results of about kDecodeTargetWorkgroups ranges of one length over the whole batch, the
// longest sequence's number of them for every sequence.  Its size, and with it what the static call takes, does not depend
// on how the matrix-core kernel cuts the sequences: that has the same number of places to give out, to whichever of them.
// Returns the number of ranges of the longest sequence.
inline int64_t decode_even_splits(const chunkkv_problem *p, bool compacted) {
  int64_t n_max = 1, n_sum = 0;
  for (int b = 0; b < p->batch; ++b) {
    const int64_t n = decode_tokens(p, compacted, b);
    n_max = n > n_max ? n : n_max;
    n_sum += n;
  }
  const int g = p->n_q_heads / p->n_kv_heads;
  const int G = p->dtype != CHUNKKV_F32 && g > 4 ? 8 : (g > 2 ? 4 : g);
  const int64_t launches = (p->batch + kMaxBatchPerLaunch - 1) / kMaxBatchPerLaunch;
  const int64_t rows = decode_even_rows(n_sum * p->n_kv_heads * ((g + G - 1) / G) / launches);
  return (n_max + rows - 1) / rows;
}
// Cuts the sequences b0 .. b0 + nb - 1 of one launch: a pure function of the problem.
inline void decode_cut(const chunkkv_problem *p, bool compacted, int b0, int nb, DecodeCut *a) {
  const bool mfma = decode_on_matrix_cores(p, compacted);
  const int g = p->n_q_heads / p->n_kv_heads;
  const int G = mfma || p->dtype == CHUNKKV_F32 ? decode_heads_per_wg(p->dtype, g) : 1;
  const int64_t per_seq = (int64_t)p->n_kv_heads * ((g + G - 1) / G);   // workgroups of one range of a sequence
  int64_t n_sum = 0, n_max = 1;
  for (int i = 0; i < nb; ++i) {
    const int64_t n = decode_tokens(p, compacted, b0 + i);
    n_sum += n;
    n_max = n > n_max ? n : n_max;
  }
  const int64_t n_even = decode_even_splits(p, compacted);
  auto ranges = [&](int64_t r) {
    int64_t w = 0;
    for (int i = 0; i < nb; ++i) w += (decode_tokens(p, compacted, b0 + i) + r - 1) / r;
    return w;
  };
  int64_t r;
  if (!mfma) {
    r = decode_even_rows(n_sum * per_seq);
    const int64_t least = (n_max + n_even - 1) / n_even;
    if (r < least) r = (least + 127) / 128 * 128;
  } else if (n_max <= kDecodeDirectRows) {
    r = kDecodeDirectRows;
  } else {
    // The shortest range length (in steps) that gives at most `target` workgroups, or one range per head.  Where there are
    // few workgroups, and places to spare, ranges of 128 rows spread a sequence over more CUs (848 tokens of 8 kv-heads 9.2 us,
    // 9.4 in ranges of 224 rows; 1500 tokens 9.3 and 10.0).
    const int64_t lo0 = (p->batch <= kMaxBatchPerLaunch && nb * per_seq <= kDecodeCUs / 4 ? kDecodeMinRows / 2 : kDecodeMinRows) / kDecodeStepRows;
    const int64_t hi0 = (n_max + kDecodeStepRows - 1) / kDecodeStepRows > lo0 ? (n_max + kDecodeStepRows - 1) / kDecodeStepRows : lo0;
    auto shortest = [&](int64_t target) {
      int64_t lo = lo0, hi = hi0;
      while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (ranges(mid * kDecodeStepRows) * per_seq <= target) hi = mid; else lo = mid + 1;
      }
      return lo * kDecodeStepRows;
    };
    int64_t rounds = (n_sum * per_seq + kDecodeRangeRows * kDecodeCUs / 2) / (kDecodeRangeRows * kDecodeCUs);
    rounds = rounds < 1 ? 1 : (rounds > kDecodeMaxRounds ? kDecodeMaxRounds : rounds);
    // no more whole rounds than there are places for the partial results of
    const int64_t places = (int64_t)p->batch * n_even * per_seq;
    while (rounds > 1 && places < rounds * kDecodeCUs) --rounds;
    r = shortest(places < kDecodeCUs ? places : rounds * kDecodeCUs);
    // Many short sequences can use up the workgroups by themselves and leave the long ones hardly cut: then the workgroups
    // are counted by rows alone.  One sequence of 4111 tokens and fifteen of 64, 32 kv-heads: 22 us, uncut 50; 88000 and
    // fifteen of 300, 60 kv-heads: 426 and 644; three of 8111 and thirteen of 400, 16 kv-heads: 47 and 103.
    const int64_t share = (n_sum * per_seq + rounds * kDecodeCUs - 1) / (rounds * kDecodeCUs);
    if (r > 2 * share) {
      const int64_t fit = shortest(places);
      r = (share + kDecodeStepRows - 1) / kDecodeStepRows * kDecodeStepRows;
      r = r > fit ? r : fit;
    }
  }
  a->n_split = 1;
  int32_t first = 0;
  for (int i = 0; i < nb; ++i) {
    const int64_t n = decode_tokens(p, compacted, b0 + i), s = n > 0 ? (n + r - 1) / r : 1;
    int64_t rows = r;
    if (mfma) {   // equal ranges, a whole number of steps
      rows = (n + s - 1) / s;
      rows = rows < 1 ? kDecodeStepRows : (rows + kDecodeStepRows - 1) / kDecodeStepRows * kDecodeStepRows;
    }
    a->rows_per_split[i] = (int32_t)rows;
    a->splits[i] = (int32_t)(n > 0 ? (n + rows - 1) / rows : 1);
    a->first_split[i] = first;
    first += a->splits[i];
    a->n_split = a->splits[i] > a->n_split ? a->splits[i] : a->n_split;
  }
  for (int i = nb; i < kMaxBatchPerLaunch; ++i) a->first_split[i] = INT32_MAX;
}
// Wavefronts of a workgroup over fp32 caches, for the sequences of one launch.  Ranges are 256 rows or more, as many as there are places for
// their partial results, and a step of four wavefronts is 32 rows of 512 bytes: few workgroups spent their time waiting for one step after
// the other.  So up to a workgroup per CU (the grid counts the ranges of all sequences) they have 16
// wavefronts, at d = 128 up to two per CU 8 (8 from the start with four heads, where 16 leave no registers), and read a step ahead.
// us of a layer, so and with four: 244 tokens of 8 kv-heads 8.3 / 25 (half of the rest is the merge launch, which one range
// does without), 3350 tokens of 2 12 / 27, five sequences of 300 of 4 kv-heads, 4 heads each 14 / 28.  At d = 64 a step is 64 rows: five sequences of
// 560 to 3200 tokens 13.2 with eight, 12.3 with four.  One sequence of 8000 tokens and seven of 300, 4 kv-heads, 4 heads each 15.6; in a
// grid with a row as long as the longest sequence's for each, all of it counted, 55; counted by the workgroups with rows, 44.
inline int decode_f32_waves(int head_dim, int g, int n_kv_heads, int nb, const DecodeCut &cut) {
  const int G = decode_heads_per_wg(CHUNKKV_F32, g);
  int64_t wgs = 0;
  for (int i = 0; i < nb; ++i) wgs += cut.splits[i];
  wgs *= (int64_t)n_kv_heads * ((g + G - 1) / G);
  if (wgs <= kDecodeCUs && !(head_dim == 128 && G == 4)) return 16;
  return head_dim == 128 && wgs <= 2 * kDecodeCUs ? 8 : 4;
}
inline void decode_plan(const chunkkv_problem *p, bool compacted, DecodePlan *pl) {
  const size_t places = (size_t)p->batch * p->n_q_heads * (size_t)decode_even_splits(p, compacted);
  pl->off_ml = 0;
  pl->off_o = align256(places * 8);
  pl->total = pl->off_o + align256(places * p->head_dim * sizeof(float));
}

}  // namespace ckv
