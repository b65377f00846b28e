// Arithmetic that the scoring kernels and their launches share.  No HIP header, so that it can be checked by itself on the host.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define CKV_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define CKV_HOST_DEVICE inline
#endif

namespace ckv {

// Buffer loads of the K rows of a head's period from key `first` on: the descriptor starts at the head's first row and ends
// with its prefix, the loads have a scalar offset.  The bounds check lets a load through whose lane offset is below
// records - scalar offset, a difference that wraps: so a period that is not there (others start before the prefix ends) has
// no scalar offset either.  A head's rows span less than 2^31 bytes.
struct RingRows {
  uint32_t records, offset;
};
CKV_HOST_DEVICE RingRows ring_rows(int first, int prefix, uint32_t pitch, uint32_t row_bytes, bool present) {
  return {present ? (uint32_t)(prefix - 1) * pitch + row_bytes : 0u, present ? (uint32_t)first * pitch : 0u};
}

// Keys of a super-tile (importance pass) of at most `keys`: whole chunks, one where none fits.  Smaller `keys` never make it
// larger.
CKV_HOST_DEVICE int super_stride(int keys, int chunk) { return chunk <= keys ? keys / chunk * chunk : chunk; }

// Units of work that a workgroup of a launch takes, from `lo` to `hi`: what makes the launch shortest on a chip that holds `slots`
// workgroups at once, if they run in rounds and a workgroup takes as long as its units and `start` more of them.  In a last round that
// leaves every second place empty a unit takes `half` as long, as its workgroup has a CU for itself; the start, a chain of
// latencies, does not.  wgs(t): workgroups of t units; extra(t): what else t costs, in units.  Looked at is the smallest t that
// fits into r rounds, for r from `least_rounds` (0: half a round, -1: a quarter and so on) to `rounds`; launches of more rounds keep
// `lo`.
// Workgroups do not take equally long, which many short ones even out: kUneven of a workgroup's units are lost at the end.
constexpr double kUneven = 0.1;
template <typename Count, typename Extra>
inline int units_per_workgroup(int lo, int hi, int slots, int least_rounds, int rounds, double half, double start, Count wgs, Extra extra) {
  if (lo >= hi || wgs(lo) > (int64_t)rounds * slots) return lo;
  int best = lo;
  double least = 1e300;
  for (int r = least_rounds; r <= rounds; ++r) {
    const int64_t target = r <= 0 ? slots >> -r : (int64_t)slots * r;
    int a = lo, b = hi;
    while (a < b) {
      const int mid = (a + b) / 2;
      if (wgs(mid) <= target) b = mid; else a = mid + 1;
    }
    const int64_t n = wgs(a), full = n / slots, rem = n % slots;
    const double last = rem == 0 ? 0.0 : (2 * rem <= slots ? half : 1.0);
    const double cost = a * ((double)full + last) + start * (double)(full + (rem != 0)) + kUneven * a + extra(a);
    if (cost < least) { least = cost; best = a; }
    if (a == lo) break;
  }
  return best;
}

}  // namespace ckv
