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

}  // namespace ckv
