// With "stride": reads "keys chunk" lines and prints the keys of a super-tile.  Otherwise:
// walks the ring loads of the single-pass scoring kernel: reads "prefix pitch row_bytes" lines from stdin and, for every
// period of the sequence and the ones behind it, those with prefix keys present and not, checks what the descriptor of that period lets
// through (a lane offset below its records less the scalar offset) against the prefix's rows.  One "ok" or the first fault per line.
#include <cstdio>

#include "score_plan.h"

static const char *walk(int prefix, uint32_t pitch, uint32_t row_bytes) {
  const uint64_t end = prefix > 0 ? (uint64_t)(prefix - 1) * pitch + row_bytes : 0;   // of the head's prefix rows
  for (int first = 0; first < prefix + 4 * 160; first += 160)
    for (int present = 0; present < (first < prefix ? 2 : 1); ++present) {
      const ckv::RingRows r = ckv::ring_rows(first, prefix, pitch, row_bytes, present != 0);
      for (int row = 0; row < 160; ++row)
        for (uint32_t seg = 0; seg < row_bytes; seg += 16) {
          const uint32_t lane = (uint32_t)row * pitch + seg;
          const bool read = lane < r.records - r.offset, wanted = present && first + row < prefix;
          if (read != wanted) return wanted ? "a row is missing" : "a row that is not there";
          if (read && (uint64_t)r.offset + lane != (uint64_t)(first + row) * pitch + seg) return "another row";
          if (read && (uint64_t)r.offset + lane + 16 > end) return "past the end";
        }
    }
  return "ok";
}

int main(int argc, char **) {
  int keys, chunk;
  while (argc > 1 && std::scanf("%d %d", &keys, &chunk) == 2) std::printf("%d\n", ckv::super_stride(keys, chunk));
  int prefix;
  unsigned pitch, row_bytes;
  while (std::scanf("%d %u %u", &prefix, &pitch, &row_bytes) == 3) std::printf("%s\n", walk(prefix, pitch, row_bytes));
  return 0;
}
