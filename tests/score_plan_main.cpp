// With "units": reads "lo hi slots least_rounds rounds half start n u1 .. un" lines, n sequences of so many units, and prints the units of a
// workgroup and how many workgroups that makes.  With "stride": reads "keys chunk" lines and prints the keys of a super-tile.  Otherwise:
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

int main(int argc, char **argv) {
  int keys, chunk, lo, hi, slots, least, rounds, n, units[16];
  double half, start;
  while (argc > 1 && argv[1][0] == 'u' && std::scanf("%d %d %d %d %d %lf %lf %d", &lo, &hi, &slots, &least, &rounds, &half, &start, &n) == 8 && n <= 16) {
    for (int i = 0; i < n; ++i)
      if (std::scanf("%d", &units[i]) != 1) return 1;
    auto wgs = [&](int t) {
      int64_t w = 0;
      for (int i = 0; i < n; ++i) w += (units[i] + t - 1) / t;
      return w;
    };
    const int t = ckv::units_per_workgroup(lo, hi, slots, least, rounds, half, start, wgs, [](int) { return 0.0; });
    std::printf("%d %lld\n", t, (long long)wgs(t));
  }
  while (argc > 1 && std::scanf("%d %d", &keys, &chunk) == 2) std::printf("%d\n", ckv::super_stride(keys, chunk));
  int prefix;
  unsigned pitch, row_bytes;
  while (std::scanf("%d %u %u", &prefix, &pitch, &row_bytes) == 3) std::printf("%s\n", walk(prefix, pitch, row_bytes));
  return 0;
}
