// Host check of last_index (csrc/common.h), the few-outputs kernel's position
// of In's last element: of the eight elements of a 16-byte chunk at an offset
// below 2^30 it names the last one where that lies in the chunk, and none
// elsewhere, however many elements follow.  Exits 1 on any mismatch.
#include <cstdio>
#include <cstdint>
#include "common.h"
using namespace cnnlib;
int main() {
  uint64_t bad = 0, n = 0;
  for (int64_t base : {(int64_t)1, (int64_t)1 << 20, (int64_t)1 << 30, (int64_t)1 << 31,
                       (int64_t)1 << 32, (int64_t)3 << 32, (int64_t)1 << 40})
    for (int64_t d = -40; d <= 40; ++d)
      for (uint32_t off : {0u, 8u, 16u, 1000u, (1u << 20) - 8, 1u << 20, (1u << 30) - 8}) {
        // elements from the row: near the base, and an offset past it
        for (int64_t elems : {base + d, base + off + d}) {
          if (elems < 1) continue;
          const uint32_t at = last_index(elems) - off;  // as the kernel compares it
          const int64_t want = elems - 1 - (int64_t)off;
          ++n;
          if ((at < 8) != (want >= 0 && want < 8) || (at < 8 && at != (uint32_t)want)) ++bad;
        }
      }
  printf("checked %llu bad %llu\n", (unsigned long long)n, (unsigned long long)bad);
  return bad != 0;
}
