// The order in which the key preparation's workgroups are dispatched (prep_grid, prep_block): every
// workgroup of a head runs exactly once, and over a batch of heads each of the 8 XCDs gets its share.
// Prints "prep grid ok".
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "twinkv_internal.h"

int main() {
  const int heads = 64;
  for (int total = 1; total <= 600; ++total) {
    const int grid = twinkv::prep_grid(total);
    int64_t work[8] = {0};
    for (int y = 0; y < heads; ++y) {
      std::vector<int> seen(total, 0);
      for (int x = 0; x < grid; ++x) {
        const int b = twinkv::prep_block(x, y, grid, total);
        if (b < 0 || (b < total && seen[b]++)) {
          std::fprintf(stderr, "total %d head %d x %d: workgroup %d\n", total, y, x, b);
          return 1;
        }
        if (b < total) ++work[(x + (int64_t)y * grid) % 8];
      }
      if (std::count(seen.begin(), seen.end(), 1) != total) {
        std::fprintf(stderr, "total %d head %d: workgroups left out\n", total, y);
        return 1;
      }
    }
    const int64_t most = *std::max_element(work, work + 8);
    if (8 * most > (int64_t)heads * total) {  // 64 heads: a multiple of 8 of each pattern, so exactly even
      std::fprintf(stderr, "total %d: one XCD has %lld of %lld workgroups\n", total, (long long)most,
                   (long long)heads * total);
      return 1;
    }
  }
  std::printf("prep grid ok\n");
  return 0;
}
