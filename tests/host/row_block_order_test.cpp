// The order of a problem's row blocks (spread_row_block): every one runs once, and over a batch of equal
// problems the work, which falls from the first row block to the last, is even over the places that
// workgroups go round: 4 shader engines of an XCD, or 8 XCDs.  Prints "row block order ok".
#include <algorithm>
#include <cstdio>
#include <vector>

#include "twinkv_internal.h"

int main() {
  for (int own = 0; own < 2; ++own) {
    const int places = own ? 4 : 8;
    for (int nb = 1; nb <= 32; ++nb) {
      std::vector<long> work(places, 0);
      for (int p = 0; p < 64; ++p) {
        std::vector<int> seen(nb, 0);
        for (int i = 0; i < nb; ++i) {
          const int rb = twinkv::spread_row_block(i, nb, p, own != 0);
          if (rb < 0 || rb >= nb || seen[rb]++) {
            std::fprintf(stderr, "nb %d problem %d place %d: row block %d\n", nb, p, i, rb);
            return 1;
          }
          work[(p * nb + i) % places] += nb - rb;
        }
      }
      long sum = 0;
      for (long w : work) sum += w;
      const long most = *std::max_element(work.begin(), work.end());
      // at most 1.2 times the mean (nb = 4 on 8 places); in order 1.33 at nb = 2, 1.6 at 4, 1.78 on 8 places at 8
      if (100 * most * places > 120 * sum) {
        std::fprintf(stderr, "nb %d, %d places: the fullest has %ld of %ld\n", nb, places, most, sum);
        return 1;
      }
    }
  }
  std::printf("row block order ok\n");
  return 0;
}
