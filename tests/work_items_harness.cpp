// Host harness for the work distribution (xcd_pair_item in common.hpp): reads
// "pairs T interleave" lines from stdin and prints, per line, "pair rank" of
// every workgroup of the launch in order, "-" where it has no item.
#include <cstdio>

#include "common.hpp"

int main() {
  int nbk, T, il;
  while (std::scanf("%d %d %d", &nbk, &T, &il) == 3) {
    const int n = bdlm::workgroups_for(nbk * T);
    std::printf("%d", n);
    for (int wg = 0; wg < n; ++wg) {
      int pair, rank;
      if (bdlm::xcd_pair_item(wg, nbk, T, il != 0, pair, rank)) std::printf(" %d,%d", pair, rank);
      else std::printf(" -");
    }
    std::printf("\n");
  }
  return 0;
}
