// CPU check of how a persistent plane kernel's items are shared: every (unit,
// plane) of a launch is visited exactly once and in range, whatever the number
// of workgroups, and with a grid of a multiple of the XCD count no XCD holds
// more than 5% over its share, unless all walk the items together.
#include <cstdint>
#include <cstdio>
#include <vector>

#define FX_HD inline
#include "item_map.hpp"

int main() {
  using namespace fx;
  const int grids[] = {1, 3, 7, 8, 16, 24, 104, 256, 512, 2304};
  for (int nz = 2; nz <= 96; nz += nz < 12 ? 1 : 3)
    for (int units = 1; units < 200; units += units < 40 ? 1 : 17)
      for (int zsplit = 0; zsplit < 2; ++zsplit)
        for (int grid : grids) {
          int G = grid < units * nz ? grid : units * nz;
          if (G >= kXcds) G -= G % kXcds;
          std::vector<int> seen(units * nz, 0);
          int share[kXcds] = {0};
          const int split = item_split(nz, units, zsplit, G);
          for (int b = 0; b < G; ++b) {
            const ItemMap m = item_map(nz, units, split, G, b);
            for (int li = m.first; li < m.total; li += m.step) {
              int u, z;
              m.at(li, &u, &z);
              if (u < 0 || u >= units || z < 0 || z >= nz) return std::printf("out of range\n"), 1;
              ++seen[z * units + u];
              ++share[b % kXcds];
            }
          }
          for (int c : seen)
            if (c != 1)
              return std::printf("nz %d units %d zsplit %d G %d: visited %d times\n", nz, units, zsplit, G, c), 1;
          if (G % kXcds == 0)
            for (int s : share)
              if (s > 1.05 * units * nz / kXcds + G / kXcds)
                return std::printf("nz %d units %d zsplit %d G %d: share %d\n", nz, units, zsplit, G, s), 1;
        }
  for (int n = 1; n < 300; ++n) {
    std::vector<int> seen(n, 0);
    for (int b = 0; b < n; ++b) {
      const int p = xcd_run(n, b);
      if (p < 0 || p >= n || seen[p]++) return std::printf("xcd_run(%d, %d) = %d\n", n, b, p), 1;
      if (b >= kXcds && p != xcd_run(n, b - kXcds) + 1) return std::printf("no run at %d of %d\n", b, n), 1;
    }
  }
  std::printf("ok\n");
  return 0;
}
