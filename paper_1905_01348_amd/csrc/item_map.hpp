// How the workgroups of a persistent plane kernel share its items, and which
// XCD takes which.  Integer logic only, for host and device (FX_HD must be
// defined before inclusion), so that it can be checked on the CPU.
#pragma once
#include <cstdint>

namespace fx {

// Work of a persistent plane kernel: `units` (pairs, or targets) x nz planes.
// Workgroups are dispatched round-robin over the XCDs, so with a grid that is
// a multiple of the XCD count workgroup b runs on XCD b % kXcds.  Each XCD
// takes either a contiguous chunk of the units (preferred with zsplit 0) or a
// contiguous range of the planes of every unit (zsplit 1), and walks its share
// z-major: the workgroups of one XCD work on the same z at the same time and
// find that plane's input data (orbital and target planes in pass A, orbital
// planes in pass C) in their shared L2 instead of reading it again from HBM.
// With the z split no two XCDs read the same input plane.
// A split whose largest share exceeds the mean by more than 5% is not taken:
// the other one is, or else all workgroups walk all items z-major.  (One target
// of 427 terms at 72 x 72 x 24 ran on a single XCD, 21.7 ms; the halved 48^3
// apply, 43 targets per launch, has shares of 5 and 6.)
constexpr int kXcds = 8;

// Position of block b of n in a tiled product's order of tiles: blocks are dealt
// round-robin to the XCDs, and each XCD takes a run of consecutive positions, so
// that the tiles in flight on it share rows of the operands in its L2.  (With
// runs for a multiple of 8 blocks only, 3556 blocks of K_ACE's first product at
// 72^3, 432 factors and right-hand sides, missed 97% of their L2 reads.)
FX_HD int xcd_run(int n, int b) {
  const int x = b % kXcds, rest = n % kXcds;
  return x * (n / kXcds) + (x < rest ? x : rest) + b / kXcds;
}

struct ItemMap {
  int u_lo, u_n, z_lo, first, step, total;
  FX_HD void at(int li, int* unit, int* z) const {
    const int zz = li / u_n;
    *z = z_lo + zz;
    *unit = u_lo + (li - zz * u_n);
  }
};

// The split of a launch of G workgroups, chosen on the host (in the kernels the
// rule's arithmetic cost the smallest calls 0.3 of 35 us): kItemsAll,
// kItemsUnits or kItemsPlanes.
enum { kItemsAll = 0, kItemsUnits = 1, kItemsPlanes = 2 };
inline int item_split(int nz, int units, int zsplit, int G) {
  if (G < kXcds || G % kXcds != 0) return kItemsAll;
  const auto even = [](int n) { return (n + kXcds - 1) / kXcds * kXcds * 20 <= 21 * n; };
  if (even(nz) && (zsplit || !even(units))) return kItemsPlanes;
  return even(units) ? kItemsUnits : kItemsAll;
}

// The items of workgroup b of G.
FX_HD ItemMap item_map(int nz, int units, int split, int G, int b) {
  ItemMap m{0, units, 0, b, G, units * nz};
  if (split == kItemsAll) return m;
  const int x = b % kXcds;
  m.first = b / kXcds;
  m.step = G / kXcds;
  if (split == kItemsPlanes) {
    m.z_lo = nz * x / kXcds;
    m.total = units * (nz * (x + 1) / kXcds - m.z_lo);
  } else {
    m.u_lo = (int)((int64_t)units * x / kXcds);
    m.u_n = (int)((int64_t)units * (x + 1) / kXcds) - m.u_lo;
    m.total = m.u_n * nz;
  }
  return m;
}

}  // namespace fx
