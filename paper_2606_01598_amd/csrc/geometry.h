// Atom bins and mesh tiles of a plan (host only): the sizes that every binning, spread and
// gather of the plan works with, and the bounds that their kernels count on.
#pragma once

#include "../../include/pme.h"
#include "kernels.h"

namespace pme {

inline int pick_bin(int N) {
  for (int c : {4, 5, 3, 6, 2})
    if (N % c == 0) return c;
  return N;
}

// Default geometry of one axis: among atom-bin sizes B that divide N (in the
// order of pick_bin) and tiles T = k B that divide N as well, the T closest to
// the target within [target / 2, 2 target] (ties: the larger B, then the
// smaller T).  Tiles that divide the mesh leave no partial tiles at the edge,
// whose shorter work and uneven spread over the CUs cost the 100^3 mesh about 7 %
// of a step (8 x 8 x 16 with 4-point bins against 10 x 10 x 20 with 5-point
// bins).  Returns false when no such tile exists.
inline bool pick_dividing_tile(int N, int target, int& B, int& T) {
  int best = -1;
  for (int c : {4, 5, 3, 6, 2}) {
    if (N % c) continue;
    for (int t = c; t <= 2 * target && t <= N; t += c) {
      if (N % t || 2 * t < target) continue;
      const int d = t > target ? t - target : target - t;
      if (best < 0 || d < best || (d == best && c > B)) {
        best = d;
        B = c;
        T = t;
      }
    }
  }
  return best >= 0;
}

// Whether tiles of T points in bins of B cells keep the kernels' bounds: the spread's
// scanned bins, its tile and its LDS, the gather's own bins (one per thread) and its two
// field regions with their row and z tables.
inline bool bins_fit(const DevPlan& d) {
  const int p = d.p;
  long range = 1, own = 1, region = 2;
  for (int a = 0; a < 3; ++a) {
    const long k = (d.T[a] + p - 1 + d.B[a] - 1) / d.B[a] + 1, nb = d.N[a] / d.B[a];
    range *= (k < nb ? k : nb);
    own *= d.T[a] / d.B[a];
    region *= d.T[a] + p - 1;
  }
  const long tpad = long(d.T[0]) * d.T[1] * (d.T[2] + 1);
  const long rows = long(d.T[0] + p - 1) * (d.T[1] + p - 1) + (d.T[2] + p - 1);
  return range <= kMaxBinRange && own <= kGatherBins && tpad <= kTileLds &&
         region * 4 + rows * 4 <= kGatherLds &&
         long(spread_lds_bytes(int(tpad), int(range), 64, p, 2)) <= kBigLds;
}

struct Bins {
  bool fit;             // false: no tile keeps the bounds
  bool spread_planes;   // planes or bands can be spread
  bool planes;          // and the bins are one cell wide in x
};

// Bins and tiles of a plan with d.N and d.p set: fills d.B, d.T, d.nb and d.nt.  cubes:
// cubic bins whatever the spread.
inline Bins plan_bins(const pme_desc_t& desc, DevPlan& d, bool cubes) {
  const int p = d.p;
  // mesh tiles of T = k B points: by default tiles near 8 x 8 x 16 that divide the mesh
  // (pick_dividing_tile); a target the descriptor sets is rounded to the first B that
  // divides N, as are axes with no dividing tile
  int target[3] = {8, 8, 16};
  const bool given = desc.tile[0] > 0 || desc.tile[1] > 0 || desc.tile[2] > 0;
  for (int a = 0; a < 3; ++a)
    if (desc.tile[a] > 0) target[a] = desc.tile[a];
  for (int a = 0; a < 3; ++a) {
    if (given || !pick_dividing_tile(d.N[a], target[a], d.B[a], d.T[a])) {
      d.B[a] = pick_bin(d.N[a]);
      int k = (target[a] + d.B[a] / 2) / d.B[a];
      if (k < 1) k = 1;
      if (k > d.N[a] / d.B[a]) k = d.N[a] / d.B[a];
      d.T[a] = k * d.B[a];
    }
  }
  // plane and band spreads need N >= p + B on every axis
  bool roomy = true;
  for (int a = 0; a < 3; ++a)
    if (d.N[a] < p + d.B[a]) roomy = false;
  const bool spread_planes = roomy && p <= 7 && !(desc.flags & PME_F_SEPARATE_SPREAD);
  // shrink tiles until the bounds are kept
  while (!bins_fit(d)) {
    int big = 0;
    for (int a = 1; a < 3; ++a)
      if (d.T[a] / d.B[a] > d.T[big] / d.B[big]) big = a;
    if (d.T[big] == d.B[big]) return Bins{false, spread_planes, false};
    d.T[big] -= d.B[big];
  }
  for (int a = 0; a < 3; ++a) d.nt[a] = (d.N[a] + d.T[a] - 1) / d.T[a];
  // Where planes or bands are spread, the atom bins are 1 x B_y x T_z mesh cells instead:
  // every atom of the p bin layers a plane takes reaches it, and a plane has few bins to
  // count (100^3: 600 of 1 x 5 x 20 with 1920 atoms, all wanted, instead of 800 of
  // 5 x 5 x 5 with 3200).  The tile spread, whose tiles test a halo in z as well, keeps
  // cubes, and so do tiles that would hold too many of the thin bins (given tiles whose
  // edge does not divide N_z: 15^3 on 27^3 is 375 of 1 x 3 x 3, 125 of 3 x 3 x 3).
  bool planes = spread_planes && !cubes;
  if (planes) {
    const int cube[3] = {d.B[0], d.B[1], d.B[2]};
    d.B[0] = 1;
    if (d.N[2] % d.T[2] == 0) d.B[2] = d.T[2];
    if (!bins_fit(d)) {
      planes = false;
      for (int a = 0; a < 3; ++a) d.B[a] = cube[a];
    }
  }
  for (int a = 0; a < 3; ++a) d.nb[a] = d.N[a] / d.B[a];
  return Bins{true, spread_planes, planes};
}

}  // namespace pme
