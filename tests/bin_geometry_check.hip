// Host build of the bins and tiles of plans (csrc/geometry.h): 5-smooth meshes with the
// default and with given tiles, orders and spreads.  Built with hipcc --offload-host-only
// by test_bin_geometry_cpu.py; prints
//   plan N_x N_y N_z p tile_x tile_y tile_z flags | T | B | planes
// for every geometry that breaks a bound its kernels count on, then "plans <count>",
// "planes <count>" and "refused <count>".
#include <stdio.h>
#include <string.h>

#include <random>
#include <vector>

#include "../paper_2606_01598_amd/csrc/geometry.h"

using pme::DevPlan;

int main() {
  std::vector<int> smooth;
  for (int n = 2; n <= 1024; ++n) {
    int m = n;
    for (int f : {2, 3, 5})
      while (m % f == 0) m /= f;
    if (m == 1) smooth.push_back(n);
  }
  const int tiles[][3] = {{0, 0, 0},    {8, 8, 16},   {8, 16, 16},  {12, 12, 16}, {16, 16, 16},
                          {8, 8, 8},    {16, 16, 8},  {8, 8, 32},   {16, 16, 32}, {32, 12, 12},
                          {64, 20, 4},  {128, 4, 16}, {16, 20, 16}, {1, 1, 1},    {1024, 1024, 1024}};
  const int fixed[][3] = {{18, 18, 18},    {27, 27, 27}, {54, 54, 54},    {54, 60, 54},
                          {81, 81, 81},    {64, 64, 64}, {100, 100, 100}, {162, 162, 162},
                          {324, 486, 243}, {27, 162, 162}};
  std::mt19937 g(5);
  auto any = [&](int n) { return int(g() % unsigned(n)); };
  long plans = 0, planes = 0, refused = 0;
  auto check = [&](const int* N, const int* tile, int p, int flags, bool cubes) {
    pme_desc_t desc;
    memset(&desc, 0, sizeof(desc));
    desc.flags = flags;
    DevPlan d;
    memset(&d, 0, sizeof(d));
    d.p = p;
    for (int a = 0; a < 3; ++a) { d.N[a] = desc.mesh[a] = N[a]; desc.tile[a] = tile[a]; }
    const pme::Bins b = pme::plan_bins(desc, d, cubes);
    ++plans;
    if (!b.fit) { ++refused; return; }
    planes += b.planes;
    bool good = !(b.planes && (!b.spread_planes || cubes || d.B[0] != 1));
    long own = 1, range = 1;
    for (int a = 0; a < 3; ++a) {
      good = good && d.B[a] >= 1 && d.T[a] >= d.B[a] && d.T[a] % d.B[a] == 0 &&
             d.N[a] % d.B[a] == 0 && d.nb[a] * d.B[a] == d.N[a] && (d.nt[a] - 1) * d.T[a] < d.N[a] &&
             d.nt[a] * d.T[a] >= d.N[a];
      own *= d.T[a] / d.B[a];
      const long k = (d.T[a] + p - 1 + d.B[a] - 1) / d.B[a] + 1;
      range *= k < d.nb[a] ? k : d.nb[a];
    }
    if (!good || own > pme::kGatherBins || range > pme::kMaxBinRange)
      printf("plan %d %d %d %d %d %d %d %d | %d %d %d | %d %d %d | %d\n", N[0], N[1], N[2], p, tile[0],
             tile[1], tile[2], flags, d.T[0], d.T[1], d.T[2], d.B[0], d.B[1], d.B[2], int(b.planes));
  };
  for (const auto& N : fixed)
    for (const auto& t : tiles)
      for (int p = 1; p <= 7; ++p) {
        check(N, t, p, 0, false);
        check(N, t, p, PME_F_SEPARATE_SPREAD, false);
        check(N, t, p, 0, true);
      }
  for (int k = 0; k < 200000; ++k) {
    int N[3], t[3];
    for (int a = 0; a < 3; ++a) {
      N[a] = smooth[any(int(smooth.size()))];
      t[a] = any(4) ? 1 + any(40) : any(1025);
    }
    const int* tile = any(3) ? t : tiles[any(15)];
    check(N, tile, 1 + any(7), any(8) ? 0 : PME_F_SEPARATE_SPREAD, any(8) == 0);
  }
  printf("plans %ld\nplanes %ld\nrefused %ld\n", plans, planes, refused);
  return 0;
}
