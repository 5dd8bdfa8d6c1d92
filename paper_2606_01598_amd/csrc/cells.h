// Cell list for the real-space pair kernels (polarizable model, dipole-head
// features): atoms binned by fractional coordinate into a grid of cells at least
// one cutoff wide, by a counting sort (count, exclusive scan, scatter).  A pair
// kernel visits, for each atom, the 3 x 3 x 3 neighbouring cells, or every cell
// along an axis with fewer than three, so that with the cutoff below half the
// smallest perpendicular width every pair within the cutoff is seen once under the
// minimum image.  The sort leaves the positions themselves in cell order
// (CellList::sp), so the candidates of a row of cells are consecutive 16-byte loads.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "../../include/pme.h"

namespace {

struct CellGrid {
  float C[9];                       // rows are lattice vectors
  float Ci[9];                      // inverse: s = r Ci
  int nc[3];
  int ncell;
};

// Several device arrays out of one allocation (each is a call into the driver): take()
// the sizes, allocate(), then ask for the addresses.
struct Carve {
  size_t bytes = 0;
  char* base = nullptr;
  template <class T>
  size_t take(size_t count) {
    const size_t at = bytes;
    bytes += (sizeof(T) * count + 255) / 256 * 256;
    return at;
  }
  hipError_t allocate() { return hipMalloc(reinterpret_cast<void**>(&base), bytes ? bytes : 256); }
  template <class T>
  T* at(size_t offset) const { return reinterpret_cast<T*>(base + offset); }
};

struct CellList {
  CellGrid g;
  char* base = nullptr;             // the allocation that holds the arrays
  int* count = nullptr;             // [ncell]
  int* start = nullptr;             // [ncell + 1]
  int* cellof = nullptr;            // [max_atoms]
  int* slot = nullptr;              // [max_atoms]
  float4* sp = nullptr;             // [max_atoms] atoms grouped by cell: position, atom (bits)
};

__device__ __forceinline__ void frac(const CellGrid& g, float x, float y, float z, float& s0,
                                     float& s1, float& s2) {
  s0 = x * g.Ci[0] + y * g.Ci[3] + z * g.Ci[6];
  s1 = x * g.Ci[1] + y * g.Ci[4] + z * g.Ci[7];
  s2 = x * g.Ci[2] + y * g.Ci[5] + z * g.Ci[8];
}

// Cell of a point (wrapped into the cell; NaN coordinates land in cell 0 of an axis).
__device__ __forceinline__ void cell_of(const CellGrid& g, float x, float y, float z, int (&c)[3]) {
  float s[3];
  frac(g, x, y, z, s[0], s[1], s[2]);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float t = s[a] - floorf(s[a]);
    const int k = int(t * float(g.nc[a]));
    c[a] = (k < 0) ? 0 : ((k >= g.nc[a]) ? g.nc[a] - 1 : k);
  }
}

// Minimum-image displacement: the nearest whole lattice vector is found through
// fractional coordinates and taken off the Cartesian difference itself, which keeps
// the difference exact for pairs of the same image (going back from fractional
// coordinates rounds at the cell's size: 3e-6 Angstrom in a 50 Angstrom box).
__device__ __forceinline__ float3 min_image(const CellGrid& g, float dx, float dy, float dz) {
  float f0, f1, f2;
  frac(g, dx, dy, dz, f0, f1, f2);
  const float n0 = -rintf(f0), n1 = -rintf(f1), n2 = -rintf(f2);
  return make_float3(fmaf(n0, g.C[0], fmaf(n1, g.C[3], fmaf(n2, g.C[6], dx))),
                     fmaf(n0, g.C[1], fmaf(n1, g.C[4], fmaf(n2, g.C[7], dy))),
                     fmaf(n0, g.C[2], fmaf(n1, g.C[5], fmaf(n2, g.C[8], dz))));
}

// Neighbour cell number `o` (0 .. min(nc, 3) - 1) along an axis of a cell c.
__device__ __forceinline__ int neighbour_cell(int c, int o, int nc) {
  return (nc >= 3) ? (c + o - 1 + nc) % nc : o;
}

// The runs of consecutive cell-ordered atoms that hold the neighbours of cell c: run e
// (0 .. 17) is segment e % 2 of row (ox, oy) = (e / 6, e / 2 % 3); a row's z cells
// c_z - 1 .. c_z + 1 are one run, or two where they wrap.  Returns an empty run where
// there is none (fewer than three cells along an axis: each cell once).
constexpr int kCellRuns = 18;
__device__ __forceinline__ int2 cell_run(const CellGrid& g, const int* start, const int (&c)[3],
                                         int e) {
  const int ox = e / 6, oy = (e >> 1) % 3, seg = e & 1;
  if (e >= kCellRuns || ox >= min(g.nc[0], 3) || oy >= min(g.nc[1], 3)) return make_int2(0, 0);
  const int row = (neighbour_cell(c[0], ox, g.nc[0]) * g.nc[1] + neighbour_cell(c[1], oy, g.nc[1])) *
                  g.nc[2];
  const int last = g.nc[2] - 1;
  int z0 = max(c[2] - 1, 0), z1 = min(c[2] + 1, last);
  if (g.nc[2] <= 3) { z0 = 0; z1 = last; }
  if (seg) {
    if (g.nc[2] <= 3 || (c[2] != 0 && c[2] != last)) return make_int2(0, 0);
    z0 = z1 = c[2] == 0 ? last : 0;
  }
  return make_int2(start[row + z0], start[row + z1 + 1]);
}

// Sum over a wavefront; every lane gets it.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// LDS written by some lanes of a wavefront, read by others of the same one: LDS
// operations of a wavefront stay in order, only the compiler has to keep them so.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The pairs of atom i (at pi) within the cutoff, by one whole wavefront: candidates are
// tested 64 at a time and those within the cutoff queued in `list` (64 + BATCH entries
// of LDS: R = r_i - r_j, atom j in bits); batch(entries, count) is called with up to
// BATCH of them.  FLAT numbers the candidates of all runs through, at about 90
// instructions a round: for cells of a few atoms, whose runs leave most lanes idle.
template <int BATCH, bool FLAT, class F>
__device__ __forceinline__ void visit_pairs(const CellGrid& g, const int* start, const float4* sp,
                                            const float4 pi, int i, float rc2, float4* list,
                                            F&& batch) {
  const int lane = threadIdx.x & 63;
  int c[3];
  cell_of(g, pi.x, pi.y, pi.z, c);
  const int2 runs = cell_run(g, start, c, lane);   // lane e holds run e
  int cnt = 0;
  auto test = [&](int k, bool in) {
    const float4 pj = sp[in ? k : 0];
    const float3 R = min_image(g, pi.x - pj.x, pi.y - pj.y, pi.z - pj.z);
    const float r2 = R.x * R.x + R.y * R.y + R.z * R.z;
    // a NaN distance is a pair too, so that it reaches the outputs
    const bool hit = in && !(r2 >= rc2) && !(r2 <= 0.0f) && __float_as_int(pj.w) != i;
    const unsigned long long m = __ballot(hit);
    const int below = int(__builtin_amdgcn_mbcnt_hi(
        uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)));
    if (hit) list[cnt + below] = make_float4(R.x, R.y, R.z, pj.w);
    cnt += __popcll(m);
    if (cnt >= BATCH) {
      wave_lds_fence();
      int o = 0;
      for (; cnt - o >= BATCH; o += BATCH) batch(list + o, BATCH);
      cnt -= o;
      float4 rest;
      if (lane < cnt) rest = list[o + lane];
      wave_lds_fence();
      if (lane < cnt) list[lane] = rest;
    }
  };
  if constexpr (FLAT) {
    const int len = runs.y - runs.x;
    int end = len;   // end of the run in the numbering, then k minus the number in it
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const int v = __shfl_up(end, o, 64);
      if (lane >= o) end += v;
    }
    const int total = __builtin_amdgcn_readlane(end, kCellRuns - 1);
    const int first = end - len, shift = runs.x - first;
    for (int b = 0; b < total; b += 64) {
      const int t = b + lane;
      int k = 0;
#pragma unroll
      for (int s = 0; s < kCellRuns; ++s)   // the last run that starts at or before t
        if (t >= __builtin_amdgcn_readlane(first, s)) k = t + __builtin_amdgcn_readlane(shift, s);
      test(k, t < total);
    }
  } else {
    for (int s = 0; s < kCellRuns; ++s) {
      const int k0 = __builtin_amdgcn_readlane(runs.x, s);
      const int k1 = __builtin_amdgcn_readlane(runs.y, s);
      for (int b = k0; b < k1; b += 64) test(b + lane, b + lane < k1);
    }
  }
  wave_lds_fence();
  if (cnt) batch(list, cnt);
}

__global__ void k_cell_clear(int* count, int ncell) {
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < ncell; c += gridDim.x * blockDim.x)
    count[c] = 0;
}

__global__ void k_cell_count(int n, const float* pos, CellGrid g, int* count, int* cellof,
                             int* slot) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int c[3];
  cell_of(g, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], c);
  const int cell = (c[0] * g.nc[1] + c[1]) * g.nc[2] + c[2];
  cellof[i] = cell;
  slot[i] = atomicAdd(&count[cell], 1);
}

// exclusive scan of the cell counts (one workgroup of 1024)
__global__ void __launch_bounds__(1024) k_cell_scan(const int* count, int* start, int ncell) {
  __shared__ int part[1024];
  const int t = threadIdx.x;
  const int seg = (ncell + 1023) / 1024;
  const int s0 = min(t * seg, ncell), s1 = min(s0 + seg, ncell);
  int acc = 0;
  for (int c = s0; c < s1; ++c) acc += count[c];
  part[t] = acc;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = (t >= o) ? part[t - o] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int run = part[t] - acc;
  for (int c = s0; c < s1; ++c) { start[c] = run; run += count[c]; }
  if (t == 1023) start[ncell] = part[1023];
}

__global__ void k_cell_fill(int n, const float* pos, const int* cellof, const int* slot,
                            const int* start, float4* sp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  sp[start[cellof[i]] + slot[i]] =
      make_float4(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], __int_as_float(i));
}

// The whole counting sort in one workgroup, the counters in LDS: up to kSortAtoms atoms
// and kSortCells cells.  At 4096 atoms the four kernels above take 13 us and four
// launches, this one 7 us and one.  The limits keep a thread's atoms in registers and
// the counters in 48 KB.
constexpr int kSortAtoms = 8192, kSortCells = 12288;
__global__ void __launch_bounds__(1024) k_cell_sort(int n, const float* pos, CellGrid g,
                                                    int* start, float4* sp) {
  __shared__ int s_count[kSortCells];
  __shared__ int s_wave[16];
  constexpr int U = kSortAtoms / 1024;
  const int t = threadIdx.x;
  for (int c = t; c < g.ncell; c += 1024) s_count[c] = 0;
  float x[U], y[U], z[U];
  int cell[U], slot[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = t + u * 1024;
    if (i < n) { x[u] = pos[3 * i]; y[u] = pos[3 * i + 1]; z[u] = pos[3 * i + 2]; }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (t + u * 1024 < n) {
      int c[3];
      cell_of(g, x[u], y[u], z[u], c);
      cell[u] = (c[0] * g.nc[1] + c[1]) * g.nc[2] + c[2];
      slot[u] = atomicAdd(&s_count[cell[u]], 1);
    }
  }
  __syncthreads();
  // exclusive scan: a segment of cells per thread, wavefront prefix sums, their totals
  const int seg = (g.ncell + 1023) / 1024;
  const int c0 = min(t * seg, g.ncell), c1 = min(c0 + seg, g.ncell);
  int acc = 0;
  for (int c = c0; c < c1; ++c) acc += s_count[c];
  int incl = acc;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if ((t & 63) >= o) incl += v;
  }
  if ((t & 63) == 63) s_wave[t >> 6] = incl;
  __syncthreads();
  int run = incl - acc;
  for (int w = 0; w < (t >> 6); ++w) run += s_wave[w];
  for (int c = c0; c < c1; ++c) {
    const int v = s_count[c];
    s_count[c] = run;
    start[c] = run;
    run += v;
  }
  if (t == 1023) start[g.ncell] = run;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = t + u * 1024;
    if (i < n) {
      sp[s_count[cell[u]] + slot[u]] = make_float4(x[u], y[u], z[u], __int_as_float(i));
    }
  }
}

inline int cell_blocks(int m, int t) { return m > 0 ? (m + t - 1) / t : 1; }

// Grid of cells for a cell (host box, rows are lattice vectors) and cutoff, and
// its device arrays.  PME_EINVAL for a singular cell or a cutoff not below half
// the smallest perpendicular width.
inline int setup_cells(CellList& cl, const double* C, double rc, int max_atoms) {
  const double det = C[0] * (C[4] * C[8] - C[5] * C[7]) - C[1] * (C[3] * C[8] - C[5] * C[6]) +
                     C[2] * (C[3] * C[7] - C[4] * C[6]);
  if (!isfinite(det) || fabs(det) < 1e-12) return PME_EINVAL;
  double Ci[9];
  Ci[0] = (C[4] * C[8] - C[5] * C[7]) / det; Ci[1] = (C[2] * C[7] - C[1] * C[8]) / det;
  Ci[2] = (C[1] * C[5] - C[2] * C[4]) / det; Ci[3] = (C[5] * C[6] - C[3] * C[8]) / det;
  Ci[4] = (C[0] * C[8] - C[2] * C[6]) / det; Ci[5] = (C[2] * C[3] - C[0] * C[5]) / det;
  Ci[6] = (C[3] * C[7] - C[4] * C[6]) / det; Ci[7] = (C[1] * C[6] - C[0] * C[7]) / det;
  Ci[8] = (C[0] * C[4] - C[1] * C[3]) / det;
  // perpendicular widths w_a = 1 / |column a of C^-1|
  double w[3];
  for (int a = 0; a < 3; ++a)
    w[a] = 1.0 / sqrt(Ci[a] * Ci[a] + Ci[3 + a] * Ci[3 + a] + Ci[6 + a] * Ci[6 + a]);
  if (!(rc > 0.0) || !isfinite(rc) || rc >= 0.5 * fmin(w[0], fmin(w[1], w[2]))) return PME_EINVAL;
  long ncell = 1;
  for (int a = 0; a < 3; ++a) {
    int k = int(floor(w[a] / rc));
    if (k < 1) k = 1;
    if (k > 128) k = 128;
    cl.g.nc[a] = k;
    ncell *= k;
  }
  cl.g.ncell = int(ncell);
  for (int k = 0; k < 9; ++k) { cl.g.C[k] = float(C[k]); cl.g.Ci[k] = float(Ci[k]); }
  const size_t m = size_t(max_atoms), c = size_t(ncell);
  Carve all;
  const size_t at_sp = all.take<float4>(m), at_count = all.take<int>(c),
               at_start = all.take<int>(c + 1), at_cellof = all.take<int>(m),
               at_slot = all.take<int>(m);
  const hipError_t e = all.allocate();
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? PME_ENOMEM : PME_EHIP;
  cl.base = all.base;
  cl.sp = all.at<float4>(at_sp);
  cl.count = all.at<int>(at_count);
  cl.start = all.at<int>(at_start);
  cl.cellof = all.at<int>(at_cellof);
  cl.slot = all.at<int>(at_slot);
  return PME_OK;
}

inline void free_cells(CellList& cl) {
  if (cl.base) (void)hipFree(cl.base);
  cl = CellList();
}

// Cell list of the current positions (one launch on `s`, or four for many atoms).
inline hipError_t build_cells(const CellList& cl, hipStream_t s, int n, const float* pos) {
  const CellGrid& g = cl.g;
  if (n <= kSortAtoms && g.ncell <= kSortCells) {
    hipLaunchKernelGGL(k_cell_sort, dim3(1), dim3(1024), 0, s, n, pos, g, cl.start, cl.sp);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_cell_clear, dim3(cell_blocks(g.ncell, 256)), dim3(256), 0, s, cl.count,
                     g.ncell);
  if (n > 0)
    hipLaunchKernelGGL(k_cell_count, dim3(cell_blocks(n, 256)), dim3(256), 0, s, n, pos, g,
                       cl.count, cl.cellof, cl.slot);
  hipLaunchKernelGGL(k_cell_scan, dim3(1), dim3(1024), 0, s, cl.count, cl.start, g.ncell);
  if (n > 0)
    hipLaunchKernelGGL(k_cell_fill, dim3(cell_blocks(n, 256)), dim3(256), 0, s, n, pos,
                       cl.cellof, cl.slot, cl.start, cl.sp);
  return hipGetLastError();
}

}  // namespace
