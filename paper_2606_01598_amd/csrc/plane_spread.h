// Pieces shared by the x-plane spreads (Sec. 2.3.2, Eq. charge_dipole_assign): the
// plane spread fused with the slab transform (fft.hip, k_spread_slab) and the band
// spread (band.hip, k_spread_band).  A workgroup of either lists the records of the
// bins whose atoms can reach its plane (or band) and adds each reaching atom's p x p
// footprint in its x-plane into 64-bit fixed-point LDS words with the tile spread's
// expressions, so that every word equals the tile spread's.
#pragma once

#include "kernels.h"
#include "pme_common.h"

namespace pme {

// body(record index) for every record of the scanned bins (bin_of(e) is the e-th of nscan:
// its number and its counter's) and of the overflow list, by a whole workgroup of up to 1024
// threads.  The slots are numbered by a scan of the bins' counts and their records listed in
// LDS (s_rec, map_cap of them at a time); a lane takes slots far from its neighbours', so
// that lanes do not add to the same mesh points at once.  Bins are one mesh cell wide in x
// (but for tiles that would hold too many of them, see plan_bins), so that apart from the
// overflow list and bands' edge rows every listed record is wanted: testing the anchors of
// wider bins, compacting the hits and scanning an item map took more instructions than
// adding the atoms.  At 1M ions on 320^3 a band spread keeps the vector units busy for 72 %
// of its time (82 % for the tangent density) and LDS for half of it.  s_wsum: one int per wavefront.
template <class BinOf, class Body>
__device__ __forceinline__ void for_each_slot(int nscan, BinOf bin_of, const int* count, int cap,
                                              const int* ovf_count, long long ovf_base,
                                              uint32_t* s_rec, int map_cap, int* s_wsum,
                                              Body body) {
  const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const int nwave = nthr >> 6;
  const int novf = *ovf_count;
  for (int w0 = 0;; w0 += map_cap) {   // windows of map_cap slots
    int total = 0;
    for (int r0 = 0; r0 < nscan; r0 += nthr) {
      const int e = r0 + tid;
      int c = 0, base = 0;
      if (e < nscan) {
        const int2 bin = bin_of(e);   // its record block and its counter
        c = min(count[bin.y], cap);
        base = bin.x * cap;
      }
      int incl = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane == 63) s_wsum[wave] = incl;
      __syncthreads();
      int before = 0, all = 0;
      for (int w = 0; w < nwave; ++w) {
        const int v = s_wsum[w];
        before += w < wave ? v : 0;
        all += v;
      }
      const int off = total + before + incl - c - w0;
      for (int k = max(0, -off); k < min(c, map_cap - off); ++k) s_rec[off + k] = uint32_t(base + k);
      total += all;
      __syncthreads();   // s_wsum has been read
    }
    {
      const int off = total - w0;
      for (int k = max(0, -off) + tid; k < min(novf, map_cap - off); k += nthr)
        s_rec[off + k] = uint32_t(ovf_base + k);
      total += novf;
    }
    __syncthreads();
    const int n = min(total - w0, map_cap);
    const int rows = (n + 63) >> 6;
    for (int r = wave; r < rows; r += nwave) {
      const int slot = lane * rows + r;
      if (slot < n) body(size_t(s_rec[slot]));
    }
    if (w0 + map_cap >= total) break;
    __syncthreads();   // s_rec has been read
  }
}

// One atom's footprint in x-plane X (nothing when its stencil misses the plane): record
// ri's weights and coefficients with the tile spread's arithmetic, and its P x P words
// added at row rows(b_y, iy) (skipped from row_limit on) and padded column b_z + iz of `plane` (rows of PZ words).  DEG 1 takes the
// forward coefficients from a forward record, or with TREC forms q and J mu from a
// tangent record; DEG 2 forms the ten tangent coefficients.  s_J holds J (DEG 2 or
// TREC), s_cw the whole-number spline pieces, scale the fixed-point unit; reaches(b_y):
// whether any of its rows is wanted.
template <int P, int DEG, bool TREC, class Reaches, class Rows>
__device__ __forceinline__ void add_atom_plane(const float* rec, size_t ri, const float* s_J,
                                               const float* s_cw, int X, int Nx, float scale,
                                               unsigned long long* plane, int PZ,
                                               Reaches reaches, Rows rows, int row_limit) {
  static_assert(!TREC || DEG == 1, "tangent records serve the forward density");
  constexpr int NC = (DEG == 1) ? 4 : 10;
  constexpr int D = (DEG == 1) ? 1 : 2;       // highest weight derivative needed
  constexpr int lo = (P - 1) / 2;
  const float4* r = reinterpret_cast<const float4*>(rec + ri * kRecWords);
  const float4 h = r[0];
  const int pk = __float_as_int(h.w);
  const int by = (pk >> 10) & 1023, bz = (pk >> 20) & 1023;
  int ix = X - (pk & 1023) + lo;
  ix += (ix < 0) ? Nx : 0;
  ix -= (ix >= Nx) ? Nx : 0;
  if (ix >= P || !reaches(by)) return;
  const float4 c0v = r[1];
  float co[NC];
  if constexpr (DEG == 2) {
    const float4 c1v = r[2];
    const float* f = rec + ri * kRecWords;   // v_mu
    float Jt[3][3];
#pragma unroll
    for (int i = 0; i < 9; ++i) Jt[i / 3][i % 3] = s_J[i];
    tangent_coeffs(Jt, c0v.x, make_float3(c0v.y, c0v.z, c0v.w), c1v.x,
                   make_float3(c1v.y, c1v.z, c1v.w), make_float3(f[12], f[13], f[14]), co);
  } else if constexpr (TREC) {
    float Jt[3][3];
#pragma unroll
    for (int i = 0; i < 9; ++i) Jt[i / 3][i % 3] = s_J[i];
    const float3 d = jmul(Jt, make_float3(c0v.y, c0v.z, c0v.w));
    co[0] = c0v.x; co[1] = d.x; co[2] = d.y; co[3] = d.z;
  } else {
    co[0] = c0v.x; co[1] = c0v.y; co[2] = c0v.z; co[3] = c0v.w;
  }
  // this plane's x weights (whole-number, times the fixed-point unit): the column ix
  // of spline_weights_whole, with the same Horner steps
  float x[D + 1];
  weight_at_lds<P, D>(s_cw, ix, h.x, x);
#pragma unroll
  for (int d = 0; d <= D; ++d) x[d] *= scale;
  // this x-plane's coefficients of the (y, z) derivative monomials
  float ax0, az1, az2 = 0.f, ay1, ay2 = 0.f, ayz = 0.f;
  if (DEG == 1) {
    ax0 = co[0] * x[0] + co[1] * x[1];   // W_y W_z
    ay1 = co[2] * x[0];                  // W_y' W_z
    az1 = co[3] * x[0];                  // W_y W_z'
  } else {
    ax0 = co[0] * x[0] + co[1] * x[1] + co[4] * x[2];
    ay1 = co[2] * x[0] + co[7] * x[1];
    az1 = co[3] * x[0] + co[8] * x[1];
    ay2 = co[5] * x[0];
    az2 = co[6] * x[0];
    ayz = co[9] * x[0];
  }
  float wy[D + 1][P], wz[D + 1][P];
  spline_weights_whole<P, D>(h.y, wy);
  spline_weights_whole<P, D>(h.z, wz);
#pragma unroll
  for (int iy = 0; iy < P; ++iy) {
    const int rr = rows(by, iy);
    if (rr >= row_limit) continue;
    const float y0 = wy[0][iy], y1 = wy[1][iy];
    float c0 = ax0 * y0 + ay1 * y1, c1 = az1 * y0, c2 = 0.f;
    if (D == 2) {
      const float y2 = wy[2][iy];
      c0 += ay2 * y2;
      c1 += ayz * y1;
      c2 = az2 * y0;
    }
    unsigned long long* row = plane + rr * PZ + bz;
#pragma unroll
    for (int iz = 0; iz < P; ++iz) {
      float v = c0 * wz[0][iz] + c1 * wz[1][iz];
      if (D == 2) v += c2 * wz[2][iz];
      atomicAdd(row + iz, to_fixed(v));
    }
  }
}

}  // namespace pme
