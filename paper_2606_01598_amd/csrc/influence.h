// The influence function g(k) of Eqs. green, influence and potential_k along one line of
// the half spectrum (fixed y and kz, any x), for the x pass that makes it value by value:
//   g(k) = (4 pi / k^2) exp(-k^2 / (4 alpha^2)) dcx(kx) dcy(ky) dcz(kz), g(0) = 0,
//   k^2 = f^T M f, M = 4 pi^2 C^-1 C^-T (reciprocal metric), f = signed frequencies;
// a Nyquist bin takes the mean of g over the bin and its Hermitian partner, whose
// non-Nyquist components change sign.
#pragma once

#include "kernels.h"
#include "pme_common.h"

namespace pme {

__device__ __forceinline__ int signed_freq(int k, int N) { return (k >= (N + 1) / 2) ? k - N : k; }

struct Influence {
  double alpha;
  const float* dc[3];   // deconvolution factors (optimal influence: 1 / denominator)
  const float* al[3];   // optimal influence: aliasing weights [3][N_a]
};

inline Influence make_influence(const DevPlan& d) {
  Influence i;
  i.alpha = d.alpha;
  for (int k = 0; k < 3; ++k) { i.dc[k] = d.deconv[k]; i.al[k] = d.alias[k]; }
  return i;
}

struct InfluenceLine {
  double M[6];        // xx yy zz xy xz yz of the metric, the mixed ones doubled
  double c0, c1;      // k^2 = c0 + f (c1 + f M_xx) at signed x frequency f
  double inv4a2;
  float ci[9];        // 2 pi (C^-1)[b][a] (cell gradient)
  int y, kz, fy, fz;
  bool ny, nz;        // Nyquist bins along y, z
  float dcy, dcz;

  __device__ __forceinline__ void set(const Influence& a, const double* box, const int (&N)[3],
                                      int y_, int kz_) {
    const Cell c = cell_from_box(box);
    auto m = [&](int p, int q) {
      return 4.0 * M_PI * M_PI *
             (c.inv[p] * c.inv[q] + c.inv[3 + p] * c.inv[3 + q] + c.inv[6 + p] * c.inv[6 + q]);
    };
    M[0] = m(0, 0); M[1] = m(1, 1); M[2] = m(2, 2);
    M[3] = 2.0 * m(0, 1); M[4] = 2.0 * m(0, 2); M[5] = 2.0 * m(1, 2);
#pragma unroll
    for (int k = 0; k < 9; ++k) ci[k] = float(2.0 * M_PI * c.inv[k]);
    y = y_; kz = kz_;
    fy = signed_freq(y, N[1]); fz = signed_freq(kz, N[2]);
    ny = ((N[1] & 1) == 0) && (2 * y == N[1]);
    nz = ((N[2] & 1) == 0) && (2 * kz == N[2]);
    inv4a2 = 1.0 / (4.0 * a.alpha * a.alpha);
    c0 = M[1] * fy * fy + M[2] * fz * fz + M[5] * fy * fz;
    c1 = M[3] * fy + M[4] * fz;
    dcy = a.dc[1][y]; dcz = a.dc[2][kz];
  }

  // (4 pi / k^2) exp(-k^2 / (4 alpha^2)).  k^2, its reciprocal and the exponent are
  // formed in double precision and rounded once each to float: constants rounded to
  // float would bias every g(k) alike (about 1e-7 relative, which the near cancellation
  // of E_recip against the self terms would amplify in E^lr).  The reciprocal is the
  // hardware estimate with two Newton steps (the rounding to float hides the rest).
  __device__ __forceinline__ float green(double k2) const {
    double r = __builtin_amdgcn_rcp(k2);
    r = fma(fma(-k2, r, 1.0), r, r);
    r = fma(fma(-k2, r, 1.0), r, r);
    return float(4.0 * M_PI * r) * expf(-float(k2 * inv4a2));
  }
  __device__ __forceinline__ float green(float px, float py, float pz) const {
    const double x = px, v = py, z = pz;
    return green(M[0] * x * x + M[1] * v * v + M[2] * z * z + M[3] * x * v + M[4] * x * z +
                 M[5] * v * z);
  }

  // g at x0 + r step, r = 0 .. R - 1.  The Nyquist bins (one x of a line, or a whole line
  // of the y or z Nyquist plane) are made again with their partners in a second pass, so
  // that the first has no branches.
  template <int R>
  __device__ __forceinline__ void values(const Influence& a, const int (&N)[3], int x0, int step,
                                         float (&g)[R]) const {
    const int half = (N[0] & 1) ? -1 : N[0] / 2;   // the x Nyquist bin
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = x0 + r * step;
      const double f = signed_freq(x, N[0]);
      g[r] = green(fma(fma(M[0], f, c1), f, c0)) * (a.dc[0][x] * dcy * dcz);
    }
    if ((y | kz) == 0 && x0 == 0) g[0] = 0.0f;
    if (ny || nz || (half >= x0 && (half - x0) % step == 0)) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int x = x0 + r * step;
        if (ny || nz || x == half) {
          const float fx = float(signed_freq(x, N[0]));
          g[r] = 0.5f * (green(fx, float(fy), float(fz)) +
                         green(x == half ? fx : -fx, float(ny ? fy : -fy), float(nz ? fz : -fz))) *
                 (a.dc[0][x] * dcy * dcz);
        }
      }
    }
  }
  __device__ __forceinline__ float value(const Influence& a, const int (&N)[3], int x) const {
    float g[1];
    values<1>(a, N, x, 1, g);
    return g[0];
  }

  // the sum over the aliases f + m N of U^2 G, over the separable denominator; a partner
  // frequency s f (s = -1 on the flipped axes) takes the weight of alias -m of f, as sinc
  // is even.  Loops, not straight-line code: the caller keeps its registers.
  __device__ __forceinline__ float optimal(const Influence& a, const int (&N)[3], int x) const {
    if ((x | y | kz) == 0) return 0.0f;
    const float fx = float(signed_freq(x, N[0]));
    const bool nx = ((N[0] & 1) == 0) && (2 * x == N[0]);
    const int terms = nx || ny || nz ? 2 : 1;
    float g = 0.0f;
#pragma unroll 1
    for (int t = 0; t < terms; ++t) {
      const int sx = t && !nx ? -1 : 1, sy = t && !ny ? -1 : 1, sz = t && !nz ? -1 : 1;
      float num = 0.0f;
#pragma unroll 1
      for (int m = 0; m < 9; ++m) {
        const int mx = m / 3 - 1, my = m % 3 - 1;
        const float uxy = a.al[0][(sx * mx + 1) * N[0] + x] * a.al[1][(sy * my + 1) * N[1] + y];
#pragma unroll
        for (int mz = -1; mz <= 1; ++mz)
          num = fmaf(uxy * a.al[2][(sz * mz + 1) * N[2] + kz],
                     green(float(sx) * fx + float(mx * N[0]), float(sy * fy) + float(my * N[1]),
                           float(sz * fz) + float(mz * N[2])), num);
      }
      g += num;
    }
    return (terms == 2 ? 0.5f * g : g) * (a.dc[0][x] * dcy * dcz);
  }

  // cell gradient: w |v|^2 G(k) D(f) (1/k^2 + 1/(4 alpha^2)) k k^T with k = 2 pi C^-1 f,
  // the mean over a Nyquist bin and its partner as for g (off the Nyquist bins g itself
  // is G D of this point; on them each of the two needs its own G)
  __device__ __forceinline__ void cell_terms(const Influence& a, const int (&N)[3], int x, float wv2,
                                             float g, float (&acc)[6]) const {
    const int fxi = signed_freq(x, N[0]);
    if ((fxi | fy | fz) == 0) return;
    const bool nx = ((N[0] & 1) == 0) && (2 * x == N[0]);
    const bool nyq = nx || ny || nz;
    const float dc = nyq ? a.dc[0][x] * dcy * dcz : 0.0f;
    const float q = float(inv4a2);
    auto add = [&](float fx, float gy, float gz, float scale) {
      const float k0 = ci[0] * fx + ci[1] * gy + ci[2] * gz;
      const float k1 = ci[3] * fx + ci[4] * gy + ci[5] * gz;
      const float k2c = ci[6] * fx + ci[7] * gy + ci[8] * gz;
      const float k2 = k0 * k0 + k1 * k1 + k2c * k2c;
      const float gk = nyq ? 4.0f * float(M_PI) / k2 * expf(-k2 * q) * dc : g;
      const float f = scale * gk * (1.0f / k2 + q);
      acc[0] = fmaf(f, k0 * k0, acc[0]);
      acc[1] = fmaf(f, k1 * k1, acc[1]);
      acc[2] = fmaf(f, k2c * k2c, acc[2]);
      acc[3] = fmaf(f, k0 * k1, acc[3]);
      acc[4] = fmaf(f, k0 * k2c, acc[4]);
      acc[5] = fmaf(f, k1 * k2c, acc[5]);
    };
    const float fx = float(fxi), gy = float(fy), gz = float(fz);
    if (nyq) {
      add(fx, gy, gz, 0.5f * wv2);
      add(nx ? fx : -fx, ny ? gy : -gy, nz ? gz : -gz, 0.5f * wv2);
    } else {
      add(fx, gy, gz, wv2);
    }
  }
};

}  // namespace pme
