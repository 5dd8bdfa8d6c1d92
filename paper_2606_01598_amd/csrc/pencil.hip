// The mesh operator K of Secs. 2.3.3-2.3.4 on meshes whose y-z planes exceed LDS: five
// passes over the half spectrum (z real-to-complex, y, x with the influence function
// and the energy, y inverse, z complex-to-real; Eqs. fft, green, influence, potential_k,
// energy_recip, ifft).
//
// The spectrum is kept in blocks of 8 kz values, so that every pass moves runs of at
// least 64 bytes and all but the y passes' far side move long ones:
//   A [kz/8][x][y][w]   written by the z pass, read by the y pass (and back)
//   B [kz/8][y][x][w]   written by the y pass, transformed in place by the x pass
// with w = 8 values, or the H mod 8 that are left in the last block.  A is the plan's
// spectrum, B lies in the array the potential goes to, which is free until then.  (With
// one [x][y][kz] array the x and y passes read and wrote 32- and 64-byte pieces of
// strided, unaligned lines.)
//
// A line of N = R0 R1 points (R0 <= 20) is transformed by a butterfly per thread: stage 0
// from memory, one LDS exchange, stage 1 to memory (fft_radix.h, two_stage).  Other
// lengths go through LDS in the stages of radix_plan.
//
// Bound by memory traffic in the y passes (the 262 MB of one at 320^3 in 54 us on average,
// 41 at best: 4.8 and 6.4 TB/s); the others issue vector instructions for about half of
// their time and wait on memory for the rest (busy: x 55 %, which makes g in double
// precision between four register DFTs; z 55 and 41).  Alone at 320^3 x 105 us, z 70 and 87;
// through LDS stage by stage, from one [x][y][kz] array, y 130, x 151, z 76 and 99.
#include "../../include/pme.h"
#include "fft_radix.h"
#include "influence.h"
#include "kernels.h"
#include "pme_common.h"

namespace pme {
namespace {

constexpr int kLineMax = 16;        // lines of a y or x workgroup
constexpr int kTwoThreads = 320;    // a two-stage workgroup at most: 16 lines x radix 20
constexpr int kStageThreads = 512;  // workgroup of the general passes

// Where the lines of a workgroup lie: kz block kb of w values, `cnt` planes (x or y) from
// p0 on, line l = plane p0 + l / w, value l % w.
struct LineGroup {
  int kb, w, p0, lines;
  size_t base;    // of the kz block
};

__device__ __forceinline__ LineGroup line_group(int blk, int H, int n, size_t plane, int lines) {
  LineGroup g;
  const int nfull = H >> 3, per = (n + (lines >> 3) - 1) / (lines >> 3);
  int each = lines >> 3;
  if (blk < nfull * per) {
    g.kb = blk / per;
    g.w = 8;
    g.p0 = (blk - g.kb * per) * each;
  } else {
    g.kb = nfull;
    g.w = H - 8 * nfull;
    each = lines / g.w;
    g.p0 = (blk - nfull * per) * each;
  }
  g.lines = min(each, n - g.p0) * g.w;
  g.base = size_t(g.kb) * 8 * plane;
  return g;
}

// Twiddles into LDS (before the first barrier of the caller)
__device__ __forceinline__ void load_twiddles(float2* dst, const float2* src, int N) {
  for (int t = threadIdx.x; t < N; t += blockDim.x) dst[t] = src[t];
}

// The stages of a radix_plan over npen lines of stride ps in LDS, ping-pong; the buffer
// that holds the result.  Starts and ends with the data behind a barrier.
__device__ __forceinline__ float2* staged_fft(float2* x, float2* y, int npen, int ps,
                                              const AxisPlan& ax, const float2* tw, float s) {
  for (int i = 0; i < ax.nst; ++i) {
    const FFTStage& st = ax.st[i];
    for (int t = threadIdx.x; t < npen * st.NR; t += blockDim.x) {
      const int pen = int(fdiv(uint32_t(t), st.nr)), j = t - pen * st.NR;
      const int jq = int(fdiv(uint32_t(j), st.ns)), k = j - jq * st.Ns;
      with_radix(st.R, [&](auto rc) {
        stockham_butterfly<decltype(rc)::value>(x + pen * ps, y + pen * ps, j, k, jq, st.Ns, st.NR,
                                                st.step, tw, s);
      });
    }
    __syncthreads();
    float2* t = x; x = y; y = t;
  }
  return x;
}

struct ZArgs {
  AxisPlan ax;
  TwoStage two;
  const float2* tw;
  int rows;        // N_x N_y
  int H;
  int pairs;       // complex lines (two real rows each) per workgroup
  FastDiv nr0, nr1;   // division by R1 and by R0 (two-stage)
  const float* src;
  float2* spec;
  float* dst;
};

// value kz of spectrum row `row` in layout A
__device__ __forceinline__ size_t spec_at(const ZArgs& a, int row, int kz) {
  const int kb = kz >> 3, w = min(8, a.H - 8 * kb);
  return size_t(kb) * 8 * a.rows + size_t(row) * w + (kz & 7);
}

// z pass, real to complex: two real rows form one complex line,
//   X_even[k] = (Z[k] + conj Z[N-k]) / 2,  X_odd[k] = (Z[k] - conj Z[N-k]) / 2i.
template <bool TWO>
__global__ void __launch_bounds__(TWO ? 256 : kStageThreads) k_pencil_r2c(ZArgs a) {
  extern __shared__ float2 sm[];
  const int N = a.ax.N, H = a.H;
  const int r0 = blockIdx.x * 2 * a.pairs;
  const int np = min(a.pairs, (a.rows - r0 + 1) / 2);
  float2* tw = sm;
  float2* X = tw + N;
  load_twiddles(tw, a.tw, N);
  const float2* Z;
  int ps;
  auto value = [&](int c, int m) {
    const int ra = r0 + 2 * c;
    return make_float2(a.src[size_t(ra) * N + m], ra + 1 < a.rows ? a.src[size_t(ra + 1) * N + m] : 0.0f);
  };
  if constexpr (TWO) {
    const int R0 = a.two.R0, R1 = a.two.R1, t = threadIdx.x;
    ps = two_stage_words(R0, R1) | 1;
    {
      const int c = int(fdiv(uint32_t(t), a.nr0)), j = t - c * R1;
      if (c < np)
        with_wide_radix(R0, [&](auto rc) {
          two_stage_first<decltype(rc)::value>([&](int m) { return value(c, m); }, X + c * ps, j, R1,
                                               -1.0f);
        });
    }
    __syncthreads();
    const int c = int(fdiv(uint32_t(t), a.nr1)), j = t - c * R0;
    with_wide_radix(R1, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      float2 v[R];
      if (c < np) {
        two_stage_column<R>(X + c * ps, v, j, R0, tw, -1.0f);
        Dft<R>::run(v, -1.0f);
      }
      __syncthreads();   // the columns have been read
      if (c < np)
#pragma unroll
        for (int r = 0; r < R; ++r) X[c * ps + j + r * R0] = v[r];
    });
    __syncthreads();
    Z = X;
  } else {
    ps = N | 1;
    for (int e = threadIdx.x; e < np * N; e += blockDim.x) {
      const int c = e / N, m = e - c * N;
      X[c * ps + m] = value(c, m);
    }
    __syncthreads();
    Z = staged_fft(X, X + a.pairs * ps, np, ps, a.ax, tw, -1.0f);
  }
  // rows fastest within a kz block: runs of 2 np rows of 64 bytes
  const int nrow = min(2 * np, a.rows - r0);
  for (int kb = 0; 8 * kb < H; ++kb) {
    const int w = min(8, H - 8 * kb);
    float2* out = a.spec + size_t(kb) * 8 * a.rows + size_t(r0) * w;
    for (int e = threadIdx.x; e < nrow * w; e += blockDim.x) {
      const int rr = w == 8 ? e >> 3 : e / w, k = 8 * kb + e - rr * w;
      const float2 zk = Z[(rr >> 1) * ps + k], zn = Z[(rr >> 1) * ps + (k ? N - k : 0)];
      out[e] = (rr & 1) == 0 ? make_float2(0.5f * (zk.x + zn.x), 0.5f * (zk.y - zn.y))
                             : make_float2(0.5f * (zk.y + zn.y), -0.5f * (zk.x - zn.x));
    }
  }
}

// z pass, complex to real: P[m] = X_even[m] + i X_odd[m], X[m] = conj X[N-m] for m >= H
template <bool TWO>
__global__ void __launch_bounds__(TWO ? 256 : kStageThreads) k_pencil_c2r(ZArgs a) {
  extern __shared__ float2 sm[];
  const int N = a.ax.N, H = a.H;
  const int r0 = blockIdx.x * 2 * a.pairs;
  const int np = min(a.pairs, (a.rows - r0 + 1) / 2);
  const bool even = (N & 1) == 0;
  float2* tw = sm;
  float2* X = tw + N;
  load_twiddles(tw, a.tw, N);
  auto value = [&](int c, int m) {
    const int k = m < H ? m : N - m, ra = r0 + 2 * c;
    float2 A = a.spec[spec_at(a, ra, k)];
    float2 B = ra + 1 < a.rows ? a.spec[spec_at(a, ra + 1, k)] : make_float2(0.f, 0.f);
    if (m >= H) { A.y = -A.y; B.y = -B.y; }
    if (m == 0 || (even && m == N / 2)) { A.y = 0.0f; B.y = 0.0f; }
    return make_float2(A.x - B.y, A.y + B.x);
  };
  auto store = [&](int c, int m, float2 v) {
    const int ra = r0 + 2 * c;
    a.dst[size_t(ra) * N + m] = v.x;
    if (ra + 1 < a.rows) a.dst[size_t(ra + 1) * N + m] = v.y;
  };
  if constexpr (TWO) {
    const int R0 = a.two.R0, R1 = a.two.R1, t = threadIdx.x;
    const int ps = two_stage_words(R0, R1) | 1;
    {
      const int c = int(fdiv(uint32_t(t), a.nr0)), j = t - c * R1;
      if (c < np)
        with_wide_radix(R0, [&](auto rc) {
          two_stage_first<decltype(rc)::value>([&](int m) { return value(c, m); }, X + c * ps, j, R1,
                                               1.0f);
        });
    }
    __syncthreads();
    const int c = int(fdiv(uint32_t(t), a.nr1)), j = t - c * R0;
    if (c < np)
      with_wide_radix(R1, [&](auto rc) {
        two_stage_second<decltype(rc)::value>(
            X + c * ps, [&](int m, float2 v) { store(c, m, v); }, j, R0, tw, 1.0f);
      });
  } else {
    const int ps = N | 1;
    for (int e = threadIdx.x; e < np * N; e += blockDim.x) {
      const int c = e / N, m = e - c * N;
      X[c * ps + m] = value(c, m);
    }
    __syncthreads();
    const float2* Z = staged_fft(X, X + a.pairs * ps, np, ps, a.ax, tw, 1.0f);
    for (int e = threadIdx.x; e < np * N; e += blockDim.x) {
      const int c = e / N, m = e - c * N;
      store(c, m, Z[c * ps + m]);
    }
  }
}

struct YArgs {
  AxisPlan ax;
  TwoStage two;
  const float2* tw;
  int Nx, H, lines;
  int sy_in, sx_in, sy_out, sx_out;   // strides in values of w: A (1, N_y), B (N_x, 1)
  const float2* in;
  float2* out;
  float sign;
};

// y pass: lines of `lines / w` x-planes of one kz block, from one layout to the other
template <bool TWO>
__global__ void __launch_bounds__(TWO ? kTwoThreads : kStageThreads) k_pencil_y(YArgs a) {
  extern __shared__ float2 sm[];
  const int N = a.ax.N;
  const LineGroup g = line_group(xcd_item(blockIdx.x, gridDim.x), a.H, a.Nx, size_t(a.Nx) * N, a.lines);
  float2* tw = sm;
  float2* X = tw + N;
  load_twiddles(tw, a.tw, N);
  // thread -> (line l, butterfly j), the line fastest
  const int mask = a.lines - 1, shift = a.lines == 16 ? 4 : 3;
  const int l = threadIdx.x & mask;
  const int xi = g.w == 8 ? l >> 3 : l / g.w, kk = l - xi * g.w;
  const float2* in = a.in + g.base + size_t(g.p0 + xi) * a.sx_in * g.w + kk;
  float2* out = a.out + g.base + size_t(g.p0 + xi) * a.sx_out * g.w + kk;
  const int si = a.sy_in * g.w, so = a.sy_out * g.w;
  const bool live = l < g.lines;
  if constexpr (TWO) {
    const int R0 = a.two.R0, R1 = a.two.R1, j = threadIdx.x >> shift;
    float2* rows = X + l * (two_stage_words(R0, R1) | 1);
    if (live && j < R1)
      with_wide_radix(R0, [&](auto rc) {
        two_stage_first<decltype(rc)::value>([&](int y) { return in[size_t(y) * si]; }, rows, j, R1,
                                             a.sign);
      });
    __syncthreads();
    if (live && j < R0)
      with_wide_radix(R1, [&](auto rc) {
        two_stage_second<decltype(rc)::value>(
            rows, [&](int y, float2 v) { out[size_t(y) * so] = v; }, j, R0, tw, a.sign);
      });
  } else {
    const int ps = N | 1, step = blockDim.x >> shift;
    if (live)
      for (int y = threadIdx.x >> shift; y < N; y += step) X[l * ps + y] = in[size_t(y) * si];
    __syncthreads();
    const float2* Z = staged_fft(X, X + a.lines * ps, g.lines, ps, a.ax, tw, a.sign);
    if (live)
      for (int y = threadIdx.x >> shift; y < N; y += step) out[size_t(y) * so] = Z[l * ps + y];
  }
}

struct XArgs {
  AxisPlan ax;
  TwoStage two;
  const float2* tw;
  int N[3];
  int H, lines;
  float2* spec;    // layout B
  Influence inf;
  const double* box;
  double* epart;   // may be null
  double* vpart;   // cell gradient (MODE 1): six sums per workgroup
  float* gcache;   // MODE 2: tables of g, [workgroup][N_x lines], and the box of each
  double* gkey;
};

// x pass in place: forward transform, x g(k) with the energy partial, inverse.  The
// inverse takes the radices in reverse, so the last forward and the first inverse stage
// of a butterfly meet in registers with g between them.  g is made in registers before
// the butterfly's column is read; with 160 registers in the place of 128 (a few spills of
// the widest radices) a step at 320^3 takes 3.6 % longer, with 96 1.3 %.
// MODE 0: the influence function of Eq. influence; 1: also the cell-gradient partials;
// 2: the optimal influence function (its alias sums kept in the plan's table by box).
template <bool TWO, int MODE>
__global__ void __launch_bounds__(TWO ? kTwoThreads : kStageThreads)
__attribute__((amdgpu_waves_per_eu(4))) k_pencil_x(XArgs a) {
  extern __shared__ float2 sm[];
  __shared__ double red[16 * 6];
  const int Nx = a.N[0], Ny = a.N[1], Nz = a.N[2];
  const int blk = xcd_item(blockIdx.x, gridDim.x);
  const LineGroup g = line_group(blk, a.H, Ny, size_t(Nx) * Ny, a.lines);
  float2* tw = sm;
  float2* X = tw + Nx;
  const int mask = a.lines - 1, shift = a.lines == 16 ? 4 : 3;
  const int l = threadIdx.x & mask;
  const int yi = g.w == 8 ? l >> 3 : l / g.w, kk = l - yi * g.w;
  const bool live = l < g.lines;
  const int y = min(g.p0 + yi, Ny - 1), kz = 8 * g.kb + kk;
  float2* line = a.spec + g.base + size_t(y) * Nx * g.w + kk;
  const int w = g.w;

  InfluenceLine gl;
  float e_acc = 0.0f;
  float vacc[6] = {0, 0, 0, 0, 0, 0};
  const float wgt = (kz == 0 || (((Nz & 1) == 0) && 2 * kz == Nz)) ? 1.0f : 2.0f;
  // MODE 2: the workgroup's table of g at [x][line].  Where it is another box's, each thread
  // first makes the values that it will read (x0, x0 + stride, ..); the transform itself is
  // then the same code either way, with the registers of one load a value.  (Made inside the
  // butterfly the 27 aliases filled 256 registers: a step of 128k ions on 160^3 353 us with
  // the table kept, 213 so; forward and product of 1M on 320^3 2584 and 1722; a forward at
  // 160^3 whose cell changes at every call 239.)
  bool cached = false;
  float* table = nullptr;
  auto g_setup = [&](int x0, int stride, bool act) {
    if constexpr (MODE == 2) {
      table = a.gcache + size_t(blk) * Nx * a.lines + l;
      const double* key = a.gkey + size_t(blk) * 9;
      cached = true;
#pragma unroll
      for (int k = 0; k < 9; ++k) cached = cached && key[k] == a.box[k];
      if (!cached && act) {
        gl.set(a.inf, a.box, a.N, y, kz);
#pragma unroll 1
        for (int x = x0; x < Nx; x += stride) table[x * a.lines] = gl.optimal(a.inf, a.N, x);
      }
    } else {
      gl.set(a.inf, a.box, a.N, y, live ? kz : 0);
    }
  };
  // v x g with its share of the energy and of the cell gradient
  auto scale = [&](int x, float gg, float2 v) {
    const float v2 = v.x * v.x + v.y * v.y;
    e_acc = fmaf(wgt * gg, v2, e_acc);
    if constexpr (MODE == 1) gl.cell_terms(a.inf, a.N, x, wgt * v2, gg, vacc);
    return make_float2(v.x * gg, v.y * gg);
  };

  if constexpr (TWO) {
    const int R0 = a.two.R0, R1 = a.two.R1, j = threadIdx.x >> shift;
    float2* rows = X + l * (two_stage_words(R0, R1) | 1);
    if constexpr (MODE == 2) g_setup(j, R0, live && j < R0);
    with_wide_radix(R0, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      float2 v[R];
      const bool act = live && j < R1;
      if (act)
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = line[size_t(j + r * R1) * w];
      load_twiddles(tw, a.tw, Nx);
      if constexpr (MODE != 2) g_setup(0, 0, false);   // while the lines are in flight
      if (act) {
        Dft<R>::run(v, -1.0f);
#pragma unroll
        for (int r = 0; r < R; ++r) rows[j * (R + 1) + r] = v[r];
      }
    });
    with_wide_radix(R1, [&](auto rc) {
      constexpr int R = decltype(rc)::value;
      const bool act = live && j < R0;
      float2 v[R];
      // g before the column is read: fewer values live at once
      float gv[R];
      if (act) {
        if constexpr (MODE == 2) {
#pragma unroll
          for (int r = 0; r < R; ++r) gv[r] = table[(j + r * R0) * a.lines];
        } else {
          gl.values<R>(a.inf, a.N, j, R0, gv);
        }
      }
      __syncthreads();
      if (act) {
        two_stage_column<R>(rows, v, j, R0, tw, -1.0f);
        Dft<R>::run(v, -1.0f);
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = scale(j + r * R0, gv[r], v[r]);
        Dft<R>::run(v, 1.0f);
      }
      __syncthreads();   // the columns have been read
      if (act)
#pragma unroll
        for (int r = 0; r < R; ++r) rows[j * (R + 1) + r] = v[r];
    });
    __syncthreads();
    if (live && j < R1)
      with_wide_radix(R0, [&](auto rc) {
        two_stage_second<decltype(rc)::value>(
            rows, [&](int x, float2 v) { line[size_t(x) * w] = v; }, j, R1, tw, 1.0f);
      });
  } else {
    const int ps = Nx | 1, step = blockDim.x >> shift, t0 = threadIdx.x >> shift;
    load_twiddles(tw, a.tw, Nx);
    if (live)
      for (int x = t0; x < Nx; x += step) X[l * ps + x] = line[size_t(x) * w];
    g_setup(t0, step, live);
    __syncthreads();
    float2* Z = staged_fft(X, X + a.lines * ps, g.lines, ps, a.ax, tw, -1.0f);
    if (live)
      for (int x = t0; x < Nx; x += step) {
        const float gg = MODE == 2 ? table[x * a.lines] : gl.value(a.inf, a.N, x);
        Z[l * ps + x] = scale(x, gg, Z[l * ps + x]);
      }
    __syncthreads();
    Z = staged_fft(Z, Z == X ? X + a.lines * ps : X, g.lines, ps, a.ax, tw, 1.0f);
    if (live)
      for (int x = t0; x < Nx; x += step) line[size_t(x) * w] = Z[l * ps + x];
  }
  if constexpr (MODE == 2) {
    // the key last: every thread has read it before (barriers above)
    if (!cached && threadIdx.x < 9) a.gkey[size_t(blk) * 9 + threadIdx.x] = a.box[threadIdx.x];
  }
  if (a.epart) {
    double e[1] = {double(e_acc)};
    block_sums<1>(e, red);
    if (threadIdx.x == 0) a.epart[blk] = e[0];
  }
  if constexpr (MODE == 1) {
    double v[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) v[k] = vacc[k];
    block_sums<6>(v, red);
    if (threadIdx.x == 0)
#pragma unroll
      for (int k = 0; k < 6; ++k) a.vpart[6 * blk + k] = v[k];
  }
}

inline int round64(int n) { return (n + 63) / 64 * 64; }

// LDS of a workgroup: twiddles and `lines` lines (one buffer of two-stage rows, or two)
size_t line_lds(int N, TwoStage t, int lines) {
  const size_t buf = t.R0 ? size_t(lines) * (two_stage_words(t.R0, t.R1) | 1)
                          : 2 * size_t(lines) * (N | 1);
  return sizeof(float2) * (N + buf);
}

template <class Args>
hipError_t run(const LaunchEvents* ev, void (*two)(Args), void (*general)(Args), int blocks,
               int threads, size_t lds, hipStream_t s, const Args& a) {
  launch_k(ev, a.two.R0 ? two : general, dim3(blocks), dim3(threads), lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pencil(const DevPlan& d, hipStream_t s, const double* box, float* out,
                         bool energy, KTimer* tm, double* vpart) {
  const LaunchEvents* er = tm ? tm->next(PME_K_FFT_R2C) : nullptr;
  const LaunchEvents* ex = tm ? tm->next(PME_K_FFT_X) : nullptr;
  const LaunchEvents* ei = tm ? tm->next(PME_K_FFT_C2R) : nullptr;
  // a kind spanning two launches records its start with the first and its stop with the
  // second
  LaunchEvents er0, er1, ei0, ei1;
  if (er) { er0.start = er->start; er1.stop = er->stop; }
  if (ei) { ei0.start = ei->start; ei1.stop = ei->stop; }
  float2* B = reinterpret_cast<float2*>(out);   // mesh_floats(d) covers N_x N_y H values
  hipError_t e;

  ZArgs z;
  z.ax = d.ax[2]; z.two = two_stage(d.N[2]); z.tw = d.twiddle[2];
  z.rows = d.N[0] * d.N[1]; z.H = d.H; z.pairs = d.zpairs;
  z.nr0 = make_fast_div(z.two.R0 ? z.two.R1 : 1); z.nr1 = make_fast_div(z.two.R0 ? z.two.R0 : 1);
  z.src = d.rho; z.spec = d.spec; z.dst = out;
  const int zb = (z.rows + 2 * z.pairs - 1) / (2 * z.pairs);
  const int zt = z.two.R0 ? round64(z.pairs * z.two.R0) : kStageThreads;
  const size_t zl = line_lds(d.N[2], z.two, z.pairs);

  YArgs y;
  y.ax = d.ax[1]; y.two = two_stage(d.N[1]); y.tw = d.twiddle[1];
  y.Nx = d.N[0]; y.H = d.H; y.lines = d.ylines;
  const int yb = line_blocks(d.H, d.N[0], d.ylines);
  const int yt = y.two.R0 ? round64(y.lines * y.two.R0) : kStageThreads;
  const size_t yl = line_lds(d.N[1], y.two, y.lines);

  XArgs x;
  x.ax = d.ax[0]; x.two = two_stage(d.N[0]); x.tw = d.twiddle[0];
  for (int k = 0; k < 3; ++k) x.N[k] = d.N[k];
  x.H = d.H; x.lines = d.ktile; x.spec = B;
  x.inf = make_influence(d);
  x.box = box;
  x.epart = energy ? d.epart : nullptr;
  x.vpart = vpart;
  x.gcache = d.gcache; x.gkey = d.gkey;
  const int xt = x.two.R0 ? round64(x.lines * x.two.R0) : kStageThreads;
  const size_t xl = line_lds(d.N[0], x.two, x.lines);

  if ((e = run(er ? &er0 : nullptr, k_pencil_r2c<true>, k_pencil_r2c<false>, zb, zt, zl, s, z)) !=
      hipSuccess)
    return e;
  y.in = d.spec; y.out = B; y.sign = -1.0f;
  y.sy_in = 1; y.sx_in = d.N[1]; y.sy_out = d.N[0]; y.sx_out = 1;
  if ((e = run(er ? &er1 : nullptr, k_pencil_y<true>, k_pencil_y<false>, yb, yt, yl, s, y)) !=
      hipSuccess)
    return e;
  const int xb = fftx_blocks(d);
  if (vpart) e = run(ex, k_pencil_x<true, 1>, k_pencil_x<false, 1>, xb, xt, xl, s, x);
  else if (d.opt) e = run(ex, k_pencil_x<true, 2>, k_pencil_x<false, 2>, xb, xt, xl, s, x);
  else e = run(ex, k_pencil_x<true, 0>, k_pencil_x<false, 0>, xb, xt, xl, s, x);
  if (e != hipSuccess) return e;
  y.in = B; y.out = d.spec; y.sign = 1.0f;
  y.sy_in = d.N[0]; y.sx_in = 1; y.sy_out = 1; y.sx_out = d.N[1];
  if ((e = run(ei ? &ei0 : nullptr, k_pencil_y<true>, k_pencil_y<false>, yb, yt, yl, s, y)) !=
      hipSuccess)
    return e;
  return run(ei ? &ei1 : nullptr, k_pencil_c2r<true>, k_pencil_c2r<false>, zb, zt, zl, s, z);
}

// Lines per workgroup: 16 where a butterfly is a thread and three such workgroups fit a
// CU's LDS, else 8 (a kz block; with 16 the far side is whole 128-byte lines, a step at
// 320^3 takes 0.7 % longer with 8); z lines so that a round fills 256 threads, or 8
// pairs in the general passes, and three workgroups fit as well (125 x 125 x 625, general: a
// forward 379 us with 8 pairs, one workgroup a CU, and 333 with 4).
void pencil_lines(DevPlan& d) {
  for (int a = 0; a < 2; ++a) {
    const TwoStage t = two_stage(d.N[a]);
    (a == 0 ? d.ktile : d.ylines) =
        t.R0 && line_lds(d.N[a], t, kLineMax) <= size_t(kLineLdsTwo) ? kLineMax : 8;
  }
  const TwoStage t = two_stage(d.N[2]);
  d.zpairs = t.R0 ? 256 / t.R0 : 8;
  while (d.zpairs > 1 && line_lds(d.N[2], t, d.zpairs) > size_t(kLineLdsTwo)) --d.zpairs;
}

hipError_t enable_pencil_lds() {
  const void* fns[] = {reinterpret_cast<const void*>(k_pencil_r2c<false>),
                       reinterpret_cast<const void*>(k_pencil_c2r<false>),
                       reinterpret_cast<const void*>(k_pencil_y<false>),
                       reinterpret_cast<const void*>(k_pencil_x<false, 0>),
                       reinterpret_cast<const void*>(k_pencil_x<false, 1>),
                       reinterpret_cast<const void*>(k_pencil_x<false, 2>)};
  for (const void* f : fns) {
    const hipError_t e =
        hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLineLdsGeneral);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace pme
