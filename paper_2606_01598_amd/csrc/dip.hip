// Learned dipole head: local features, the SiLU MLP forward and backward, the
// training loss against the polarizable teacher and Adam (definitions in dip.h).
//
// Features give a wavefront to an atom over the cell list of cells.h: the pairs within
// the cutoff are queued, their radial functions are made a pair per lane, and then each
// lane sums one of the atom's 64 channels over the queued pairs.  The networks run 16
// atoms per workgroup in fp32 matrix instructions.  Parameter gradients are summed per
// workgroup, then over workgroups in a fixed order.
#include <math.h>
#include <stdio.h>

#include <new>

#include "../../include/dip.h"
#include "cells.h"

namespace {

constexpr int NR = 8, NS = 2, NCH = DIP_NCH, NF = DIP_NFEAT, HID = DIP_HIDDEN;
constexpr int NP = DIP_NPARAM;
constexpr int oW1 = 0, ob1 = oW1 + HID * NF, oW2 = ob1 + HID, ob2 = oW2 + HID * HID;
constexpr int oW3 = ob2 + HID, ob3 = oW3 + NCH * HID;
static_assert(ob3 + NCH == NP, "parameter layout");
static_assert(NCH == NR * NS && NF == 2 * NCH + NS, "feature layout");

constexpr int kFeatThreads = 256;
constexpr int kFeatAtoms = kFeatThreads / 64;   // one wavefront per atom
constexpr int kFeatBatch = 32;                  // pairs whose radial functions are held at once

struct FeatArgs {
  int n;
  const float* pos;
  const float* q;
  CellGrid g;
  const int* start;
  const float4* sp;
  float rc;
  float* feat;
  float* vec;
};

// Radial functions of one pair, R_k = norm sin((k+1) pi x) env / r, and with dR their
// r-derivatives; sin and cos of the multiples by the Chebyshev recurrences.
__device__ __forceinline__ void radial(float r, float ir, float irc, float (&Rk)[NR], float* dR) {
  const float norm = sqrtf(2.0f * irc), kpi = float(M_PI) * irc;
  const float x = r * irc, x2 = x * x, x4 = x2 * x2, x5 = x4 * x;
  const float env = 1.0f - 21.0f * x5 + 35.0f * x5 * x - 15.0f * x5 * x2;
  const float denv = (-105.0f * x4 + 210.0f * x5 - 105.0f * x5 * x) * irc;
  float sn, cs;
  sincospif(x, &sn, &cs);
  float s_prev = 0.0f, s_cur = sn, c_prev = 1.0f, c_cur = cs;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    Rk[k] = norm * s_cur * env * ir;
    if (dR)
      dR[k] = norm * ((k + 1) * kpi * c_cur * env * ir - s_cur * env * ir * ir + s_cur * ir * denv);
    const float s_next = 2.0f * cs * s_cur - s_prev;
    const float c_next = 2.0f * cs * c_cur - c_prev;
    s_prev = s_cur;
    s_cur = s_next;
    c_prev = c_cur;
    c_cur = c_next;
  }
}

// Channel (component, species, k) of a lane: component 0 is the scalar G, 1..3 are V.
// Bound by latency and issue: at 4096 ions and 5 Angstrom an atom has 110 candidates and
// 17 pairs.  With 16 lanes an atom the long radial body ran for an eighth of its lanes,
// and 64 sums a lane were shuffled together at the end; here a pair's radial functions
// are made once and the sums need no shuffle: 31 -> 9 us.
__global__ void __launch_bounds__(kFeatThreads) k_features(FeatArgs a) {
  __shared__ float4 s_pair[kFeatAtoms][64 + kFeatBatch];
  __shared__ float s_R[kFeatAtoms][kFeatBatch][NR];
  __shared__ float4 s_w[kFeatAtoms][kFeatBatch];       // (1, q_j u)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int at = blockIdx.x * kFeatAtoms + wave;
  if (at >= a.n) return;   // no workgroup barrier below
  const float4 pi = a.sp[at];
  const int i = __builtin_amdgcn_readfirstlane(__float_as_int(pi.w));
  const int k = lane & 7, s = (lane >> 3) & 1, comp = lane >> 4;
  float acc = 0.0f;
  visit_pairs<kFeatBatch, true>(
      a.g, a.start, a.sp, pi, i, a.rc * a.rc, s_pair[wave], [&](const float4* l, int nb) {
        float qj = 0.0f;
        if (lane < nb) {
          const float4 p = l[lane];
          const float r = sqrtf(p.x * p.x + p.y * p.y + p.z * p.z), ir = 1.0f / r;
          float Rk[NR];
          radial(r, ir, 1.0f / a.rc, Rk, nullptr);
#pragma unroll
          for (int m = 0; m < NR; ++m) s_R[wave][lane][m] = Rk[m];
          qj = a.q[__float_as_int(p.w)];
          s_w[wave][lane] = make_float4(1.0f, qj * p.x * ir, qj * p.y * ir, qj * p.z * ir);
        }
        const unsigned long long other = __ballot(qj > 0.0f) ^ (s ? 0ull : ~0ull);
        wave_lds_fence();
        const float* R = &s_R[wave][0][k];
        const float* w = reinterpret_cast<const float*>(&s_w[wave][0]) + comp;
        // left out, not multiplied by zero: a NaN stays in its species' channels
        for (int m = 0; m < nb; ++m) {
          const float sum = fmaf(R[NR * m], w[4 * m], acc);
          acc = (other >> m) & 1 ? acc : sum;
        }
        wave_lds_fence();
      });
  float v2 = acc * acc;   // |V|^2 of (species, k): the sum over the three components
  v2 = __shfl(v2, 16 + (lane & 15), 64) + __shfl(v2, 32 + (lane & 15), 64) +
       __shfl(v2, 48 + (lane & 15), 64);
  float* f = a.feat + size_t(i) * NF;
  if (comp == 0) {
    f[lane] = acc;
    f[NCH + lane] = v2;
  } else {
    a.vec[size_t(i) * NCH * 3 + 3 * (lane & 15) + comp - 1] = acc;
  }
  if (lane < NS) f[2 * NCH + lane] = (a.q[i] > 0.0f) == (lane == 0) ? 1.0f : 0.0f;
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

__device__ __forceinline__ float d2silu(float z) {
  const float s = 1.0f / (1.0f + expf(-z));
  return s * (1.0f - s) * (2.0f + z * (1.0f - 2.0f * s));
}

// ---- the networks on the matrix cores -------------------------------------------
//
// One workgroup of four wavefronts runs 16 atoms.  Every layer is out^T = W in^T in
// 16 x 16 x 4 fp32 matrix instructions: wavefront w makes hidden units 16 w .. 16 w + 15
// of the 16 atoms, lane l = 16 g + a holding units 4 g + r (r = 0..3) of atom a, and the
// next layer contracts them in that same order (k = 16 T + 4 g + r in step (T, r)), so
// that activations pass through LDS as they lie and the weights come straight from
// memory, one value a lane and step.  Bound by latency: a layer is at most 16 dependent
// matrix instructions of 32 cycles.  One wavefront of 64 hidden units per workgroup with
// the weights staged through LDS took 36 to 63 us a kernel at 4096 atoms; these take 5
// to 8 us, the parameter gradient of the dual network 16 us.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kNetThreads = 256;
constexpr int HS = HID + 4;           // LDS row of hidden units: 16-byte rows, no conflicts
constexpr int CS = NCH + 4;

__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

struct NetLane {
  int l16, g, w;
  __device__ __forceinline__ NetLane()
      : l16(threadIdx.x & 15), g((threadIdx.x >> 4) & 3),
        w(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {}
};

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }

// f(z) of the four units a lane holds
template <class F>
__device__ __forceinline__ f32x4 map4(f32x4 z, F f) {
  return f32x4{f(z[0]), f(z[1]), f(z[2]), f(z[3])};
}

// The inputs of atom a0 + l16 as the second operand of layer 1 (zeros past na or for a
// NULL array): k = 16 T + 4 g + r, then k = 32 + g.
struct NetIn {
  float v[9];
  __device__ __forceinline__ void load(const NetLane& L, const float* feat, int a0, int na) {
    const bool in = feat && L.l16 < na;
    const float* f = feat + size_t(a0 + L.l16) * NF;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = in ? f[16 * (k >> 2) + 4 * L.g + (k & 3)] : 0.0f;
    v[8] = in && L.g < NF - 32 ? f[32 + L.g] : 0.0f;
  }
};

// Layer 1 weights of the lane's row (hidden unit 16 w + l16) in the same order
struct NetW1 {
  float v[9];
  __device__ __forceinline__ void load(const NetLane& L, const float* W) {
    const float* f = W + (16 * L.w + L.l16) * NF;
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = f[16 * (k >> 2) + 4 * L.g + (k & 3)];
    v[8] = L.g < NF - 32 ? f[32 + L.g] : 0.0f;
  }
};

__device__ __forceinline__ f32x4 layer1(const NetW1& W, const NetIn& x, f32x4 acc) {
#pragma unroll
  for (int k = 0; k < 9; ++k) acc = mma(W.v[k], x.v[k], acc);
  return acc;
}

__device__ __forceinline__ f32x4 bias4(const NetLane& L, const float* b) {
  const float* f = b + 16 * L.w + 4 * L.g;
  return f32x4{f[0], f[1], f[2], f[3]};
}

// the lane's four units of its atom into a [16][HS] LDS matrix
__device__ __forceinline__ void put_units(const NetLane& L, float (*m)[HS], f32x4 v) {
  *reinterpret_cast<f32x4*>(&m[L.l16][16 * L.w + 4 * L.g]) = v;
}

// sum over the 64 units of m: acc += W m^T with the weights in w4 (k = 16 T + 4 g + r)
__device__ __forceinline__ f32x4 contract64(const NetLane& L, const float (&w4)[16],
                                            const float (*m)[HS], f32x4 acc) {
#pragma unroll
  for (int T = 0; T < 4; ++T) {
    const f32x4 h = *reinterpret_cast<const f32x4*>(&m[L.l16][16 * T + 4 * L.g]);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = mma(w4[4 * T + r], h[r], acc);
  }
  return acc;
}

// Partial results of the four wavefronts (16 rows 4 g + r of atom l16 each) added up;
// every wavefront gets the sum.  Two barriers; `part` is free after the second.
__device__ __forceinline__ f32x4 sum_waves(const NetLane& L, float (*part)[16][CS], f32x4 v) {
  *reinterpret_cast<f32x4*>(&part[L.w][L.l16][4 * L.g]) = v;
  __syncthreads();
  f32x4 s = zero4();
#pragma unroll
  for (int w = 0; w < 4; ++w) s += *reinterpret_cast<const f32x4*>(&part[w][L.l16][4 * L.g]);
  __syncthreads();
  return s;
}

// Weights of the dipole head a lane feeds forward, loaded at once
struct NetWeights {
  NetW1 w1;
  float w2[16], w3[4];
  f32x4 b1, b2, b3;
  __device__ __forceinline__ void load(const NetLane& L, const float* P) {
    w1.load(L, P + oW1);
    const float* r2 = P + oW2 + (16 * L.w + L.l16) * HID;
    const float* r3 = P + oW3 + L.l16 * HID + 16 * L.w;
#pragma unroll
    for (int k = 0; k < 16; ++k) w2[k] = r2[16 * (k >> 2) + 4 * L.g + (k & 3)];
#pragma unroll
    for (int r = 0; r < 4; ++r) w3[r] = r3[4 * L.g + r];
    b1 = bias4(L, P + ob1);
    b2 = bias4(L, P + ob2);
    b3 = f32x4{P[ob3 + 4 * L.g], P[ob3 + 4 * L.g + 1], P[ob3 + 4 * L.g + 2], P[ob3 + 4 * L.g + 3]};
  }
};

struct NetLds {
  float h1[16][HS];
  float part[4][16][CS];
};
template <bool DUAL>
struct NetLdsT : NetLds {
  float h1d[DUAL ? 16 : 1][HS];
};

// What the forward pass leaves in registers: pre-activations, activations and the
// output weights w (channels 4 g + r of atom l16, in every wavefront); with DUAL their
// tangents along feat_dot.
template <bool DUAL>
struct NetState {
  f32x4 z1, z2, h2, w;
  f32x4 z1d, z2d, h2d, wd;
};

template <bool DUAL>
__device__ __forceinline__ void net_forward(const NetLane& L, const NetWeights& W, const NetIn& x,
                                            const NetIn& xd, NetLdsT<DUAL>& m,
                                            NetState<DUAL>& s) {
  s.z1 = layer1(W.w1, x, W.b1);
  put_units(L, m.h1, map4(s.z1, silu));
  if constexpr (DUAL) {
    s.z1d = layer1(W.w1, xd, zero4());
    put_units(L, m.h1d, map4(s.z1, dsilu) * s.z1d);
  }
  __syncthreads();
  s.z2 = contract64(L, W.w2, m.h1, W.b2);
  s.h2 = map4(s.z2, silu);
  f32x4 w = zero4(), wd = zero4();
#pragma unroll
  for (int r = 0; r < 4; ++r) w = mma(W.w3[r], s.h2[r], w);
  if constexpr (DUAL) {
    s.z2d = contract64(L, W.w2, m.h1d, zero4());
    s.h2d = map4(s.z2, dsilu) * s.z2d;
#pragma unroll
    for (int r = 0; r < 4; ++r) wd = mma(W.w3[r], s.h2d[r], wd);
  }
  s.w = sum_waves(L, m.part, w) + W.b3;
  if constexpr (DUAL) s.wd = sum_waves(L, m.part, wd);
}

// Component d of the vector channels 4 g + r of atom a0 + l16 (zeros past na)
__device__ __forceinline__ f32x4 channels(const NetLane& L, const float* vec, int a0, int na,
                                          int d) {
  f32x4 v = zero4();
  if (vec && L.l16 < na) {
    const float* f = vec + size_t(a0 + L.l16) * NCH * 3 + 12 * L.g + d;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = f[3 * r];
  }
  return v;
}
__device__ __forceinline__ float sum_groups(float v) {   // over g, the four 16-lane groups
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float dot4(f32x4 a, f32x4 b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + a[3] * b[3];
}
__device__ __forceinline__ float of3(const float* p, size_t k) { return p ? p[k] : 0.0f; }

// mu = sum_c w_c V_c and with DUAL mu_dot = sum_c (wd_c V_c + w_c Vd_c); 16 atoms per
// workgroup, component d by wavefront d.
template <bool DUAL>
__global__ void __launch_bounds__(kNetThreads) k_mlp_forward(int n, const float* P,
                                                             const float* feat, const float* vec,
                                                             const float* feat_dot,
                                                             const float* vec_dot, float* mu,
                                                             float* mud) {
  __shared__ __attribute__((aligned(16))) NetLdsT<DUAL> m;
  const NetLane L;
  const int a0 = blockIdx.x * 16, na = min(16, n - a0);
  NetWeights W;
  NetIn x, xd;
  x.load(L, feat, a0, na);
  if constexpr (DUAL) xd.load(L, feat_dot, a0, na);
  W.load(L, P);
  const int d = min(L.w, 2);
  const f32x4 V = channels(L, vec, a0, na, d);
  f32x4 Vd = zero4();
  if constexpr (DUAL) Vd = channels(L, vec_dot, a0, na, d);
  NetState<DUAL> s;
  net_forward<DUAL>(L, W, x, xd, m, s);
  const float v = sum_groups(dot4(s.w, V));
  float vd = 0.0f;
  if constexpr (DUAL) vd = sum_groups(dot4(s.wd, V) + dot4(s.w, Vd));
  if (L.w < 3 && L.g == 0 && L.l16 < na) {
    const size_t k = size_t(a0 + L.l16) * 3 + d;
    if (mu) mu[k] = v;
    if (DUAL && mud) mud[k] = vd;
  }
}

// The transposed products of the backward passes, weights loaded at once: W3 for
// gh2 = W3^T gw (units 16 w + l16, channels 4 g + r), W2 for gh1 = W2^T gz2.
struct NetBack {
  float w3[4], w2[16];
  __device__ __forceinline__ void load(const NetLane& L, const float* P) {
    const int u = 16 * L.w + L.l16;
#pragma unroll
    for (int r = 0; r < 4; ++r) w3[r] = P[oW3 + (4 * L.g + r) * HID + u];
#pragma unroll
    for (int k = 0; k < 16; ++k) w2[k] = P[oW2 + (16 * (k >> 2) + 4 * L.g + (k & 3)) * HID + u];
  }
};

// Layer 1 transposed over the wavefront's own 16 units: its share of dL/dx_k for the
// inputs 16 kt + 4 g + r (the species one-hot does not move)
struct NetInBack {
  float w[2][4];
  __device__ __forceinline__ void load(const NetLane& L, const float* W1) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) w[kt][r] = W1[(16 * L.w + 4 * L.g + r) * NF + 16 * kt + L.l16];
  }
  __device__ __forceinline__ f32x4 run(int kt, f32x4 gz) const {
    f32x4 acc = zero4();
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = mma(w[kt][r], gz[r], acc);
    return acc;
  }
};

// Feature cotangents of the position vector-Jacobian product for dL/dmu = u:
// fbar[i] = [dL/dG_i (16) | dL/dV_i (16 x 3)], with dL/dw_c = u . V_c run back through
// the network to its inputs and dL/dV_c = w_c u + 2 (dL/dx_{16+c}) V_c.
__global__ void __launch_bounds__(kNetThreads) k_mlp_input_grad(int n, const float* P,
                                                                const float* feat,
                                                                const float* vec, const float* u,
                                                                float* fbar) {
  __shared__ __attribute__((aligned(16))) NetLdsT<false> m;
  const NetLane L;
  const int a0 = blockIdx.x * 16, na = min(16, n - a0);
  NetWeights W;
  NetBack B;
  NetInBack I;
  NetIn x;
  x.load(L, feat, a0, na);
  W.load(L, P);
  B.load(L, P);
  I.load(L, P + oW1);
  f32x4 V[3], gw = zero4();
  float uu[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    V[d] = channels(L, vec, a0, na, d);
    uu[d] = L.l16 < na ? u[size_t(a0 + L.l16) * 3 + d] : 0.0f;
    gw += uu[d] * V[d];
  }
  NetState<false> s;
  net_forward<false>(L, W, x, x, m, s);
  f32x4 g = zero4();
#pragma unroll
  for (int r = 0; r < 4; ++r) g = mma(B.w3[r], gw[r], g);
  put_units(L, m.h1, g * map4(s.z2, dsilu));   // h1 was last read before sum_waves' barriers
  __syncthreads();
  g = contract64(L, B.w2, m.h1, zero4()) * map4(s.z1, dsilu);
  const f32x4 gG = sum_waves(L, m.part, I.run(0, g));
  const f32x4 gS = sum_waves(L, m.part, I.run(1, g));
  // wavefront w writes channel 4 g + w
  if (L.l16 < na) {
    float* f = fbar + size_t(a0 + L.l16) * 4 * NCH;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r == L.w) {
        const int c = 4 * L.g + r;
        f[c] = gG[r];
#pragma unroll
        for (int d = 0; d < 3; ++d) f[NCH + 3 * c + d] = s.w[r] * uu[d] + 2.0f * gS[r] * V[d][r];
      }
  }
}

// sum_a A[a][row] B[a][col] over the 16 atoms: rows 16 rt + l16 of an LDS matrix (its
// stride S) against b(atom, t) = B[4 g + t][col of the lane]
template <int S, class Bf>
__device__ __forceinline__ f32x4 outer16(const NetLane& L, const float (*A)[S], int row0, Bf b,
                                         f32x4 acc) {
#pragma unroll
  for (int t = 0; t < 4; ++t) acc = mma(A[4 * L.g + t][row0 + L.l16], b(4 * L.g + t), acc);
  return acc;
}

// Outer products of hidden-unit cotangents gz (LDS, the wavefront's rows 16 w ..) with
// the 34 inputs, into three tiles of 16 columns
__device__ __forceinline__ void outer_inputs(const NetLane& L, const float (*gz)[HS],
                                             const float* feat, int a0, int na, f32x4 (&acc)[3]) {
  if (!feat) return;
#pragma unroll
  for (int T = 0; T < 3; ++T) {
    const int k = 16 * T + L.l16;
    acc[T] = outer16<HS>(L, gz, 16 * L.w,
                         [&](int a) { return k < NF && a < na ? feat[size_t(a0 + a) * NF + k] : 0.0f; },
                         acc[T]);
  }
}

// the lane's rows 16 w + 4 g + r, columns 16 T + l16 < cols of a row-major array
template <int T>
__device__ __forceinline__ void put_rows(const NetLane& L, float* out, int cols,
                                         const f32x4 (&acc)[T]) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int k = 16 * t + L.l16;
    if (k < cols)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(16 * L.w + 4 * L.g + r) * cols + k] = acc[t][r];
  }
}
// sums over the atoms of the lane's units (lanes of one group), written by its first lane
__device__ __forceinline__ void put_sums(const NetLane& L, float* out, f32x4 v) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v[r] += __shfl_xor(v[r], o, 16);
    if (L.l16 == 0) out[4 * L.g + r] = v[r];
  }
}

template <bool DUAL>
struct GradLds : NetLdsT<DUAL> {
  float h2[16][HS], gz1[16][HS], gz2[16][HS];
  float gw[16][CS];
  float h2d[DUAL ? 16 : 1][HS], gz1d[DUAL ? 16 : 1][HS], gz2d[DUAL ? 16 : 1][HS];
  float gwd[DUAL ? 16 : 1][CS];
};

// Dipole-head parameter gradient.  Cotangents on w: gw_c = (g0 + g1 + g2) . V_c, and
// with DUAL + u . Vd_c on w and gwd_c = u . V_c on wd, run back through the primal and
// the tangent activations (silu'' couples them).  The workgroup walks the 16-atom tiles
// blockIdx.x, + gridDim.x, ..; the weight gradients are outer products over its atoms,
// kept in matrix accumulators and written once to the workgroup's partial row.
template <bool DUAL>
__global__ void __launch_bounds__(kNetThreads) k_mlp_backward(
    int n, const float* P, const float* feat, const float* vec, const float* feat_dot,
    const float* vec_dot, const float* g0, const float* g1, const float* g2, const float* u,
    float* part) {
  __shared__ __attribute__((aligned(16))) GradLds<DUAL> m;
  const NetLane L;
  NetWeights W;
  NetBack B;
  W.load(L, P);
  B.load(L, P);
  f32x4 aW1[3], aW2[4], aW3[1], ab1 = zero4(), ab2 = zero4(), ab3 = zero4();
#pragma unroll
  for (int t = 0; t < 4; ++t) aW2[t] = zero4();
#pragma unroll
  for (int t = 0; t < 3; ++t) aW1[t] = zero4();
  aW3[0] = zero4();
  const int tiles = (n + 15) / 16;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int a0 = tile * 16, na = min(16, n - a0);
    NetIn x, xd;
    x.load(L, feat, a0, na);
    if constexpr (DUAL) xd.load(L, feat_dot, a0, na);
    f32x4 gw = zero4(), gwd = zero4();
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const f32x4 V = channels(L, vec, a0, na, d);
      const size_t k = size_t(a0 + L.l16) * 3 + d;
      const bool in = L.l16 < na;
      gw += (in ? of3(g0, k) + of3(g1, k) + of3(g2, k) : 0.0f) * V;
      if constexpr (DUAL) {
        const float ud = in ? of3(u, k) : 0.0f;
        gw += ud * channels(L, vec_dot, a0, na, d);
        gwd += ud * V;
      }
    }
    __syncthreads();   // the previous tile's outer products are done with the LDS
    NetState<DUAL> s;
    net_forward<DUAL>(L, W, x, xd, m, s);
    put_units(L, m.h2, s.h2);
    if constexpr (DUAL) put_units(L, m.h2d, s.h2d);
    if (L.w == 0) {
      *reinterpret_cast<f32x4*>(&m.gw[L.l16][4 * L.g]) = gw;
      if constexpr (DUAL) *reinterpret_cast<f32x4*>(&m.gwd[L.l16][4 * L.g]) = gwd;
      ab3 += gw;
    }
    f32x4 g = zero4(), gd = zero4();
#pragma unroll
    for (int r = 0; r < 4; ++r) g = mma(B.w3[r], gw[r], g);
    f32x4 ds = map4(s.z2, dsilu);
    f32x4 gz2 = g * ds;
    if constexpr (DUAL) {
#pragma unroll
      for (int r = 0; r < 4; ++r) gd = mma(B.w3[r], gwd[r], gd);
      gz2 += gd * map4(s.z2, d2silu) * s.z2d;
      put_units(L, m.gz2d, gd * ds);
    }
    put_units(L, m.gz2, gz2);
    ab2 += gz2;
    __syncthreads();
    g = contract64(L, B.w2, m.gz2, zero4());
    ds = map4(s.z1, dsilu);
    f32x4 gz1 = g * ds;
    if constexpr (DUAL) {
      gd = contract64(L, B.w2, m.gz2d, zero4());
      gz1 += gd * map4(s.z1, d2silu) * s.z1d;
      put_units(L, m.gz1d, gd * ds);
    }
    put_units(L, m.gz1, gz1);
    ab1 += gz1;
    __syncthreads();
    outer_inputs(L, m.gz1, feat, a0, na, aW1);
#pragma unroll
    for (int T = 0; T < 4; ++T)
      aW2[T] = outer16<HS>(L, m.gz2, 16 * L.w, [&](int a) { return m.h1[a][16 * T + L.l16]; }, aW2[T]);
    aW3[0] = outer16<CS>(L, m.gw, 0, [&](int a) { return m.h2[a][16 * L.w + L.l16]; }, aW3[0]);
    if constexpr (DUAL) {
      outer_inputs(L, m.gz1d, feat_dot, a0, na, aW1);
#pragma unroll
      for (int T = 0; T < 4; ++T)
        aW2[T] = outer16<HS>(L, m.gz2d, 16 * L.w, [&](int a) { return m.h1d[a][16 * T + L.l16]; },
                             aW2[T]);
      aW3[0] = outer16<CS>(L, m.gwd, 0, [&](int a) { return m.h2d[a][16 * L.w + L.l16]; }, aW3[0]);
    }
  }
  float* out = part + size_t(blockIdx.x) * NP;
  put_rows(L, out + oW1, NF, aW1);
  put_rows(L, out + oW2, HID, aW2);
#pragma unroll
  for (int r = 0; r < 4; ++r) out[oW3 + (4 * L.g + r) * HID + 16 * L.w + L.l16] = aW3[0][r];
  put_sums(L, out + ob1 + 16 * L.w, ab1);
  put_sums(L, out + ob2 + 16 * L.w, ab2);
  if (L.w == 0) put_sums(L, out + ob3, ab3);
}

struct VjpArgs {
  int n;
  const float* pos;
  const float* q;
  CellGrid g;
  const int* start;
  const float4* sp;
  float rc;
  const float* fbar;   // [n][64] feature cotangents
  const float* base;   // [n][3] added to the output, or NULL
  float* g_pos;        // [n][3] out
};

// d/dR of the features of the centre atom of a pair (R = r_c - r_o, neighbour o
// with charge qo) contracted with the cotangents cg[k], cv[k][3] of the neighbour's
// species: sum_k cg R_k' u + qo [R_k' (cv.u) u + R_k / r (cv - (cv.u) u)].  c points at
// 16-byte aligned cg; cv follows `to_v` floats later.
__device__ __forceinline__ float3 pair_vjp(const float* c, int to_v, float qo, float ux, float uy,
                                           float uz, const float (&Rk)[NR], const float (&dR)[NR],
                                           float ir) {
  float cg[NR], cv[3 * NR];
#pragma unroll
  for (int k = 0; k < NR; k += 4)
    *reinterpret_cast<float4*>(cg + k) = *reinterpret_cast<const float4*>(c + k);
#pragma unroll
  for (int k = 0; k < 3 * NR; k += 4)
    *reinterpret_cast<float4*>(cv + k) = *reinterpret_cast<const float4*>(c + to_v + k);
  float fx = 0.0f, fy = 0.0f, fz = 0.0f;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    const float vx = cv[3 * k], vy = cv[3 * k + 1], vz = cv[3 * k + 2];
    const float cu = vx * ux + vy * uy + vz * uz;
    const float a = cg[k] * dR[k] + qo * (dR[k] - Rk[k] * ir) * cu;
    const float b = qo * Rk[k] * ir;
    fx += a * ux + b * vx;
    fy += a * uy + b * vy;
    fz += a * uz + b * vz;
  }
  return make_float3(fx, fy, fz);
}

// g_i = sum_j [d/dr_i of the features of i, with i's cotangents] + [d/dr_i of the
// features of j, with j's cotangents]: the pair (i, j) is visited from i only, so no
// atomics are needed.  A wavefront per atom, a queued pair per lane (52 -> 10 us at 4096
// ions against 16 lanes an atom with the pairs evaluated where they are found).
__global__ void __launch_bounds__(kFeatThreads) k_features_vjp(VjpArgs a) {
  __shared__ float4 s_pair[kFeatAtoms][128];
  __shared__ __attribute__((aligned(16))) float s_f[kFeatAtoms][4 * NCH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int at = blockIdx.x * kFeatAtoms + wave;
  if (at >= a.n) return;   // no workgroup barrier below
  const float4 pi = a.sp[at];
  const int i = __builtin_amdgcn_readfirstlane(__float_as_int(pi.w));
  const float* fi = s_f[wave];
  s_f[wave][lane] = a.fbar[size_t(i) * 4 * NCH + lane];
  wave_lds_fence();
  const float qi = a.q[i];
  const int si = qi > 0.0f ? 0 : 1;
  float gx = 0.0f, gy = 0.0f, gz = 0.0f;
  visit_pairs<64, true>(
      a.g, a.start, a.sp, pi, i, a.rc * a.rc, s_pair[wave], [&](const float4* l, int nb) {
        if (lane >= nb) return;
        const float4 p = l[lane];
        const int j = __float_as_int(p.w);
        const float r = sqrtf(p.x * p.x + p.y * p.y + p.z * p.z), ir = 1.0f / r;
        const float ux = p.x * ir, uy = p.y * ir, uz = p.z * ir;
        float Rk[NR], dR[NR];
        radial(r, ir, 1.0f / a.rc, Rk, dR);
        const float qj = a.q[j];
        const int sj = qj > 0.0f ? 0 : 1;
        // features of i (neighbour j of species sj), R_ij = R; then features of j
        // (neighbour i of species si), R_ji = -R
        const float3 f1 = pair_vjp(fi + sj * NR, NCH + 2 * sj * NR, qj, ux, uy, uz, Rk, dR, ir);
        const float3 f2 = pair_vjp(a.fbar + size_t(j) * 4 * NCH + si * NR, NCH + 2 * si * NR, qi,
                                   -ux, -uy, -uz, Rk, dR, ir);
        gx += f1.x - f2.x;
        gy += f1.y - f2.y;
        gz += f1.z - f2.z;
      });
  gx = wave_sum(gx);
  gy = wave_sum(gy);
  gz = wave_sum(gz);
  if (lane < 3) {
    const float g = lane == 0 ? gx : (lane == 1 ? gy : gz);
    a.g_pos[3 * i + lane] = a.base ? g + a.base[3 * i + lane] : g;
  }
}

// ---- Charge head ------------------------------------------------------------------
//
// c_i = w2 . silu(W1 x_i + b1) on the same tiles: layer 1 by matrix instructions, the
// output sum over the units of a lane, its group and the four wavefronts.

constexpr int NQP = DIP_NQPARAM;
constexpr int oQW1 = 0, oQb1 = HID * NF, oQw2 = oQb1 + HID;
static_assert(oQw2 + HID == NQP, "charge head layout");
constexpr int kGradBlocks = 256;      // cap on the workgroups of the parameter gradients

// c and its tangent c_dot along feat_dot (uncentred), and their sums over the tile's
// atoms into csum[2 blockIdx.x ..] (FP64; k_qcentre adds them up)
__global__ void __launch_bounds__(kNetThreads) k_qhead_forward(int n, const float* P,
                                                               const float* feat,
                                                               const float* feat_dot, float* c,
                                                               float* cd, double* csum) {
  __shared__ float part[2][4][16];
  const NetLane L;
  const int a0 = blockIdx.x * 16, na = min(16, n - a0);
  NetW1 W;
  NetIn x, xd;
  x.load(L, feat, a0, na);
  xd.load(L, feat_dot, a0, na);
  W.load(L, P + oQW1);
  const f32x4 w2 = bias4(L, P + oQw2);
  const f32x4 z = layer1(W, x, bias4(L, P + oQb1)), zd = layer1(W, xd, zero4());
  const float s = sum_groups(dot4(w2, map4(z, silu)));
  const float sd = sum_groups(dot4(w2, map4(z, dsilu) * zd));
  if (L.g == 0) {
    part[0][L.w][L.l16] = s;
    part[1][L.w][L.l16] = sd;
  }
  __syncthreads();
  if (threadIdx.x < 32) {   // lanes 0..15: c of atom l16, lanes 16..31: c_dot
    const int which = threadIdx.x >> 4;
    const float* p = part[which][0] + L.l16;
    const float v = (p[0] + p[16]) + (p[32] + p[48]);
    if (L.l16 < na) (which ? cd : c)[a0 + L.l16] = v;
    double t = L.l16 < na ? double(v) : 0.0;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o, 16);
    if (L.l16 == 0) csum[2 * blockIdx.x + which] = t;
  }
}

// out[0] = mean of (a0 + a1), out[1] = mean of b (NULL arrays are zero); one workgroup
__global__ void __launch_bounds__(1024) k_means(int n, const float* a0, const float* a1,
                                                const float* b, double* out) {
  __shared__ double r0[1024], r1[1024];
  double s0 = 0.0, s1 = 0.0;
  for (int k = threadIdx.x; k < n; k += 1024) {
    s0 += double(a0 ? a0[k] : 0.0f) + double(a1 ? a1[k] : 0.0f);
    s1 += double(b ? b[k] : 0.0f);
  }
  r0[threadIdx.x] = s0;
  r1[threadIdx.x] = s1;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      r0[threadIdx.x] += r0[threadIdx.x + o];
      r1[threadIdx.x] += r1[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = n > 0 ? r0[0] / n : 0.0;
    out[1] = n > 0 ? r1[0] / n : 0.0;
  }
}

// q = z + c - mean c; q_dot = c_dot - mean c_dot (either output may be NULL).  Every
// workgroup adds up the tiles' sums, in the same order.
__global__ void __launch_bounds__(256) k_qcentre(int n, const float* z, const float* c,
                                                 const float* cd, const double* csum, float* q,
                                                 float* qd) {
  __shared__ double red[2][4];
  const int t = threadIdx.x;
  double s[2] = {0.0, 0.0};
  for (int k = t; k < (n + 15) / 16; k += 256) {
    s[0] += csum[2 * k];
    s[1] += csum[2 * k + 1];
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[m] += __shfl_xor(s[m], o, 64);
    if ((t & 63) == 0) red[m][t >> 6] = s[m];
  }
  __syncthreads();
  double mean[2];
#pragma unroll
  for (int m = 0; m < 2; ++m) mean[m] = ((red[m][0] + red[m][1]) + (red[m][2] + red[m][3])) / n;
  const int i = blockIdx.x * 256 + t;
  if (i >= n) return;
  if (q) q[i] = z[i] + (c[i] - float(mean[0]));
  if (qd) qd[i] = cd[i] - float(mean[1]);
}

// Feature cotangents of the charge head for a charge cotangent g (centred with
// mean[1]): dL/dx = sum_o (g - mean) w2_o silu'(z_o) W1q[o][:], mapped to
// fbar = [dL/dG (16) | dL/dV (16 x 3)] with dL/dV_c = 2 (dL/dx_{16+c}) V_c; added
// to fbar when `accumulate`.
__global__ void __launch_bounds__(kNetThreads) k_qhead_input_grad(int n, const float* P,
                                                                  const float* feat,
                                                                  const float* vec,
                                                                  const float* g,
                                                                  const double* mean,
                                                                  float* fbar, int accumulate) {
  __shared__ __attribute__((aligned(16))) float part[4][16][CS];
  const NetLane L;
  const int a0 = blockIdx.x * 16, na = min(16, n - a0);
  NetW1 W;
  NetInBack I;
  NetIn x;
  x.load(L, feat, a0, na);
  W.load(L, P + oQW1);
  I.load(L, P + oQW1);
  const float ga = L.l16 < na ? g[a0 + L.l16] - float(mean[1]) : 0.0f;
  const f32x4 z = layer1(W, x, bias4(L, P + oQb1));
  const f32x4 gz = ga * bias4(L, P + oQw2) * map4(z, dsilu);
  const f32x4 gG = sum_waves(L, part, I.run(0, gz));
  const f32x4 gS = sum_waves(L, part, I.run(1, gz));
  if (L.l16 < na) {
    float* f = fbar + size_t(a0 + L.l16) * 4 * NCH;
    const float* V = vec + size_t(a0 + L.l16) * NCH * 3;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (r == L.w) {
        const int c = 4 * L.g + r;
        f[c] = accumulate ? f[c] + gG[r] : gG[r];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int k = NCH + 3 * c + d;
          const float v = 2.0f * gS[r] * V[3 * c + d];
          f[k] = accumulate ? f[k] + v : v;
        }
      }
  }
}

// Charge-head parameter gradient from cotangents (g_q0 + g_q1 - mean[0]) on c and
// (cq - mean[1]) on c_dot; tiles and partial rows as in k_mlp_backward.
__global__ void __launch_bounds__(kNetThreads) k_qhead_backward(int n, const float* P,
                                                                const float* feat,
                                                                const float* feat_dot,
                                                                const float* g_q0,
                                                                const float* g_q1,
                                                                const float* cq,
                                                                const double* mean,
                                                                float* part) {
  __shared__ __attribute__((aligned(16))) float gzs[16][HS], gzds[16][HS];
  const NetLane L;
  NetW1 W;
  W.load(L, P + oQW1);
  const f32x4 b1 = bias4(L, P + oQb1), w2 = bias4(L, P + oQw2);
  const float m0 = float(mean[0]), m1 = float(mean[1]);
  f32x4 aW[3] = {zero4(), zero4(), zero4()}, ab = zero4(), aw2 = zero4();
  const int tiles = (n + 15) / 16;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int a0 = tile * 16, na = min(16, n - a0);
    NetIn x, xd;
    x.load(L, feat, a0, na);
    xd.load(L, feat_dot, a0, na);
    const size_t i = size_t(a0 + L.l16);
    const bool in = L.l16 < na;
    const float gc = in ? of3(g_q0, i) + of3(g_q1, i) - m0 : 0.0f;
    const float gcd = in ? of3(cq, i) - m1 : 0.0f;
    const f32x4 z = layer1(W, x, b1), zd = layer1(W, xd, zero4());
    const f32x4 ds = map4(z, dsilu);
    aw2 += gc * map4(z, silu) + gcd * ds * zd;
    const f32x4 gz = gc * w2 * ds + gcd * w2 * map4(z, d2silu) * zd;
    ab += gz;
    __syncthreads();   // the previous tile's outer products are done with the LDS
    put_units(L, gzs, gz);
    put_units(L, gzds, gcd * w2 * ds);
    __syncthreads();
    outer_inputs(L, gzs, feat, a0, na, aW);
    outer_inputs(L, gzds, feat_dot, a0, na, aW);
  }
  float* out = part + size_t(blockIdx.x) * NQP;
  put_rows(L, out + oQW1, NF, aW);
  put_sums(L, out + oQb1 + 16 * L.w, ab);
  put_sums(L, out + oQw2 + 16 * L.w, aw2);
}

struct FeatJvpArgs {
  int n;
  const float* pos;
  const float* q;
  CellGrid g;
  const int* start;
  const float4* sp;
  float rc;
  const float* vec;    // [n][16][3] features of dip_features
  const float* v;      // [n][3] position tangent
  float* feat_dot;     // [n][34]
  float* vec_dot;      // [n][16][3]
};

// Directional derivative of the features along v, laid out as k_features (39 -> 11 us at
// 4096 ions).  Pair R = r_i - r_j, w = v_i - v_j, u = R/r, r_dot = u . w:
//   G_dot += R_k' r_dot,  V_dot += q_j [R_k' r_dot u + R_k/r (w - r_dot u)].
__global__ void __launch_bounds__(kFeatThreads) k_features_jvp(FeatJvpArgs a) {
  __shared__ float4 s_pair[kFeatAtoms][64 + kFeatBatch];
  __shared__ float s_R[kFeatAtoms][kFeatBatch][2 * NR];         // R_k' r_dot, R_k / r
  __shared__ float4 s_w[kFeatAtoms][kFeatBatch][2];             // their factors
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int at = blockIdx.x * kFeatAtoms + wave;
  if (at >= a.n) return;   // no workgroup barrier below
  const float4 pi = a.sp[at];
  const int i = __builtin_amdgcn_readfirstlane(__float_as_int(pi.w));
  const float vix = a.v[3 * i], viy = a.v[3 * i + 1], viz = a.v[3 * i + 2];
  const int k = lane & 7, s = (lane >> 3) & 1, comp = lane >> 4;
  float acc = 0.0f;
  visit_pairs<kFeatBatch, true>(
      a.g, a.start, a.sp, pi, i, a.rc * a.rc, s_pair[wave], [&](const float4* l, int nb) {
        float qj = 0.0f;
        if (lane < nb) {
          const float4 p = l[lane];
          const int j = __float_as_int(p.w);
          const float r = sqrtf(p.x * p.x + p.y * p.y + p.z * p.z), ir = 1.0f / r;
          const float ux = p.x * ir, uy = p.y * ir, uz = p.z * ir;
          const float wx = vix - a.v[3 * j], wy = viy - a.v[3 * j + 1], wz = viz - a.v[3 * j + 2];
          const float rd = ux * wx + uy * wy + uz * wz;
          float Rk[NR], dR[NR];
          radial(r, ir, 1.0f / a.rc, Rk, dR);
#pragma unroll
          for (int m = 0; m < NR; ++m) {
            s_R[wave][lane][m] = dR[m] * rd;
            s_R[wave][lane][NR + m] = Rk[m] * ir;
          }
          qj = a.q[j];
          s_w[wave][lane][0] = make_float4(1.0f, qj * ux, qj * uy, qj * uz);
          s_w[wave][lane][1] = make_float4(0.0f, qj * (wx - rd * ux), qj * (wy - rd * uy),
                                           qj * (wz - rd * uz));
        }
        const unsigned long long other = __ballot(qj > 0.0f) ^ (s ? 0ull : ~0ull);
        wave_lds_fence();
        const float* R = &s_R[wave][0][k];
        const float* w = reinterpret_cast<const float*>(&s_w[wave][0][0]) + comp;
        for (int m = 0; m < nb; ++m) {
          const float sum = fmaf(R[2 * NR * m], w[8 * m], fmaf(R[2 * NR * m + NR], w[8 * m + 4], acc));
          acc = (other >> m) & 1 ? acc : sum;
        }
        wave_lds_fence();
      });
  // d|V|^2 = 2 V . V_dot of (species, k)
  float vd = 0.0f;
  if (comp) vd = a.vec[size_t(i) * NCH * 3 + 3 * (lane & 15) + comp - 1] * acc;
  vd = __shfl(vd, 16 + (lane & 15), 64) + __shfl(vd, 32 + (lane & 15), 64) +
       __shfl(vd, 48 + (lane & 15), 64);
  float* f = a.feat_dot + size_t(i) * NF;
  if (comp == 0) {
    f[lane] = acc;
    f[NCH + lane] = 2.0f * vd;
  } else {
    a.vec_dot[size_t(i) * NCH * 3 + 3 * (lane & 15) + comp - 1] = acc;
  }
  if (lane < NS) f[2 * NCH + lane] = 0.0f;
}

// g[p] = sum over nb partial rows of width `width`, in a fixed order: 32 columns and 8
// groups of rows per workgroup.  A thread per column alone left 30 workgroups walking
// 512 rows each (91 us for the 7440 parameters; now 4 us).
__global__ void __launch_bounds__(256) k_rows_reduce(int nb, int width, const float* part,
                                                     float* g) {
  __shared__ float s_part[8][32];
  const int col = threadIdx.x & 31, grp = threadIdx.x >> 5;
  const int p = blockIdx.x * 32 + col;
  float s = 0.0f;
  if (p < width)
#pragma unroll 8
    for (int b = grp; b < nb; b += 8) s += part[size_t(b) * width + p];
  s_part[grp][col] = s;
  __syncthreads();
  if (grp == 0 && p < width) {
    float t = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) t += s_part[k][col];
    g[p] = t;
  }
}

__global__ void __launch_bounds__(1024) k_loss(int n, const double* Us, const double* Ut,
                                               const float* ds, const float* dt, const float* mu,
                                               const float* mut, const float* dmu,
                                               const float* dq, double lE, double lF, double lmu,
                                               double* loss, float* vpos, float* gmu, float* gq) {
  __shared__ double rF[1024], rM[1024];
  const int m = 3 * n;
  const double dE = (n > 0) ? (Us[0] - Ut[0]) / double(n) : 0.0;
  const double cE = (n > 0) ? 2.0 * lE * dE / double(n) : 0.0;
  const double inv = (m > 0) ? 1.0 / double(m) : 0.0;
  double sF = 0.0, sM = 0.0;
  // kLossUnroll elements' loads in flight before their stores (which the compiler could
  // not move them across): the loop is a chain of memory round trips, 11.3 us at 4096
  // atoms one element at a time, 8.7 so.  The sums keep their order.
  constexpr int kLossUnroll = 6;
  for (int k0 = threadIdx.x; k0 < m; k0 += kLossUnroll * 1024) {
    float dF[kLossUnroll], dM[kLossUnroll], gm[kLossUnroll], gc[kLossUnroll];
#pragma unroll
    for (int u = 0; u < kLossUnroll; ++u) {
      const int k = k0 + u * 1024;
      dF[u] = dM[u] = gm[u] = gc[u] = 0.0f;
      if (k < m) {
        dF[u] = ds[k] - dt[k];
        if (mut) dM[u] = mu[k] - mut[k];
        gm[u] = dmu[k];
        if (gq && k < n) gc[u] = dq[k];
      }
    }
#pragma unroll
    for (int u = 0; u < kLossUnroll; ++u) {
      const int k = k0 + u * 1024;
      if (k >= m) break;
      sF += double(dF[u]) * dF[u];
      sM += double(dM[u]) * dM[u];
      vpos[k] = float(2.0 * lF * inv) * dF[u];
      gmu[k] = float(cE) * gm[u] + float(2.0 * lmu * inv) * dM[u];
      if (gq && k < n) gq[k] = float(cE) * gc[u];
    }
  }
  rF[threadIdx.x] = sF;
  rM[threadIdx.x] = sM;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      rF[threadIdx.x] += rF[threadIdx.x + o];
      rM[threadIdx.x] += rM[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[0] = lE * dE * dE + lF * rF[0] * inv + lmu * rM[0] * inv;
}

__global__ void k_adam(int count, float lr, float b1, float b2, float eps, float c1, float c2,
                       float* p, const float* g, float* m, float* v) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  const float gk = g[k];
  const float mk = b1 * m[k] + (1.0f - b1) * gk;
  const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

thread_local char g_dip_err[256] = "";

int dip_fail(hipError_t e) {
  snprintf(g_dip_err, sizeof(g_dip_err), "%s", hipGetErrorString(e));
  return PME_EHIP;
}

inline int mlp_blocks(int n) { return n > 0 ? (n + 15) / 16 : 1; }
inline int grad_blocks(int n) { return mlp_blocks(n) < kGradBlocks ? mlp_blocks(n) : kGradBlocks; }

// add up nb partial rows
void launch_reduce(hipStream_t s, int nb, int width, const float* part, float* g) {
  hipLaunchKernelGGL(k_rows_reduce, dim3((width + 31) / 32), dim3(256), 0, s, nb, width, part, g);
}

}  // namespace

struct dip_plan_s {
  dip_desc_t desc;
  CellList cells;
  char* base = nullptr;      // the allocation that holds the arrays
  float* part = nullptr;     // [grad_blocks(max_atoms)][NP] dipole-head partials
  float* qpart = nullptr;    // [grad_blocks(max_atoms)][NQP] charge-head partials
  float* fbar = nullptr;     // [max_atoms][64] feature cotangents (position VJP)
  float* qbuf = nullptr;     // [2][max_atoms] charge-head outputs c, c_dot
  double* csum = nullptr;    // [mlp_blocks(max_atoms)][2] their sums per tile
  double* means = nullptr;   // [2]
};

namespace {

void dip_free(dip_plan_s* pl) {
  free_cells(pl->cells);
  if (pl->base) (void)hipFree(pl->base);
  delete pl;
}

}  // namespace

extern "C" {

int dip_plan_create(const dip_desc_t* desc, dip_plan_t* out) {
  if (!desc || !out) return PME_EINVAL;
  *out = nullptr;
  if (desc->max_atoms < 1 || desc->flags != 0) return PME_EINVAL;
  dip_plan_s* pl = new (std::nothrow) dip_plan_s();
  if (!pl) return PME_ENOMEM;
  pl->desc = *desc;
  int rc = setup_cells(pl->cells, desc->box, desc->cutoff, desc->max_atoms);
  hipError_t e = hipSuccess;
  if (rc == PME_OK) {
    const size_t n = size_t(desc->max_atoms), nb = size_t(grad_blocks(desc->max_atoms));
    Carve all;
    const size_t at_part = all.take<float>(nb * NP), at_qpart = all.take<float>(nb * NQP),
                 at_fbar = all.take<float>(n * 4 * NCH), at_qbuf = all.take<float>(2 * n),
                 at_csum = all.take<double>(2 * size_t(mlp_blocks(desc->max_atoms))),
                 at_means = all.take<double>(2);
    if ((e = all.allocate()) == hipSuccess) {
      pl->base = all.base;
      pl->part = all.at<float>(at_part);
      pl->qpart = all.at<float>(at_qpart);
      pl->fbar = all.at<float>(at_fbar);
      pl->qbuf = all.at<float>(at_qbuf);
      pl->csum = all.at<double>(at_csum);
      pl->means = all.at<double>(at_means);
    }
  }
  if (rc != PME_OK || e != hipSuccess) {
    dip_free(pl);
    return rc != PME_OK ? rc : (e == hipErrorOutOfMemory ? PME_ENOMEM : dip_fail(e));
  }
  *out = pl;
  return PME_OK;
}

void dip_plan_destroy(dip_plan_t plan) {
  if (!plan) return;
  (void)hipDeviceSynchronize();
  dip_free(plan);
}

int dip_features(dip_plan_t plan, void* stream, int32_t n, const float* pos, const float* q,
                 float* feat, float* vec) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || (n > 0 && (!pos || !q || !feat || !vec)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return dip_fail(e);
  FeatArgs a;
  a.n = n; a.pos = pos; a.q = q; a.g = plan->cells.g;
  a.start = plan->cells.start; a.sp = plan->cells.sp;
  a.rc = float(plan->desc.cutoff); a.feat = feat; a.vec = vec;
  const int per = kFeatAtoms;
  hipLaunchKernelGGL(k_features, dim3((n + per - 1) / per), dim3(kFeatThreads), 0, s, a);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_forward(dip_plan_t plan, void* stream, int32_t n, const float* params, const float* feat,
                const float* vec, float* mu) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || (n > 0 && (!params || !feat || !vec || !mu)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_mlp_forward<false>, dim3(mlp_blocks(n)), dim3(kNetThreads), 0, s, n,
                     params, feat, vec, nullptr, nullptr, mu, nullptr);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_backward(dip_plan_t plan, void* stream, int32_t n, const float* params, const float* feat,
                 const float* vec, const float* g_mu0, const float* g_mu1, const float* g_mu2,
                 float* g_params) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || !g_params ||
      (n > 0 && (!params || !feat || !vec)))
    return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nb = n > 0 ? grad_blocks(n) : 0;
  if (n > 0)
    hipLaunchKernelGGL(k_mlp_backward<false>, dim3(nb), dim3(kNetThreads), 0, s, n, params, feat,
                       vec, nullptr, nullptr, g_mu0, g_mu1, g_mu2, nullptr, plan->part);
  launch_reduce(s, nb, NP, plan->part, g_params);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_position_vjp(dip_plan_t plan, void* stream, int32_t n, const float* params,
                     const float* qparams, const float* pos, const float* q, const float* feat,
                     const float* vec, const float* u, const float* c, const float* base,
                     float* g_pos) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || (u && !params) || (c && !qparams) ||
      (n > 0 && ((!u && !c) || !pos || !q || !feat || !vec || !g_pos)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return dip_fail(e);
  if (u)
    hipLaunchKernelGGL(k_mlp_input_grad, dim3(mlp_blocks(n)), dim3(kNetThreads), 0, s, n, params,
                       feat, vec, u, plan->fbar);
  if (c) {
    hipLaunchKernelGGL(k_means, dim3(1), dim3(1024), 0, s, n, nullptr, nullptr, c, plan->means);
    hipLaunchKernelGGL(k_qhead_input_grad, dim3(mlp_blocks(n)), dim3(kNetThreads), 0, s, n,
                       qparams, feat, vec, c, plan->means, plan->fbar, u ? 1 : 0);
  }
  VjpArgs a;
  a.n = n; a.pos = pos; a.q = q; a.g = plan->cells.g;
  a.start = plan->cells.start; a.sp = plan->cells.sp;
  a.rc = float(plan->desc.cutoff); a.fbar = plan->fbar; a.base = base; a.g_pos = g_pos;
  const int per = kFeatAtoms;
  hipLaunchKernelGGL(k_features_vjp, dim3((n + per - 1) / per), dim3(kFeatThreads), 0, s, a);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_features_jvp(dip_plan_t plan, void* stream, int32_t n, const float* pos, const float* q,
                     const float* vec, const float* v, float* feat_dot, float* vec_dot) {
  if (!plan || n < 0 || n > plan->desc.max_atoms ||
      (n > 0 && (!pos || !q || !vec || !v || !feat_dot || !vec_dot)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return dip_fail(e);
  FeatJvpArgs a;
  a.n = n; a.pos = pos; a.q = q; a.g = plan->cells.g;
  a.start = plan->cells.start; a.sp = plan->cells.sp;
  a.rc = float(plan->desc.cutoff); a.vec = vec; a.v = v;
  a.feat_dot = feat_dot; a.vec_dot = vec_dot;
  const int per = kFeatAtoms;
  hipLaunchKernelGGL(k_features_jvp, dim3((n + per - 1) / per), dim3(kFeatThreads), 0, s, a);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_charges(dip_plan_t plan, void* stream, int32_t n, const float* qparams, const float* z,
                const float* feat, const float* feat_dot, float* q, float* q_dot) {
  if (!plan || n < 0 || n > plan->desc.max_atoms ||
      (n > 0 && ((!q && !q_dot) || !qparams || !z || !feat)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* c = plan->qbuf;
  float* cd = plan->qbuf + plan->desc.max_atoms;
  hipLaunchKernelGGL(k_qhead_forward, dim3(mlp_blocks(n)), dim3(kNetThreads), 0, s, n, qparams,
                     feat, feat_dot, c, cd, plan->csum);
  hipLaunchKernelGGL(k_qcentre, dim3((n + 255) / 256), dim3(256), 0, s, n, z, c, cd, plan->csum,
                     q, q_dot);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_forward_jvp(dip_plan_t plan, void* stream, int32_t n, const float* params,
                    const float* feat, const float* vec, const float* feat_dot,
                    const float* vec_dot, float* mu, float* mu_dot) {
  if (!plan || n < 0 || n > plan->desc.max_atoms ||
      (n > 0 && ((!mu && !mu_dot) || !params || !feat || !vec)))
    return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_mlp_forward<true>, dim3(mlp_blocks(n)), dim3(kNetThreads), 0, s, n, params,
                     feat, vec, feat_dot, vec_dot, mu, mu_dot);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_backward_jvp(dip_plan_t plan, void* stream, int32_t n, const float* params,
                     const float* qparams, const float* feat, const float* vec,
                     const float* feat_dot, const float* vec_dot, const float* g_mu0,
                     const float* g_mu1, const float* u, const float* g_q0, const float* g_q1,
                     const float* c, float* g_params, float* g_qparams) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || (!g_params && !g_qparams) ||
      (g_params && !params) || (g_qparams && !qparams) || (n > 0 && (!feat || !vec)))
    return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nb = n > 0 ? grad_blocks(n) : 0;
  if (g_params) {
    if (n > 0)
      hipLaunchKernelGGL(k_mlp_backward<true>, dim3(nb), dim3(kNetThreads), 0, s, n, params, feat,
                         vec, feat_dot, vec_dot, g_mu0, g_mu1, nullptr, u, plan->part);
    launch_reduce(s, nb, NP, plan->part, g_params);
  }
  if (g_qparams) {
    if (n > 0) {
      hipLaunchKernelGGL(k_means, dim3(1), dim3(1024), 0, s, n, g_q0, g_q1, c, plan->means);
      hipLaunchKernelGGL(k_qhead_backward, dim3(nb), dim3(kNetThreads), 0, s, n, qparams, feat,
                         feat_dot, g_q0, g_q1, c, plan->means, plan->qpart);
    }
    launch_reduce(s, nb, NQP, plan->qpart, g_qparams);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_loss(dip_plan_t plan, void* stream, int32_t n, const double* U_s, const double* U_t,
             const float* dUdr_s, const float* dUdr_t, const float* mu, const float* mu_t,
             const float* dUdmu_s, const float* dUdq_s, double lE, double lF, double lmu,
             double* loss, float* v_pos, float* g_mu, float* g_q) {
  if (!plan || n < 0 || n > plan->desc.max_atoms || !U_s || !U_t || !loss ||
      (n > 0 && (!dUdr_s || !dUdr_t || !mu || !dUdmu_s || !v_pos || !g_mu)) ||
      (lmu != 0.0 && !mu_t) || (!g_q != !dUdq_s))
    return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_loss, dim3(1), dim3(1024), 0, s, n, U_s, U_t, dUdr_s, dUdr_t, mu, mu_t,
                     dUdmu_s, dUdq_s, lE, lF, lmu, loss, v_pos, g_mu, g_q);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

int dip_adam(void* stream, int32_t count, int32_t t, double lr, double beta1, double beta2,
             double eps, float* params, const float* grad, float* m, float* v) {
  if (count < 0 || t < 1 || !params || !grad || !m || !v) return PME_EINVAL;
  if (count == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const float c1 = float(1.0 - pow(beta1, double(t))), c2 = float(1.0 - pow(beta2, double(t)));
  hipLaunchKernelGGL(k_adam, dim3((count + 255) / 256), dim3(256), 0, s, count, float(lr),
                     float(beta1), float(beta2), float(eps), c1, c2, params, grad, m, v);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? PME_OK : dip_fail(e);
}

}  // extern "C"
