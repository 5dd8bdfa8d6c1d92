// Thole-damped polarizable point-charge model: cell list, real-space pair
// kernels and the preconditioned-conjugate-gradient induced-dipole solve whose
// matrix-vector product is the PME field of the dipoles (pme::dipole_response) plus the
// real-space dipole tensor.  The model and its conventions are documented in pol.h.
//
// Pair kernels give a wavefront to an atom: the lanes test the atoms of the
// neighbouring cells, compact the pairs within the cutoff into LDS, evaluate them 64 at
// a time and combine their partial sums with wavefront shuffles.
// The screened functions follow the recursion of the explicit Ewald sum,
//     B0 = erfc(a r)/r,  B_l = [(2l-1) B_{l-1} + (2a^2)^l exp(-a^2 r^2)/(a sqrt(pi))] / r^2,
// and the damped B_l^t keep grad B_l^t = -R B_{l+1}^t, so every gradient has the
// undamped form with B -> B^t.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <new>

#include "../../include/pol.h"
#include "cells.h"
#include "kernels.h"

namespace {

constexpr int kPairThreads = 256;
constexpr int kPairAtoms = kPairThreads / 64;   // one wavefront per atom

enum PairMode { kEnergyGrad = 0, kMuGrad = 1, kMixed = 2, kHvp = 3 };

struct PairArgs {
  int n;
  const float* pos;
  const float* q;
  const float* mu;
  const float* pol;
  const float* vpos;
  const float* vq;   // charge and dipole tangents (kHvp)
  const float* vmu;
  CellGrid g;
  const int* start;
  const float4* sp;
  float alpha;
  float rc2;
  float A;
  float pf;
  float* o_pos;      // dE/dr
  float* o_q;        // dE/dq (or the q row of the Hessian product)
  float* o_mu;       // dE/dmu (or the mixed block, or the mu row)
  // added to the outputs (the long-range part; may be the outputs themselves) and, to
  // o_mu, the polarization term (pf / a) p_mu; NULL = nothing
  const float* b_pos;
  const float* b_q;
  const float* b_mu;
  const float* p_mu;
  double* epart;     // [blocks] energy partials, with p_mu including |mu|^2 / (2 a); or
                     // (kMuGrad) partials of mu . o_mu
};

__device__ __forceinline__ float3 ld3(const float* p, int i) {
  return p ? make_float3(p[3 * i], p[3 * i + 1], p[3 * i + 2]) : make_float3(0.f, 0.f, 0.f);
}
__device__ __forceinline__ float dot3(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }

// Bound by vector issue: a pair within the cutoff costs about 150 instructions (erfc,
// two exponentials, the screened functions), a candidate about 35, and at a 10 Angstrom
// cutoff only one candidate in seven is within it.  So candidates (consecutive loads in
// cell order) are only tested, and the pairs that pass are queued until 64 lanes of work
// are there.  Evaluating each pair where it is found, 16 lanes an atom, ran the long
// body at an eighth of its lanes on one wavefront per SIMD: 67 to 82 us at 4096 ions
// against 16 to 22 us.
template <int MODE>
__global__ void __launch_bounds__(kPairThreads) k_pair(PairArgs a) {
  __shared__ double red[kPairAtoms];
  __shared__ float4 s_pair[kPairAtoms][128];   // R, neighbour (bits)
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  // wavefronts take atoms in cell order, so that those of a workgroup share candidates
  const int at = blockIdx.x * kPairAtoms + wave;
  const bool live = at < a.n;
  const float4 pi = a.sp[live ? at : 0];
  const int i = __builtin_amdgcn_readfirstlane(__float_as_int(pi.w));
  const float qi = a.q ? a.q[i] : 0.0f;
  const float3 mi = ld3(a.mu, i);
  const float ai = a.pol[i];
  const float3 vi =
      (MODE == kMixed || MODE == kHvp) ? ld3(a.vpos, i) : make_float3(0.f, 0.f, 0.f);
  const float sqpi = 1.7724538509055159f;
  const float t2 = 2.0f * a.alpha * a.alpha;
  float e = 0.f, gx = 0.f, gy = 0.f, gz = 0.f, mx = 0.f, my = 0.f, mz = 0.f, gq = 0.f;
  float4* list = s_pair[wave];

  auto pair = [&](const float4 ent) {
    const float3 R = make_float3(ent.x, ent.y, ent.z);
    const int j = __float_as_int(ent.w);
    const float r2 = dot3(R, R);
    const float r = sqrtf(r2), ir = 1.0f / r, ir2 = ir * ir;
    const float ar = a.alpha * r;
    const float gexp = expf(-ar * ar) / (a.alpha * sqpi);
    const float B0 = erfcf(ar) * ir;
    const float B1 = (B0 + t2 * gexp) * ir2;
    const float B2 = (3.0f * B1 + t2 * t2 * gexp) * ir2;
    const float B3 = (5.0f * B2 + t2 * t2 * t2 * gexp) * ir2;
    float B1t = B1, B2t = B2, B3t = B3;
    const float aj = a.pol[j];
    const float pp = ai * aj;
    if (a.A > 0.0f && pp > 0.0f) {
      const float au3 = a.A * r2 * r * rsqrtf(pp);
      const float ex = expf(-au3);
      const float ir3 = ir2 * ir;
      B1t = B1 - ex * ir3;
      B2t = B2 - 3.0f * (1.0f + au3) * ex * ir3 * ir2;
      B3t = B3 - 15.0f * (1.0f + au3 + 0.6f * au3 * au3) * ex * ir3 * ir2 * ir2;
    }
    const float qj = a.q ? a.q[j] : 0.0f;
    const float3 mj = ld3(a.mu, j);
    const float mjr = dot3(mj, R);
    if (MODE == kHvp || MODE == kMixed) {
      // r column: d/dR of dE/dmu_i (and dE/dq_i) along w = v_i - v_j (grad B0 = -R B1
      // undamped)
      const float3 vj = ld3(a.vpos, j);
      const float3 w = make_float3(vi.x - vj.x, vi.y - vj.y, vi.z - vj.z);
      const float rw = dot3(R, w), mjw = dot3(mj, w);
      const float cw = -qj * B1t - mjr * B2t;
      float cR = qj * rw * B2t - mjw * B2t + rw * mjr * B3t;
      const float cm = -rw * B2t;
      float3 vmj = make_float3(0.f, 0.f, 0.f);
      if (MODE == kHvp) {
        // (q, mu) columns: the bilinear gradients with charges vq and dipoles vmu
        const float vqj = a.vq ? a.vq[j] : 0.0f;
        vmj = ld3(a.vmu, j);
        const float vmjr = dot3(vmj, R);
        gq += -qj * B1 * rw + B1t * mjw - mjr * B2t * rw + vqj * B0 + vmjr * B1t;
        cR += -vqj * B1t - vmjr * B2t;
      }
      mx += cw * w.x + cR * R.x + cm * mj.x + B1t * vmj.x;
      my += cw * w.y + cR * R.y + cm * mj.y + B1t * vmj.y;
      mz += cw * w.z + cR * R.z + cm * mj.z + B1t * vmj.z;
      return;
    }
    // dE/dmu_i
    const float cRm = -qj * B1t - mjr * B2t;
    mx += cRm * R.x + B1t * mj.x;
    my += cRm * R.y + B1t * mj.y;
    mz += cRm * R.z + B1t * mj.z;
    if (MODE == kEnergyGrad) {
      gq += qj * B0 + mjr * B1t;
      const float mir = dot3(mi, R), mm = dot3(mi, mj);
      const float cross = qi * mjr - qj * mir;
      e += 0.5f * (qi * qj * B0 + cross * B1t + mm * B1t - mir * mjr * B2t);
      const float cR = -qi * qj * B1 - cross * B2t - mm * B2t + mir * mjr * B3t;
      gx += cR * R.x + B1t * (qi * mj.x - qj * mi.x) - B2t * (mi.x * mjr + mj.x * mir);
      gy += cR * R.y + B1t * (qi * mj.y - qj * mi.y) - B2t * (mi.y * mjr + mj.y * mir);
      gz += cR * R.z + B1t * (qi * mj.z - qj * mi.z) - B2t * (mi.z * mjr + mj.z * mir);
    }
  };

  if (live)
    visit_pairs<64, false>(a.g, a.start, a.sp, pi, i, a.rc2, list,
                           [&](const float4* l, int nb) { if (lane < nb) pair(l[lane]); });
  mx = wave_sum(mx); my = wave_sum(my); mz = wave_sum(mz);
  if (MODE == kEnergyGrad || MODE == kHvp) gq = wave_sum(gq);
  if (MODE == kEnergyGrad) {
    e = wave_sum(e);
    gx = wave_sum(gx); gy = wave_sum(gy); gz = wave_sum(gz);
  }
  double part = double(e);
  if (live && lane == 0) {
    auto add = [](const float* b, int k, float v) { return b ? b[k] + v : v; };
    if (a.o_mu) {
      float o[3] = {add(a.b_mu, 3 * i, a.pf * mx), add(a.b_mu, 3 * i + 1, a.pf * my),
                    add(a.b_mu, 3 * i + 2, a.pf * mz)};
      if (a.p_mu)
#pragma unroll
        for (int d = 0; d < 3; ++d) o[d] += a.pf * a.p_mu[3 * i + d] / ai;
#pragma unroll
      for (int d = 0; d < 3; ++d) a.o_mu[3 * i + d] = o[d];
      if (MODE == kMuGrad) part = double(mi.x) * o[0] + double(mi.y) * o[1] + double(mi.z) * o[2];
    }
    if (MODE == kEnergyGrad && a.p_mu)
      part += (double(mi.x) * mi.x + double(mi.y) * mi.y + double(mi.z) * mi.z) / (2.0 * double(ai));
    if ((MODE == kEnergyGrad || MODE == kHvp) && a.o_q) a.o_q[i] = add(a.b_q, i, a.pf * gq);
    if (MODE == kEnergyGrad && a.o_pos) {
      const float o[3] = {add(a.b_pos, 3 * i, a.pf * gx), add(a.b_pos, 3 * i + 1, a.pf * gy),
                          add(a.b_pos, 3 * i + 2, a.pf * gz)};
#pragma unroll
      for (int d = 0; d < 3; ++d) a.o_pos[3 * i + d] = o[d];
    }
  }
  if ((MODE == kEnergyGrad || MODE == kMuGrad) && a.epart) {
    if (lane == 0) red[wave] = live ? part : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (int k = 0; k < kPairAtoms; ++k) sum += red[k];
      a.epart[blockIdx.x] = sum;
    }
  }
}

// Sum of n doubles (stride `by`) by a workgroup of 256, in a fixed order; every thread
// gets it.  `red` holds 4 values and is free after the call.
__device__ __forceinline__ double sum256(const double* p, int n, int by, double* red) {
  double s = 0.0;
  for (int k = threadIdx.x; k < n; k += 256) s += p[size_t(by) * k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  s = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return s;
}

// energy = pf * sum of block partials, plus the three long-range terms (one workgroup)
__global__ void __launch_bounds__(256) k_energy_sum(const double* part, int nb, double pf,
                                                    const double* e_lr, double* energy) {
  __shared__ double red[4];
  const double s = sum256(part, nb, 1, red);
  if (threadIdx.x == 0) energy[0] = (e_lr ? e_lr[0] + e_lr[1] + e_lr[2] : 0.0) + pf * s;
}

// ---- PCG vector kernels (length m = 3n) ----
//
// Dot products are FP64 partials per workgroup, added up in the same order by every
// workgroup of the kernel that needs them: an iteration is the product (its pair kernel
// leaves the partials of p . A p) and two launches, where single-workgroup dot products,
// a copy of the scalars and the vector sums took six (25 us of an iteration at 4096
// ions, now 10).  Grids are at most kPcgBlocks workgroups, so the partials stay few.
constexpr int kPcgBlocks = 64;

struct PcgResidual {   // in host memory: a workgroup's z . z and the step it belongs to
  double zz;
  unsigned long long step;
};

// block sums of (a, b) into part[2 blk ..], and b to the host with its step number
__device__ __forceinline__ void pcg_partials(double a, double b, double* part, PcgResidual* host,
                                             unsigned long long step, double* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = a;
    red[2 * (threadIdx.x >> 6) + 1] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double sa = (red[0] + red[2]) + (red[4] + red[6]);
    const double sb = (red[1] + red[3]) + (red[5] + red[7]);
    part[2 * blockIdx.x] = sa;
    part[2 * blockIdx.x + 1] = sb;
    if (host) {
      PcgResidual* h = host + blockIdx.x;
      *reinterpret_cast<volatile double*>(&h->zz) = sb;
      __threadfence_system();
      *reinterpret_cast<volatile unsigned long long*>(&h->step) = step;
    }
  }
}

// r = -g - (warm ? Ax : 0); x = warm ? x : 0; z = (a / pf) r; p = z; partials of r.z, z.z
__global__ void __launch_bounds__(256) k_pcg_start(int m, float pf, const float* pol,
                                                   const float* g, const float* Ax, float* x,
                                                   float* r, float* z, float* p, int warm,
                                                   double* part, PcgResidual* host,
                                                   unsigned long long step) {
  __shared__ double red[8];
  double rz = 0.0, zz = 0.0;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < m; k += gridDim.x * 256) {
    float rk = -g[k];
    if (warm) rk -= Ax[k];
    else x[k] = 0.0f;
    const float zk = pol[k / 3] / pf * rk;
    r[k] = rk;
    z[k] = zk;
    p[k] = zk;
    rz += double(rk) * zk;
    zz += double(zk) * zk;
  }
  pcg_partials(rz, zz, part, host, step, red);
}

// alpha = r.z / p.Ap; x += alpha p; r -= alpha Ap; z = (a / pf) r; partials of the new
// r.z and z.z (old: npart workgroups' partials of the old ones; pap: npap of p . Ap)
__global__ void __launch_bounds__(256) k_pcg_step(int m, float pf, const float* pol,
                                                  const double* old, int npart,
                                                  const double* pap, int npap, const float* p,
                                                  const float* Ap, float* x, float* r, float* z,
                                                  double* part, PcgResidual* host,
                                                  unsigned long long step) {
  __shared__ double red[8];
  const double rz0 = sum256(old, npart, 2, red), pAp = sum256(pap, npap, 1, red);
  const float al = pAp != 0.0 ? float(rz0 / pAp) : 0.0f;
  double rz = 0.0, zz = 0.0;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < m; k += gridDim.x * 256) {
    x[k] += al * p[k];
    const float rk = r[k] - al * Ap[k];
    const float zk = pol[k / 3] / pf * rk;
    r[k] = rk;
    z[k] = zk;
    rz += double(rk) * zk;
    zz += double(zk) * zk;
  }
  pcg_partials(rz, zz, part, host, step, red);
}

// beta = new r.z / old r.z; p = z + beta p
__global__ void __launch_bounds__(256) k_pcg_dir(int m, const double* old, const double* now,
                                                 int npart, const float* z, float* p) {
  __shared__ double red[4];
  const double rz0 = sum256(old, npart, 2, red), rz = sum256(now, npart, 2, red);
  const float be = rz0 != 0.0 ? float(rz / rz0) : 0.0f;
  for (int k = blockIdx.x * 256 + threadIdx.x; k < m; k += gridDim.x * 256)
    p[k] = z[k] + be * p[k];
}

__global__ void __launch_bounds__(256) k_copy(int m, const float* from, float* to) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < m) to[k] = from[k];
}

}  // namespace

struct pol_plan_s {
  pol_desc_t desc;
  CellList cells;
  char* base = nullptr;      // the allocation that holds the arrays
  double* epart = nullptr;   // [pair_blocks(max_atoms)]
  double* scal = nullptr;    // [0..2] long-range energy terms; from 8: PCG partials
  float* vec = nullptr;      // 6 work vectors of 3 max_atoms floats
  PcgResidual* host = nullptr;        // [kPcgBlocks] pinned, written by the device
  unsigned long long steps = 0;       // PCG steps launched (their numbers are never reused)
};

namespace {

thread_local char g_pol_err[256] = "";

int pol_hip_fail(hipError_t e) {
  snprintf(g_pol_err, sizeof(g_pol_err), "%s", hipGetErrorString(e));
  return PME_EHIP;
}

void pol_free(pol_plan_s* p) {
  free_cells(p->cells);
  if (p->base) (void)hipFree(p->base);
  if (p->host) (void)hipHostFree(p->host);
  delete p;
}

inline int blocks_for(int m, int t) { return cell_blocks(m, t); }

PairArgs pair_args(const pol_plan_s* pl, int n, const float* pos, const float* q, const float* mu,
                   const float* pol) {
  PairArgs a;
  a.n = n; a.pos = pos; a.q = q; a.mu = mu; a.pol = pol;
  a.vpos = nullptr; a.vq = nullptr; a.vmu = nullptr;
  a.g = pl->cells.g;
  a.start = pl->cells.start; a.sp = pl->cells.sp;
  a.alpha = float(pl->desc.alpha);
  a.rc2 = float(pl->desc.cutoff * pl->desc.cutoff);
  a.A = float(pl->desc.thole_a);
  a.pf = float(pl->desc.prefactor);
  a.o_pos = nullptr; a.o_q = nullptr; a.o_mu = nullptr; a.epart = nullptr;
  a.b_pos = nullptr; a.b_q = nullptr; a.b_mu = nullptr; a.p_mu = nullptr;
  return a;
}

int pair_blocks(int n) { return blocks_for(n, kPairAtoms); }

// base + dE_real/dmu (dipole field of mu and q) on the cell list of these positions;
// with p_mu also the polarization term and, in plan->epart, the partials of mu . out
hipError_t real_mu_grad(pol_plan_s* pl, hipStream_t s, int n, const float* pos, const float* q,
                        const float* mu, const float* pol, const float* base, const float* p_mu,
                        float* out) {
  PairArgs a = pair_args(pl, n, pos, q, mu, pol);
  a.o_mu = out;
  a.b_mu = base;
  a.p_mu = p_mu;
  a.epart = p_mu ? pl->epart : nullptr;
  hipLaunchKernelGGL(k_pair<kMuGrad>, dim3(pair_blocks(n)), dim3(kPairThreads), 0, s, a);
  return hipGetLastError();
}

// Wait for every workgroup's residual of PCG step `step` and add them up.  The device
// writes them to host memory as the step ends, so the wait costs no copy and no wake-up
// (about 15 us an iteration); a stream that has ended without them, or is not running
// (being captured), is an error.
int wait_residual(pol_plan_s* pl, hipStream_t s, int nb, unsigned long long step, double& zz) {
  auto arrived = [&](int& k) {
    while (k < nb && *static_cast<volatile unsigned long long*>(&pl->host[k].step) == step) ++k;
    return k == nb;
  };
  int k = 0;
  for (unsigned spin = 1; !arrived(k); ++spin) {
    __builtin_ia32_pause();
    if (spin % 4096 == 0) {
      const hipError_t e = hipStreamQuery(s);
      if (e == hipErrorNotReady) {
        (void)hipGetLastError();   // not an error of the launches that follow
        continue;
      }
      if (e != hipSuccess) return pol_hip_fail(e);
      if (!arrived(k)) return pol_hip_fail(hipErrorUnknown);
    }
  }
  __atomic_thread_fence(__ATOMIC_ACQUIRE);
  zz = 0.0;
  for (int b = 0; b < nb; ++b) zz += *static_cast<volatile double*>(&pl->host[b].zz);
  return PME_OK;
}

// Outputs of the model calls that lie in the place of inputs (an update of v_mu by H v, say):
// both the long-range part and the pair kernel write outputs while inputs are still to be
// read, so such calls work in the plan's vectors and copy.
struct Range { const void* p; size_t floats; };

bool overlap(const Range* out, int nout, const Range* in, int nin) {
  for (int o = 0; o < nout; ++o)
    for (int i = 0; i < nin; ++i) {
      if (!out[o].p || !in[i].p) continue;
      const uintptr_t a = reinterpret_cast<uintptr_t>(out[o].p), b = reinterpret_cast<uintptr_t>(in[i].p);
      if (a < b + 4 * in[i].floats && b < a + 4 * out[o].floats) return true;
    }
  return false;
}

hipError_t copy_out(hipStream_t s, int m, const float* from, float* to) {
  if (!to || m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy, dim3(blocks_for(m, 256)), dim3(256), 0, s, m, from, to);
  return hipGetLastError();
}

bool check_common(const pol_plan_s* pl, int n, const float* pos, const float* pol) {
  return pl && n >= 0 && n <= pl->desc.max_atoms && (n == 0 || (pos && pol));
}

}  // namespace

extern "C" {

int pol_plan_create(const pol_desc_t* desc, pol_plan_t* out) {
  if (!desc || !out) return PME_EINVAL;
  *out = nullptr;
  if (desc->max_atoms < 1 || (desc->flags & ~(POL_F_WARM_START | POL_F_FIXED_ITERS)))
    return PME_EINVAL;
  if (!(desc->alpha > 0.0) || !isfinite(desc->alpha) || !(desc->thole_a >= 0.0) ||
      !isfinite(desc->thole_a) || !isfinite(desc->prefactor) || desc->prefactor == 0.0)
    return PME_EALPHA;
  pol_plan_s* pl = new (std::nothrow) pol_plan_s();
  if (!pl) return PME_ENOMEM;
  pl->desc = *desc;
  int rc0 = setup_cells(pl->cells, desc->box, desc->cutoff, desc->max_atoms);
  if (rc0 != PME_OK) {
    pol_free(pl);
    return rc0;
  }
  const size_t m = size_t(desc->max_atoms);
  Carve all;
  const size_t at_epart = all.take<double>(size_t(pair_blocks(int(m)))),
               at_scal = all.take<double>(8 + 4 * kPcgBlocks), at_vec = all.take<float>(6 * 3 * m);
  hipError_t e = all.allocate();
  if (e == hipSuccess) {
    pl->base = all.base;
    pl->epart = all.at<double>(at_epart);
    pl->scal = all.at<double>(at_scal);
    pl->vec = all.at<float>(at_vec);
    e = hipHostMalloc(reinterpret_cast<void**>(&pl->host), sizeof(PcgResidual) * kPcgBlocks,
                      hipHostMallocCoherent);
  }
  if (e == hipSuccess) memset(pl->host, 0, sizeof(PcgResidual) * kPcgBlocks);
  if (e != hipSuccess) {
    pol_free(pl);
    return e == hipErrorOutOfMemory ? PME_ENOMEM : pol_hip_fail(e);
  }
  *out = pl;
  return PME_OK;
}

void pol_plan_destroy(pol_plan_t plan) {
  if (!plan) return;
  (void)hipDeviceSynchronize();
  pol_free(plan);
}

int pol_real(pol_plan_t plan, void* stream, int32_t n, const float* pos, const float* q,
             const float* mu, const float* pol, double* energy, float* dE_dpos, float* dE_dq,
             float* dE_dmu) {
  if (!check_common(plan, n, pos, pol)) return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return pol_hip_fail(e);
  PairArgs a = pair_args(plan, n, pos, q, mu, pol);
  a.o_pos = dE_dpos;
  a.o_q = dE_dq;
  a.o_mu = dE_dmu;
  a.epart = energy ? plan->epart : nullptr;
  const int nb = n > 0 ? pair_blocks(n) : 0;
  if (n > 0) hipLaunchKernelGGL(k_pair<kEnergyGrad>, dim3(nb), dim3(kPairThreads), 0, s, a);
  if (energy)
    hipLaunchKernelGGL(k_energy_sum, dim3(1), dim3(256), 0, s, plan->epart, nb,
                       plan->desc.prefactor, nullptr, energy);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : pol_hip_fail(e);
}

int pol_real_mixed(pol_plan_t plan, void* stream, int32_t n, const float* pos, const float* q,
                   const float* mu, const float* pol, const float* v_pos, float* g_mu) {
  if (!check_common(plan, n, pos, pol) || !g_mu || (n > 0 && !v_pos)) return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return pol_hip_fail(e);
  PairArgs a = pair_args(plan, n, pos, q, mu, pol);
  a.vpos = v_pos;
  a.o_mu = g_mu;
  if (n > 0)
    hipLaunchKernelGGL(k_pair<kMixed>, dim3(pair_blocks(n)), dim3(kPairThreads), 0, s, a);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : pol_hip_fail(e);
}

int pol_model(pol_plan_t plan, pme_plan_t pme, void* stream, int32_t n, const float* pos,
              const float* q, const float* mu, const float* pol, const double* box,
              double* energy, float* dU_dpos, float* dU_dq, float* dU_dmu) {
  if (!check_common(plan, n, pos, pol) || !pme || !box) return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // the long-range gradients go straight into the outputs, to which the pair kernel adds
  // the real-space part and the polarization term
  const size_t n1 = size_t(n), n3 = 3 * n1, stride = size_t(3) * plan->desc.max_atoms;
  const Range outs[] = {{dU_dpos, n3}, {dU_dq, n1}, {dU_dmu, n3}};
  const Range ins[] = {{pos, n3}, {q, n1}, {mu, n3}, {pol, n1}};
  const bool apart = overlap(outs, 3, ins, 4);
  float* o_pos = apart && dU_dpos ? plan->vec : dU_dpos;
  float* o_q = apart && dU_dq ? plan->vec + stride : dU_dq;
  float* o_mu = apart && dU_dmu ? plan->vec + 2 * stride : dU_dmu;
  int rc = pme_forward(pme, stream, n, pos, q, mu, box, energy ? plan->scal : nullptr, o_pos, o_q,
                       o_mu);
  if (rc != PME_OK) return rc;
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return pol_hip_fail(e);
  PairArgs a = pair_args(plan, n, pos, q, mu, pol);
  a.o_pos = o_pos; a.o_q = o_q; a.o_mu = o_mu;
  a.b_pos = o_pos; a.b_q = o_q; a.b_mu = o_mu;
  a.p_mu = mu;
  a.epart = energy ? plan->epart : nullptr;
  const int nb = n > 0 ? pair_blocks(n) : 0;
  if (n > 0) hipLaunchKernelGGL(k_pair<kEnergyGrad>, dim3(nb), dim3(kPairThreads), 0, s, a);
  if (energy)
    hipLaunchKernelGGL(k_energy_sum, dim3(1), dim3(256), 0, s, plan->epart, nb,
                       plan->desc.prefactor, plan->scal, energy);
  if (apart && ((e = copy_out(s, 3 * n, o_pos, dU_dpos)) != hipSuccess ||
                (e = copy_out(s, n, o_q, dU_dq)) != hipSuccess ||
                (e = copy_out(s, 3 * n, o_mu, dU_dmu)) != hipSuccess))
    return pol_hip_fail(e);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : pol_hip_fail(e);
}

int pol_model_hvp(pol_plan_t plan, pme_plan_t pme, void* stream, int32_t n, const float* pos,
                  const float* q, const float* mu, const float* pol, const double* box,
                  const float* v_pos, const float* v_q, const float* v_mu, float* g_q,
                  float* g_mu) {
  if (!check_common(plan, n, pos, pol) || !pme || !box || !g_q || !g_mu) return PME_EINVAL;
  if (n == 0) return PME_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t n1 = size_t(n), n3 = 3 * n1;
  const Range outs[] = {{g_q, n1}, {g_mu, n3}};
  const Range ins[] = {{pos, n3}, {q, n1}, {mu, n3}, {pol, n1}, {v_pos, n3}, {v_q, n1}, {v_mu, n3}};
  const bool apart = overlap(outs, 2, ins, 7);
  float* o_q = apart ? plan->vec : g_q;
  float* o_mu = apart ? plan->vec + size_t(3) * plan->desc.max_atoms : g_mu;
  int rc = pme_backward(pme, stream, n, pos, q, mu, box, v_pos, v_q, v_mu, nullptr, o_q, o_mu);
  if (rc != PME_OK) return rc;
  hipError_t e = build_cells(plan->cells, s, n, pos);
  if (e != hipSuccess) return pol_hip_fail(e);
  PairArgs a = pair_args(plan, n, pos, q, mu, pol);
  a.vpos = v_pos; a.vq = v_q; a.vmu = v_mu;
  a.o_q = o_q; a.o_mu = o_mu;
  a.b_q = o_q; a.b_mu = o_mu;
  a.p_mu = v_mu;   // the polarization term adds (pf / a) v_mu
  hipLaunchKernelGGL(k_pair<kHvp>, dim3(pair_blocks(n)), dim3(kPairThreads), 0, s, a);
  if (apart && ((e = copy_out(s, n, o_q, g_q)) != hipSuccess ||
                (e = copy_out(s, 3 * n, o_mu, g_mu)) != hipSuccess))
    return pol_hip_fail(e);
  e = hipGetLastError();
  return e == hipSuccess ? PME_OK : pol_hip_fail(e);
}

int pol_scf(pol_plan_t plan, pme_plan_t pme, void* stream, int32_t n, const float* pos,
            const float* q, const float* pol, const double* box, double tol, int32_t max_iter,
            float* mu, int32_t* iters, double* resid) {
  if (!check_common(plan, n, pos, pol) || !pme || !box || !mu || max_iter < 0 || !(tol >= 0.0))
    return PME_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int m = 3 * n;
  const size_t stride = size_t(3) * plan->desc.max_atoms;
  float* g1 = plan->vec;
  float* g2 = g1 + stride;
  float* r = g2 + stride;
  float* z = r + stride;
  float* p = z + stride;
  float* Ap = p + stride;
  double* part[2] = {plan->scal + 8, plan->scal + 8 + 2 * kPcgBlocks};
  const float pf = float(plan->desc.prefactor);
  const bool warm = (plan->desc.flags & POL_F_WARM_START) != 0;
  const bool fixed = (plan->desc.flags & POL_F_FIXED_ITERS) != 0;
  int vb = blocks_for(m, 256);
  if (vb > kPcgBlocks) vb = kPcgBlocks;
  int rc;
  hipError_t e;
  if (iters) *iters = 0;
  if (resid) *resid = 0.0;
  if (n == 0) return PME_OK;
  // the positions do not move during the solve: one cell list serves every product
  if ((e = build_cells(plan->cells, s, n, pos)) != hipSuccess) return pol_hip_fail(e);
  // A v = (pf / a) v + H_pme v + H_real v, and the partials of v . A v
  auto matvec = [&](const float* v, float* out) -> int {
    const int rr = pme::dipole_response(pme, s, n, pos, v, box, g1);
    if (rr != PME_OK) return rr;
    const hipError_t he = real_mu_grad(plan, s, n, pos, nullptr, v, pol, g1, v, out);
    return he == hipSuccess ? PME_OK : pol_hip_fail(he);
  };
  if (warm && (rc = matvec(mu, Ap)) != PME_OK) return rc;
  // right-hand side: -(dE_lr/dmu + dE_real/dmu) at mu = 0 (charges only)
  if ((rc = pme_forward(pme, stream, n, pos, q, nullptr, box, nullptr, nullptr, nullptr, g1)) !=
      PME_OK)
    return rc;
  if ((e = real_mu_grad(plan, s, n, pos, q, nullptr, pol, g1, nullptr, g2)) != hipSuccess)
    return pol_hip_fail(e);
  // with a fixed count (capturable) the residual does not go to the host
  PcgResidual* host = fixed ? nullptr : plan->host;
  hipLaunchKernelGGL(k_pcg_start, dim3(vb), dim3(256), 0, s, m, pf, pol, g2, Ap, mu, r, z, p,
                     warm ? 1 : 0, part[0], host, ++plan->steps);
  if ((e = hipGetLastError()) != hipSuccess) return pol_hip_fail(e);
  int it = 0;
  double rms = 0.0;
  for (;;) {
    if (fixed) {
      // no host round trip: exactly max_iter iterations
      if (it >= max_iter) {
        rms = -1.0;
        break;
      }
    } else {
      double zz;
      if ((rc = wait_residual(plan, s, vb, plan->steps, zz)) != PME_OK) return rc;
      rms = sqrt(zz / double(m));   // of squares: NaN where a residual is
      if (!isfinite(rms) || rms < tol || it >= max_iter) {
        // the residual arrives before its kernel ends and k_pcg_dir runs: the caller gets
        // the solution with nothing in flight (a solve and its forces at 4096 ions: 791 us,
        // 768 where the next call is queued behind them)
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return pol_hip_fail(e);
        if (!isfinite(rms)) return PME_ENONFINITE;
        break;
      }
    }
    const double* old = part[it & 1];
    double* now = part[(it & 1) ^ 1];
    if ((rc = matvec(p, Ap)) != PME_OK) return rc;
    hipLaunchKernelGGL(k_pcg_step, dim3(vb), dim3(256), 0, s, m, pf, pol, old, vb, plan->epart,
                       pair_blocks(n), p, Ap, mu, r, z, now, host, ++plan->steps);
    hipLaunchKernelGGL(k_pcg_dir, dim3(vb), dim3(256), 0, s, m, old, now, vb, z, p);
    if ((e = hipGetLastError()) != hipSuccess) return pol_hip_fail(e);
    ++it;
  }
  if (iters) *iters = it;
  if (resid) *resid = rms;
  return PME_OK;
}

}  // extern "C"
