// Kernels of the gradient of L = Re <chi, y_k> with respect to b, mu and the
// links, for the two-sided Lanczos approximation of Section 4 without
// deflation, y_k = |b| V_k sgn(G_k) e_1 (eq. 2sLapp with m = 0).
//
// The driver (gradient.cpp) runs the Lanczos recurrences forward storing the
// FP64 bases V, W (or checkpoints), then walks them backwards.  Every vector
// step is a pass over stored fields, short linear combinations with fused dot
// products (k_pass_*; k_lin, k_lin_multi for the first and last steps); the
// per-source scalar steps run at the start of the pass that uses their
// coefficient rows; the pairs of A and A^dagger applications
// are the dual stencil; the link and mu derivatives are accumulated by
// k_gforce (one step) and k_gforce_group (a group of steps).  Reductions
// are fixed-order.
#include <cmath>

#include "ovs_common.h"
#include "ovs_device.h"
#include "ovs_grad.h"
#include "ovs_spin.h"

namespace ovs {

// ---- linear combinations with fused dots -------------------------------------

// Workgroups per source of the linear combinations: up to 1024 (four per CU),
// so that one source's pass keeps enough waves in flight to stream from HBM.
int lin_nchunk(long stride) {
  long c = (stride + kWG - 1) / kWG;
  if (c > 1024) c = 1024;
  if (c < 1) c = 1;
  return (int)c;
}

__device__ __forceinline__ void lin_body(const LinArgs& a, long stride, int nrhs, double* lds) {
  const int r = blockIdx.y;
  const long off = (long)r * stride;
  Cx<double> c[kLinTerms];
#pragma unroll
  for (int j = 0; j < kLinTerms; ++j)
    c[j] = (j < a.nterm) ? c64(a.coef[(long)j * nrhs + r]) : Cx<double>{0.0, 0.0};
  double part[2 * kLinDots];
#pragma unroll
  for (int q = 0; q < 2 * kLinDots; ++q) part[q] = 0.0;
  for (long e = (long)blockIdx.x * kWG + threadIdx.x; e < stride; e += (long)gridDim.x * kWG) {
    Cx<double> v = {0.0, 0.0};
    if (a.accumulate) v = c64(a.out[off + e]);
#pragma unroll
    for (int j = 0; j < kLinTerms; ++j)
      if (j < a.nterm) v = cfma(c[j], c64(a.x[j][off + e]), v);
    if (a.out) a.out[off + e] = d2(v);
#pragma unroll
    for (int q = 0; q < kLinDots; ++q) {
      if (q < a.ndot) {
        const Cx<double> y = a.y[q] ? c64(a.y[q][off + e]) : v;
        const Cx<double> p = cmulc(y, v);
        part[2 * q] += p.re;
        part[2 * q + 1] += p.im;
      }
    }
  }
  if (a.ndot == 0) return;  // uniform over the workgroup
  block_sum<2 * kLinDots>(part, lds);
  if (threadIdx.x == 0) {
    double* dst = a.partials + ((long)r * gridDim.x + blockIdx.x) * 2 * kLinDots;
#pragma unroll
    for (int q = 0; q < 2 * kLinDots; ++q) dst[q] = part[q];
  }
}

__global__ void __launch_bounds__(kWG) k_lin(LinArgs a, long stride, int nrhs) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  lin_body(a, stride, nrhs, lds);
}

// Several linear combinations in one launch: each is computed as k_lin
// computes it (same grid, same per-element arithmetic, its own partial sums),
// so the results equal those of separate launches bit for bit.  A thread
// visits the same elements in every combination, so a combination may read
// an earlier one's output at the element it is computing (written by the same
// thread); no other element of another's output.
__global__ void __launch_bounds__(kWG) k_lin_multi(LinMulti m, long stride, int nrhs) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  for (int j = 0; j < m.n; ++j) {
    __syncthreads();  // lds of the previous combination
    lin_body(m.a[j], stride, nrhs, lds);
  }
}

void launch_lin(const LinArgs& a, long stride, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL(k_lin, dim3(lin_nchunk(stride), nrhs), dim3(kWG), 0, s, a, stride, nrhs);
}

void launch_lin_multi(const LinMulti& m, long stride, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL(k_lin_multi, dim3(lin_nchunk(stride), nrhs), dim3(kWG), 0, s, m, stride,
                     nrhs);
}

// Workgroup of the per-source scalar kernels: one per source, the dot sums
// over the chunks reduced by all its threads.
constexpr int kScalarWG = 256;

// Fixed-order sums over the chunks of ND dots of source r (dot q[d] of the
// partials parts[d]): strided over the chunks by the workgroup, then a
// fixed-order workgroup sum; every thread receives the results.
template <int ND>
__device__ void wg_dot_sums(const double* const (&parts)[ND], const int (&q)[ND], int r,
                            int nchunk, Cx<double> (&out)[ND]) {
  __shared__ double lds[(kScalarWG / 64) * 2 * ND];
  __shared__ double res[2 * ND];
  double v[2 * ND];
#pragma unroll
  for (int j = 0; j < 2 * ND; ++j) v[j] = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += blockDim.x) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      const double* pp = parts[d] + ((long)r * nchunk + c) * 2 * kLinDots + 2 * q[d];
      v[2 * d] += pp[0];
      v[2 * d + 1] += pp[1];
    }
  }
  block_sum<2 * ND>(v, lds);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < 2 * ND; ++j) res[j] = v[j];
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < ND; ++d) out[d] = {res[2 * d], res[2 * d + 1]};
}

__device__ __forceinline__ void set_coef(const GradScalars& s, int t, int j, int r, Cx<double> v) {
  s.coef[((long)t * kLinTerms + j) * s.nrhs + r] = d2(v);
}

// Where a scalar step puts the coefficient rows it forms for source r: the
// LDS table of the pass that follows it in the same launch
// (`lds`, read by all of that launch's threads), and/or the global tables
// (`coef`) for later launches.  `wr`: the step also writes its scalars
// (alpha, beta, ...) to global memory; in a pass only its first workgroup
// of each source does.
struct TabOut {
  double2 (*lds)[kLinTerms];
  double2* coef;
  int nrhs;
  int r;
  bool wr;
  __device__ void put(int t, int j, Cx<double> v) const {
    if (lds) lds[t][j] = d2(v);
    if (coef) coef[((long)t * kLinTerms + j) * nrhs + r] = d2(v);
  }
};

// ---- forward scalar steps ------------------------------------------------------

__global__ void __launch_bounds__(kScalarWG) k_gf_norm(GradScalars s, const double* part, int nchunk) {
  const int r = blockIdx.x;
  Cx<double> d[1];
  wg_dot_sums<1>({part}, {0}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const double nb = sqrt(d[0].re);
  s.nb[r] = nb;
  s.status[r] = 0;
  set_coef(s, kTabNorm, 0, r, {nb > 0.0 ? 1.0 / nb : 0.0, 0.0});
}

__global__ void __launch_bounds__(kScalarWG) k_gf_start(GradScalars s, const double* part,
                                                         const double* part_b, int nchunk) {
  const int r = blockIdx.x;
  Cx<double> d[3];
  wg_dot_sums<3>({part, part, part_b}, {0, 1, 0}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const double nb = sqrt(d[0].re);
  const Cx<double> sig = d[1];
  s.nb[r] = nb;
  s.sigma[r] = d2(sig);
  s.status[r] = 0;
  set_coef(s, kTabNorm, 0, r, {nb > 0.0 ? 1.0 / nb : 0.0, 0.0});
  // |b_R| <= 1e-12 |b|: the source lies in span R (the solve drops the Krylov
  // part there); like a start with no biorthogonal partner, it has no gradient
  const bool ok = nb > 1e-12 * sqrt(d[2].re) && (sig.re != 0.0 || sig.im != 0.0);
  set_coef(s, kTabStartW, 0, r, ok ? cdiv(Cx<double>{nb, 0.0}, cconj(sig)) : Cx<double>{0.0, 0.0});
  if (!ok) s.status[r] = 2;
}

// alpha_i = w_i^dagger t_i (dot 0), |t_i|^2 (dot 1); coefficient rows of the
// update.  All threads of the workgroup take part (the dot sums); thread 0
// forms the rows.
__device__ void step_gf_alpha(const GradScalars& s, int i, const double* part, int nchunk,
                              const TabOut& o) {
  const int r = o.r;
  Cx<double> d[2];
  wg_dot_sums<2>({part, part}, {0, 1}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const long rk = (long)r * s.kmax;
  const Cx<double> al = d[0];
  if (o.wr) {
    s.alpha[rk + i] = d2(al);
    s.tnorm2[rk + i] = d[1].re;
  }
  const Cx<double> gprev = (i > 0) ? c64(s.gamma[rk + i - 1]) : Cx<double>{0.0, 0.0};
  const double bprev = (i > 0) ? s.beta[rk + i - 1] : 0.0;
  o.put(kTabV, 0, {1.0, 0.0});
  o.put(kTabV, 1, -al);
  o.put(kTabV, 2, -gprev);
  o.put(kTabW, 0, {1.0, 0.0});
  o.put(kTabW, 1, -cconj(al));
  o.put(kTabW, 2, {-bprev, 0.0});
}
__global__ void __launch_bounds__(kScalarWG) k_gf_alpha(GradScalars s, int i, const double* part, int nchunk) {
  step_gf_alpha(s, i, part, nchunk, TabOut{nullptr, s.coef, s.nrhs, (int)blockIdx.x, true});
}

// beta_i = |v~|, delta_i = w~^dagger v~, gamma_i = delta_i / beta_i, with the
// breakdown tests of the forward recurrences (lucky: |v~| <= 1e-14 |t|;
// serious: |delta| <= 1e-13 |v~| |w~|).
__device__ void step_gf_beta(const GradScalars& s, int i, const double* part_v,
                             const double* part_w, int nchunk, const TabOut& o) {
  const int r = o.r;
  Cx<double> d[3];
  wg_dot_sums<3>({part_v, part_w, part_w}, {0, 0, 1}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const long rk = (long)r * s.kmax;
  const double vn = sqrt(d[0].re);
  const Cx<double> delta = cconj(d[1]);  // dot 0 of part_w = v~^dagger w~
  const double wn = sqrt(d[2].re);
  const Cx<double> g = vn > 0.0 ? scale(1.0 / vn, delta) : Cx<double>{0.0, 0.0};
  if (o.wr) {
    if (s.status[r] == 0) {
      if (vn <= 1e-14 * sqrt(s.tnorm2[rk + i])) s.status[r] = 1;
      else if (cabs1(delta) <= 1e-13 * vn * wn) s.status[r] = 2;
    }
    s.beta[rk + i] = vn;
    s.gamma[rk + i] = d2(g);
  }
  o.put(kTabSV, 0, {vn > 0.0 ? 1.0 / vn : 0.0, 0.0});
  const bool gz = g.re == 0.0 && g.im == 0.0;
  o.put(kTabSW, 0, gz ? Cx<double>{0.0, 0.0} : cdiv({1.0, 0.0}, cconj(g)));
}

void launch_gf_norm(const GradScalars& s, const double* part, int nchunk, hipStream_t st) {
  hipLaunchKernelGGL(k_gf_norm, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, part, nchunk);
}
void launch_gf_start(const GradScalars& s, const double* part, const double* part_b, int nchunk,
                     hipStream_t st) {
  hipLaunchKernelGGL(k_gf_start, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, part, part_b, nchunk);
}
void launch_gf_alpha(const GradScalars& s, int i, const double* part, int nchunk, hipStream_t st) {
  hipLaunchKernelGGL(k_gf_alpha, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, i, part, nchunk);
}

// ---- reverse scalar steps ------------------------------------------------------
// Adjoint rules used below (zbar = dL/dRe z + i dL/dIm z, dL = Re <zbar, dz>):
//   z = c u         : ubar += conj(c) zbar,   cbar += u^dagger zbar
//   z = u^dagger v  : vbar += zbar u,         ubar += conj(zbar) v
//   z = u / conj(c) : ubar += zbar / c,       cbar += -(zbar^dagger z) / conj(c)
//   r = |u| (real)  : ubar += rbar u / r

// Last step (i = k-1): only t = A v_{k-1} and alpha_{k-1} = w_{k-1}^dagger t exist.
__global__ void k_gr_first(GradScalars s) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= s.nrhs) return;  // scalar only: one thread per source
  const int i = s.kmax - 1;
  const long rk = (long)r * s.kmax;
  const Cx<double> ab = c64(s.abar[rk + i]);
  set_coef(s, kTabSV, 0, r, ab);                                           // tbar = abar w_i
  set_coef(s, kTabSW, 0, r, scale(s.nb[r], cconj(c64(s.x[rk + i]))));     // vbar = nb conj(x_i) chi
  set_coef(s, kTabWB, 0, r, cconj(ab));                                    // wbar = conj(abar) t_i
  set_coef(s, kTabY, 0, r, scale(s.nb[r], c64(s.x[rk + i])));              // y += nb x_i v_i
}

// Step i < k-1, first half.  Inputs: dots of the completed vbar_{i+1}, wbar_{i+1}
// with v_{i+1}, w_{i+1}.  Through v_{i+1} = v~/beta_i, w_{i+1} = w~/conj(gamma_i),
// gamma_i = delta_i/beta_i, beta_i = |v~|, delta_i = w~^dagger v~:
//   gbar_i += -(wbar_{i+1}^dagger w_{i+1}) / conj(gamma_i)
//   bbar_i += -Re(vbar_{i+1}^dagger v_{i+1}) / beta_i - Re(conj(gbar_i) gamma_i) / beta_i
//   dbar    = gbar_i / beta_i
//   vbar~_i = vbar_{i+1}/beta_i + bbar_i v_{i+1} + dbar conj(gamma_i) w_{i+1}
//   wbar~_i = wbar_{i+1}/gamma_i + conj(dbar) beta_i v_{i+1}
// gbar_i and bbar_i are read here and used nowhere after this step, so the
// updated values are not written back (a combination launch that forms them
// in every workgroup could not write them without racing its own reads).
__device__ void step_gr_s1(const GradScalars& s, int i, const double* part_v, const double* part_w,
                           int nchunk, const TabOut& o) {
  const int r = o.r;
  Cx<double> d[2];
  wg_dot_sums<2>({part_v, part_w}, {0, 0}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const long rk = (long)r * s.kmax;
  const Cx<double> d2v = cconj(d[0]);  // vbar^dagger v
  const Cx<double> d1w = cconj(d[1]);  // wbar^dagger w
  const double be = s.beta[rk + i];
  const Cx<double> ga = c64(s.gamma[rk + i]);
  Cx<double> gb = c64(s.gbar[rk + i]);
  double bb = s.bbar[rk + i];
  gb = gb - cdiv(d1w, cconj(ga));
  bb -= d2v.re / be;
  const Cx<double> db = scale(1.0 / be, gb);
  bb -= (gb.re * ga.re + gb.im * ga.im) / be;  // Re(conj(gbar) gamma)
  o.put(kTabV, 0, {1.0 / be, 0.0});
  o.put(kTabV, 1, {bb, 0.0});
  o.put(kTabV, 2, cmul(db, cconj(ga)));
  o.put(kTabW, 0, cdiv({1.0, 0.0}, ga));
  o.put(kTabW, 1, scale(be, cconj(db)));
}

// Step i < k-1, second half.  Inputs: v_i^dagger vbar~ (d5), v_{i-1}^dagger vbar~
// (d6), w_i^dagger wbar~ (conj d4), w_{i-1}^dagger wbar~ (d3).  Through
// v~ = t_i - alpha_i v_i - gamma_{i-1} v_{i-1}, w~ = s_i - conj(alpha_i) w_i -
// beta_{i-1} w_{i-1} and alpha_i = w_i^dagger t_i:
//   abar_i += -d4 - d5;  bbar_{i-1} += -Re d3;  gbar_{i-1} += -d6
//   tbar_i = vbar~_i + abar_i w_i                (then vbar_i += A^dagger tbar_i)
//   sbar_i = wbar~_i                              (then wbar_i += A sbar_i)
//   vbar_i = nb conj(x_i) chi - conj(gamma_i) vbar~_{i+1} - conj(alpha_i) vbar~_i
//   wbar_i = -beta_i wbar~_{i+1} - alpha_i wbar~_i + conj(abar_i) t_i,
//            t_i = beta_i v_{i+1} + alpha_i v_i + gamma_{i-1} v_{i-1}
// abar_i is read here and used nowhere after this step (not written back, as
// gbar_i in step 1); bbar_{i-1}, gbar_{i-1} are written for step i-1.
__device__ void step_gr_s2(const GradScalars& s, int i, const double* part_v, const double* part_w,
                           int nchunk, const TabOut& o) {
  const int r = o.r;
  // dots 1 exist for i > 0 only; at i = 0 their sums are formed and not used
  Cx<double> d[4];
  wg_dot_sums<4>({part_v, part_w, part_v, part_w}, {0, 0, 1, 1}, r, nchunk, d);
  if (threadIdx.x != 0) return;
  const long rk = (long)r * s.kmax;
  const Cx<double> d5 = d[0];
  const Cx<double> d4 = cconj(d[1]);
  const Cx<double> ab = c64(s.abar[rk + i]) - d4 - d5;
  if (o.wr && i > 0) {
    const Cx<double> d6 = d[2];
    const Cx<double> d3 = d[3];
    s.bbar[rk + i - 1] -= d3.re;
    s.gbar[rk + i - 1] = d2(c64(s.gbar[rk + i - 1]) - d6);
  }
  const Cx<double> al = c64(s.alpha[rk + i]);
  const Cx<double> ga = c64(s.gamma[rk + i]);
  const double be = s.beta[rk + i];
  const Cx<double> gprev = (i > 0) ? c64(s.gamma[rk + i - 1]) : Cx<double>{0.0, 0.0};
  o.put(kTabSV, 0, {1.0, 0.0});
  o.put(kTabSV, 1, ab);
  o.put(kTabSW, 0, scale(s.nb[r], cconj(c64(s.x[rk + i]))));
  o.put(kTabSW, 1, -cconj(ga));
  o.put(kTabSW, 2, -cconj(al));
  const Cx<double> cab = cconj(ab);
  o.put(kTabWB, 0, {-be, 0.0});
  o.put(kTabWB, 1, -al);
  o.put(kTabWB, 2, scale(be, cab));
  o.put(kTabWB, 3, cmul(cab, al));
  o.put(kTabWB, 4, cmul(cab, gprev));
  o.put(kTabY, 0, scale(s.nb[r], c64(s.x[rk + i])));
}

// v_1 = w_1 = b/|b|: grad_b = ubar/|b| + nbar v_1 with ubar = vbar_1 + wbar_1 and
// nbar = Re(chi^dagger y)/|b| - Re(ubar^dagger v_1)/|b|, chi^dagger y = sum_i x_i conj(xbar_i).
__global__ void __launch_bounds__(kScalarWG) k_gr_final(GradScalars s, const double* part, int nchunk) {
  __shared__ double lds[kScalarWG / 64];
  const int r = blockIdx.x;
  const long rk = (long)r * s.kmax;
  Cx<double> d[1];
  wg_dot_sums<1>({part}, {0}, r, nchunk, d);
  double cy[1] = {0.0};
  for (int i = threadIdx.x; i < s.kmax; i += blockDim.x) {
    const Cx<double> p = cmulc(c64(s.xbar[rk + i]), c64(s.x[rk + i]));
    cy[0] += p.re;
  }
  block_sum<1>(cy, lds);
  if (threadIdx.x != 0) return;
  const double nb = s.nb[r];
  const double uv = d[0].re;  // Re(v_1^dagger ubar)
  const double nbar = (cy[0] - uv) / nb;
  set_coef(s, kTabFin, 0, r, {1.0 / nb, 0.0});
  set_coef(s, kTabFin, 1, r, {nbar, 0.0});
}

__global__ void __launch_bounds__(kScalarWG) k_gr_final_defl(GradScalars s, const double* part_v,
                                                             const double* part_w, int nchunk) {
  __shared__ double lds[kScalarWG / 64];
  const int r = blockIdx.x;
  const long rk = (long)r * s.kmax;
  Cx<double> d[2];
  wg_dot_sums<2>({part_v, part_w}, {0, 0}, r, nchunk, d);
  double cy[1] = {0.0};
  for (int i = threadIdx.x; i < s.kmax; i += blockDim.x) {
    const Cx<double> p = cmulc(c64(s.xbar[rk + i]), c64(s.x[rk + i]));
    cy[0] += p.re;
  }
  block_sum<1>(cy, lds);
  if (threadIdx.x != 0) return;
  const double nb = s.nb[r];
  const Cx<double> sig = c64(s.sigma[r]);
  const Cx<double> rho = cconj(d[1]);           // wbar_1^dagger w_1
  const double nbar = (cy[0] - d[0].re + rho.re) / nb;
  const Cx<double> tau = -cdiv(rho, cconj(sig));
  set_coef(s, kTabFin, 0, r, {1.0 / nb, 0.0});
  set_coef(s, kTabFin, 1, r, tau);
  set_coef(s, kTabFin, 2, r, {nbar / nb, 0.0});
  set_coef(s, kTabFinW, 0, r, cdiv(Cx<double>{nb, 0.0}, sig));
  set_coef(s, kTabFinW, 1, r, cconj(tau));
}

void launch_gr_final_defl(const GradScalars& s, const double* part_v, const double* part_w,
                          int nchunk, hipStream_t st) {
  hipLaunchKernelGGL(k_gr_final_defl, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, part_v, part_w,
                     nchunk);
}

void launch_gr_first(const GradScalars& s, hipStream_t st) {
  hipLaunchKernelGGL(k_gr_first, dim3((s.nrhs + 63) / 64), dim3(64), 0, st, s);
}
void launch_gr_final(const GradScalars& s, const double* part, int nchunk, hipStream_t st) {
  hipLaunchKernelGGL(k_gr_final, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, part, nchunk);
}

// ---- source projections and replay coefficients -----------------------------

__device__ void step_gf_xbar(const GradScalars& s, int i, const double* part, int nchunk,
                             const TabOut& o) {
  const int r = o.r;
  Cx<double> d[1];
  wg_dot_sums<1>({part}, {0}, r, nchunk, d);  // chi^dagger v_i
  if (threadIdx.x != 0 || !o.wr) return;
  s.xbar[(long)r * s.kmax + i] = d2(scale(s.nb[r], cconj(d[0])));
}
__global__ void __launch_bounds__(kScalarWG) k_gf_xbar(GradScalars s, int i, const double* part, int nchunk) {
  step_gf_xbar(s, i, part, nchunk, TabOut{nullptr, nullptr, s.nrhs, (int)blockIdx.x, true});
}

void launch_gf_xbar(const GradScalars& s, int i, const double* part, int nchunk, hipStream_t st) {
  hipLaunchKernelGGL(k_gf_xbar, dim3(s.nrhs), dim3(kScalarWG), 0, st, s, i, part, nchunk);
}

// The rows of the forward update and normalisation of step i from the stored
// coefficients, with the arithmetic of steps alpha and beta (one thread).
__device__ void gp_coef_rows(const GradScalars& s, int i, const TabOut& o) {
  const int r = o.r;
  const long rk = (long)r * s.kmax;
  const Cx<double> al = c64(s.alpha[rk + i]);
  const Cx<double> gprev = (i > 0) ? c64(s.gamma[rk + i - 1]) : Cx<double>{0.0, 0.0};
  const double bprev = (i > 0) ? s.beta[rk + i - 1] : 0.0;
  o.put(kTabV, 0, {1.0, 0.0});
  o.put(kTabV, 1, -al);
  o.put(kTabV, 2, -gprev);
  o.put(kTabW, 0, {1.0, 0.0});
  o.put(kTabW, 1, -cconj(al));
  o.put(kTabW, 2, {-bprev, 0.0});
  const double vn = s.beta[rk + i];
  const Cx<double> g = c64(s.gamma[rk + i]);
  o.put(kTabSV, 0, {vn > 0.0 ? 1.0 / vn : 0.0, 0.0});
  const bool gz = g.re == 0.0 && g.im == 0.0;
  o.put(kTabSW, 0, gz ? Cx<double>{0.0, 0.0} : cdiv({1.0, 0.0}, cconj(g)));
}


// ---- passes preceded by their scalar step --------------------------------------
// Every workgroup of source r forms the step's coefficient rows itself (the
// same dot sums in the same order, kWG = kScalarWG threads, so the same
// values as the separate scalar kernel) and keeps them in LDS; the first
// workgroup of each source also writes the step's scalars.  That saves the
// scalar kernel's launch.
// Every value a step reads is written by earlier launches and none is
// written in this one, except the scalars of workgroup 0, which no other
// workgroup of the launch reads.
__device__ void run_step(const ScalarStep& st, double2 (*tab)[kLinTerms]) {
  const bool first = blockIdx.x == 0;
  const TabOut o{tab, nullptr, st.s.nrhs, (int)blockIdx.y, first};
  switch (st.kind) {
    case kStepAlpha: step_gf_alpha(st.s, st.i, st.pa, st.nchunk, o); break;
    case kStepBeta: step_gf_beta(st.s, st.i, st.pa, st.pb, st.nchunk, o); break;
    case kStepXbar: step_gf_xbar(st.s, st.i, st.pa, st.nchunk, o); break;
    case kStepCoef:
      if (threadIdx.x == 0) gp_coef_rows(st.s, st.i, o);
      break;
    case kStepS1: step_gr_s1(st.s, st.i, st.pa, st.pb, st.nchunk, o); break;
    case kStepS2: step_gr_s2(st.s, st.i, st.pa, st.pb, st.nchunk, o); break;
    default: break;
  }
  __syncthreads();  // the rows in LDS for every thread
}

// ---- the vector passes of a Lanczos step and of its reverse -----------------------
// One kernel per pass, each doing what launches of k_lin with the same
// coefficient rows and dots do, bit for bit (every output element and every
// thread's share of a dot by the same operations in the same order, the same
// grid).  An element's loads are all issued before its arithmetic, the first
// element's before the scalar step, the next one's before the current one's
// stores: on small lattices a pass is one memory latency, the dot sums of the
// scalar step and one reduction, on large ones it streams.  (A general kernel
// over a run-time list of combinations waited for each term's load in turn and
// for its arguments: the five passes of a step took 9.1 us on average at 8^4 and
// 27 us at 16^4.)

// Sweeps this workgroup's elements: cur holds the first one's loads.
template <class E, class Fetch, class Body>
__device__ __forceinline__ void sweep(long stride, E& cur, Fetch fetch, Body body) {
  long e = (long)blockIdx.x * kWG + threadIdx.x;
  while (e < stride) {
    const E c = cur;
    const long n = e + (long)gridDim.x * kWG;
    if (n < stride) fetch(n, cur);
    body(e, c);
    e = n;
  }
}
template <class E, class Fetch>
__device__ __forceinline__ void sweep_begin(long stride, E& cur, Fetch fetch) {
  const long e = (long)blockIdx.x * kWG + threadIdx.x;
  if (e < stride) fetch(e, cur);
}

// Adds conj(y) v to a dot's running sums.
__device__ __forceinline__ void dot_acc(double* p, Cx<double> y, Cx<double> v) {
  const Cx<double> d = cmulc(y, v);
  p[0] += d.re;
  p[1] += d.im;
}

// The workgroup's share of two dots to the partials of source r.
__device__ __forceinline__ void put_dots(double (&part)[2 * kLinDots], double* lds,
                                         double* partials) {
  block_sum<2 * kLinDots>(part, lds);
  if (threadIdx.x == 0) {
    double* dst = partials + ((long)blockIdx.y * gridDim.x + blockIdx.x) * 2 * kLinDots;
#pragma unroll
    for (int q = 0; q < 2 * kLinDots; ++q) dst[q] = part[q];
  }
}

// Dots w^dagger t and |t|^2; the first workgroup of a source also runs the step
// (xbar of the iteration, from the previous pass's dots).
__global__ void __launch_bounds__(kWG) k_pass_dots(const double2* t, const double2* w,
                                                   double* partials, long stride, ScalarStep st) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  const long off = (long)blockIdx.y * stride;
  struct E {
    double2 t, w;
  } cur;
  auto fetch = [&](long e, E& v) {
    v.t = t[off + e];
    v.w = w[off + e];
  };
  sweep_begin(stride, cur, fetch);
  if (st.kind == kStepXbar && blockIdx.x == 0) run_step(st, nullptr);
  double part[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0};
  sweep(stride, cur, fetch, [&](long, const E& c) {
    // the combination 1 t
    const Cx<double> v = cfma(Cx<double>{1.0, 0.0}, c64(c.t), Cx<double>{0.0, 0.0});
    dot_acc(part, c64(c.w), v);
    dot_acc(part + 2, v, v);
  });
  put_dots(part, lds, partials);
}

struct StepElem {
  double2 t, v, vm, s, w, wm;
};
__device__ __forceinline__ void fetch_step(const StepFields& f, long e, StepElem& c) {
  c.t = f.t[e];
  c.v = f.v[e];
  c.s = f.s[e];
  c.w = f.w[e];
  if (f.vm) {
    c.vm = f.vm[e];
    c.wm = f.wm[e];
  }
}
__device__ __forceinline__ void step_vectors(const StepFields& f, const StepElem& c,
                                             const double2 (*tab)[kLinTerms], Cx<double>& v,
                                             Cx<double>& w) {
  const Cx<double> zero = {0.0, 0.0};
  v = cfma(c64(tab[kTabV][1]), c64(c.v), cfma(c64(tab[kTabV][0]), c64(c.t), zero));
  w = cfma(c64(tab[kTabW][1]), c64(c.w), cfma(c64(tab[kTabW][0]), c64(c.s), zero));
  if (f.vm) {
    v = cfma(c64(tab[kTabV][2]), c64(c.vm), v);
    w = cfma(c64(tab[kTabW][2]), c64(c.wm), w);
  }
}

// alpha, then v~ and w~ with |v~|^2 (pv), v~^dagger w~ and |w~|^2 (pw).
__global__ void __launch_bounds__(kWG) k_pass_update(StepFields f, double2* vn, double2* wn,
                                                     double* pv, double* pw, long stride,
                                                     ScalarStep st) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  __shared__ double2 tab[kCoefTables][kLinTerms];
  const long off = (long)blockIdx.y * stride;
  StepElem cur;
  auto fetch = [&](long e, StepElem& c) { fetch_step(f, off + e, c); };
  sweep_begin(stride, cur, fetch);
  run_step(st, tab);
  double a[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0}, b[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0};
  sweep(stride, cur, fetch, [&](long e, const StepElem& c) {
    Cx<double> v, w;
    step_vectors(f, c, tab, v, w);
    vn[off + e] = d2(v);
    wn[off + e] = d2(w);
    dot_acc(a, v, v);
    dot_acc(b, v, w);
    dot_acc(b + 2, w, w);
  });
  put_dots(a, lds, pv);
  put_dots(b, lds, pw);
}

// beta and gamma, then the normalisation of v~ and w~ in place with chi^dagger v
// (chi null: no dot).
__global__ void __launch_bounds__(kWG) k_pass_norm(double2* vn, double2* wn, const double2* chi,
                                                   double* pchi, long stride, ScalarStep st) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  __shared__ double2 tab[kCoefTables][kLinTerms];
  const long off = (long)blockIdx.y * stride;
  struct E {
    double2 v, w, chi;
  } cur;
  auto fetch = [&](long e, E& c) {
    c.v = vn[off + e];
    c.w = wn[off + e];
    if (chi) c.chi = chi[off + e];
  };
  sweep_begin(stride, cur, fetch);
  run_step(st, tab);
  const Cx<double> cv = c64(tab[kTabSV][0]), cw = c64(tab[kTabSW][0]);
  double part[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0};
  sweep(stride, cur, fetch, [&](long e, const E& c) {
    const Cx<double> v = cfma(cv, c64(c.v), Cx<double>{0.0, 0.0});
    vn[off + e] = d2(v);
    wn[off + e] = d2(cfma(cw, c64(c.w), Cx<double>{0.0, 0.0}));
    if (chi) dot_acc(part, c64(c.chi), v);
  });
  if (chi) put_dots(part, lds, pchi);
}

// The replayed step: v~, w~ and their normalisation with the stored rows.
__global__ void __launch_bounds__(kWG) k_pass_replay(StepFields f, double2* vn, double2* wn,
                                                     long stride, ScalarStep st) {
  __shared__ double2 tab[kCoefTables][kLinTerms];
  const long off = (long)blockIdx.y * stride;
  StepElem cur;
  auto fetch = [&](long e, StepElem& c) { fetch_step(f, off + e, c); };
  sweep_begin(stride, cur, fetch);
  run_step(st, tab);
  const Cx<double> cv = c64(tab[kTabSV][0]), cw = c64(tab[kTabSW][0]);
  sweep(stride, cur, fetch, [&](long e, const StepElem& c) {
    Cx<double> v, w;
    step_vectors(f, c, tab, v, w);
    vn[off + e] = d2(cfma(cv, v, Cx<double>{0.0, 0.0}));
    wn[off + e] = d2(cfma(cw, w, Cx<double>{0.0, 0.0}));
  });
}

// Reverse step 1.
__global__ void __launch_bounds__(kWG) k_pass_rev1(Rev1Fields f, double* pv, double* pw,
                                                   long stride, ScalarStep st) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  __shared__ double2 tab[kCoefTables][kLinTerms];
  const long off = (long)blockIdx.y * stride;
  struct E {
    double2 vb, v1, w1, wb, v, vm, w, wm;
  } cur;
  auto fetch = [&](long e, E& c) {
    c.vb = f.vb[off + e];
    c.v1 = f.v1[off + e];
    c.w1 = f.w1[off + e];
    c.wb = f.wb[off + e];
    c.v = f.v[off + e];
    c.w = f.w[off + e];
    if (f.vm) {
      c.vm = f.vm[off + e];
      c.wm = f.wm[off + e];
    }
  };
  sweep_begin(stride, cur, fetch);
  run_step(st, tab);
  double a[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0}, b[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0};
  sweep(stride, cur, fetch, [&](long e, const E& c) {
    const Cx<double> zero = {0.0, 0.0};
    Cx<double> v = cfma(c64(tab[kTabV][0]), c64(c.vb), zero);
    v = cfma(c64(tab[kTabV][1]), c64(c.v1), v);
    v = cfma(c64(tab[kTabV][2]), c64(c.w1), v);
    Cx<double> w = cfma(c64(tab[kTabW][0]), c64(c.wb), zero);
    w = cfma(c64(tab[kTabW][1]), c64(c.v1), w);
    f.vtb[off + e] = d2(v);
    f.sb[off + e] = d2(w);
    dot_acc(a, c64(c.v), v);
    dot_acc(b, c64(c.w), w);
    if (f.vm) {
      dot_acc(a + 2, c64(c.vm), v);
      dot_acc(b + 2, c64(c.wm), w);
    }
  });
  put_dots(a, lds, pv);
  put_dots(b, lds, pw);
}

// Reverse step 2.
__global__ void __launch_bounds__(kWG) k_pass_rev2(Rev2Fields f, long stride, ScalarStep st) {
  __shared__ double2 tab[kCoefTables][kLinTerms];
  const long off = (long)blockIdx.y * stride;
  struct E {
    double2 vtb, vtbn, w, chi, sbn, sb, v1, v, vm, ya;
  } cur;
  auto fetch = [&](long e, E& c) {
    c.vtb = f.vtb[off + e];
    c.vtbn = f.vtbn[off + e];
    c.w = f.w[off + e];
    c.chi = f.chi[off + e];
    c.sbn = f.sbn[off + e];
    c.sb = f.sb[off + e];
    c.v1 = f.v1[off + e];
    c.v = f.v[off + e];
    if (f.vm) c.vm = f.vm[off + e];
    if (f.ya) c.ya = f.ya[off + e];
  };
  sweep_begin(stride, cur, fetch);
  run_step(st, tab);
  sweep(stride, cur, fetch, [&](long e, const E& c) {
    const Cx<double> zero = {0.0, 0.0};
    Cx<double> t = cfma(c64(tab[kTabSV][0]), c64(c.vtb), zero);
    t = cfma(c64(tab[kTabSV][1]), c64(c.w), t);
    Cx<double> v = cfma(c64(tab[kTabSW][0]), c64(c.chi), zero);
    v = cfma(c64(tab[kTabSW][1]), c64(c.vtbn), v);
    v = cfma(c64(tab[kTabSW][2]), c64(c.vtb), v);
    Cx<double> w = cfma(c64(tab[kTabWB][0]), c64(c.sbn), zero);
    w = cfma(c64(tab[kTabWB][1]), c64(c.sb), w);
    w = cfma(c64(tab[kTabWB][2]), c64(c.v1), w);
    w = cfma(c64(tab[kTabWB][3]), c64(c.v), w);
    if (f.vm) w = cfma(c64(tab[kTabWB][4]), c64(c.vm), w);
    f.tb[off + e] = d2(t);
    f.vb[off + e] = d2(v);
    f.wb[off + e] = d2(w);
    if (f.ya) f.ya[off + e] = d2(cfma(c64(tab[kTabY][0]), c64(c.v), c64(c.ya)));
  });
}

// vbar += A^dagger tbar and wbar += A sbar with their dots with v_i and w_i.
__global__ void __launch_bounds__(kWG) k_pass_add(double2* vb, const double2* t1, const double2* v,
                                                  double* pv, double2* wb, const double2* t2,
                                                  const double2* w, double* pw, long stride) {
  __shared__ double lds[(kWG / 64) * 2 * kLinDots];
  const long off = (long)blockIdx.y * stride;
  struct E {
    double2 vb, t1, v, wb, t2, w;
  } cur;
  auto fetch = [&](long e, E& c) {
    c.vb = vb[off + e];
    c.t1 = t1[off + e];
    c.v = v[off + e];
    c.wb = wb[off + e];
    c.t2 = t2[off + e];
    c.w = w[off + e];
  };
  sweep_begin(stride, cur, fetch);
  double a[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0}, b[2 * kLinDots] = {0.0, 0.0, 0.0, 0.0};
  sweep(stride, cur, fetch, [&](long e, const E& c) {
    const Cx<double> one = {1.0, 0.0};
    const Cx<double> x = cfma(one, c64(c.t1), c64(c.vb)), y = cfma(one, c64(c.t2), c64(c.wb));
    vb[off + e] = d2(x);
    wb[off + e] = d2(y);
    dot_acc(a, c64(c.v), x);
    dot_acc(b, c64(c.w), y);
  });
  put_dots(a, lds, pv);
  put_dots(b, lds, pw);
}

#define OVS_PASS(kernel, ...) \
  hipLaunchKernelGGL(kernel, dim3(lin_nchunk(stride), nrhs), dim3(kWG), 0, s, __VA_ARGS__)
void launch_pass_dots(const double2* t, const double2* w, double* partials, long stride, int nrhs,
                      const ScalarStep& st, hipStream_t s) {
  OVS_PASS(k_pass_dots, t, w, partials, stride, st);
}
void launch_pass_update(const StepFields& f, double2* vn, double2* wn, double* pv, double* pw,
                        long stride, int nrhs, const ScalarStep& st, hipStream_t s) {
  OVS_PASS(k_pass_update, f, vn, wn, pv, pw, stride, st);
}
void launch_pass_norm(double2* vn, double2* wn, const double2* chi, double* pchi, long stride,
                      int nrhs, const ScalarStep& st, hipStream_t s) {
  OVS_PASS(k_pass_norm, vn, wn, chi, pchi, stride, st);
}
void launch_pass_replay(const StepFields& f, double2* vn, double2* wn, long stride, int nrhs,
                        const ScalarStep& st, hipStream_t s) {
  OVS_PASS(k_pass_replay, f, vn, wn, stride, st);
}
void launch_pass_rev1(const Rev1Fields& f, double* pv, double* pw, long stride, int nrhs,
                      const ScalarStep& st, hipStream_t s) {
  OVS_PASS(k_pass_rev1, f, pv, pw, stride, st);
}
void launch_pass_rev2(const Rev2Fields& f, long stride, int nrhs, const ScalarStep& st,
                      hipStream_t s) {
  OVS_PASS(k_pass_rev2, f, stride, st);
}
void launch_pass_add(double2* vb, const double2* t1, const double2* v, double* pv, double2* wb,
                     const double2* t2, const double2* w, double* pw, long stride, int nrhs,
                     hipStream_t s) {
  OVS_PASS(k_pass_add, vb, t1, v, pv, wb, t2, w, pw, stride);
}
#undef OVS_PASS

// ---- inner sign and its vector-Jacobian product -----------------------------------
// One thread per (node, sign): LU with row interchanges of the tridiagonal
// M = G + i sigma (sigma = +-tau), then q = M^{-1} e_1 and p = M^{-H} xbar.
// Per-thread arrays live in scratch as [entry][thread] (coalesced).

struct VjpScratch {
  double2 *dl, *d, *du, *du2, *q, *p;
  unsigned char* piv;
};

static VjpScratch carve(void* base, int k, int nthr) {
  VjpScratch v;
  double2* b = (double2*)base;
  const long n = (long)k * nthr;
  v.dl = b;
  v.d = b + n;
  v.du = b + 2 * n;
  v.du2 = b + 3 * n;
  v.q = b + 4 * n;
  v.p = b + 5 * n;
  v.piv = (unsigned char*)(b + 6 * n);
  return v;
}

size_t isign_vjp_scratch_bytes(int k, int nnode) {
  const long n = (long)k * 2 * nnode;
  return (size_t)n * (6 * sizeof(double2) + 1) + 256;
}

// Bound by the latency of one wave's serial chain (the nodes fill a few dozen
// waves): two sweeps over the rows, the way down factors and solves L q = e_1 and
// U^H p = xbar as the rows become final, the way back finishes both.  What a row
// needs from its neighbours stays in registers, the coefficients of 64 rows sit
// in the lanes of the wave, loaded a block ahead, and the way back loads its rows
// four ahead.  (Five sweeps, each waiting for the previous row's entries from
// memory, took 840 us at k = 200.)
__global__ void __launch_bounds__(64) k_isign_vjp(const double2* alpha, const double* beta,
                                                  const double2* gamma, const double2* xbar,
                                                  int k, double h, int n0, int nnode,
                                                  VjpScratch sc) {
  const int nthr = 2 * nnode;
  const int lane = threadIdx.x;
  const int tt = blockIdx.x * 64 + lane;
  const bool live = tt < nthr;
  const int t = live ? tt : nthr - 1;  // the spare lanes repeat the last solve, unstored
  const double tau = exp((double)(n0 + (t >> 1)) * h);
  const double sigma = (t & 1) ? -tau : tau;
#define AT(arr, i) arr[(long)(i) * nthr + t]
  const Cx<double> zero = {0.0, 0.0};
  // lane l of a block holds alpha_{i0+l+1}, beta, gamma_{i0+l+1}, xbar of row i0+l
  struct Block {
    double2 a, g, x;
    double b;
  };
  auto load_block = [&](int i0) {
    const int i = i0 + lane;
    Block o;
    o.a = alpha[min(i + 1, k - 1)];
    o.b = beta[min(i, k - 1)];
    o.g = gamma[min(i + 1, k - 1)];
    o.x = xbar[min(i, k - 1)];
    return o;
  };
  Cx<double> d = {alpha[0].x, alpha[0].y + sigma};  // row i's diagonal, as updated
  Cx<double> du = c64(gamma[0]);                     // row i's superdiagonal, as updated
  Cx<double> q = {1.0, 0.0};                         // entry i of the right-hand side
  Cx<double> dum = zero, du2m = zero, du2mm = zero;  // du_{i-1}, du2_{i-1}, du2_{i-2}
  Cx<double> pm = zero, pmm = zero;                  // p_{i-1}, p_{i-2}
  Block nxt = load_block(0);
  for (int i0 = 0; i0 < k; i0 += 64) {
    const Block cur = nxt;
    nxt = load_block(i0 + 64);
    const int n = min(64, k - i0);
    for (int l = 0; l < n; ++l) {
      const int i = i0 + l;
      const bool last = i == k - 1;
      const Cx<double> dn = {lane_value(cur.a.x, l), lane_value(cur.a.y, l) + sigma};
      const Cx<double> un = {lane_value(cur.g.x, l), lane_value(cur.g.y, l)};
      const double li = lane_value(cur.b, l);
      const Cx<double> xb = {lane_value(cur.x.x, l), lane_value(cur.x.y, l)};
      // rows i and i + 1 interchanged when |beta_i| > |d|
      Cx<double> f = zero, df = d, duf = du, du2f = zero, qf = q, dnext = zero, dunext = un,
                 qnext = zero;
      bool sw = false;
      if (!last) {  // uniform
        f = pivot_quotient(li, d, sw);
        const Cx<double> fm = cmul(f, csel(sw, dn, du));
        dnext = csel(sw, du, dn) - fm;
        df = csel(sw, Cx<double>{li, 0.0}, d);
        duf = csel(sw, dn, du);
        if (i < k - 2) {
          du2f = csel(sw, un, zero);
          dunext = csel(sw, -cmul(f, un), un);
        }
        // entry i + 1 of e_1 is still zero here
        qf = csel(sw, zero, q);
        qnext = csel(sw, q - cmul(f, zero), zero - cmul(f, q));
      }
      Cx<double> b = xb;
      if (i >= 1) b = b - cmulc(dum, pm);
      if (i >= 2) b = b - cmulc(du2mm, pmm);
      const Cx<double> p = cdiv_fast(b, cconj(df));
      if (live) {
        AT(sc.d, i) = d2(df);
        AT(sc.du, i) = d2(duf);
        AT(sc.du2, i) = d2(du2f);
        AT(sc.dl, i) = d2(f);
        AT(sc.q, i) = d2(qf);
        AT(sc.p, i) = d2(p);
        AT(sc.piv, i) = sw ? 1 : 0;
      }
      d = dnext;
      du = dunext;
      q = qnext;
      du2mm = du2m;
      du2m = du2f;
      dum = duf;
      pmm = pm;
      pm = p;
    }
  }
  // the way back: U q = (.), L^H p = (.); four rows' entries loaded together,
  // one group ahead
  constexpr int kGroup = 4;
  struct Row {
    double2 d, du, du2, f, q, p;
    unsigned char piv;
  };
  Row rn[kGroup], rc[kGroup];
  auto load_rows = [&](int i) {  // rows i, i - 1, ... (clamped to row 0)
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int j = max(i - u, 0);
      rn[u].d = AT(sc.d, j);
      rn[u].du = AT(sc.du, j);
      rn[u].du2 = AT(sc.du2, j);
      rn[u].f = AT(sc.dl, j);
      rn[u].q = AT(sc.q, j);
      rn[u].p = AT(sc.p, j);
      rn[u].piv = AT(sc.piv, j);
    }
  };
  Cx<double> q1 = zero, q2 = zero, pc = zero;  // q_{i+1}, q_{i+2}; p_{i+1} so far
  load_rows(k - 1);
  for (int i0 = k - 1; i0 >= 0; i0 -= kGroup) {
#pragma unroll
    for (int u = 0; u < kGroup; ++u) rc[u] = rn[u];
    load_rows(i0 - kGroup);
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int i = i0 - u;
      if (i >= 0) {  // uniform
        Cx<double> b = c64(rc[u].q);
        if (i + 1 < k) b = b - cmul(c64(rc[u].du), q1);
        if (i + 2 < k) b = b - cmul(c64(rc[u].du2), q2);
        const Cx<double> qi = cdiv_fast(b, c64(rc[u].d));
        if (live) AT(sc.q, i) = d2(qi);
        q2 = q1;
        q1 = qi;
        if (i == k - 1) {
          pc = c64(rc[u].p);
        } else {
          const Cx<double> v = c64(rc[u].p) - cmulc(c64(rc[u].f), pc);
          const bool sw = rc[u].piv != 0;
          if (live) AT(sc.p, i + 1) = d2(csel(sw, v, pc));
          pc = csel(sw, pc, v);
        }
      }
    }
  }
  if (live) AT(sc.p, 0) = d2(pc);
#undef AT
}

// Sums over nodes (fixed order) with the trapezoid weights h tau / pi.  With
// coarse.x set, also the rule of step 2h (the nodes of even index, weights
// 2 h tau / pi) into coarse (x, gd, gsup), for the first comparison of two
// levels without a launch at step 2h.
// One wave per row: the lanes load and weight 64 solves at a time (coalesced),
// then one lane per sum adds them in order from LDS.  (One thread per row,
// walking its row of memory by itself, took 540 us at k = 200.)
__global__ void __launch_bounds__(64) k_isign_vjp_reduce(int k, double h, int n0, int nnode,
                                                         VjpScratch sc, IsignVjpOut out,
                                                         IsignVjpOut coarse) {
  constexpr int kSums = 13;  // x, gd, Re gs, gu; coarse x, gd, gu
  __shared__ double term[kSums][65];
  const int i = blockIdx.x;
  const int lane = threadIdx.x;
  const int nthr = 2 * nnode;
  const bool two = coarse.x != nullptr, up = i + 1 < k;
  double acc = 0.0;
  for (int t0 = 0; t0 < nthr; t0 += 64) {
    const int t = min(t0 + lane, nthr - 1);
    const int node = n0 + (t >> 1);
    const Cx<double> qi = c64(sc.q[(long)i * nthr + t]), pi_ = c64(sc.p[(long)i * nthr + t]);
    Cx<double> qn = {0.0, 0.0}, pn = {0.0, 0.0};
    if (up) {
      qn = c64(sc.q[(long)(i + 1) * nthr + t]);
      pn = c64(sc.p[(long)(i + 1) * nthr + t]);
    }
    const double w = h * exp((double)node * h) / M_PI;
    const bool even = two && (node & 1) == 0;
    const Cx<double> x = scale(w, qi), gd = scale(w, cmulc(qi, pi_));
    const Cx<double> gs = scale(w, cmulc(qi, pn));   // -Gbar_{i+1,i} = p_{i+1} conj(q_i)
    const Cx<double> gu = scale(w, cmulc(qn, pi_));  // -Gbar_{i,i+1} = p_i conj(q_{i+1})
    const Cx<double> xc = scale(2.0 * w, qi), gdc = scale(2.0 * w, cmulc(qi, pi_)),
                     guc = scale(2.0 * w, cmulc(qn, pi_));
    __syncthreads();
    const double v[kSums] = {x.re,
                             x.im,
                             -gd.re,
                             -gd.im,
                             -gs.re,
                             -gu.re,
                             -gu.im,
                             even ? xc.re : 0.0,
                             even ? xc.im : 0.0,
                             even ? -gdc.re : 0.0,
                             even ? -gdc.im : 0.0,
                             even ? -guc.re : 0.0,
                             even ? -guc.im : 0.0};
#pragma unroll
    for (int s = 0; s < kSums; ++s) term[s][lane] = v[s];
    __syncthreads();
    if (lane < kSums) {
      const int n = min(64, nthr - t0);
      int l = 0;
      for (; l + 16 <= n; l += 16) {
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += term[lane][l + u];
      }
      for (; l < n; ++l) acc += term[lane][l];
    }
  }
  double* const dst[kSums] = {&out.x[i].x, &out.x[i].y, &out.gd[i].x, &out.gd[i].y,
                              up ? &out.gsub_re[i] : nullptr, up ? &out.gsup[i].x : nullptr,
                              up ? &out.gsup[i].y : nullptr, two ? &coarse.x[i].x : nullptr,
                              two ? &coarse.x[i].y : nullptr, two ? &coarse.gd[i].x : nullptr,
                              two ? &coarse.gd[i].y : nullptr,
                              two && up ? &coarse.gsup[i].x : nullptr,
                              two && up ? &coarse.gsup[i].y : nullptr};
#pragma unroll
  for (int s = 0; s < kSums; ++s)
    if (lane == s && dst[s]) *dst[s] = acc;
}

void launch_isign_vjp(const double2* alpha, const double* beta, const double2* gamma,
                      const double2* xbar, int k, double h, int n0, int nnode, void* scratch,
                      const IsignVjpOut& out, hipStream_t st, const IsignVjpOut* coarse) {
  const int nthr = 2 * nnode;
  const VjpScratch sc = carve(scratch, k, nthr);
  hipLaunchKernelGGL(k_isign_vjp, dim3((nthr + 63) / 64), dim3(64), 0, st, alpha, beta, gamma,
                     xbar, k, h, n0, nnode, sc);
  const IsignVjpOut none{};
  hipLaunchKernelGGL(k_isign_vjp_reduce, dim3(k), dim3(64), 0, st, k, h, n0, nnode, sc,
                     out, coarse ? *coarse : none);
}

// ---- link force -----------------------------------------------------------------
// For Re <pbar, A p>, A = gamma5 Dw with hop coefficient k eta on packed links
// U~ (boundary signs folded in), the gradient with respect to U~_nu(x) is
//   forward hop into x+nu : -k eta+ sum_s [(1+g_nu) g5 pbar(x+nu)]_s [p(x)]_s^dagger
//   backward hop into x   : -k eta- sum_s [(1-g_nu) p(x+nu)]_s [g5 pbar(x)]_s^dagger
// (colour outer products summed over spin).  With (1 +- g_nu) = E P, P the
// two-row projection of the stencil and E = P^dagger, each sum reduces to two
// outer products of projected half spinors.

struct HopPair {
  double fA[4], bA[4], fAd[4], bAd[4];
};

__device__ __forceinline__ void load_sp(const double2* f, long Vs, int s, bool g5,
                                        Cx<double> (&p)[12]) {
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    p[c] = c64(f[fidx(c, s, Vs)]);
    if (g5 && c >= 6) p[c] = -p[c];
  }
}

// F[a][b] += c * sum_k h_k[a] conj(g_k[b])
__device__ __forceinline__ void outer_acc(Cx<double> (&F)[9], const Cx<double> (&h)[6],
                                          const Cx<double> (&g)[6], double c) {
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const Cx<double> v = cmulc(g[b], h[a]) + cmulc(g[3 + b], h[3 + a]);
      F[3 * a + b] = F[3 * a + b] + scale(c, v);
    }
}

// forward and backward hop terms of one (adjoint, input) pair
template <int NU>
__device__ __forceinline__ void force_pair(Cx<double> (&Ff)[9], Cx<double> (&Fb)[9],
                                           const double2* bar, const double2* in, long Vs, int s,
                                           int sf, double cf, double cb) {
  Cx<double> a[12], b[12], h[6], g[6];
  load_sp(bar, Vs, sf, true, a);
  project<double, NU, +1>(a, h);
  load_sp(in, Vs, s, false, b);
  project<double, NU, +1>(b, g);
  outer_acc(Ff, h, g, -cf);
  load_sp(in, Vs, sf, false, a);
  project<double, NU, -1>(a, h);
  load_sp(bar, Vs, s, true, b);
  project<double, NU, -1>(b, g);
  outer_acc(Fb, h, g, -cb);
}

template <int NU>
__device__ __forceinline__ void force_dir(double2* F, const double2* pbar, const double2* p,
                                          const double2* qbar, const double2* q, long stride,
                                          int nrhs, const Geometry& g, int s, int sf,
                                          const HopPair& hp) {
  const long Vs = g.Vs;
  Cx<double> fp[9], fm[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) fp[e] = fm[e] = {0.0, 0.0};
  for (int r = 0; r < nrhs; ++r) {
    const long o = (long)r * stride;
    // A(mu): forward carries e^{+mu}, backward e^{-mu}
    if constexpr (NU == 3) force_pair<NU>(fp, fm, pbar + o, p + o, Vs, s, sf, hp.fA[NU], hp.bA[NU]);
    else force_pair<NU>(fp, fp, pbar + o, p + o, Vs, s, sf, hp.fA[NU], hp.bA[NU]);
    if (qbar) {
      // A(mu)^dagger = A(-mu): forward carries e^{-mu}, backward e^{+mu}
      if constexpr (NU == 3)
        force_pair<NU>(fm, fp, qbar + o, q + o, Vs, s, sf, hp.fAd[NU], hp.bAd[NU]);
      else force_pair<NU>(fp, fp, qbar + o, q + o, Vs, s, sf, hp.fAd[NU], hp.bAd[NU]);
    }
  }
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    double2* dst = F + ((long)NU * 9 + e) * Vs + s;
    *dst = d2(c64(*dst) + fp[e]);
  }
  if constexpr (NU == 3) {
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      double2* dst = F + ((long)4 * 9 + e) * Vs + s;
      *dst = d2(c64(*dst) + fm[e]);
    }
  }
}

// Site and direction of a thread: one thread per site and direction (each
// direction writes only its own slots of F, so the directions are independent),
// a workgroup takes 64 sites in the four directions (a wave each), and each XCD
// a contiguous range of the lattice: the spinors that the directions of a site
// and its neighbours share are then in one L1 and one L2 (16^4, ten steps: 460 us
// with the directions in workgroups of their own, spread over the XCDs).
__device__ __forceinline__ bool force_site(const Geometry& g, int& s, int& dir) {
  const int ntile = (g.V + 63) / 64, per = (ntile + 7) / 8;
  const int tile = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
  s = tile * 64 + ((int)threadIdx.x & 63);
  dir = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  return tile < ntile && s < g.V;
}
static dim3 force_grid(const Geometry& g) { return dim3(8 * (((g.V + 63) / 64 + 7) / 8)); }

__global__ void __launch_bounds__(kWG) k_gforce(double2* F, const double2* pbar, const double2* p,
                                                const double2* qbar, const double2* q, long stride,
                                                int nrhs, Geometry g, HopPair hp) {
  int s, dir;
  if (!force_site(g, s, dir)) return;
  const Nbr nb = neighbours(s, g);
  switch (dir) {
    case 0: force_dir<0>(F, pbar, p, qbar, q, stride, nrhs, g, s, nb.f[0], hp); break;
    case 1: force_dir<1>(F, pbar, p, qbar, q, stride, nrhs, g, s, nb.f[1], hp); break;
    case 2: force_dir<2>(F, pbar, p, qbar, q, stride, nrhs, g, s, nb.f[2], hp); break;
    default: force_dir<3>(F, pbar, p, qbar, q, stride, nrhs, g, s, nb.f[3], hp); break;
  }
}

static HopPair hop_pair(const Hop& hA, const Hop& hAd) {
  HopPair hp;
  for (int nu = 0; nu < 4; ++nu) {
    hp.fA[nu] = hA.fwd[nu];
    hp.bA[nu] = hA.bwd[nu];
    hp.fAd[nu] = hAd.fwd[nu];
    hp.bAd[nu] = hAd.bwd[nu];
  }
  return hp;
}

void launch_gforce(double2* F, const double2* pbar, const double2* p, const double2* qbar,
                   const double2* q, long stride, int nrhs, const Geometry& g, const Hop& hA,
                   const Hop& hAd, hipStream_t st) {
  const HopPair hp = hop_pair(hA, hAd);
  hipLaunchKernelGGL(k_gforce, force_grid(g), dim3(kWG), 0, st, F, pbar, p, qbar,
                     q, stride, nrhs, g, hp);
}

// The force of n consecutive reverse steps in one pass: the contributions of
// every step and source are summed in registers (steps in order, then
// sources, as force_dir sums the sources of one step) and F is read and
// written once, not once per step.  Step j's fields are at pbar0 + j *
// step_stride etc.
template <int NU>
__device__ __forceinline__ void force_dir_group(double2* F, const double2* pbar0,
                                                const double2* p0, const double2* qbar0,
                                                const double2* q0, int nsteps, long step_stride,
                                                long stride, int nrhs, const Geometry& g, int s,
                                                int sf, const HopPair& hp) {
  const long Vs = g.Vs;
  Cx<double> fp[9], fm[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) fp[e] = fm[e] = {0.0, 0.0};
  for (int j = 0; j < nsteps; ++j) {
    const long js = (long)j * step_stride;
    for (int r = 0; r < nrhs; ++r) {
      const long o = js + (long)r * stride;
      if constexpr (NU == 3) {
        force_pair<NU>(fp, fm, pbar0 + o, p0 + o, Vs, s, sf, hp.fA[NU], hp.bA[NU]);
        force_pair<NU>(fm, fp, qbar0 + o, q0 + o, Vs, s, sf, hp.fAd[NU], hp.bAd[NU]);
      } else {
        force_pair<NU>(fp, fp, pbar0 + o, p0 + o, Vs, s, sf, hp.fA[NU], hp.bA[NU]);
        force_pair<NU>(fp, fp, qbar0 + o, q0 + o, Vs, s, sf, hp.fAd[NU], hp.bAd[NU]);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    double2* dst = F + ((long)NU * 9 + e) * Vs + s;
    *dst = d2(c64(*dst) + fp[e]);
  }
  if constexpr (NU == 3) {
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      double2* dst = F + ((long)4 * 9 + e) * Vs + s;
      *dst = d2(c64(*dst) + fm[e]);
    }
  }
}

__global__ void __launch_bounds__(kWG) k_gforce_group(double2* F, const double2* pbar0,
                                                      const double2* p0, const double2* qbar0,
                                                      const double2* q0, int nsteps,
                                                      long step_stride, long stride, int nrhs,
                                                      Geometry g, HopPair hp) {
  int s, dir;
  if (!force_site(g, s, dir)) return;
  const Nbr nb = neighbours(s, g);
  switch (dir) {
    case 0: force_dir_group<0>(F, pbar0, p0, qbar0, q0, nsteps, step_stride, stride, nrhs, g, s, nb.f[0], hp); break;
    case 1: force_dir_group<1>(F, pbar0, p0, qbar0, q0, nsteps, step_stride, stride, nrhs, g, s, nb.f[1], hp); break;
    case 2: force_dir_group<2>(F, pbar0, p0, qbar0, q0, nsteps, step_stride, stride, nrhs, g, s, nb.f[2], hp); break;
    default: force_dir_group<3>(F, pbar0, p0, qbar0, q0, nsteps, step_stride, stride, nrhs, g, s, nb.f[3], hp); break;
  }
}

void launch_gforce_group(double2* F, const double2* pbar0, const double2* p0,
                         const double2* qbar0, const double2* q0, int nsteps, long step_stride,
                         long stride, int nrhs, const Geometry& g, const Hop& hA, const Hop& hAd,
                         hipStream_t st) {
  const HopPair hp = hop_pair(hA, hAd);
  hipLaunchKernelGGL(k_gforce_group, force_grid(g), dim3(kWG), 0, st, F, pbar0,
                     p0, qbar0, q0, nsteps, step_stride, stride, nrhs, g, hp);
}

__global__ void __launch_bounds__(kWG) k_gforce_out(const double2* F, const double2* links,
                                                    Geometry g, int bc0, int bc1, int bc2, int bc3,
                                                    double2* grad_U, double* partials) {
  __shared__ double lds[(kWG / 64)];
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  double part[1] = {0.0};
  if (s < g.V) {
    const int x = s % g.lx, y = (s / g.lx) % g.ly, z = (s / (g.lx * g.ly)) % g.lz,
              t = s / (g.lx * g.ly * g.lz);
    const int coord[4] = {x, y, z, t};
    const int ext[4] = {g.lx, g.ly, g.lz, g.lt};
    const int bc[4] = {bc0, bc1, bc2, bc3};
    for (int nu = 0; nu < 4; ++nu) {
      const double sg = (coord[nu] == ext[nu] - 1 && bc[nu] < 0) ? -1.0 : 1.0;
      for (int e = 0; e < 9; ++e) {
        Cx<double> v = c64(F[((long)nu * 9 + e) * g.Vs + s]);
        if (nu == 3) {
          const Cx<double> vm = c64(F[((long)4 * 9 + e) * g.Vs + s]);
          const Cx<double> u = c64(links[lidx(3, e, s, g.Vs)]);
          part[0] += cmulc(v, u).re - cmulc(vm, u).re;
          v = v + vm;
        }
        grad_U[((long)s * 4 + nu) * 9 + e] = d2(scale(sg, v));
      }
    }
  }
  block_sum<1>(part, lds);
  if (threadIdx.x == 0) partials[blockIdx.x] = part[0];
}

__global__ void k_sum_partials(const double* partials, int n, double* out) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  double a = 0.0;
  for (int i = 0; i < n; ++i) a += partials[i];
  *out = a;
}

void launch_gforce_out(const double2* F, const double2* links, const Geometry& g, const int bc[4],
                       double2* grad_U, double* partials, double* grad_mu, hipStream_t st) {
  const int nb = (g.V + kWG - 1) / kWG;
  hipLaunchKernelGGL(k_gforce_out, dim3(nb), dim3(kWG), 0, st, F, links, g, bc[0], bc[1], bc[2],
                     bc[3], grad_U, partials);
  hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(1), 0, st, partials, nb, grad_mu);
}

}  // namespace ovs

namespace ovs {

// ---- su(3) link force ------------------------------------------------------
// F = -TA(U G^dagger) per link, TA(M) = (M - M^dagger)/2 - tr(M - M^dagger)/6:
// the force of a real L(U) for U -> exp(eps X) U, X in su(3), from its link
// gradient G = dL/dRe U + i dL/dIm U.  Canonical layout [V][4][3][3].
__global__ void __launch_bounds__(kWG) k_link_force(const double2* __restrict__ U,
                                                    const double2* __restrict__ G,
                                                    double2* __restrict__ F, long nlinks) {
  const long n = (long)blockIdx.x * kWG + threadIdx.x;
  if (n >= nlinks) return;
  Cx<double> u[9], g[9], m[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    u[e] = c64(U[n * 9 + e]);
    g[e] = c64(G[n * 9 + e]);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      Cx<double> s = {0.0, 0.0};
#pragma unroll
      for (int c = 0; c < 3; ++c) s = cfmac(g[b * 3 + c], u[a * 3 + c], s);  // U_ac conj(G_bc)
      m[a * 3 + b] = s;
    }
  // trace of the anti-Hermitian part: i Im tr M
  const double imtr = (m[0].im + m[4].im + m[8].im) / 3.0;
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const Cx<double> x = m[a * 3 + b], y = m[b * 3 + a];
      Cx<double> t = {0.5 * (x.re - y.re), 0.5 * (x.im + y.im)};  // (M - M^dagger)/2
      if (a == b) t.im -= imtr;
      F[n * 9 + a * 3 + b] = d2(-t);
    }
}

void launch_link_force(const double2* U, const double2* G, double2* F, long nlinks,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_link_force, dim3((unsigned)((nlinks + kWG - 1) / kWG)), dim3(kWG), 0, s,
                     U, G, F, nlinks);
}

}  // namespace ovs
