// Krylov-side kernels: LR deflation (Section 3), the two-sided Lanczos update
// and coefficient steps (Section 4), the Arnoldi Gram-Schmidt steps
// (Section 2), the combination |b_R| V_k x (eq. 2sLapp / Arnapp) and the
// inner sign sgn(T) e_1 of the small projected matrix.
//
// All inner products and norms accumulate in FP64 and are reduced in a fixed
// order (per-workgroup partials, then one pass over the partials), so results
// are bitwise repeatable from run to run.
#include <algorithm>

#include "ovs_common.h"
#include "ovs_device.h"
#include "ovs_krylov.h"
#include "ovs_lanczos.h"

namespace ovs {

static inline int cdiv_i(long a, long b) { return (int)((a + b - 1) / b); }

// ===========================================================================
// Generic fixed-order reduction of per-workgroup partials.
// partials: [nslots][nparts][nv]; out: [nslots][nv].  One workgroup per slot.
// ===========================================================================
template <int NV>
__global__ void __launch_bounds__(256) k_reduce_partials(const double* __restrict__ partials,
                                                         int nparts, double* __restrict__ out) {
  __shared__ double lds[4 * NV];
  const long slot = blockIdx.x;
  double v[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) v[j] = 0.0;
  for (int p = threadIdx.x; p < nparts; p += blockDim.x) {
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] += partials[(slot * nparts + p) * NV + j];
  }
  block_sum<NV>(v, lds);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) out[slot * NV + j] = v[j];
  }
}

// ===========================================================================
// LR deflation (Section 3 and eq. 2sLapp):
//   C = L^dag b, D = R^dag b, b_R = b - R C, b_L = b - L D, y_ex = R sgn(Lam) C
// ===========================================================================
constexpr int kDeflRhs = 8;  // sources per thread in the dot kernel

// partials [m][nrhs][nchunk][4] = (C.re, C.im, D.re, D.im)
__global__ void __launch_bounds__(256) k_defl_dots(const double2* __restrict__ R,
                                                   const double2* __restrict__ L,
                                                   const double2* __restrict__ B, int nrhs, long N,
                                                   int nchunk, double* __restrict__ partials) {
  __shared__ double lds[4 * 4 * kDeflRhs];
  const int j = blockIdx.y;
  const int r0 = blockIdx.z * kDeflRhs;
  const int nr = min(kDeflRhs, nrhs - r0);
  double v[4 * kDeflRhs];
#pragma unroll
  for (int q = 0; q < 4 * kDeflRhs; ++q) v[q] = 0.0;
  const double2* Rj = R + (long)j * N;
  const double2* Lj = L + (long)j * N;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    const Cx<double> rr = c64(Rj[e]), ll = c64(Lj[e]);
#pragma unroll
    for (int q = 0; q < kDeflRhs; ++q) {
      if (q < nr) {
        const Cx<double> bb = c64(B[(long)(r0 + q) * N + e]);
        const Cx<double> c = cmulc(ll, bb), d = cmulc(rr, bb);
        v[4 * q + 0] += c.re;
        v[4 * q + 1] += c.im;
        v[4 * q + 2] += d.re;
        v[4 * q + 3] += d.im;
      }
    }
  }
  const double a = block_sums(v, lds);
  const int q = threadIdx.x;
  if (q < 4 * nr)
    partials[(((long)j * nrhs + r0 + (q >> 2)) * nchunk + blockIdx.x) * 4 + (q & 3)] = a;
}

// CD: [m][nrhs][4] reduced (C, D); sgn: [m] sign of Re lambda.
__global__ void __launch_bounds__(256) k_defl_axpy(const double2* __restrict__ R,
                                                   const double2* __restrict__ L,
                                                   const double2* __restrict__ B,
                                                   const double* __restrict__ CD,
                                                   const double* __restrict__ sgn, int m, int nrhs,
                                                   long N, double2* __restrict__ bR,
                                                   double2* __restrict__ bL,
                                                   double2* __restrict__ yex) {
  const int r = blockIdx.y;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    const Cx<double> b = c64(B[(long)r * N + e]);
    Cx<double> pr = {0, 0}, pl = {0, 0}, py = {0, 0};
    for (int j = 0; j < m; ++j) {
      const double* cd = CD + ((long)j * nrhs + r) * 4;
      const Cx<double> c = {cd[0], cd[1]}, d = {cd[2], cd[3]};
      const Cx<double> rr = c64(R[(long)j * N + e]), ll = c64(L[(long)j * N + e]);
      pr = cfma(rr, c, pr);
      pl = cfma(ll, d, pl);
      if (yex) py = cfma(rr, scale(sgn[j], c), py);
    }
    if (bR) bR[(long)r * N + e] = d2(b - pr);
    if (bL) bL[(long)r * N + e] = d2(b - pl);
    if (yex) yex[(long)r * N + e] = d2(py);
  }
}

// D[j][r] -= kappa[r][j] (the bL output of k_defl_axpy then gains + L kappa)
__global__ void k_cd_shift(double* __restrict__ CD, const double2* __restrict__ kappa, int m,
                           int nrhs) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m * nrhs) return;
  const int j = e / nrhs, r = e % nrhs;
  const double2 k = kappa[(long)r * m + j];
  CD[(long)e * 4 + 2] -= k.x;
  CD[(long)e * 4 + 3] -= k.y;
}

// per-source partials of |b_R|^2 and b_L^dag b_R: [nrhs][nchunk][3]
__global__ void __launch_bounds__(256) k_start_dots(const double2* __restrict__ bR,
                                                    const double2* __restrict__ bL, long N,
                                                    int nchunk, double* __restrict__ partials) {
  __shared__ double lds[4 * 3];
  const int r = blockIdx.y;
  double v[3] = {0, 0, 0};
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    const Cx<double> a = c64(bR[(long)r * N + e]), l = c64(bL[(long)r * N + e]);
    v[0] += cnorm2(a);
    const Cx<double> s = cmulc(l, a);
    v[1] += s.re;
    v[2] += s.im;
  }
  block_sum<3>(v, lds);
  if (threadIdx.x == 0)
    for (int t = 0; t < 3; ++t) partials[((long)r * nchunk + blockIdx.x) * 3 + t] = v[t];
}

// Start vectors v_1 = b_R / n_b, w_1 = b_L n_b / conj(sigma) (stored in
// storage precision) from sums[r] = (|b_R|^2, sigma.re, sigma.im).
template <typename T2>
__global__ void k_start_vectors(const double2* __restrict__ bR, const double2* __restrict__ bL,
                                const double* __restrict__ sums, long N, T2* __restrict__ V0,
                                T2* __restrict__ W0) {
  const int r = blockIdx.y;
  const double nb = sqrt(sums[r * 3 + 0]);
  const Cx<double> sig = {sums[r * 3 + 1], sums[r * 3 + 2]};
  const double inv = nb > 0 ? 1.0 / nb : 0.0;
  Cx<double> fw = {0, 0};
  if (nb > 0 && (sig.re != 0 || sig.im != 0)) fw = cdiv(Cx<double>{nb, 0}, Cx<double>{sig.re, -sig.im});
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    if (V0) st64(V0 + (long)r * N + e, scale(inv, c64(bR[(long)r * N + e])));
    if (W0) st64(W0 + (long)r * N + e, cmul(fw, c64(bL[(long)r * N + e])));
  }
}

// ===========================================================================
// Two-sided Lanczos coefficient steps (Section 4).  The iteration index lives
// in device memory (*it) so a captured chunk of iterations can be replayed.
// ===========================================================================

// ---- per-step kernels (bodies in ovs_lanczos.h) ----------------------------

__global__ void __launch_bounds__(256) k_alpha(const double* __restrict__ partials, int nparts,
                                               int quad, CoefArrays co, const int* __restrict__ it,
                                               int off,
                                               const int* __restrict__ rhs_map,
                                               const int* __restrict__ n_active) {
  alpha_body(blockIdx.x, *it + off, partials, nparts, quad, co, rhs_map, *n_active);
}

template <typename T2>
__global__ void __launch_bounds__(256) k_update(const T2* __restrict__ T, const T2* __restrict__ S,
                                                T2* __restrict__ basis, long basis_stride,
                                                T2* __restrict__ wbuf, long slot_stride, long N,
                                                CoefArrays co, const int* __restrict__ it, int off,
                                                const int* __restrict__ rhs_map,
                                                const int* __restrict__ n_active,
                                                double* __restrict__ partials, int two_pass_ring,
                                                const double* __restrict__ apart, int anparts,
                                                int quad, int nt) {
  update_body<T2>(blockIdx.x, blockIdx.y, gridDim.x, *it + off, T, S, basis, basis_stride, wbuf,
                  slot_stride, N, co, rhs_map, *n_active, partials, two_pass_ring, apart, anparts,
                  quad, nt);
}

// beta_body of iteration *it + adv - 1 for one source slot per workgroup, then
// the iteration index advances by adv: the last workgroup to finish (a ticket
// counter, reset by that workgroup, so it is zero between launches) adds it,
// after every workgroup has read *it.  Ends a run of adv iterations; the beta
// steps before run beside the next iteration's dual stencil (BetaArgs).
template <typename T2>
__global__ void __launch_bounds__(256) k_beta_tail(const double* __restrict__ partials, int nparts,
                                                   CoefArrays co, int* __restrict__ it, int adv,
                                                   const int* __restrict__ rhs_map,
                                                   const int* __restrict__ n_active,
                                                   int* __restrict__ ticket,
                                                   const T2* __restrict__ basis, long basis_stride,
                                                   long N, int ring, const int* __restrict__ idx,
                                                   int P, double2* __restrict__ probes) {
  const int base = *it;
  beta_body<T2>(blockIdx.x, base + adv - 1, partials, nparts, co, rhs_map, *n_active, basis, basis_stride, N,
                ring, idx, P, probes);
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    if (atomicAdd(ticket, 1) == (int)gridDim.x - 1) {
      *ticket = 0;
      *it = base + adv;
    }
  }
}

// Probe sketch for the convergence estimate: the entries idx[0..P) of the
// stored Lanczos vector V~_j (j = *it + 1, or j = 0 before the first step) of
// every active source are copied to probes[slot][j][P] in FP64.
template <typename T2>
__global__ void __launch_bounds__(256) k_probe_gather(const T2* __restrict__ basis, long basis_stride,
                                                      long N, int ring, const int* __restrict__ it,
                                                      int first, const int* __restrict__ idx, int P,
                                                      int kmax, const int* __restrict__ rhs_map,
                                                      const int* __restrict__ n_active,
                                                      double2* __restrict__ probes) {
  const int jj = blockIdx.y;
  if (jj >= *n_active) return;
  const int slot = rhs_map[jj];
  const int j = first ? 0 : *it + 1;
  if (j >= kmax) return;
  const long sl = ring ? (j % 3) : j;
  const T2* v = basis + sl * basis_stride + (long)slot * N;
  for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x)
    probes[((long)slot * kmax + j) * P + p] = d2(ld64(v + idx[p]));
}

// yp[r][p] = yex[r][idx[p]] + sum_{i < k_r} c_i probes[r][i][p] with the
// combination's coefficients c_i = n_b x[r][i] sv[r][i] (k_make_coef's), formed
// for 64 terms at a time by the workgroup.  Bound by memory latency along i:
// the loads of 16 terms are issued before their multiply-adds (k = 375: 22 us a
// launch with eight, behind a launch that formed the coefficients).
__global__ void __launch_bounds__(64) k_probe_y(const double2* __restrict__ probes,
                                                const double2* __restrict__ x,
                                                const double* __restrict__ sv,
                                                const double* __restrict__ nb,
                                                const int* __restrict__ kvec, int kmax,
                                                const double2* __restrict__ yex, long N,
                                                const int* __restrict__ idx, int P,
                                                double2* __restrict__ yp) {
  __shared__ double2 cs[64];
  const int r = blockIdx.y;
  const int k = kvec[r];
  const int p = blockIdx.x * 64 + threadIdx.x;
  const int pc = min(p, P - 1);
  const double n_b = nb[r];
  const double2* xr = x + (long)r * kmax;
  const double* svr = sv ? sv + (long)r * (kmax + 1) : nullptr;
  const double2* pr = probes + (long)r * kmax * P + pc;
  Cx<double> acc = yex ? c64(yex[(long)r * N + idx[pc]]) : Cx<double>{0, 0};
  for (int i0 = 0; i0 < k; i0 += 64) {
    const int n = min(64, k - i0);
    __syncthreads();
    if ((int)threadIdx.x < n) {
      const int i = i0 + threadIdx.x;
      cs[threadIdx.x] = d2(scale(n_b * (svr ? svr[i] : 1.0), c64(xr[i])));
    }
    __syncthreads();
    int t = 0;
    for (; t + 16 <= n; t += 16) {
      double2 q[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) q[u] = pr[(long)(i0 + t + u) * P];
#pragma unroll
      for (int u = 0; u < 16; ++u) acc = cfma(c64(cs[t + u]), c64(q[u]), acc);
    }
    for (; t < n; ++t) acc = cfma(c64(cs[t]), c64(pr[(long)(i0 + t) * P]), acc);
  }
  if (p < P) yp[(long)r * P + p] = d2(acc);
}

__global__ void k_advance(int* it) { *it += 1; }

// ===========================================================================
// Combination y = y_ex + sum_i coef_i V~_i   (coef_i = n_b x_i sv_i)
// ===========================================================================
template <typename T2>
__global__ void __launch_bounds__(256) k_combine(const T2* __restrict__ basis, long basis_stride,
                                                 long N, const double2* __restrict__ coef, int kmax,
                                                 const int* __restrict__ kused,
                                                 const double2* __restrict__ yex,
                                                 double2* __restrict__ y) {
  const int r = blockIdx.y;
  const int kr = kused[r];
  const double2* cr = coef + (long)r * kmax;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    Cx<double> acc = yex ? c64(yex[(long)r * N + e]) : Cx<double>{0, 0};
    const T2* br = basis + (long)r * N + e;
    // the same sequential sum as one term per step, with the loads of eight
    // basis vectors issued before their multiply-adds: one load in flight per
    // wave would leave the sweep over the k_used stored vectors latency-bound
    int i = 0;
    for (; i + 8 <= kr; i += 8) {
      Cx<double> q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = ld64(br + (long)(i + u) * basis_stride);
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = cfma(c64(cr[i + u]), q[u], acc);
    }
    for (; i < kr; ++i) acc = cfma(c64(cr[i]), ld64(br + (long)i * basis_stride), acc);
    y[(long)r * N + e] = d2(acc);
  }
}

// coef[r][i] = n_b x[r][i] sv[r][i] for i < kused[r], else 0
__global__ void k_make_coef(const double2* __restrict__ x, const double* __restrict__ sv,
                            const double* __restrict__ nb, int kmax, int nrhs,
                            double2* __restrict__ coef) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (e >= (long)nrhs * kmax) return;
  const long r = e / kmax, i = e % kmax;
  coef[e] = d2(scale(nb[r] * (sv ? sv[r * (kmax + 1) + i] : 1.0), c64(x[e])));
}

// Second pass of the small-memory evaluation: replay v_{i+1} from the stored
// coefficients (identical arithmetic to k_update) and accumulate y.
template <typename T2>
__global__ void __launch_bounds__(256) k_replay(const T2* __restrict__ T, T2* __restrict__ ring,
                                                long ring_stride, long N, CoefArrays co, int i,
                                                const double2* __restrict__ coef,
                                                const int* __restrict__ kused,
                                                double2* __restrict__ y) {
  const int r = blockIdx.y;
  const int kr = kused[r];
  if (i >= kr) return;
  const long ks = co.kmax;
  const bool prev = i > 0;
  const bool next = i + 1 < kr;
  const Cx<double> a = c64(co.alpha[r * ks + i]);
  const double svi = co.sv[r * (ks + 1) + i];
  const double svm = prev ? co.sv[r * (ks + 1) + i - 1] : 0.0;
  const Cx<double> gm = prev ? c64(co.gamma[r * ks + i - 1]) : Cx<double>{0, 0};
  const Cx<double> c1 = {svi, 0.0};
  const Cx<double> c2 = scale(-svi, a);
  const Cx<double> c3 = scale(-svm, gm);
  const Cx<double> ci = c64(coef[r * ks + i]);
  const T2* Vi = ring + (long)(i % 3) * ring_stride + (long)r * N;
  const T2* Vm = ring + (long)((i + 2) % 3) * ring_stride + (long)r * N;
  T2* Vn = ring + (long)((i + 1) % 3) * ring_stride + (long)r * N;
  const T2* Ts = T + (long)r * N;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    const Cx<double> vi = ld64(Vi + e);
    y[(long)r * N + e] = d2(cfma(ci, vi, c64(y[(long)r * N + e])));
    if (next) {
      Cx<double> vt = cmul(c1, ld64(Ts + e));
      vt = cfma(c2, vi, vt);
      if (prev) vt = cfma(c3, ld64(Vm + e), vt);
      st64(Vn + e, vt);
    }
  }
}

// y <- b + gamma5 y  (D_ov b, eq. (1.1)); fields [nrhs][12][V] FP64
__global__ void k_overlap(const double2* __restrict__ b, double2* __restrict__ y, long N, int V) {
  // V: the padded plane stride Vs; component c of offset e (layout of fidx)
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    const long loc = e % (12L * V);
    const int c = (int)(2 * ((loc >> 1) / V) + (loc & 1));
    Cx<double> v = c64(y[e]);
    if (c >= 6) v = -v;
    y[e] = d2(c64(b[e]) + v);
  }
}

// ===========================================================================
// Arnoldi (Section 2): classical Gram-Schmidt applied twice.
// ===========================================================================
constexpr int kArnVec = 8;  // basis vectors per workgroup in the dot kernel

// partials [nrhs][nvec][nchunk][2] of v_i^dag t, i < nvec; npart != nullptr: the
// last workgroups (in z) form the partials [nrhs][nchunk] of |t|^2 instead.
// Bound by the basis' traffic: the loads of an element's eight vectors issue
// together, past the last vector from the last one (each under a branch of its own
// and with the sums by thread 0: 19.2 us for 100 vectors of 8^4, now 15.0, 5.3 TB/s).
template <typename T2>
__global__ void __launch_bounds__(256) k_block_dots(const T2* __restrict__ basis, long basis_stride,
                                                    const T2* __restrict__ T, long N, int nvec,
                                                    int nchunk, double* __restrict__ partials,
                                                    double* __restrict__ npart) {
  __shared__ double lds[4 * 2 * kArnVec];
  const int r = blockIdx.y;
  const int i0 = blockIdx.z * kArnVec;
  if (i0 >= nvec) {
    norm2_part(T + (long)r * N, N, blockIdx.x, nchunk, npart + (long)r * nchunk);
    return;
  }
  const int ni = min(kArnVec, nvec - i0);
  double v[2 * kArnVec];
#pragma unroll
  for (int q = 0; q < 2 * kArnVec; ++q) v[q] = 0.0;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x) {
    T2 b[kArnVec];
    const T2* bv = basis + i0 * basis_stride + (long)r * N + e;
#pragma unroll
    for (int q = 0; q < kArnVec; ++q) b[q] = bv[min(q, ni - 1) * basis_stride];
    const Cx<double> t = ld64(T + (long)r * N + e);
#pragma unroll
    for (int q = 0; q < kArnVec; ++q) {
      const Cx<double> p = cmulc(ld64(&b[q]), t);
      v[2 * q] += p.re;
      v[2 * q + 1] += p.im;
    }
  }
  const double a = block_sums(v, lds);
  const int q = threadIdx.x;
  if (q < 2 * ni)
    partials[(((long)r * nvec + i0 + (q >> 1)) * nchunk + blockIdx.x) * 2 + (q & 1)] = a;
}

// h_i from its nparts partials (workgroup i of source r): H[r][j][i] += h_i
// (column-major: column j of H_r), hcur[r][i] = h_i
__global__ void __launch_bounds__(256) k_arn_accum(const double* __restrict__ partials, int nparts,
                                                   int kmax, int j, int first,
                                                   double2* __restrict__ H,
                                                   double2* __restrict__ hcur) {
  __shared__ double lds[4 * 2];
  const int i = blockIdx.x, r = blockIdx.y;
  const double* p = partials + ((long)r * gridDim.x + i) * nparts * 2;
  double v[2] = {0.0, 0.0};
  for (int q = threadIdx.x; q < nparts; q += blockDim.x) {
    v[0] += p[2 * q];
    v[1] += p[2 * q + 1];
  }
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) {
    const Cx<double> h = {v[0], v[1]};
    double2* hij = H + ((long)r * kmax + j) * kmax + i;
    *hij = first ? d2(h) : d2(c64(*hij) + h);
    hcur[(long)r * kmax + i] = d2(h);
  }
}

// T -= sum_i hcur_i V_i ; partials of |T|^2 [nrhs][nchunk] (if given).  A small
// lattice gives one workgroup per CU at most, so bound by latency unless enough
// loads are in flight: two groups of 16 vectors take turns, one loading while the
// other is subtracted, and the coefficients come from LDS (8^4, 100 vectors: 20.4 us with
// scalar loads of them, now 15.7, 5.1 TB/s; a plain read 11.8).  One term after the other.
constexpr int kArnAhead = 16;
template <typename T2>
__global__ void __launch_bounds__(256) k_block_axpy(const T2* __restrict__ basis, long basis_stride,
                                                    T2* __restrict__ T, long N, int nvec,
                                                    const double2* __restrict__ hcur, int kmax,
                                                    double* __restrict__ partials) {
  __shared__ double lds[4];
  __shared__ double2 h[kHessMaxK];
  const int r = blockIdx.y;
  double v[1] = {0.0};
  T2 qa[kArnAhead], qb[kArnAhead];
  auto load = [&](T2 (&q)[kArnAhead], long e, int i) {
    if (i >= nvec) return;
    const T2* br = basis + (long)r * N + e;
#pragma unroll
    for (int u = 0; u < kArnAhead; ++u) q[u] = br[(long)min(i + u, nvec - 1) * basis_stride];
  };
  const long e0 = blockIdx.x * (long)blockDim.x + threadIdx.x;
  load(qa, min(e0, N - 1), 0);
  for (int i = threadIdx.x; i < nvec; i += blockDim.x) h[i] = hcur[(long)r * kmax + i];
  __syncthreads();
  for (long e = e0; e < N; e += (long)gridDim.x * blockDim.x) {
    if (e != e0) load(qa, e, 0);
    Cx<double> t = ld64(T + (long)r * N + e);
    auto subtract = [&](const T2 (&q)[kArnAhead], int i) {
      if (i + kArnAhead <= nvec) {
#pragma unroll
        for (int u = 0; u < kArnAhead; ++u) t = t - cmul(c64(h[i + u]), ld64(&q[u]));
      } else {
#pragma unroll
        for (int u = 0; u < kArnAhead; ++u)
          if (i + u < nvec) t = t - cmul(c64(h[i + u]), ld64(&q[u]));
      }
    };
    for (int i = 0; i < nvec; i += 2 * kArnAhead) {
      load(qb, e, i + kArnAhead);
      subtract(qa, i);
      load(qa, e, i + 2 * kArnAhead);
      subtract(qb, i + kArnAhead);
    }
    st64(T + (long)r * N + e, t);
    v[0] += cnorm2(round_to(T, t));
  }
  if (!partials) return;
  block_sum<1>(v, lds);
  if (threadIdx.x == 0) partials[(long)r * gridDim.x + blockIdx.x] = v[0];
}

// partials of |T|^2 [nrhs][nchunk]
template <typename T2>
__global__ void __launch_bounds__(256) k_norm2(const T2* __restrict__ T, long N,
                                               double* __restrict__ partials) {
  const int r = blockIdx.y;
  norm2_part(T + (long)r * N, N, blockIdx.x, gridDim.x, partials + (long)r * gridDim.x);
}

// V_{j+1} = T / h, h = |T| from the subtraction's partials (every workgroup sums
// them; the first of a source writes H[j+1][j] = h); zero after the lucky
// breakdown h <= 1e-14 |A v_j| (its norm from the dots' partials), which stops the
// source at k = j+1.  Workgroups that read the status of this step or of the one
// before take the same branch.
template <typename T2>
__global__ void __launch_bounds__(256) k_arn_next(const T2* __restrict__ T, T2* __restrict__ out,
                                                  long N, const double* __restrict__ npart,
                                                  const double* __restrict__ tnpart, int nparts,
                                                  double2* __restrict__ H, int kmax, int j,
                                                  int* __restrict__ kstop,
                                                  int* __restrict__ status) {
  __shared__ double lds[4 * 2];
  __shared__ double scl;
  const int r = blockIdx.y;
  double v[2] = {0.0, 0.0};
  for (int q = threadIdx.x; q < nparts; q += blockDim.x) {
    v[0] += npart[(long)r * nparts + q];
    v[1] += tnpart[(long)r * nparts + q];
  }
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) {
    const double h = sqrt(v[0]), tn = sqrt(v[1]);
    const bool stopped = status[r] != 0;
    const bool ok = !stopped && h > 1e-14 * tn;
    scl = ok ? 1.0 / h : 0.0;
    if (blockIdx.x == 0) {
      H[((long)r * kmax + j) * kmax + (j + 1)] = make_double2(ok ? h : 0.0, 0.0);
      if (!stopped && !ok) {
        status[r] = 1;
        kstop[r] = j + 1;
      }
    }
  }
  __syncthreads();
  const double s = scl;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < N; e += (long)gridDim.x * blockDim.x)
    st64(out + (long)r * N + e, scale(s, ld64(T + (long)r * N + e)));
}

// ===========================================================================
// Inner sign: x = sgn(T) e_1 for a small non-Hermitian T with no eigenvalue
// on the imaginary axis, from sgn(z) = (1/pi) int_0^inf [1/(z+i tau) +
// 1/(z-i tau)] d tau, tau = e^u, trapezoidal rule in u:
//   x ~= (h/pi) sum_n e^{u_n} [ (T + i e^{u_n})^{-1} e_1 + (T - i e^{u_n})^{-1} e_1 ].
// The nodes with even n form the rule with step 2h; their difference gives
// the error estimate.
// ===========================================================================

// One thread per (source r, shifted solve q): q = 2*node + (0: +tau, 1: -tau).
// Tridiagonal T_r = tridiag(beta, alpha, gamma) of size k_r, with the rules of
// source r (task[r]: one or two steps, each source its own): the waves of the
// first rule, then those of the second.  Wave results are reduced over lanes:
// part[r][wave][2][kmax] complex (fine rule, coarse rule), wave = wave0 +
// blockIdx.x of nwave in all; waves beyond a source's nodes write nothing.  A
// launch covers one chunk of waves; the minors of a chunk live in minor
// [r][blockIdx.x][kmax][64] and their exponents in expo, which the next chunk
// (ordered on the stream) reuses.
//
// (T + i sigma) y = e_1 by the trailing principal minors theta_j of T + i sigma
// (rows and columns j to k-1; Usmani, Linear Algebra Appl. 212/213 (1994) 413):
//   theta_j = a_j theta_{j+1} - gamma_j beta_j theta_{j+2},  theta_k = 1,
//   y_j = (-1)^j beta_0 ... beta_{j-1} theta_{j+1} / theta_0.
// A computed theta_j is the exact combination of the two before it for entries
// changed by a few rounding errors each, and every a_j and gamma_j beta_j enters
// one of them only: the computed minors are those of a matrix equal to T + i sigma
// to rounding, entry by entry, also through zero or tiny minors, so no pivoting;
// y_j adds one relative rounding error per factor.  The pair of minors is scaled
// by a power of two every kMinors steps (exact), expo holding the exponents.
//
// Bound by the latency and issue of one wave's serial chain, whatever the number
// of waves: a step is two dependent fused multiply-adds, with the coefficients of
// 64 steps in the lanes of the wave, loaded a block ahead and read by readlane.
// The rows have no chain; their minors load a block of 16 ahead.  One source, k =
// 375 on average (the checks of an 8^4 solve): 149 us a launch by elimination
// with column pivoting (two dependent quotients a step), 65 us so; against 113-bit
// arithmetic both are within 3e-15 for Lanczos matrices of 4^4 and 6^4 (k to 600).
constexpr int kMinors = 8;
__global__ void __launch_bounds__(64) k_isign_tri(const double2* __restrict__ alpha,
                                                  const double* __restrict__ beta,
                                                  const double2* __restrict__ gamma, int kmax,
                                                  const IsignTask* __restrict__ task,
                                                  const int* __restrict__ kstop,
                                                  int wave0, int nwave,
                                                  double2* __restrict__ minor,
                                                  int* __restrict__ expo,
                                                  double2* __restrict__ part) {
  const int r = blockIdx.y;
  const IsignTask tk = task[r];
  const int wave = wave0 + blockIdx.x;
  const int lane = threadIdx.x;
  const int k = kstop ? min(tk.k, kstop[r]) : tk.k;
  const int nw0 = (2 * tk.rule[0].nnode + 63) / 64;
  const QuadNodes qn = wave < nw0 ? tk.rule[0] : tk.rule[1];
  const int first = (wave < nw0 ? wave : wave - nw0) * 64;
  const int nq = 2 * qn.nnode;
  if (k <= 0 || first >= nq) return;  // uniform over the wave
  const int q = first + lane;
  const bool live = q < nq;
  const int node = qn.n0 + (live ? q / 2 : 0);
  const double tau = exp(node * qn.h);
  const double sig = live ? ((q & 1) ? -tau : tau) : 1.0;
  const double wfine = live ? qn.h / M_PI * tau : 0.0;
  const double2* al = alpha + (long)r * kmax;
  const double* be = beta + (long)r * kmax;
  const double2* ga = gamma + (long)r * kmax;
  const long wbase = (long)(r * gridDim.x + blockIdx.x);
  double2* th = minor + wbase * kmax * 64 + lane;             // theta_j at [j * 64]
  int* ex = expo + wbase * isign_expo_words(kmax) * 64 + lane;  // by (k - 1 - j) / kMinors
  double2* part_r = part + ((long)r * nwave + wave) * 2 * kmax;
  // lane l of a block starting at row j0 holds the entries of row j0 - l (below
  // row 0: clamped loads, never used): a_j without the shift and gamma_j beta_j
  struct Block {
    double2 a, g;
    double b;
  };
  auto load_block = [&](int j0) {
    const int j = max(j0 - lane, 0);
    Block o;
    o.a = al[j];
    o.b = be[j];
    o.g = ga[j];
    if (j >= k - 1) {  // theta_{k+1} = 0; the last row's couplings may be unset
      o.g = make_double2(0.0, 0.0);
      o.b = 0.0;
    }
    return o;
  };
  Cx<double> t1 = {1.0, 0.0}, t2 = {0.0, 0.0};  // theta_{j+1}, theta_{j+2} times 2^-e
  int e = 0;
  Block nxt = load_block(k - 1);
  for (int j0 = k - 1; j0 >= 0; j0 -= 64) {
    const Block cur = nxt;
    nxt = load_block(j0 - 64);
    const double cre = cur.b * cur.g.x, cim = cur.b * cur.g.y;
    const int n = min(64, j0 + 1);
    auto step = [&](int l) {
      const double are = lane_value(cur.a.x, l), aim = lane_value(cur.a.y, l) + sig;
      const double gr = lane_value(cre, l), gi = lane_value(cim, l);
      const double ur = fma(gi, t2.im, -(gr * t2.re)), ui = -fma(gr, t2.im, gi * t2.re);
      const Cx<double> t0 = {fma(are, t1.re, fma(-aim, t1.im, ur)),
                             fma(are, t1.im, fma(aim, t1.re, ui))};
      th[(long)(j0 - l) * 64] = d2(t0);
      t2 = t1;
      t1 = t0;
    };
    for (int l0 = 0; l0 < n; l0 += kMinors) {
      if (l0 + kMinors <= n) {
#pragma unroll
        for (int l = 0; l < kMinors; ++l) step(l0 + l);
      } else {
        for (int l = l0; l < n; ++l) step(l);
      }
      ex[(long)((k - 1 - j0 + l0) / kMinors) * 64] = e;
      const double top = fmax(fmax(fabs(t1.re), fabs(t1.im)), fmax(fabs(t2.re), fabs(t2.im)));
      const int s = __builtin_amdgcn_frexp_exp(top);
      t1 = {__builtin_amdgcn_ldexp(t1.re, -s), __builtin_amdgcn_ldexp(t1.im, -s)};
      t2 = {__builtin_amdgcn_ldexp(t2.re, -s), __builtin_amdgcn_ldexp(t2.im, -s)};
      e += s;
    }
  }
  const Cx<double> inv = scale(wfine, cdiv(Cx<double>{1.0, 0.0}, t1));  // weight / theta_0
  const int e0 = e;
  // The weighted rows of the 64 lanes are buffered in LDS for two groups of minors
  // at a time and summed over the lanes of even nodes and of odd nodes (the coarse
  // rule takes the even ones at twice the weight), in a fixed order, one (row,
  // part, parity) per lane.  Row j takes theta_{j+1}: the blocks start ahead of
  // row 0 where that aligns them with the groups.
  constexpr int kRows = 2 * kMinors;
  static_assert(kRows == 16);
  __shared__ double rows[kRows][2][65];  // [row][re, im][lane]
  // a block's minors and the exponents of its groups, loaded together and one
  // block ahead of their use (clamped outside the matrix)
  double2 mb[kRows], mn[kRows];
  int sb[2], sn[2];
  double bb, bn;  // lane t: beta_{j-1} of row j = j0 + t
  auto load_rows = [&](int j0) {
#pragma unroll
    for (int t = 0; t < kRows; ++t) mn[t] = th[(long)min(max(j0 + t + 1, 0), k - 1) * 64];
#pragma unroll
    for (int u = 0; u < 2; ++u) sn[u] = ex[(long)(max(k - 2 - j0 - u * kMinors, 0) / kMinors) * 64];
    const int jb = j0 + (lane & (kRows - 1)) - 1;
    bn = be[min(max(jb, 0), k - 1)];
    if (jb < 0) bn = -1.0;
  };
  const int parity = qn.n0 & 1;
  double bm = 1.0;  // (-1)^j beta_0 ... beta_{j-1} = bm 2^bx
  int bx = 0;
  const int start = -((kMinors + 1 - k % kMinors) % kMinors);  // (k - 2 - start) % kMinors == kMinors - 1
  load_rows(start);
  for (int j0 = start; j0 < k; j0 += kRows) {
#pragma unroll
    for (int t = 0; t < kRows; ++t) mb[t] = mn[t];
    sb[0] = sn[0];
    sb[1] = sn[1];
    bb = bn;
    if (j0 + kRows < k) load_rows(j0 + kRows);
    // rows before 0 and from k on are formed from clamped entries and not read
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int s = __builtin_amdgcn_frexp_exp(bm);
      bm = __builtin_amdgcn_ldexp(bm, -s);
      bx += s;
      const bool end = j0 + u * kMinors >= k - 1;  // row k - 1: theta_k = 1
      const int eg = bx + (end ? 0 : sb[u]) - e0;
      const Cx<double> ig = {__builtin_amdgcn_ldexp(inv.re, eg), __builtin_amdgcn_ldexp(inv.im, eg)};
      if (end) mb[u * kMinors] = make_double2(1.0, 0.0);
#pragma unroll
      for (int v = 0; v < kMinors; ++v) {
        const int t = u * kMinors + v;
        bm = -(bm * lane_value(bb, t));
        const Cx<double> y = cmul(c64(mb[t]), ig);
        rows[t][0][lane] = bm * y.re;
        rows[t][1][lane] = bm * y.im;
      }
    }
    __syncthreads();
    {
      const int t = lane & (kRows - 1), c = (lane >> 4) & 1, odd = lane >> 5;
      const double* row = rows[t][c] + 2 * (odd ^ parity);
      double acc = 0.0;
#pragma unroll
      for (int l = 0; l < 64; l += 4) {
        acc += row[l];
        acc += row[l + 1];
      }
      const double other = __shfl_xor(acc, 32);
      const int j = j0 + t;
      if (j >= 0 && j < k) {
        double* out = reinterpret_cast<double*>(part_r + (odd ? kmax : 0) + j);
        out[c] = odd ? 2.0 * other : acc + other;
      }
    }
    __syncthreads();
  }
}

// For each source with a task (k > 0): x[r][j] = sum over the first rule's waves
// (fixed order) and its error |x_fine - x_coarse| / |x_fine|; if that misses the
// target and the step is not the finest allowed, the same with the second rule.
// The result says which rule was accepted (-1: none, x is then not final), its
// error, and the source's k, kstop and status.  A source without a task keeps
// its row, or gets a zero row in the first round.  kout (optional): k of each
// source in the first round.
// One workgroup per source, bound by memory latency: the loads of eight waves
// are issued before their additions, 1024 rows at a time (22 waves, k = 375:
// 21 us one load at a time and 256 rows).  The error sums keep the order of
// 256 threads striding over the rows.
__global__ void __launch_bounds__(1024) k_isign_final(const double2* __restrict__ part, int nwave,
                                                      int kmax, const IsignTask* __restrict__ task,
                                                      const int* __restrict__ kstop,
                                                      const int* __restrict__ status, int first,
                                                      double2* __restrict__ x,
                                                      int* __restrict__ kout,
                                                      IsignResult* __restrict__ res) {
  __shared__ double lds[4 * 2];
  __shared__ double sq[2][1024];
  __shared__ double err_s;
  const int r = blockIdx.x;
  const int tid = threadIdx.x;
  const IsignTask tk = task[r];
  const int ks = kstop ? kstop[r] : tk.k;
  const int k = min(tk.k, ks);
  double2* xr = x + (long)r * kmax;
  if (tid == 0 && kout && first) kout[r] = max(k, 0);
  if (k <= 0) {  // uniform over the workgroup
    if (first)
      for (int j = tid; j < kmax; j += 1024) xr[j] = make_double2(0.0, 0.0);
    if (tid == 0) res[r] = IsignResult{0.0, 0, 0, ks, status ? status[r] : 0};
    return;
  }
  const int nw0 = (2 * tk.rule[0].nnode + 63) / 64, nw1 = (2 * tk.rule[1].nnode + 63) / 64;
  int level = -1;
  double err = 0.0;
  for (int lev = 0; lev < 2 && level < 0; ++lev) {
    const int nw = lev ? nw1 : nw0;
    if (nw == 0) break;
    double v[2] = {0, 0};
    for (int j0 = 0; j0 < kmax; j0 += 1024) {
      const int j = j0 + tid;
      if (j < kmax) {
        Cx<double> f = {0, 0}, c = {0, 0};
        if (j < k) {
          const double2* p = part + ((long)r * nwave + (lev ? nw0 : 0)) * 2 * kmax + j;
          int w = 0;
          for (; w + 8 <= nw; w += 8) {
            double2 a[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              a[u] = p[(long)(w + u) * 2 * kmax];
              b[u] = p[(long)(w + u) * 2 * kmax + kmax];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              f = f + c64(a[u]);
              c = c + c64(b[u]);
            }
          }
          for (; w < nw; ++w) {
            f = f + c64(p[(long)w * 2 * kmax]);
            c = c + c64(p[(long)w * 2 * kmax + kmax]);
          }
        }
        xr[j] = d2(f);
        sq[0][tid] = cnorm2(f - c);
        sq[1][tid] = cnorm2(f);
      }
      __syncthreads();
      if (tid < 256)
        for (int t = tid; t < 1024 && j0 + t < kmax; t += 256) {
          v[0] += sq[0][t];
          v[1] += sq[1][t];
        }
      __syncthreads();
    }
    block_sum<2>(v, lds, 4);
    if (tid == 0) err_s = v[1] > 0 ? sqrt(v[0] / v[1]) : 0.0;
    __syncthreads();
    err = err_s;
    // NaN stays unaccepted until the finest step
    if (err <= tk.target || tk.rule[lev].h <= tk.hmin) level = lev;
    __syncthreads();
  }
  if (tid == 0) res[r] = IsignResult{err, level, k, ks, status ? status[r] : 0};
}

// Hessenberg variant: one workgroup per (source r, shifted solve q), q = q0 +
// blockIdx.x for a chunk of gridDim.x solves.  The current column lives in
// LDS; H is column-major [r][kmax][kmax].
// Output ys[r][blockIdx.x][kmax] = (H + i sigma)^{-1} e_1 (unweighted).
constexpr int kHessMax = 1536;

__global__ void __launch_bounds__(256) k_isign_hess(const double2* __restrict__ H, int kmax,
                                                    const int* __restrict__ kvec, QuadNodes qn,
                                                    int q0, double2* __restrict__ ys) {
  __shared__ double2 c[kHessMax];
  __shared__ double2 mlt[kHessMax];
  __shared__ unsigned char swv[kHessMax];
  __shared__ double2 bc_m;
  __shared__ int bc_sw;
  const int q = q0 + blockIdx.x;
  const int r = blockIdx.y;
  const int k = kvec[r];
  const int node = qn.n0 + q / 2;
  const double tau = exp(node * qn.h);
  const double sig = (q & 1) ? -tau : tau;
  const double2* Hr = H + (long)r * kmax * kmax;
  double2* y = ys + ((long)r * gridDim.x + blockIdx.x) * kmax;
  if (k <= 0) return;
  // current column k-1 (rows 0..k-1)
  for (int i = threadIdx.x; i < k; i += blockDim.x) {
    Cx<double> v = c64(Hr[(long)(k - 1) * kmax + i]);
    if (i == k - 1) v.im += sig;
    c[i] = d2(v);
  }
  __syncthreads();
  for (int j = k - 1; j >= 1; --j) {
    const double2* dcol = Hr + (long)(j - 1) * kmax;
    if (threadIdx.x == 0) {
      const Cx<double> cd = c64(c[j]);
      const Cx<double> dd = c64(dcol[j]);  // subdiagonal entry H[j][j-1]
      const bool sw = cabs1(dd) > cabs1(cd);
      const Cx<double> m = sw ? cdiv(cd, dd) : cdiv(dd, cd);
      bc_m = d2(m);
      bc_sw = sw;
      mlt[j] = d2(m);
      swv[j] = sw;
    }
    __syncthreads();
    const Cx<double> m = c64(bc_m);
    const bool sw = bc_sw;
    for (int i = threadIdx.x; i < j; i += blockDim.x) {
      Cx<double> d = c64(dcol[i]);
      if (i == j - 1) d.im += sig;
      const Cx<double> ci = c64(c[i]);
      c[i] = d2(sw ? ci - cmul(m, d) : d - cmul(m, ci));
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    Cx<double> cur = cdiv(Cx<double>{1.0, 0.0}, c64(c[0]));
    for (int j = 1; j < k; ++j) {
      const Cx<double> nw = -cmul(c64(mlt[j]), cur);
      if (swv[j]) {
        y[j - 1] = d2(nw);
      } else {
        y[j - 1] = d2(cur);
        cur = nw;
      }
    }
    y[k - 1] = d2(cur);
  }
}

// acc[r][0][j] += sum over the chunk's solves of w_q ys (fine rule),
// acc[r][1][j] the same over the coarse rule's nodes; solves in order, so the
// sums are the same for every run.  first: the chunk starts the sums.
__global__ void __launch_bounds__(256) k_isign_hess_accum(const double2* __restrict__ ys, int q0,
                                                          int nq_chunk, int kmax,
                                                          const int* __restrict__ kvec,
                                                          QuadNodes qn, int first,
                                                          double2* __restrict__ acc) {
  const int r = blockIdx.y;
  const int k = kvec[r];
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= kmax) return;
  double2* a = acc + (long)r * 2 * kmax;
  Cx<double> f = first ? Cx<double>{0, 0} : c64(a[j]);
  Cx<double> c = first ? Cx<double>{0, 0} : c64(a[kmax + j]);
  if (j < k) {
    for (int qq = 0; qq < nq_chunk; ++qq) {
      const int node = qn.n0 + (q0 + qq) / 2;
      const double tau = exp(node * qn.h);
      const Cx<double> yv = c64(ys[((long)r * nq_chunk + qq) * kmax + j]);
      f = f + scale(qn.h / M_PI * tau, yv);
      if ((node & 1) == 0) c = c + scale(2.0 * qn.h / M_PI * tau, yv);
    }
  }
  a[j] = d2(f);
  a[kmax + j] = d2(c);
}

// x[r] = fine sums; err[r] = |x_fine - x_coarse| / |x_fine|
__global__ void __launch_bounds__(256) k_isign_hess_final(const double2* __restrict__ acc, int kmax,
                                                          const int* __restrict__ kvec,
                                                          double2* __restrict__ x,
                                                          double* __restrict__ err) {
  __shared__ double lds[4 * 2];
  const int r = blockIdx.x;
  const int k = kvec[r];
  double v[2] = {0, 0};
  for (int j = threadIdx.x; j < kmax; j += blockDim.x) {
    Cx<double> f = {0, 0}, c = {0, 0};
    if (j < k) {
      f = c64(acc[(long)r * 2 * kmax + j]);
      c = c64(acc[(long)r * 2 * kmax + kmax + j]);
    }
    x[(long)r * kmax + j] = d2(f);
    v[0] += cnorm2(f - c);
    v[1] += cnorm2(f);
  }
  block_sum<2>(v, lds);
  if (threadIdx.x == 0) err[r] = v[1] > 0 ? sqrt(v[0] / v[1]) : 0.0;
}

// ===========================================================================
// Host-side launchers
// ===========================================================================

static int chunks_for(long N, int cap = 1024) {
  long b = (N + 255) / 256;
  if (b > cap) b = cap;
  if (b < 1) b = 1;
  return (int)b;
}

// chunks of the deflation dots: at least 16 entries per thread, so that the
// per-workgroup reduction of 4 kDeflRhs values does not dominate (one entry
// per thread made the dots latency-bound: 107 us for m = 30 at 8^4)
int defl_nchunk(long N) {
  long c = (N + 256L * 16 - 1) / (256L * 16);
  if (c > 512) c = 512;
  if (c < 1) c = 1;
  return (int)c;
}

void launch_defl(const double2* R, const double2* L, const double2* B, const double* sgn, int m,
                 int nrhs, long N, double* partials, double* CD, double2* bR, double2* bL,
                 double2* yex, hipStream_t s) {
  const int nch = defl_nchunk(N);
  hipLaunchKernelGGL(k_defl_dots, dim3(nch, m, cdiv_i(nrhs, kDeflRhs)), dim3(256), 0, s, R, L, B,
                     nrhs, N, nch, partials);
  hipLaunchKernelGGL(k_reduce_partials<4>, dim3(m * nrhs), dim3(256), 0, s, partials, nch, CD);
  hipLaunchKernelGGL(k_defl_axpy, dim3(chunks_for(N, 4096), nrhs), dim3(256), 0, s, R, L, B, CD,
                     sgn, m, nrhs, N, bR, bL, yex);
}

void launch_defl_proj(const double2* R, const double2* L, const double2* X, int m, int nrhs, long N,
                      double* partials, double* CD, const double2* kappa, double2* outQ,
                      double2* outQd, hipStream_t s) {
  const int nch = defl_nchunk(N);
  hipLaunchKernelGGL(k_defl_dots, dim3(nch, m, cdiv_i(nrhs, kDeflRhs)), dim3(256), 0, s, R, L, X,
                     nrhs, N, nch, partials);
  hipLaunchKernelGGL(k_reduce_partials<4>, dim3(m * nrhs), dim3(256), 0, s, partials, nch, CD);
  if (kappa)
    hipLaunchKernelGGL(k_cd_shift, dim3(cdiv_i(m * nrhs, 256)), dim3(256), 0, s, CD, kappa, m, nrhs);
  hipLaunchKernelGGL(k_defl_axpy, dim3(chunks_for(N, 4096), nrhs), dim3(256), 0, s, R, L, X, CD,
                     (const double*)nullptr, m, nrhs, N, outQ, outQd, (double2*)nullptr);
}

void launch_defl_cd(const double2* R, const double2* L, const double2* B, int m, int nrhs, long N,
                    double* partials, double* CD, hipStream_t s) {
  const int nch = defl_nchunk(N);
  hipLaunchKernelGGL(k_defl_dots, dim3(nch, m, cdiv_i(nrhs, kDeflRhs)), dim3(256), 0, s, R, L, B,
                     nrhs, N, nch, partials);
  hipLaunchKernelGGL(k_reduce_partials<4>, dim3(m * nrhs), dim3(256), 0, s, partials, nch, CD);
}

void launch_start(const double2* bR, const double2* bL, int nrhs, long N, double* partials,
                  double* sums, void* V0, void* W0, bool f32, hipStream_t s) {
  const int nch = chunks_for(N, 512);
  hipLaunchKernelGGL(k_start_dots, dim3(nch, nrhs), dim3(256), 0, s, bR, bL, N, nch, partials);
  hipLaunchKernelGGL(k_reduce_partials<3>, dim3(nrhs), dim3(256), 0, s, partials, nch, sums);
  if (!V0 && !W0) return;  // norms only
  if (f32)
    hipLaunchKernelGGL(k_start_vectors<float2>, dim3(chunks_for(N, 4096), nrhs), dim3(256), 0, s,
                       bR, bL, sums, N, (float2*)V0, (float2*)W0);
  else
    hipLaunchKernelGGL(k_start_vectors<double2>, dim3(chunks_for(N, 4096), nrhs), dim3(256), 0, s,
                       bR, bL, sums, N, (double2*)V0, (double2*)W0);
}

// 256 workgroups per source: each reduces the dual stencil's partials for alpha
// first, so fewer and longer-running workgroups keep that head cheap.
int update_nwg(long N) { return chunks_for(N, 256); }

void launch_alpha(const double* partials, int nparts, bool quad, const CoefArrays& co, const int* it,
                  int off, const int* rhs_map, const int* n_active, int nslots, hipStream_t s) {
  hipLaunchKernelGGL(k_alpha, dim3(nslots), dim3(256), 0, s, partials, nparts, (int)quad, co, it,
                     off, rhs_map, n_active);
}

void launch_update(bool f32, const void* T, const void* S, void* basis, long basis_stride,
                   void* wbuf, long N, const CoefArrays& co, const int* it, int off,
                   const int* rhs_map, const int* n_active, int nslots, double* partials, bool ring,
                   const double* apart, int anparts, bool quad, int nt, hipStream_t s) {
  dim3 grid(update_nwg(N), nslots);
  if (f32)
    hipLaunchKernelGGL(k_update<float2>, grid, dim3(256), 0, s, (const float2*)T, (const float2*)S,
                       (float2*)basis, basis_stride, (float2*)wbuf, N, N, co, it, off, rhs_map, n_active,
                       partials, (int)ring, apart, anparts, (int)quad, nt);
  else
    hipLaunchKernelGGL(k_update<double2>, grid, dim3(256), 0, s, (const double2*)T,
                       (const double2*)S, (double2*)basis, basis_stride, (double2*)wbuf, N, N, co,
                       it, off, rhs_map, n_active, partials, (int)ring, apart, anparts, (int)quad, nt);
}

void launch_beta_tail(bool f32, const double* partials, int nparts, const CoefArrays& co, int* it,
                      int adv, const int* rhs_map, const int* n_active, int nslots, int* ticket,
                      const void* basis, long basis_stride, long N, bool ring, const int* idx,
                      int P, double2* probes, hipStream_t s) {
  if (f32)
    hipLaunchKernelGGL(k_beta_tail<float2>, dim3(nslots), dim3(256), 0, s, partials, nparts, co, it,
                       adv, rhs_map, n_active, ticket, (const float2*)basis, basis_stride, N, (int)ring,
                       idx, P, probes);
  else
    hipLaunchKernelGGL(k_beta_tail<double2>, dim3(nslots), dim3(256), 0, s, partials, nparts, co, it,
                       adv, rhs_map, n_active, ticket, (const double2*)basis, basis_stride, N, (int)ring,
                       idx, P, probes);
}

void launch_probe_gather(bool f32, const void* basis, long basis_stride, long N, bool ring,
                         const int* it, bool first, const int* idx, int P, int kmax,
                         const int* rhs_map, const int* n_active, int nslots, double2* probes,
                         hipStream_t s) {
  dim3 grid(cdiv_i(P, 256), nslots);
  if (f32)
    hipLaunchKernelGGL(k_probe_gather<float2>, grid, dim3(256), 0, s, (const float2*)basis,
                       basis_stride, N, (int)ring, it, (int)first, idx, P, kmax, rhs_map, n_active,
                       probes);
  else
    hipLaunchKernelGGL(k_probe_gather<double2>, grid, dim3(256), 0, s, (const double2*)basis,
                       basis_stride, N, (int)ring, it, (int)first, idx, P, kmax, rhs_map, n_active,
                       probes);
}

void launch_probe_y(const double2* probes, const double2* x, const double* sv, const double* nb,
                    const int* kvec, int kmax, const double2* yex, long N, const int* idx, int P,
                    double2* yp, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL(k_probe_y, dim3(cdiv_i(P, 64), nrhs), dim3(64), 0, s, probes, x, sv, nb, kvec,
                     kmax, yex, N, idx, P, yp);
}

void launch_advance(int* it, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(1), 0, s, it);
}

void launch_make_coef(const double2* x, const double* sv, const double* nb, int kmax, int nrhs,
                      double2* coef, hipStream_t s) {
  long n = (long)nrhs * kmax;
  hipLaunchKernelGGL(k_make_coef, dim3(cdiv_i(n, 256)), dim3(256), 0, s, x, sv, nb, kmax, nrhs, coef);
}

void launch_combine(bool f32, const void* basis, long basis_stride, long N, const double2* coef,
                    int kmax, const int* kused, const double2* yex, double2* y, int nrhs,
                    hipStream_t s) {
  dim3 grid(chunks_for(N, 4096), nrhs);
  if (f32)
    hipLaunchKernelGGL(k_combine<float2>, grid, dim3(256), 0, s, (const float2*)basis, basis_stride,
                       N, coef, kmax, kused, yex, y);
  else
    hipLaunchKernelGGL(k_combine<double2>, grid, dim3(256), 0, s, (const double2*)basis,
                       basis_stride, N, coef, kmax, kused, yex, y);
}

void launch_replay(bool f32, const void* T, void* ring, long ring_stride, long N,
                   const CoefArrays& co, int i, const double2* coef, const int* kused, double2* y,
                   int nrhs, hipStream_t s) {
  dim3 grid(chunks_for(N, 4096), nrhs);
  if (f32)
    hipLaunchKernelGGL(k_replay<float2>, grid, dim3(256), 0, s, (const float2*)T, (float2*)ring,
                       ring_stride, N, co, i, coef, kused, y);
  else
    hipLaunchKernelGGL(k_replay<double2>, grid, dim3(256), 0, s, (const double2*)T, (double2*)ring,
                       ring_stride, N, co, i, coef, kused, y);
}

void launch_overlap(const double2* b, double2* y, long N, int V, hipStream_t s) {
  hipLaunchKernelGGL(k_overlap, dim3(chunks_for(N, 8192)), dim3(256), 0, s, b, y, N, V);
}

int arn_nchunk(long N) { return chunks_for(N, 256); }

void launch_arn_dots(bool f32, const void* basis, long basis_stride, const void* T, long N,
                     int nvec, int nrhs, double* partials, double* npart, hipStream_t s) {
  const int nch = arn_nchunk(N);
  dim3 grid(nch, nrhs, cdiv_i(nvec, kArnVec) + (npart ? 1 : 0));
  if (f32)
    hipLaunchKernelGGL(k_block_dots<float2>, grid, dim3(256), 0, s, (const float2*)basis,
                       basis_stride, (const float2*)T, N, nvec, nch, partials, npart);
  else
    hipLaunchKernelGGL(k_block_dots<double2>, grid, dim3(256), 0, s, (const double2*)basis,
                       basis_stride, (const double2*)T, N, nvec, nch, partials, npart);
}

void launch_block_dots(bool f32, const void* basis, long basis_stride, const void* T, long N,
                       int nvec, int nrhs, double* partials, double* red, hipStream_t s) {
  launch_arn_dots(f32, basis, basis_stride, T, N, nvec, nrhs, partials, nullptr, s);
  hipLaunchKernelGGL(k_reduce_partials<2>, dim3(nrhs * nvec), dim3(256), 0, s, partials,
                     arn_nchunk(N), red);
}

void launch_gram(const double2* X, int nx, const double2* Y, int ny, long N, double* partials,
                 double2* G, hipStream_t s) {
  for (int j = 0; j < ny; ++j)
    launch_block_dots(false, X, N, Y + (long)j * N, N, nx, 1, partials, (double*)(G + (long)j * nx), s);
}

void launch_arn_accum(const double* partials, long N, int nvec, int kmax, int j, bool first,
                      double2* H, double2* hcur, int nrhs, hipStream_t s) {
  hipLaunchKernelGGL(k_arn_accum, dim3(nvec, nrhs), dim3(256), 0, s, partials, arn_nchunk(N), kmax,
                     j, (int)first, H, hcur);
}

void launch_arn_axpy(bool f32, const void* basis, long basis_stride, void* T, long N, int nvec,
                     const double2* hcur, int kmax, int nrhs, double* npart, hipStream_t s) {
  dim3 grid(arn_nchunk(N), nrhs);
  if (f32)
    hipLaunchKernelGGL(k_block_axpy<float2>, grid, dim3(256), 0, s, (const float2*)basis,
                       basis_stride, (float2*)T, N, nvec, hcur, kmax, npart);
  else
    hipLaunchKernelGGL(k_block_axpy<double2>, grid, dim3(256), 0, s, (const double2*)basis,
                       basis_stride, (double2*)T, N, nvec, hcur, kmax, npart);
}

static void launch_norm2_parts(bool f32, const void* T, long N, int nrhs, double* partials,
                               hipStream_t s) {
  dim3 grid(arn_nchunk(N), nrhs);
  if (f32)
    hipLaunchKernelGGL(k_norm2<float2>, grid, dim3(256), 0, s, (const float2*)T, N, partials);
  else
    hipLaunchKernelGGL(k_norm2<double2>, grid, dim3(256), 0, s, (const double2*)T, N, partials);
}

void launch_norm2(bool f32, const void* T, long N, int nrhs, double* partials, double* red,
                  hipStream_t s) {
  launch_norm2_parts(f32, T, N, nrhs, partials, s);
  hipLaunchKernelGGL(k_reduce_partials<1>, dim3(nrhs), dim3(256), 0, s, partials, arn_nchunk(N), red);
}

void launch_norm2_part(bool f32, const void* T, long N, double* partials, hipStream_t s) {
  launch_norm2_parts(f32, T, N, 1, partials, s);
}

void launch_arn_next(bool f32, const void* T, void* out, long N, const double* npart,
                     const double* tnpart, double2* H, int kmax, int j, int* kstop, int* status,
                     int nrhs, hipStream_t s) {
  const int nch = arn_nchunk(N);
  dim3 grid(chunks_for(N, 4096), nrhs);
  if (f32)
    hipLaunchKernelGGL(k_arn_next<float2>, grid, dim3(256), 0, s, (const float2*)T, (float2*)out, N,
                       npart, tnpart, nch, H, kmax, j, kstop, status);
  else
    hipLaunchKernelGGL(k_arn_next<double2>, grid, dim3(256), 0, s, (const double2*)T,
                       (double2*)out, N, npart, tnpart, nch, H, kmax, j, kstop, status);
}

int isign_tri_nwave(int nnode) { return cdiv_i(2L * nnode, 64); }

void launch_isign_tri(const double2* alpha, const double* beta, const double2* gamma, int kmax,
                      const IsignTask* task, const int* kstop, const int* status, int nrhs,
                      int nwave, int chunk, bool first, double2* minor, int* expo,
                      double2* part, double2* x, int* kout, IsignResult* res, hipStream_t s) {
  for (int w0 = 0; w0 < nwave; w0 += chunk)
    hipLaunchKernelGGL(k_isign_tri, dim3(std::min(chunk, nwave - w0), nrhs), dim3(64), 0, s, alpha,
                       beta, gamma, kmax, task, kstop, w0, nwave, minor, expo, part);
  hipLaunchKernelGGL(k_isign_final, dim3(nrhs), dim3(1024), 0, s, part, nwave, kmax, task, kstop,
                     status, (int)first, x, kout, res);
}

void launch_isign_hess(const double2* H, int kmax, const int* kvec, int nrhs, double h, int n0,
                       int nnode, double2* ys, double2* acc, double2* x, double* err,
                       hipStream_t s) {
  QuadNodes qn{h, n0, nnode};
  const int nq = 2 * nnode;
  for (int q0 = 0; q0 < nq; q0 += kIsignHessChunk) {
    const int nc = std::min(kIsignHessChunk, nq - q0);
    hipLaunchKernelGGL(k_isign_hess, dim3(nc, nrhs), dim3(256), 0, s, H, kmax, kvec, qn, q0, ys);
    hipLaunchKernelGGL(k_isign_hess_accum, dim3(cdiv_i(kmax, 256), nrhs), dim3(256), 0, s, ys, q0,
                       nc, kmax, kvec, qn, (int)(q0 == 0), acc);
  }
  hipLaunchKernelGGL(k_isign_hess_final, dim3(nrhs), dim3(256), 0, s, acc, kmax, kvec, x, err);
}

}  // namespace ovs
