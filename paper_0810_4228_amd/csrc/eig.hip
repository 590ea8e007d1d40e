// Elementwise kernels of the deflation eigensolver (blocks of nb FP64 fields,
// each of padded length Np = 12*Vs).
#include "ovs_common.h"
#include "ovs_device.h"
#include "ovs_eig.h"

namespace ovs {

static int egrid(long n) {
  long b = (n + 255) / 256;
  if (b > 16384) b = 16384;
  if (b < 1) b = 1;
  return (int)b;
}

// Counter-based fill: the entry at flat offset e of a block gets (u1, u2)
// uniform in [-1, 1) from splitmix64 of (seed, e); pad entries are zero.
__device__ __forceinline__ unsigned long long splitmix(unsigned long long x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

__global__ void k_fill_random(double2* __restrict__ X, long nfields, int V, int Vs,
                              unsigned long long seed) {
  const long n = nfields * 12 * Vs;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const int s = (int)(((e % (12L * Vs)) >> 1) % Vs);  // site of the pair layout
    if (s >= V) {
      X[e] = make_double2(0.0, 0.0);
      continue;
    }
    const unsigned long long h1 = splitmix(seed * 0x100000001B3ull + 2 * (unsigned long long)e);
    const unsigned long long h2 = splitmix(seed * 0x100000001B3ull + 2 * (unsigned long long)e + 1);
    const double u1 = (double)(h1 >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    const double u2 = (double)(h2 >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
    X[e] = make_double2(u1, u2);
  }
}

// Y_new = alpha (MY - c Y) + beta Y_old   (Y_old may be null): scaling and axpby
__global__ void k_cheb(double2* __restrict__ Ynew, const double2* __restrict__ MY,
                       const double2* __restrict__ Y, const double2* __restrict__ Yold, double alpha,
                       double c, double beta, long n) {
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const double2 my = MY[e], y = Y[e];
    double re = alpha * (my.x - c * y.x), im = alpha * (my.y - c * y.y);
    if (Yold) {
      const double2 yo = Yold[e];
      re += beta * yo.x;
      im += beta * yo.y;
    }
    Ynew[e] = make_double2(re, im);
  }
}

// D_j = AR_j - theta_j R_j for nb fields of length Np (theta: device complex [nb])
__global__ void k_resid(double2* __restrict__ D, const double2* __restrict__ AR,
                        const double2* __restrict__ R, const double2* __restrict__ theta, long Np) {
  const int j = blockIdx.y;
  const Cx<double> th = c64(theta[j]);
  const long off = (long)j * Np;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < Np; e += (long)gridDim.x * blockDim.x)
    D[off + e] = d2(c64(AR[off + e]) - cmul(th, c64(R[off + e])));
}

__global__ void k_divide(double2* __restrict__ c, const double* __restrict__ d, int n) {
  for (int j = threadIdx.x; j < n; j += blockDim.x) c[j] = make_double2(c[j].x / d[j], c[j].y / d[j]);
}

// Conjugate gradients on the normal equations M^H M x = M^H y (one source, field
// of Np entries).  With rr = |r|^2 and tt = |M p|^2 of the step (the sum of ntt
// partials, formed by every workgroup): alpha = rr / tt, x += alpha p,
// r -= alpha w (w = M^H M p), and per-workgroup partials of the new |r|^2.
// Bound by latency on the small lattices this is for: the first four elements of
// a thread (all of them up to 2^18 entries) load ahead of the sum's two barriers,
// and the sum costs no launch of its own (4^3 x 8: 2.0 + 3.9 us before).
constexpr int kCgAhead = 4;
__global__ void __launch_bounds__(256) k_cg_xr(double2* __restrict__ X, double2* __restrict__ R,
                                               const double2* __restrict__ P,
                                               const double2* __restrict__ W,
                                               const double* __restrict__ rr,
                                               const double* __restrict__ ttpart, int ntt, long Np,
                                               double* __restrict__ part) {
  __shared__ double lds[4];
  __shared__ double alpha;
  const double num = *rr;
  double t[1] = {0.0};
  for (int q = threadIdx.x; q < ntt; q += 256) t[0] += ttpart[q];
  const long st = gridDim.x * 256L, e0 = blockIdx.x * 256L + threadIdx.x;
  double2 p[kCgAhead], w[kCgAhead], x[kCgAhead], r[kCgAhead];
#pragma unroll
  for (int k = 0; k < kCgAhead; ++k) {
    const long e = e0 + k * st < Np ? e0 + k * st : Np - 1;
    p[k] = P[e];
    w[k] = W[e];
    x[k] = X[e];
    r[k] = R[e];
  }
  block_sum<1>(t, lds);
  if (threadIdx.x == 0) alpha = t[0] > 0.0 ? num / t[0] : 0.0;
  __syncthreads();
  const double a = alpha;
  double v[1] = {0.0};
  auto step = [&](long e, double2 pe, double2 we, double2 xe, double2 re) {
    X[e] = make_double2(xe.x + a * pe.x, xe.y + a * pe.y);
    const double2 rn = make_double2(re.x - a * we.x, re.y - a * we.y);
    R[e] = rn;
    v[0] += rn.x * rn.x + rn.y * rn.y;
  };
#pragma unroll
  for (int k = 0; k < kCgAhead; ++k)
    if (e0 + k * st < Np) step(e0 + k * st, p[k], w[k], x[k], r[k]);
  for (long e = e0 + kCgAhead * st; e < Np; e += st) step(e, P[e], W[e], X[e], R[e]);
  block_sum<1>(v, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = v[0];
}

// beta = rr' / rr with rr' the sum of k_cg_xr's partials (every workgroup
// forms it; workgroup 0 stores it in rr_next); next = r + beta p.
__global__ void __launch_bounds__(256) k_cg_p(double2* __restrict__ next,
                                              const double2* __restrict__ P,
                                              const double2* __restrict__ R,
                                              const double* __restrict__ rr,
                                              double* __restrict__ rr_next,
                                              const double* __restrict__ part, int nch, long Np) {
  __shared__ double lds[4];
  __shared__ double beta;
  double v[1] = {0.0};
  for (int q = threadIdx.x; q < nch; q += 256) v[0] += part[q];
  block_sum<1>(v, lds);
  if (threadIdx.x == 0) {
    beta = *rr > 0.0 ? v[0] / *rr : 0.0;
    if (blockIdx.x == 0) *rr_next = v[0];
  }
  __syncthreads();
  const double b = beta;
  for (long e = blockIdx.x * 256L + threadIdx.x; e < Np; e += gridDim.x * 256L) {
    const double2 r = R[e], p = P[e];
    next[e] = make_double2(r.x + b * p.x, r.y + b * p.y);
  }
}

// The state ahead of a first step, from rr = |r|^2: partials that sum to it, and
// an infinite predecessor, so that beta = 0 and the direction is r.
__global__ void k_cg_start(double* __restrict__ rr, double* __restrict__ part, int nch) {
  if ((int)threadIdx.x < nch) part[threadIdx.x] = threadIdx.x == 0 ? *rr : 0.0;
  __syncthreads();
  if (threadIdx.x == 0) *rr = __builtin_inf();
}

int cg_nchunk(long Np) {
  long b = (Np + 1023) / 1024;
  if (b > 256) b = 256;
  if (b < 1) b = 1;
  return (int)b;
}

void launch_cg_xr(double2* X, double2* R, const double2* P, const double2* W, const double* rr,
                  const double* ttpart, int ntt, long Np, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_xr, dim3(cg_nchunk(Np)), dim3(256), 0, s, X, R, P, W, rr, ttpart, ntt, Np,
                     part);
}

void launch_cg_p(double2* next, const double2* P, const double2* R, const double* rr,
                 double* rr_next, const double* part, long Np, hipStream_t s) {
  const int nch = cg_nchunk(Np);
  hipLaunchKernelGGL(k_cg_p, dim3(nch), dim3(256), 0, s, next, P, R, rr, rr_next, part, nch, Np);
}

void launch_cg_start(double* rr, double* part, long Np, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_start, dim3(1), dim3(256), 0, s, rr, part, cg_nchunk(Np));
}

void launch_fill_random(double2* X, long nfields, const Geometry& g, unsigned long long seed,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_fill_random, dim3(egrid(nfields * 12 * g.Vs)), dim3(256), 0, s, X, nfields,
                     g.V, g.Vs, seed);
}

void launch_cheb(double2* Ynew, const double2* MY, const double2* Y, const double2* Yold,
                 double alpha, double c, double beta, long n, hipStream_t s) {
  hipLaunchKernelGGL(k_cheb, dim3(egrid(n)), dim3(256), 0, s, Ynew, MY, Y, Yold, alpha, c, beta, n);
}

void launch_divide(double2* c, const double* d, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_divide, dim3(1), dim3(64), 0, s, c, d, n);
}

void launch_resid(double2* D, const double2* AR, const double2* R, const double2* theta, int nb,
                  long Np, hipStream_t s) {
  long b = (Np + 255) / 256;
  if (b > 1024) b = 1024;
  hipLaunchKernelGGL(k_resid, dim3((int)b, nb), dim3(256), 0, s, D, AR, R, theta, Np);
}

}  // namespace ovs
