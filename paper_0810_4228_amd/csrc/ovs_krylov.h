// Launchers of the Krylov-side kernels (krylov.hip).
#pragma once

#include "ovs_common.h"

namespace ovs {

constexpr int kHessMaxK = 1536;   // largest Arnoldi size of the Hessenberg inner sign

int defl_nchunk(long N);
void launch_defl(const double2* R, const double2* L, const double2* B, const double* sgn, int m,
                 int nrhs, long N, double* partials, double* CD, double2* bR, double2* bL,
                 double2* yex, hipStream_t s);
// Projections of X (nrhs fields) against the deflation space: outQ = X - R
// (L^dag X) and outQd = X - L (R^dag X) + L kappa (kappa [nrhs][m] or null);
// either output may be null.  CD [m][nrhs][4] receives the dots.
void launch_defl_proj(const double2* R, const double2* L, const double2* X, int m, int nrhs, long N,
                      double* partials, double* CD, const double2* kappa, double2* outQ,
                      double2* outQd, hipStream_t s);
// CD[j][r] = (L_j^dag B_r, R_j^dag B_r) only (used to check L^dag R = I)
void launch_defl_cd(const double2* R, const double2* L, const double2* B, int m, int nrhs, long N,
                    double* partials, double* CD, hipStream_t s);
void launch_start(const double2* bR, const double2* bL, int nrhs, long N, double* partials,
                  double* sums, void* V0, void* W0, bool f32, hipStream_t s);

int update_nwg(long N);
// quad: the dual stencil's sums per 64-site quarter of a tile (DualArgs::pair 6).
void launch_alpha(const double* partials, int nparts, bool quad, const CoefArrays& co, const int* it,
                  int off, const int* rhs_map, const int* n_active, int nslots, hipStream_t s);
// apart != nullptr: alpha is formed from the dual stencil's anparts partials
// inside the update (k_alpha is then not launched).  nt: streaming stores of
// the new vectors.
void launch_update(bool f32, const void* T, const void* S, void* basis, long basis_stride,
                   void* wbuf, long N, const CoefArrays& co, const int* it, int off,
                   const int* rhs_map, const int* n_active, int nslots, double* partials, bool ring,
                   const double* apart, int anparts, bool quad, int nt, hipStream_t s);
// beta and the probe gather (probes != nullptr) of iteration *it + adv - 1 and
// the advance of *it by adv in one launch; *ticket must be zero before the first
// launch and stays zero after each.
void launch_beta_tail(bool f32, const double* partials, int nparts, const CoefArrays& co, int* it,
                      int adv, const int* rhs_map, const int* n_active, int nslots, int* ticket,
                      const void* basis, long basis_stride, long N, bool ring, const int* idx,
                      int P, double2* probes, hipStream_t s);
void launch_advance(int* it, hipStream_t s);
void launch_probe_gather(bool f32, const void* basis, long basis_stride, long N, bool ring,
                         const int* it, bool first, const int* idx, int P, int kmax,
                         const int* rhs_map, const int* n_active, int nslots, double2* probes,
                         hipStream_t s);
// yp[r][p]: the result at the sampled entries from the coefficients
// n_b x[r][i] sv[r][i] (sv null: 1) of the k_r first basis vectors.
void launch_probe_y(const double2* probes, const double2* x, const double* sv, const double* nb,
                    const int* kvec, int kmax, const double2* yex, long N, const int* idx, int P,
                    double2* yp, int nrhs, hipStream_t s);

void launch_make_coef(const double2* x, const double* sv, const double* nb, int kmax, int nrhs,
                      double2* coef, hipStream_t s);
void launch_combine(bool f32, const void* basis, long basis_stride, long N, const double2* coef,
                    int kmax, const int* kused, const double2* yex, double2* y, int nrhs,
                    hipStream_t s);
void launch_replay(bool f32, const void* T, void* ring, long ring_stride, long N,
                   const CoefArrays& co, int i, const double2* coef, const int* kused, double2* y,
                   int nrhs, hipStream_t s);
void launch_overlap(const double2* b, double2* y, long N, int V, hipStream_t s);

int arn_nchunk(long N);
// partials of V_i^H T (i < nvec), [nrhs][nvec][arn_nchunk(N)]; npart (may be null):
// those of |T|^2, [nrhs][arn_nchunk(N)]
void launch_arn_dots(bool f32, const void* basis, long basis_stride, const void* T, long N,
                     int nvec, int nrhs, double* partials, double* npart, hipStream_t s);
// the dots themselves: red[nrhs][nvec]
void launch_block_dots(bool f32, const void* basis, long basis_stride, const void* T, long N,
                       int nvec, int nrhs, double* partials, double* red, hipStream_t s);
// G = X^H Y (nx x ny, column-major) for column-major FP64 blocks with
// leading dimension N: one dot launch per column of Y (tall-skinny products
// that library GEMMs tile poorly); partials hold nx * arn_nchunk(N) * 2.
void launch_gram(const double2* X, int nx, const double2* Y, int ny, long N, double* partials,
                 double2* G, hipStream_t s);
void launch_arn_accum(const double* partials, long N, int nvec, int kmax, int j, bool first,
                      double2* H, double2* hcur, int nrhs, hipStream_t s);
// T -= sum_i hcur_i V_i; npart (may be null): partials of |T|^2 as above
void launch_arn_axpy(bool f32, const void* basis, long basis_stride, void* T, long N, int nvec,
                     const double2* hcur, int kmax, int nrhs, double* npart, hipStream_t s);
// out = T / |T| and H[j+1][j] = |T| from the partials of |T|^2; tnpart: those of
// the vector before its orthogonalisation (lucky breakdown)
void launch_arn_next(bool f32, const void* T, void* out, long N, const double* npart,
                     const double* tnpart, double2* H, int kmax, int j, int* kstop, int* status,
                     int nrhs, hipStream_t s);
// partials of |T|^2 of one source, arn_nchunk(N) of them
void launch_norm2_part(bool f32, const void* T, long N, double* partials, hipStream_t s);
void launch_norm2(bool f32, const void* T, long N, int nrhs, double* partials, double* red,
                  hipStream_t s);

// Inner sign by the tau = e^u trapezoid rule.  The tridiagonal form runs its
// shifted solves in launches of at most `chunk` waves of 64 solves per source
// (kIsignWaveChunk or isign_wave_chunk(nrhs); minor: [nrhs][chunk][kmax][64]; expo:
// [nrhs][chunk][isign_expo_words(kmax)][64]; part: [nrhs][all waves][2][kmax]); the Hessenberg
// form kIsignHessChunk solves per source (ys: [nrhs][kIsignHessChunk][kmax];
// acc: [nrhs][2][kmax]).
constexpr int kIsignHessChunk = 1024;
// A trapezoid rule in u: nodes u = n h for n0 <= n < n0 + nnode.
struct QuadNodes {
  double h;   // step in u
  int n0;     // first node index (u = n h)
  int nnode;  // number of nodes
};
// What the inner sign of one source tries in a launch: one or two steps (rule[1]
// is the next finer one, or has no nodes), for its leading k x k block (k = 0:
// nothing; capped by kstop where that is given).
struct IsignTask {
  QuadNodes rule[2];
  double target, hmin;
  int k;
};
struct IsignResult {
  double err;   // of the accepted rule (or the last one tried)
  int level;    // rule accepted, or -1
  int k, kstop, status;
};
int isign_tri_nwave(int nnode);
// A launch takes about k sequential steps of the minors whatever its number of
// waves, until the waves of a compute unit's SIMDs share their issue slots, and a
// wave takes 1 KiB a source and Krylov step.  The narrow chunk holds every solve of
// the rules down to step 1/16 (43 waves); it is what a call needs, and never more
// for a part of a batch than for the batch.  Where there is room, up to five sources
// take a wide one, with 512 KiB a step for the solves of 1/32 (86 waves) or 1/64 (171)
// in one launch: 8^4 in FP64 to 1e-10, 1 / 2 / 5 sources 12.4 / 14.9 / 22.4 ms against
// 13.7 / 17.1 / 24.3.  From six on 512 KiB would still gain (6: 25.3 against 27.0), but
// the two halves of a batch of 12 would hold 1 MiB a step, 2.8 times the FP32 basis
// of 4^4 (the narrow ones 1.6).
constexpr int kIsignWaveChunk = 48;
inline int isign_wave_chunk(int nrhs) {
  const int c = 512 / nrhs;
  return nrhs > 5 ? kIsignWaveChunk : c > 172 ? 172 : c;
}
// exponents of kmax minors, one for each eight
__host__ __device__ inline int isign_expo_words(int kmax) { return (kmax + 7) / 8; }
// task, res: [nrhs] (readable and writable by the device); nwave: the largest
// number of waves of a source's rules together (the part stride).
void launch_isign_tri(const double2* alpha, const double* beta, const double2* gamma, int kmax,
                      const IsignTask* task, const int* kstop, const int* status, int nrhs,
                      int nwave, int chunk, bool first, double2* minor, int* expo,
                      double2* part, double2* x, int* kout, IsignResult* res, hipStream_t s);
void launch_isign_hess(const double2* H, int kmax, const int* kvec, int nrhs, double h, int n0,
                       int nnode, double2* ys, double2* acc, double2* x, double* err,
                       hipStream_t s);

}  // namespace ovs
