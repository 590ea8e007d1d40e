// C-ABI of libovsign: lattice handles, operator application, LR deflation and
// the sign-function drivers (two-sided Lanczos and Arnoldi).  The drivers
// enqueue the HIP kernels of stencil.hip and krylov.hip on the lattice's own
// stream; the host only makes the decisions that need a global view
// (convergence checks, quadrature refinement, breakdown bookkeeping).
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstring>
#include <functional>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "ovs_common.h"
#include "dense.h"
#include "ovs_eig.h"
#include "ovs_host.h"
#include "ovs_krylov.h"

using namespace ovs;

namespace ovs {
static thread_local char g_last_error[512] = "";
void record_error(const char* what, int line, hipError_t e) {
  snprintf(g_last_error, sizeof(g_last_error), "%s (line %d): %s", what, line, hipGetErrorString(e));
}
}  // namespace ovs

namespace ovs {

// Batches of this many sources or more are solved as two concurrent halves
// (run_batch); the autotuner times the dual stencil the same way.
constexpr int kSplitMin = 8;

// kappa * eta^{+-}_nu (Section 1): e^{+-mu} on the time hops only.
Hop make_hop(double m_w, double mu) {
  Hop h;
  const double k = 1.0 / (8.0 + 2.0 * m_w);
  for (int nu = 0; nu < 4; ++nu) {
    h.fwd[nu] = (nu == 3) ? k * std::exp(mu) : k;
    h.bwd[nu] = (nu == 3) ? k * std::exp(-mu) : k;
    h.f32_fwd[nu] = (float)h.fwd[nu];
    h.f32_bwd[nu] = (float)h.bwd[nu];
  }
  return h;
}

void op_setup(const ovs_lattice_s* l, ovs_op op, Hop& h, bool& g5in, bool& g5out) {
  switch (op) {
    case OVS_OP_DW: h = make_hop(l->m_w, l->mu); g5in = false; g5out = false; break;
    case OVS_OP_A: h = make_hop(l->m_w, l->mu); g5in = false; g5out = true; break;
    case OVS_OP_A_DAG: h = make_hop(l->m_w, -l->mu); g5in = false; g5out = true; break;
    default: h = make_hop(l->m_w, -l->mu); g5in = true; g5out = true; break;  // Dw^dag
  }
}

bool valid_op(int op) { return op >= 0 && op <= 3; }

size_t elem_bytes(const ovs_lattice_s* l) { return l->prec == OVS_F32_STORE ? 8 : 16; }


// The configuration set for batches of nrhs sources, or the default of a launch
// of `launch` of them (0: all).
Tuning get_tuning(const ovs_lattice_s* l, int nrhs, int launch) {
  for (auto& p : l->tuning)
    if (p.first == nrhs) return p.second;
  return default_tuning(l->prec == OVS_F32_STORE, l->g, launch > 0 ? launch : nrhs);
}

Tuning get_dual_tuning(const ovs_lattice_s* l, int nrhs, int launch = 0) {
  for (auto& p : l->dual_tuning)
    if (p.first == nrhs) return p.second;
  return default_dual_tuning(l->prec == OVS_F32_STORE, l->g, launch > 0 ? launch : nrhs);
}

void set_tuning(ovs_lattice_s* l, int nrhs, const Tuning& t) {
  for (auto& p : l->tuning)
    if (p.first == nrhs) { p.second = t; return; }
  l->tuning.push_back({nrhs, t});
}
void set_dual_tuning(ovs_lattice_s* l, int nrhs, const Tuning& t) {
  for (auto& p : l->dual_tuning)
    if (p.first == nrhs) { p.second = t; return; }
  l->dual_tuning.push_back({nrhs, t});
}

// Occupancy caps tried by the autotuner: dynamic LDS per workgroup in KiB
// (0 = none; 40, 53, 80, 160 allow 4, 3, 2, 1 workgroups per CU of 160 KiB).
std::vector<int> lds_candidates(const ovs_lattice_s* l) {
  std::vector<int> c;
  for (int kb : {0, 40, 53, 80, 159})
    if (kb <= l->lds_max_kb - 1) c.push_back(kb);
  return c;
}

// The two halves of a split batch run on two host threads.  While one
// captures its chunk of iterations as a graph, the other must not free or
// allocate device memory (hipFree synchronises the device), so captures and
// the growth of cached buffers hold this lock.
static std::mutex g_capture_mu;

// Memory that single kernels on the caller's stream may still use (the workspace,
// fields, links) is freed by hipFree alone, which waits for the whole device: the
// caller's stream may be gone by then, so it is not waited for by name.
ovs_status ensure_ws(ovs_lattice_s* l, size_t bytes) {
  if (l->ws && l->ws_bytes >= bytes) return OVS_OK;
  std::lock_guard<std::mutex> lock(g_capture_mu);
  if (l->ws) {
    OVS_HIP(hipStreamSynchronize(l->stream));
    (void)hipFree(l->ws);
    l->ws = nullptr;
    l->ws_bytes = 0;
  }
  if (hipMalloc(&l->ws, bytes) != hipSuccess) {
    (void)hipGetLastError();
    l->ws = nullptr;
    return OVS_ERR_ALLOC;
  }
  l->ws_bytes = bytes;
  return OVS_OK;
}

// Grows the handle's pinned host buffer to at least bytes.  Kernels read their
// small inputs from it and write their small results to it directly; the host
// looks at results after a stream synchronisation.
static ovs_status ensure_pin(ovs_lattice_s* l, size_t bytes) {
  if (l->pin_bytes >= bytes) return OVS_OK;
  std::lock_guard<std::mutex> lock(g_capture_mu);
  if (l->pin) {
    OVS_HIP(hipStreamSynchronize(l->stream));
    (void)hipHostFree(l->pin);
    l->pin = nullptr;
    l->pin_bytes = 0;
  }
  if (hipHostMalloc(&l->pin, bytes, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    l->pin = nullptr;
    return OVS_ERR_ALLOC;
  }
  l->pin_bytes = bytes;
  return OVS_OK;
}

void pack_field(const ovs_lattice_s* l, const void* canon, void* field, int nrhs, hipStream_t s) {
  if (l->prec == OVS_F32_STORE)
    launch_pack_f32((const double2*)canon, (float2*)field, nrhs, l->g, s);
  else
    launch_pack_f64((const double2*)canon, (double2*)field, nrhs, l->g, s);
}
void unpack_field(const ovs_lattice_s* l, const void* field, void* canon, int nrhs, hipStream_t s) {
  if (l->prec == OVS_F32_STORE)
    launch_unpack_f32((const float2*)field, (double2*)canon, nrhs, l->g, s);
  else
    launch_unpack_f64((const double2*)field, (double2*)canon, nrhs, l->g, s);
}

bool ready(const ovs_lattice_s* l) { return l && l->links_set && l->params_set; }

Ranges::Ranges(const ovs_lattice_s* l, const char* call)
    : on_(l && (l->debug_flags & OVS_DEBUG_RANGES)) {
  if (on_) roctxRangePushA(call);
}
Ranges::~Ranges() {
  if (!on_) return;
  if (inner_) roctxRangePop();
  roctxRangePop();
}
void Ranges::phase(const char* name) {
  if (!on_) return;
  if (inner_) roctxRangePop();
  roctxRangePushA(name);
  inner_ = true;
}

// ---- inner sign with step refinement ----------------------------------------
constexpr double kULo = -40.0, kUHi = 45.0;  // u range of the tau = e^u quadrature
constexpr double kHStart = 0.25, kHMin = 1.0 / 64;
// Target of the coarse/fine difference of x = sgn(G) e_1 (the error of the
// rule with step 2h, an upper bound of the error of step h while the rule
// converges exponentially): kQuadAccept, and a tenth of the source's
// tolerance when that is smaller, but not below kQuadFloor: the FP64
// rounding of thousands of node solves puts differences of ~1e-13 between
// two converged levels, which say nothing about the sign.  The error of step
// s behaves like exp(-2 pi d / s) for a Ritz value at angle d from the
// imaginary axis, so a target missed at h = 1/64 means a Ritz value within a
// few degrees of it: the sign is ambiguous there (sgn(z) = sgn(Re z) jumps
// across the axis).
constexpr double kQuadAccept = 3e-7;
constexpr double kQuadFloor = 1e-12;
constexpr int kProbe = 512;           // sampled entries per source for the convergence estimate
constexpr int kBasisFirst = 256;      // first capacity (vectors) of a growable one-pass basis
constexpr int kCheckEvery = 25;       // iterations between convergence checks
constexpr int kStallChecks = 6;       // checks without the estimate halving: FP32 stall

// Distinct sampled field positions fidx(c, s) (s < V), sorted; a fixed
// sequence, the same for all calls.
std::vector<int> probe_positions(const Geometry& g, int P) {
  const long N = 12L * g.V;
  std::vector<int> idx;
  idx.reserve(P);
  std::vector<char> used(N, 0);
  unsigned long long st = 0x9E3779B97F4A7C15ull;
  while ((int)idx.size() < P) {
    st = st * 6364136223846793005ull + 1442695040888963407ull;
    const long p = (long)((st >> 17) % (unsigned long long)N);
    if (!used[p]) {
      used[p] = 1;
      idx.push_back((int)fidx((int)(p / g.V), p % g.V, g.Vs));
    }
  }
  std::sort(idx.begin(), idx.end());
  return idx;
}


void quad_range(double h, int& n0, int& nnode) {
  n0 = (int)std::floor(kULo / h);
  const int n1 = (int)std::ceil(kUHi / h);
  nnode = n1 - n0 + 1;
}
int max_nodes() {
  int n0, nn;
  quad_range(kHMin, n0, nn);
  return nn;
}

// Scratch of the inner sign (sizes in ovs_krylov.h): minor, expo (of `chunk`
// waves a launch), part for the tridiagonal form; ys, acc, and xtmp [nrhs][kmax],
// kv [nrhs] for the refinement levels, of the Hessenberg form.
struct InnerScratch {
  double2* minor = nullptr;
  int* expo = nullptr;
  double2* part = nullptr;
  double2* ys = nullptr;
  double2* acc = nullptr;
  double2* xtmp = nullptr;
  int* kv = nullptr;
  int chunk = 0;
};

// Quadrature target of each source (see kQuadAccept); tol may be NULL.
std::vector<double> quad_targets(const double* tol, int nrhs) {
  std::vector<double> t(nrhs, kQuadAccept);
  if (tol)
    for (int r = 0; r < nrhs; ++r) t[r] = std::min(kQuadAccept, std::max(kQuadFloor, 0.1 * tol[r]));
  return t;
}

// x[r] = sgn(T_r) e_1 for the sources with kcap[r] > 0 (rows of the others
// are zero), T_r of size min(kcap[r], kstop[r]) (kstop: device, or null).  Runs
// the quadrature at h = 0.25 and halves h for the sources whose coarse/fine
// difference is above their target, down to h = kHMin; each source keeps the x
// of the first step that met its target (or of the finest), so its result does
// not depend on the other sources of the batch.  out[r]: that step's difference,
// and the source's k, kstop and status (device array, or null).
//
// h_level (optional, per source, in and out): on entry the step at which the
// source's refinement starts (kHStart or a power-of-two fraction of it), on
// return the step it was accepted at.  Without it every source starts at
// kHStart.  Every round takes each unaccepted source at its own step and, where
// both fit the scratch, the next finer one in the same launch: a launch takes
// the time of one sweep of minors however many solves it holds, and the device
// picks the first step that meets the target.  A source's steps depend only on
// its own differences, so its x, and with it the convergence checks that pass
// their levels from one check to the next, do not depend on the rest of the
// batch.
//
// kout: device [nrhs], the sizes of the first round, or null.  then (optional):
// enqueues work that uses x and kout; called after the launches of the first
// round, and again if a later round changed x.
ovs_status inner_sign_tri(ovs_lattice_s* l, const double2* alpha, const double* beta,
                          const double2* gamma, int kmax, const std::vector<int>& kcap,
                          const int* kstop, const int* status, int nrhs, InnerScratch& sc,
                          double2* x, int* kout, const std::vector<double>& target,
                          std::vector<IsignResult>& out, std::vector<double>* h_level = nullptr,
                          const std::function<ovs_status()>& then = nullptr) {
  hipStream_t s = l->stream;
  const size_t tb = sizeof(IsignTask) * (size_t)nrhs;
  ovs_status st = ensure_pin(l, tb + sizeof(IsignResult) * (size_t)nrhs);
  if (st != OVS_OK) return st;
  IsignTask* task = (IsignTask*)l->pin;
  IsignResult* res = (IsignResult*)((char*)l->pin + tb);
  out.assign(nrhs, IsignResult{0.0, 0, 0, 0, 0});
  const bool lev = h_level && (int)h_level->size() >= nrhs;
  std::vector<double> cur(nrhs, kHStart);
  std::vector<char> open(nrhs, 0);
  for (int r = 0; r < nrhs; ++r) {
    open[r] = kcap[r] > 0;
    if (lev) cur[r] = std::max(kHMin, std::min(kHStart, (*h_level)[r]));
  }
  const int cap = isign_tri_nwave(max_nodes());
  for (bool first = true;; first = false) {
    int nw = 0;
    for (int r = 0; r < nrhs; ++r) {
      IsignTask& t = task[r];
      t = IsignTask{};
      t.k = open[r] ? kcap[r] : 0;
      t.target = target[r];
      t.hmin = kHMin;
      if (!open[r]) continue;
      int w = 0;
      for (int q = 0; q < 2; ++q) {
        const double h = q ? 0.5 * cur[r] : cur[r];
        int n0, nn;
        quad_range(h, n0, nn);
        if (q && (h < kHMin || w + isign_tri_nwave(nn) > cap)) break;
        t.rule[q] = QuadNodes{h, n0, nn};
        w += isign_tri_nwave(nn);
      }
      nw = std::max(nw, w);
    }
    launch_isign_tri(alpha, beta, gamma, kmax, task, kstop, status, nrhs, nw,
                     sc.chunk, first, sc.minor, sc.expo, sc.part, x, kout, res, s);
    OVS_HIP(hipGetLastError());
    if (then) {
      st = then();
      if (st != OVS_OK) return st;
    }
    OVS_HIP(hipStreamSynchronize(s));
    bool any = false;
    for (int r = 0; r < nrhs; ++r) {
      if (first) out[r] = res[r];
      if (!open[r]) continue;
      out[r] = res[r];
      if (res[r].k <= 0) {
        open[r] = 0;
      } else if (res[r].level >= 0) {
        if (lev) (*h_level)[r] = task[r].rule[res[r].level].h;
        open[r] = 0;
      } else {
        cur[r] = 0.5 * (task[r].rule[1].nnode ? task[r].rule[1].h : task[r].rule[0].h);
        any = true;
      }
    }
    if (!any) return OVS_OK;
  }
}

// The same for upper Hessenberg matrices of size kvec[r] (Arnoldi), one launch
// per distinct step of a round.
ovs_status inner_sign_hess(ovs_lattice_s* l, const double2* H, int kmax,
                           const std::vector<int>& kvec, int nrhs, InnerScratch& sc, double2* x,
                           double* err_dev, const std::vector<double>& target,
                           std::vector<double>& err_host) {
  hipStream_t s = l->stream;
  std::vector<int> klev(kvec.begin(), kvec.begin() + nrhs);
  std::vector<int> kl(nrhs, 0);
  std::vector<double> eh(nrhs, 0.0), cur(nrhs, kHStart);
  err_host.assign(nrhs, 0.0);
  bool first = true;  // the first launch writes every row of x
  // accept or refine the sources that took part in the launch just read back
  auto settle = [&](const std::vector<int>& part_in) -> ovs_status {
    for (int r = 0; r < nrhs; ++r) {
      if (part_in[r] <= 0) continue;
      if ((eh[r] <= target[r]) || cur[r] <= kHMin) {  // NaN stays unaccepted until the last step
        if (!first)
          OVS_HIP(hipMemcpyAsync(x + (size_t)r * kmax, sc.xtmp + (size_t)r * kmax,
                                 sizeof(double2) * kmax, hipMemcpyDeviceToDevice, s));
        err_host[r] = eh[r];
        klev[r] = 0;
      } else {
        cur[r] *= 0.5;
      }
    }
    return OVS_OK;
  };
  for (;;) {
    bool any = false;
    for (int r = 0; r < nrhs; ++r) any = any || klev[r] > 0;
    if (!any && !first) break;
    // one launch per distinct step of the round, coarsest first
    std::vector<double> steps;
    for (int r = 0; r < nrhs; ++r)
      if (klev[r] > 0 && std::find(steps.begin(), steps.end(), cur[r]) == steps.end())
        steps.push_back(cur[r]);
    if (steps.empty()) steps.push_back(kHStart);  // no active source: zero rows
    std::sort(steps.begin(), steps.end(), std::greater<double>());
    for (double h : steps) {
      for (int r = 0; r < nrhs; ++r) kl[r] = (klev[r] > 0 && cur[r] == h) ? klev[r] : 0;
      int n0, nn;
      quad_range(h, n0, nn);
      OVS_HIP(hipMemcpyAsync(sc.kv, kl.data(), sizeof(int) * nrhs, hipMemcpyHostToDevice, s));
      launch_isign_hess(H, kmax, sc.kv, nrhs, h, n0, nn, sc.ys, sc.acc, first ? x : sc.xtmp,
                        err_dev, s);
      OVS_HIP(hipGetLastError());
      OVS_HIP(hipMemcpyAsync(eh.data(), err_dev, sizeof(double) * nrhs, hipMemcpyDeviceToHost, s));
      OVS_HIP(hipStreamSynchronize(s));
      const ovs_status sst = settle(kl);
      if (sst != OVS_OK) return sst;
      first = false;
    }
  }
  OVS_HIP(hipStreamSynchronize(s));  // host vector lifetimes
  return OVS_OK;
}

}  // namespace ovs

// ============================================================================
extern "C" {

const char* ovs_last_error(void) { return g_last_error; }

const char* ovs_status_string(ovs_status s) {
  switch (s) {
    case OVS_OK: return "ok";
    case OVS_WARN_NOT_CONVERGED: return "not converged within k_max";
    case OVS_WARN_BREAKDOWN: return "serious Lanczos breakdown";
    case OVS_WARN_SIGN_AMBIGUOUS: return "inner sign quadrature not converged (eigenvalue near the imaginary axis)";
    case OVS_ERR_ARG: return "invalid argument";
    case OVS_ERR_HIP: return "HIP runtime error";
    case OVS_ERR_ALLOC: return "device allocation failed";
    case OVS_ERR_STATE: return "handle not ready (links or parameters not set)";
    default: return "unknown status";
  }
}

ovs_status ovs_lattice_create(const int32_t dims[4], const int32_t bc[4], ovs_precision prec,
                              void* hip_stream, ovs_lattice* out) {
  if (!dims || !bc || !out) return OVS_ERR_ARG;
  *out = nullptr;
  long v = 1;
  for (int i = 0; i < 4; ++i) {
    if (dims[i] < 2 || dims[i] > 4096) return OVS_ERR_ARG;
    if (bc[i] != 1 && bc[i] != -1) return OVS_ERR_ARG;
    v *= dims[i];
  }
  if (v > (1L << 24)) return OVS_ERR_ARG;  // 32-bit byte offsets within a source field
  if (prec != OVS_F64 && prec != OVS_F32_STORE) return OVS_ERR_ARG;
  ovs_lattice_s* l = new (std::nothrow) ovs_lattice_s();
  if (!l) return OVS_ERR_ALLOC;
  l->g = Geometry{dims[0], dims[1], dims[2], dims[3], (int)v, (int)(((v + 63) / 64) * 64 + 64)};
  for (int i = 0; i < 4; ++i) l->bc[i] = bc[i];
  l->prec = prec;
  l->user_stream = (hipStream_t)hip_stream;
  if (hipGetDevice(&l->device) != hipSuccess ||
      hipStreamCreateWithFlags(&l->stream, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&l->ev_in, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&l->ev_out, hipEventDisableTiming) != hipSuccess) {
    delete l;
    return OVS_ERR_HIP;
  }
  {
    int optin = 0, dflt = 0;
    (void)hipDeviceGetAttribute(&optin, hipDeviceAttributeSharedMemPerBlockOptin, l->device);
    (void)hipDeviceGetAttribute(&dflt, hipDeviceAttributeMaxSharedMemoryPerBlock, l->device);
    const int kb = std::max(optin, dflt) / 1024;
    l->lds_max_kb = kb > 0 ? kb : 64;
    set_lds_limit(l->lds_max_kb);
    (void)hipGetLastError();
  }
  const size_t lb = 4ul * kLinkSlots * l->g.Vs * elem_bytes(l);
  if (hipMalloc(&l->links, lb) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipStreamDestroy(l->stream);
    delete l;
    return OVS_ERR_ALLOC;
  }
  *out = l;
  return OVS_OK;
}

static void destroy_shadow(ovs_lattice_s* l) {
  ovs_lattice_s* sh = l->shadow64;
  if (!sh) return;
  if (sh->ws) (void)hipFree(sh->ws);
  if (sh->bbuf) (void)hipFree(sh->bbuf);
  if (sh->pin) (void)hipHostFree(sh->pin);
  (void)hipEventDestroy(sh->ev_in);
  (void)hipEventDestroy(sh->ev_out);
  delete sh;  // links (the parent's links64) and stream belong to the parent
  l->shadow64 = nullptr;
}

static void destroy_worker(ovs_lattice_s* l) {
  ovs_lattice_s* w = l->worker;
  if (!w) return;
  (void)hipStreamSynchronize(w->stream);
  if (w->ws) (void)hipFree(w->ws);
  if (w->bbuf) (void)hipFree(w->bbuf);
  if (w->pin) (void)hipHostFree(w->pin);
  (void)hipEventDestroy(w->ev_in);
  (void)hipEventDestroy(w->ev_out);
  (void)hipStreamDestroy(w->stream);
  delete w;  // links belong to the parent
  l->worker = nullptr;
}

ovs_status ovs_lattice_destroy(ovs_lattice l) {
  if (!l || l->parent) return OVS_ERR_ARG;
  (void)hipStreamSynchronize(l->stream);
  destroy_worker(l);
  destroy_shadow(l);
  if (l->split_buf) (void)hipFree(l->split_buf);
  if (l->ev_fork) (void)hipEventDestroy(l->ev_fork);
  if (l->links) (void)hipFree(l->links);
  if (l->links64) (void)hipFree(l->links64);
  if (l->ws) (void)hipFree(l->ws);
  if (l->bbuf) (void)hipFree(l->bbuf);
  if (l->pin) (void)hipHostFree(l->pin);
  (void)hipEventDestroy(l->ev_in);
  (void)hipEventDestroy(l->ev_out);
  (void)hipStreamDestroy(l->stream);
  delete l;
  return OVS_OK;
}

ovs_status ovs_set_links(ovs_lattice l, const void* U, int32_t on_device) {
  if (!l || !U) return OVS_ERR_ARG;
  StreamScope sc(l);
  const double2* src = (const double2*)U;
  void* tmp = nullptr;
  if (!on_device) {
    const size_t bytes = 36ul * l->g.V * sizeof(double2);
    if (hipMalloc(&tmp, bytes) != hipSuccess) {
      (void)hipGetLastError();
      return OVS_ERR_ALLOC;
    }
    if (hipMemcpyAsync(tmp, U, bytes, hipMemcpyHostToDevice, l->stream) != hipSuccess) {
      (void)hipFree(tmp);
      return OVS_ERR_HIP;
    }
    src = (const double2*)tmp;
  }
  struct TmpFree {
    void* p;
    hipStream_t s;
    ~TmpFree() {
      if (p) {
        (void)hipStreamSynchronize(s);
        (void)hipFree(p);
      }
    }
  } tf{tmp, l->stream};
  launch_pack_links(src, l->links, l->prec == OVS_F32_STORE, l->g, l->bc, l->stream);
  if (l->prec == OVS_F32_STORE) {
    if (!l->links64 &&
        hipMalloc(&l->links64, 4ul * kLinkSlots * l->g.Vs * sizeof(double2)) != hipSuccess) {
      (void)hipGetLastError();
      l->links64 = nullptr;
      return OVS_ERR_ALLOC;
    }
    launch_pack_links(src, l->links64, false, l->g, l->bc, l->stream);
  }
  OVS_HIP(hipGetLastError());
  l->links_set = true;
  return OVS_OK;
}

ovs_status ovs_set_params(ovs_lattice l, double m_w, double mu) {
  if (!l) return OVS_ERR_ARG;
  if (!std::isfinite(m_w) || !std::isfinite(mu) || !(8.0 + 2.0 * m_w > 0.0)) return OVS_ERR_ARG;
  l->m_w = m_w;
  l->mu = mu;
  l->params_set = true;
  return OVS_OK;
}

ovs_status ovs_set_debug(ovs_lattice l, int32_t flags, int32_t breakdown_at) {
  if (!l || l->parent ||
      (flags & ~(OVS_DEBUG_CHECKS | OVS_DEBUG_PROGRESS | OVS_DEBUG_RANGES)) || breakdown_at < -1)
    return OVS_ERR_ARG;
  l->debug_flags = flags;
  l->debug_breakdown_at = breakdown_at;
  return OVS_OK;
}

// Single kernels (operator applications, conversions) go on the caller's stream
// itself: every call that uses the library stream leaves the caller's stream
// waiting for it and starts behind the caller's, so the order is the same, and
// the two event records and waits of StreamScope (4^4: more than the kernel)
// are not needed.
ovs_status ovs_apply(ovs_lattice l, ovs_op op, const void* x, void* y, int32_t nrhs) {
  if (!l || !x || !y || x == y || nrhs < 1 || nrhs > kMaxNrhs || !valid_op(op)) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  const size_t fb = (size_t)nrhs * 12 * l->g.Vs * elem_bytes(l);
  ovs_status st = ensure_ws(l, 2 * fb + 512);
  if (st != OVS_OK) return st;
  (void)hipGetLastError();  // as StreamScope: drop a stale error
  Arena a{(char*)l->ws};
  void* fin = a.take<char>(fb);
  void* fout = a.take<char>(fb);
  Hop h;
  bool g5in, g5out;
  op_setup(l, op, h, g5in, g5out);
  OVS_HIP(launch_apply(l->prec == OVS_F32_STORE, l->links, (const double2*)x, (double2*)y, fin,
                       fout, nrhs, l->g, h, g5in, g5out, get_tuning(l, nrhs), l->user_stream));
  return OVS_OK;
}

// ---- resident fields ---------------------------------------------------------

ovs_status ovs_field_create(ovs_lattice l, int32_t nrhs, ovs_field* out) {
  if (!l || !out || nrhs < 1 || nrhs > kMaxNrhs) return OVS_ERR_ARG;
  ovs_field_s* f = new (std::nothrow) ovs_field_s();
  if (!f) return OVS_ERR_ALLOC;
  f->lat = l;
  f->nrhs = nrhs;
  if (hipMalloc(&f->data, (size_t)nrhs * 12 * l->g.Vs * elem_bytes(l)) != hipSuccess) {
    (void)hipGetLastError();
    delete f;
    return OVS_ERR_ALLOC;
  }
  *out = f;
  return OVS_OK;
}

ovs_status ovs_field_destroy(ovs_field f) {
  if (!f) return OVS_ERR_ARG;
  (void)hipStreamSynchronize(f->lat->stream);
  (void)hipFree(f->data);
  delete f;
  return OVS_OK;
}

ovs_status ovs_field_import(ovs_field f, const void* x) {
  if (!f || !x) return OVS_ERR_ARG;
  (void)hipGetLastError();
  pack_field(f->lat, x, f->data, f->nrhs, f->lat->user_stream);
  OVS_HIP(hipGetLastError());
  return OVS_OK;
}

ovs_status ovs_field_export(ovs_field f, void* x) {
  if (!f || !x) return OVS_ERR_ARG;
  (void)hipGetLastError();
  unpack_field(f->lat, f->data, x, f->nrhs, f->lat->user_stream);
  OVS_HIP(hipGetLastError());
  return OVS_OK;
}

static ovs_status field_apply_nosync(ovs_lattice l, ovs_op op, ovs_field in, ovs_field out,
                                     const Tuning& tn, hipStream_t s) {
  Hop h;
  bool g5in, g5out;
  op_setup(l, op, h, g5in, g5out);
  OVS_HIP(launch_wilson(l->prec == OVS_F32_STORE, l->links, in->data, out->data, in->nrhs, l->g, h,
                        g5in, g5out, tn, s));
  return OVS_OK;
}

static bool fields_ok(ovs_lattice l, ovs_op op, ovs_field in, ovs_field out) {
  return l && in && out && in != out && in->lat == l && out->lat == l && in->nrhs == out->nrhs &&
         valid_op(op);
}

ovs_status ovs_field_apply(ovs_lattice l, ovs_op op, ovs_field in, ovs_field out) {
  if (!fields_ok(l, op, in, out)) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  (void)hipGetLastError();
  return field_apply_nosync(l, op, in, out, get_tuning(l, in->nrhs), l->user_stream);
}

static ovs_status timed_loop(ovs_lattice l, ovs_op op, ovs_field in, ovs_field out, int iters,
                             const Tuning& tn, double* ms) {
  hipEvent_t e0, e1;
  OVS_HIP(hipEventCreate(&e0));
  OVS_HIP(hipEventCreate(&e1));
  ovs_status st = OVS_OK;
  (void)hipEventRecord(e0, l->stream);
  for (int i = 0; i < iters && st == OVS_OK; ++i) st = field_apply_nosync(l, op, in, out, tn, l->stream);
  (void)hipEventRecord(e1, l->stream);
  (void)hipEventSynchronize(e1);
  float f = 0.f;
  (void)hipEventElapsedTime(&f, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms = (double)f / iters;
  return st;
}

ovs_status ovs_field_apply_timed(ovs_lattice l, ovs_op op, ovs_field in, ovs_field out,
                                 int32_t iters, double* ms_per_apply) {
  if (!fields_ok(l, op, in, out) || iters < 1 || !ms_per_apply) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  StreamScope sc(l);
  return timed_loop(l, op, in, out, iters, get_tuning(l, in->nrhs), ms_per_apply);
}

ovs_status ovs_dual_apply_timed(ovs_lattice l, ovs_field v, int32_t iters, double* ms_per_apply) {
  if (!l || !v || v->lat != l || iters < 1 || !ms_per_apply) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  StreamScope sc(l);
  const bool f32 = l->prec == OVS_F32_STORE;
  const int nrhs = v->nrhs;
  const long N = 12L * l->g.Vs;
  const size_t fb = (size_t)nrhs * N * elem_bytes(l);
  const int nwg = dual_num_wg(l->g);
  Arena a{nullptr};
  a.take<char>(fb); a.take<char>(fb); a.take<char>(fb);
  a.take<double>((size_t)nrhs * nwg * 12); a.take<int>(nrhs); a.take<int>(2);
  ovs_status st = ensure_ws(l, a.off + 4096);
  if (st != OVS_OK) return st;
  Arena b{(char*)l->ws};
  void* T = b.take<char>(fb);
  void* S = b.take<char>(fb);
  void* Wt = b.take<char>(fb);  // w~: a copy of v in its own memory, as in the solve
  double* part = b.take<double>((size_t)nrhs * nwg * 12);
  int* map = b.take<int>(nrhs);
  int* ints = b.take<int>(2);
  std::vector<int> hmap(nrhs);
  for (int i = 0; i < nrhs; ++i) hmap[i] = i;
  const int hints[2] = {0, nrhs};  // iteration 0, all sources active
  OVS_HIP(hipMemcpyAsync(map, hmap.data(), sizeof(int) * nrhs, hipMemcpyHostToDevice, l->stream));
  OVS_HIP(hipMemcpyAsync(ints, hints, sizeof(hints), hipMemcpyHostToDevice, l->stream));
  OVS_HIP(hipMemcpyAsync(Wt, v->data, fb, hipMemcpyDeviceToDevice, l->stream));
  OVS_HIP(hipStreamSynchronize(l->stream));
  const Tuning dt = get_dual_tuning(l, nrhs);
  // V~ = the field, W~ = its copy: distinct memory, so the A and A^dag
  // workgroups of a tile do not share spinor fetches (iteration 0 reads slot 0)
  const DualArgs da{l->links, v->data, Wt, (long)nrhs * N, false, ints, T, S, part, map,
                    ints + 1, nrhs, dt.lds_kb, dt.order, dt.nt & 1, dual_pair_of(dt)};
  const Hop hA = make_hop(l->m_w, l->mu), hAd = make_hop(l->m_w, -l->mu);
  hipEvent_t e0, e1;
  OVS_HIP(hipEventCreate(&e0));
  OVS_HIP(hipEventCreate(&e1));
  hipError_t e = hipEventRecord(e0, l->stream);
  for (int i = 0; i < iters && e == hipSuccess; ++i)
    e = launch_dual(f32, da, l->g, hA, hAd, dt.rhs_block, l->stream);
  if (e == hipSuccess) e = hipEventRecord(e1, l->stream);
  if (e == hipSuccess) e = hipEventSynchronize(e1);
  float f = 0.f;
  if (e == hipSuccess) e = hipEventElapsedTime(&f, e0, e1);
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (e != hipSuccess) {
    ovs::record_error("dual stencil timing", __LINE__, e);
    return OVS_ERR_HIP;
  }
  *ms_per_apply = (double)f / iters;
  return OVS_OK;
}

ovs_status ovs_get_tuning(ovs_lattice l, int32_t nrhs, int32_t* rhs_block, int32_t* wg_size) {
  if (!l || nrhs < 1) return OVS_ERR_ARG;
  Tuning t = get_tuning(l, nrhs);
  if (rhs_block) *rhs_block = t.rhs_block;
  if (wg_size) *wg_size = t.wg;
  return OVS_OK;
}

ovs_status ovs_get_tuning_ex(ovs_lattice l, int32_t nrhs, int32_t out[8]) {
  if (!l || nrhs < 1 || !out) return OVS_ERR_ARG;
  // (of a batch that runs as two halves, the operator pair's launch is a half's)
  const Tuning t = get_tuning(l, nrhs);
  const Tuning d = get_dual_tuning(l, nrhs, nrhs >= kSplitMin ? nrhs / 2 : nrhs);
  out[0] = t.stage * 1000 + t.rhs_block * 100 + (t.hops ? 0 : t.g) * 10 + t.nt;
  out[1] = t.wg;
  out[2] = t.lds_kb;
  out[3] = t.order;
  out[4] = d.rhs_block * 100 + (dual_pair_of(d) + 1) * 10 + d.nt;
  out[5] = (d.hops || d.g == 2 || d.g == 3) ? 512 : 256;
  out[6] = d.lds_kb;
  out[7] = d.order;
  return OVS_OK;
}

ovs_status ovs_set_tuning_ex(ovs_lattice l, int32_t nrhs, const int32_t cfg[8]) {
  if (!l || nrhs < 1 || !cfg) return OVS_ERR_ARG;
  const bool f32 = l->prec == OVS_F32_STORE;
  Tuning t, d;
  t.stage = cfg[0] / 1000;
  t.rhs_block = (cfg[0] / 100) % 10;
  t.g = (cfg[0] / 10) % 10;
  t.nt = cfg[0] % 10;
  t.wg = cfg[1];
  t.lds_kb = cfg[2];
  t.order = cfg[3];
  d.rhs_block = cfg[4] / 100;
  d.g = (cfg[4] / 10) % 10;
  d.nt = cfg[4] % 10;
  d.lds_kb = cfg[6];
  d.order = cfg[7];
  t.hops = t.g == 0;
  d.hops = d.g == kDualHops + 1;
  const bool blk_ok = f32 ? (t.rhs_block == 1 || t.rhs_block == 2 || t.rhs_block == 3 ||
                             t.rhs_block == 4 || t.rhs_block == 6)
                          : (t.rhs_block >= 1 && t.rhs_block <= 3);
  // one wave per hop has one form: 64 sites and one source a workgroup
  const bool g_ok = (t.hops && t.rhs_block == 1 && t.wg == 64 && !t.stage && !t.nt && !t.lds_kb &&
                     !t.order) ||
                    t.g == 1 || ((t.g == 2 || t.g == 4 || t.g == 8) && t.rhs_block == 1);
  // the staged tile (B 12 256 values) fits for B <= 4 in FP32 and B <= 2 in FP64
  const bool stage_ok = t.stage == 0 || (t.stage == 1 && t.g == 1 && t.rhs_block <= (f32 ? 4 : 2));
  const bool wg_ok = t.wg == 64 || t.wg == 128 || t.wg == 256;
  // variant 6 marches along t: FP32 storage, one source per thread, xy planes
  // of 256 sites, Lt % 8 == 0
  const bool march_ok = f32 && l->g.lx * l->g.ly == 256 && l->g.lt % 8 == 0;
  const bool d_ok = d.rhs_block >= 1 && d.rhs_block <= (f32 ? 4 : 2) && d.g >= 1 &&
                    (d.g <= 6 || (d.hops && d.rhs_block == 1 && !(d.nt & 1) && !d.lds_kb && !d.order)) &&
                    (d.g != 3 || d.rhs_block <= (f32 ? 2 : 1)) &&
                    (d.g != 6 || (d.rhs_block == 1 && march_ok));
  if (!blk_ok || !g_ok || !stage_ok || !wg_ok || !d_ok || t.nt < 0 || t.nt > 1 || d.nt < 0 || d.nt > 3 ||
      t.lds_kb < 0 || t.lds_kb >= l->lds_max_kb || d.lds_kb < 0 || d.lds_kb >= l->lds_max_kb ||
      t.order < 0 || t.order > 7 || d.order < 0 || d.order > 7)
    return OVS_ERR_ARG;
  if (t.hops) t.g = 1;
  if (d.hops) d.g = 1;
  t.tuned = d.tuned = true;
  set_tuning(l, nrhs, t);
  set_dual_tuning(l, nrhs, d);
  return OVS_OK;
}

ovs_status ovs_autotune(ovs_lattice l, int32_t nrhs) {
  if (!l || nrhs < 1 || nrhs > kMaxNrhs) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  const bool f32 = l->prec == OVS_F32_STORE;
  ovs_field fi = nullptr, fo = nullptr;
  ovs_status st = ovs_field_create(l, nrhs, &fi);
  if (st != OVS_OK) return st;
  st = ovs_field_create(l, nrhs, &fo);
  if (st != OVS_OK) { ovs_field_destroy(fi); return st; }
  {
    StreamScope sc(l);
    // deterministic non-zero contents: zero then the links' bytes do not matter for timing
    (void)hipMemsetAsync(fi->data, 0, (size_t)nrhs * 12 * l->g.Vs * elem_bytes(l), l->stream);
    const int blocks_f32[] = {1, 2, 3, 4, 6};
    const int blocks_f64[] = {1, 2, 3};
    const int wgs[] = {64, 128, 256};
    Tuning best;
    double best_ms = 1e300;
    const int* bl = f32 ? blocks_f32 : blocks_f64;
    const int nb = f32 ? 5 : 3;
    // candidates: source blocking in registers (g = 1, block b) or lanes per
    // site (g > 1, block 1)
    // (block, lanes per site, staged tile)
    std::vector<std::array<int, 3>> shapes;
    for (int ib = 0; ib < nb; ++ib)
      if (bl[ib] <= nrhs || bl[ib] == 1) {
        shapes.push_back({bl[ib], 1, 0});
        if (bl[ib] <= (f32 ? 4 : 2)) shapes.push_back({bl[ib], 1, 1});
      }
    for (int gg : {2, 4, 8})
      if (gg <= nrhs) shapes.push_back({1, gg, 0});
    for (auto sh : shapes) {
      for (int w : wgs)
        for (int kb : lds_candidates(l))
          for (int order = 0; order < 8; ++order)
            for (int nt = 0; nt < 2; ++nt) {
            Tuning t;
            t.rhs_block = sh[0];
            t.g = sh[1];
            t.stage = sh[2];
            t.nt = nt;
            t.wg = w;
            t.lds_kb = kb;
            t.order = order;
            double ms = 0;
            if (timed_loop(l, OVS_OP_A, fi, fo, 2, t, &ms) != OVS_OK ||
                timed_loop(l, OVS_OP_A, fi, fo, 8, t, &ms) != OVS_OK) {
              (void)hipGetLastError();  // configuration rejected at launch: skip it
              continue;
            }
            if (ms < best_ms) { best_ms = ms; best = t; }
          }
    }
    // one wave per hop, where it is the default, unless a candidate beats it
    double def_ms = 1e300;
    const Tuning def = default_tuning(f32, l->g, nrhs);
    if (timed_loop(l, OVS_OP_A, fi, fo, 2, def, &def_ms) != OVS_OK ||
        timed_loop(l, OVS_OP_A, fi, fo, 8, def, &def_ms) != OVS_OK)
      def_ms = 1e300;
    if (def.hops && def_ms <= best_ms) best = def;
    best.tuned = true;
    if (st == OVS_OK) set_tuning(l, nrhs, best);
    // dual-stencil source block for the Lanczos step
    if (st == OVS_OK) {
      const long N = 12L * l->g.Vs;
      const size_t fb = (size_t)nrhs * N * elem_bytes(l);
      const int nwg = dual_num_wg(l->g);
      Arena a{nullptr};
      a.take<char>(fb); a.take<char>(3 * fb); a.take<char>(fb); a.take<char>(fb);
      a.take<double>((size_t)nrhs * nwg * 12); a.take<int>(nrhs); a.take<int>(4);
      st = ensure_ws(l, a.off + 4096);
      if (st == OVS_OK) {
        Arena b{(char*)l->ws};
        void* basis = b.take<char>(fb);
        void* wbuf = b.take<char>(3 * fb);
        void* T = b.take<char>(fb);
        void* S = b.take<char>(fb);
        double* part = b.take<double>((size_t)nrhs * nwg * 12);
        int* map = b.take<int>(nrhs);
        int* ints = b.take<int>(4);
        std::vector<int> hmap(nrhs);
        for (int i = 0; i < nrhs; ++i) hmap[i] = i;
        // batches the solve splits run as two concurrent halves (run_batch):
        // the candidates are timed that way, each half on its own stream
        const bool halves = nrhs >= kSplitMin;
        const int n1 = halves ? nrhs / 2 : nrhs, n2 = nrhs - n1;
        int hints[4] = {0, nrhs, n1, n2};
        hipStream_t s2 = nullptr;
        hipEvent_t fork = nullptr, join = nullptr;
        if (halves && (hipStreamCreateWithFlags(&s2, hipStreamNonBlocking) != hipSuccess ||
                       hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess ||
                       hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess))
          st = OVS_ERR_HIP;
        (void)hipMemcpyAsync(map, hmap.data(), sizeof(int) * nrhs, hipMemcpyHostToDevice, l->stream);
        (void)hipMemcpyAsync(ints, hints, sizeof(hints), hipMemcpyHostToDevice, l->stream);
        (void)hipMemsetAsync(basis, 0, fb, l->stream);
        (void)hipMemsetAsync(wbuf, 0, 3 * fb, l->stream);
        const Hop hA = make_hop(l->m_w, l->mu), hAd = make_hop(l->m_w, -l->mu);
        Tuning dbest;
        double bms = 1e300;
        const bool with_hops = default_dual_tuning(f32, l->g, n1).hops;
        for (int pair = 0; pair <= (with_hops ? kDualHops : 5); ++pair)
        for (int bb = 1; bb <= (f32 ? 4 : 2); ++bb) {
          if (bb > nrhs && bb != 1) continue;
          if (pair == 5 && (bb != 1 || !f32)) continue;  // the t march: FP32, one source per thread
          if (pair == kDualHops && bb != 1) continue;    // one configuration, the default
          for (int kb : lds_candidates(l))
            for (int order = 0; order < (pair == 5 ? 2 : 8); ++order)
              for (int nt = 0; nt < 2; ++nt) {
              if (pair == kDualHops && (kb || order || nt)) continue;
              const size_t eb = elem_bytes(l);
              DualArgs da{l->links, basis, wbuf, (long)nrhs * N, false, ints, T, S, part, map,
                          halves ? ints + 2 : ints + 1, n1, kb, order, nt, pair};
              DualArgs db{l->links, (char*)basis + n1 * N * eb, (char*)wbuf + n1 * N * eb,
                          (long)nrhs * N, false, ints, (char*)T + n1 * N * eb,
                          (char*)S + n1 * N * eb, part + (size_t)n1 * nwg * 12, map, ints + 3,
                          n2, kb, order, nt, pair};
              auto launch = [&]() {
                if (launch_dual(f32, da, l->g, hA, hAd, bb, l->stream) != hipSuccess) return false;
                if (!halves) return true;
                return hipEventRecord(fork, l->stream) == hipSuccess &&
                       hipStreamWaitEvent(s2, fork, 0) == hipSuccess &&
                       launch_dual(f32, db, l->g, hA, hAd, bb, s2) == hipSuccess &&
                       hipEventRecord(join, s2) == hipSuccess &&
                       hipStreamWaitEvent(l->stream, join, 0) == hipSuccess;
              };
              hipEvent_t e0, e1;
              (void)hipEventCreate(&e0);
              (void)hipEventCreate(&e1);
              bool ok = st == OVS_OK;
              for (int w = 0; w < 2 && ok; ++w) ok = launch();
              (void)hipEventRecord(e0, l->stream);
              for (int w = 0; w < 6 && ok; ++w) ok = launch();
              (void)hipEventRecord(e1, l->stream);
              (void)hipEventSynchronize(e1);
              float f = 0;
              (void)hipEventElapsedTime(&f, e0, e1);
              (void)hipEventDestroy(e0);
              (void)hipEventDestroy(e1);
              if (!ok) {
                (void)hipGetLastError();
                continue;
              }
              if (f < bms) {
                bms = f;
                dbest.rhs_block = bb;
                dbest.lds_kb = kb;
                dbest.order = order;
                dbest.nt = nt;
                dbest.g = pair + 1;
              }
            }
        }
        // the update's new vectors are read back only by the next dual stencil,
        // after T and S and the other vectors have passed through the caches:
        // streaming stores measured ~1% faster over whole solves at 16^3 x 32
        dbest.nt |= 2;
        if (dbest.g == kDualHops + 1) dbest = default_dual_tuning(f32, l->g, n1);
        dbest.tuned = true;
        if (st == OVS_OK) set_dual_tuning(l, nrhs, dbest);
        if (s2) (void)hipStreamSynchronize(s2);
        if (fork) (void)hipEventDestroy(fork);
        if (join) (void)hipEventDestroy(join);
        if (s2) (void)hipStreamDestroy(s2);
      }
    }
    (void)hipStreamSynchronize(l->stream);
  }
  ovs_field_destroy(fi);
  ovs_field_destroy(fo);
  return st;
}

// ---- deflation -------------------------------------------------------------------

ovs_status ovs_deflation_set(ovs_lattice l, int32_t m, const double* lambda, const void* R,
                             const void* L, ovs_deflation* out) {
  if (!l || !out || m < 1 || m > kMaxDefl || !lambda || !R || !L) return OVS_ERR_ARG;
  *out = nullptr;
  for (int j = 0; j < 2 * m; ++j)
    if (!std::isfinite(lambda[j])) return OVS_ERR_ARG;
  const long N = 12L * l->g.Vs;  // padded field length
  ovs_deflation_s* d = new (std::nothrow) ovs_deflation_s();
  if (!d) return OVS_ERR_ALLOC;
  d->lat = l;
  d->m = m;
  d->lambda.assign(lambda, lambda + 2 * m);
  d->R = d->L = nullptr;
  d->sgn = nullptr;
  if (hipMalloc(&d->R, sizeof(double2) * m * N) != hipSuccess ||
      hipMalloc(&d->L, sizeof(double2) * m * N) != hipSuccess ||
      hipMalloc(&d->sgn, sizeof(double) * m) != hipSuccess) {
    (void)hipGetLastError();
    ovs_deflation_destroy(d);
    return OVS_ERR_ALLOC;
  }
  ovs_status st = OVS_OK;
  {
    StreamScope sc(l);
    launch_pack_f64((const double2*)R, d->R, m, l->g, l->stream);
    launch_pack_f64((const double2*)L, d->L, m, l->g, l->stream);
    std::vector<double> sg(m);
    for (int j = 0; j < m; ++j) sg[j] = (lambda[2 * j] >= 0.0) ? 1.0 : -1.0;
    (void)hipMemcpyAsync(d->sgn, sg.data(), sizeof(double) * m, hipMemcpyHostToDevice, l->stream);
    // check L^dagger R = I
    double *part = nullptr, *cd = nullptr;
    const int nch = defl_nchunk(N);
    if (hipMalloc(&part, sizeof(double) * (size_t)m * m * nch * 4) != hipSuccess ||
        hipMalloc(&cd, sizeof(double) * (size_t)m * m * 4) != hipSuccess) {
      (void)hipGetLastError();
      st = OVS_ERR_ALLOC;
    } else {
      launch_defl_cd(d->R, d->L, d->R, m, m, N, part, cd, l->stream);
      std::vector<double> h((size_t)m * m * 4);
      (void)hipMemcpyAsync(h.data(), cd, h.size() * sizeof(double), hipMemcpyDeviceToHost, l->stream);
      if (hipStreamSynchronize(l->stream) != hipSuccess) st = OVS_ERR_HIP;
      double dev = 0.0;
      for (int j = 0; j < m; ++j)
        for (int r = 0; r < m; ++r) {
          const double* c = &h[((size_t)j * m + r) * 4];
          const double re = c[0] - (j == r ? 1.0 : 0.0);
          dev = std::max(dev, std::hypot(re, c[1]));
        }
      if (st == OVS_OK && !(dev <= 1e-8)) st = OVS_ERR_ARG;
    }
    if (part) (void)hipFree(part);
    if (cd) (void)hipFree(cd);
  }
  if (st != OVS_OK) {
    ovs_deflation_destroy(d);
    return st;
  }
  *out = d;
  return OVS_OK;
}

ovs_status ovs_deflation_compute(ovs_lattice l, int32_t m, double tol, int32_t max_iter,
                                 ovs_deflation* out) {
  if (!l || !out || m < 1 || m > kMaxDefl || !(tol > 0.0) || max_iter < 1) return OVS_ERR_ARG;
  if (!ready(l)) return OVS_ERR_STATE;
  *out = nullptr;
  const long N = 12L * l->g.Vs;
  ovs_deflation_s* d = new (std::nothrow) ovs_deflation_s();
  if (!d) return OVS_ERR_ALLOC;
  d->lat = l;
  d->m = m;
  d->R = d->L = nullptr;
  d->sgn = nullptr;
  if (hipMalloc(&d->R, sizeof(double2) * m * N) != hipSuccess ||
      hipMalloc(&d->L, sizeof(double2) * m * N) != hipSuccess ||
      hipMalloc(&d->sgn, sizeof(double) * m) != hipSuccess) {
    (void)hipGetLastError();
    ovs_deflation_destroy(d);
    return OVS_ERR_ALLOC;
  }
  d->lambda.assign(2 * m, 0.0);
  ovs_status st;
  {
    StreamScope sc(l);
    st = compute_eigentriples(l, m, tol, max_iter, d->R, d->L, d->lambda.data(), d->info);
    if (st == OVS_OK) {
      std::vector<double> sg(m);
      for (int j = 0; j < m; ++j) sg[j] = (d->lambda[2 * j] >= 0.0) ? 1.0 : -1.0;
      if (hipMemcpyAsync(d->sgn, sg.data(), sizeof(double) * m, hipMemcpyHostToDevice, l->stream) != hipSuccess ||
          hipStreamSynchronize(l->stream) != hipSuccess)
        st = OVS_ERR_HIP;
    }
  }
  if (st != OVS_OK) {
    ovs_deflation_destroy(d);
    return st;
  }
  *out = d;
  // residual above the requested tolerance or poor biorthogonality: usable, flagged
  return (d->info[0] <= tol && d->info[1] <= 1e-6) ? OVS_OK : OVS_WARN_NOT_CONVERGED;
}

ovs_status ovs_deflation_get(ovs_deflation d, double* lambda, void* R, void* L, double* info) {
  if (!d) return OVS_ERR_ARG;
  ovs_lattice_s* l = d->lat;
  if (lambda) std::memcpy(lambda, d->lambda.data(), sizeof(double) * 2 * d->m);
  if (info) std::memcpy(info, d->info, sizeof(d->info));
  StreamScope sc(l);
  if (R) launch_unpack_f64(d->R, (double2*)R, d->m, l->g, l->stream);
  if (L) launch_unpack_f64(d->L, (double2*)L, d->m, l->g, l->stream);
  OVS_HIP(hipGetLastError());
  OVS_HIP(hipStreamSynchronize(l->stream));
  return OVS_OK;
}

ovs_status ovs_deflation_destroy(ovs_deflation d) {
  if (!d) return OVS_ERR_ARG;
  (void)hipStreamSynchronize(d->lat->stream);
  if (d->R) (void)hipFree(d->R);
  if (d->L) (void)hipFree(d->L);
  if (d->sgn) (void)hipFree(d->sgn);
  delete d;
  return OVS_OK;
}

// ---- sign function ------------------------------------------------------------------

// tune_key: the batch size whose tuned kernel configuration is used (the
// whole batch when this call runs one part of it).
// ws_bytes: if not NULL, only the workspace this call needs is computed and
// stored there (b, y, tol and info are not used).
// user_ws: the caller's workspace for this call (user_ws_bytes of it), or
// NULL for the handle's cached workspace.
static ovs_status sign_apply_impl(ovs_lattice l, ovs_deflation defl, int32_t n_defl,
                                  const void* b, void* y, int32_t nrhs, int32_t k_max,
                                  const double* tol, ovs_method method, int32_t flags,
                                  ovs_rhs_info* info, int tune_key, size_t* ws_bytes = nullptr,
                                  void* user_ws = nullptr, size_t user_ws_bytes = 0) {
  if (!l || (!ws_bytes && (!b || !y || b == y)) || nrhs < 1 || nrhs > kMaxNrhs || k_max < 1)
    return OVS_ERR_ARG;
  if (!ws_bytes && !ready(l)) return OVS_ERR_STATE;  // sizing needs no links
  if (method != OVS_2SL && method != OVS_ARNOLDI) return OVS_ERR_ARG;
  if (flags & ~(OVS_FLAG_TWO_PASS | OVS_FLAG_GRAPH | OVS_FLAG_OVERLAP | OVS_FLAG_NO_SPLIT |
                OVS_FLAG_PERSISTENT))
    return OVS_ERR_ARG;
  if (k_max > 12L * l->g.V) return OVS_ERR_ARG;
  const long N = 12L * l->g.Vs;  // padded field length of one source
  int m = 0;
  if (defl) {
    if ((defl->lat != l && defl->lat != l->parent) || n_defl < 0 || n_defl > defl->m)
      return OVS_ERR_ARG;
    m = n_defl;
  }
  const bool arn = method == OVS_ARNOLDI;
  Ranges rg(ws_bytes ? nullptr : l, "ovs_sign_apply");
  const bool two_pass = (flags & OVS_FLAG_TWO_PASS) != 0;
  const bool use_persist = (flags & OVS_FLAG_PERSISTENT) != 0;
  const bool use_graph = (flags & OVS_FLAG_GRAPH) != 0 && !use_persist;
  if (arn && (two_pass || k_max > kHessMaxK)) return OVS_ERR_ARG;
  if (tol)
    for (int r = 0; r < nrhs; ++r)
      if (!(tol[r] > 0.0)) return OVS_ERR_ARG;
  const bool f32 = l->prec == OVS_F32_STORE;
  const size_t es = elem_bytes(l);
  const int K = k_max, nr = nrhs;
  const int nslots = two_pass ? 3 : K;
  // One-pass 2sL in the handle's workspace keeps the basis in its own buffer,
  // grown in doubling steps as the iteration needs it (not sized by k_max up
  // front); in a caller's workspace it is laid out for k_max.
  const bool grow = !ws_bytes && !user_ws && !two_pass && !arn;
  const int nwg_d = dual_num_wg(l->g), nwg_u = update_nwg(N);
  const int nwave_max = isign_tri_nwave(max_nodes());
  const int nq_chunk = std::min(kIsignHessChunk, 2 * max_nodes());
  const int nch_start = 512, nch_arn = arn_nchunk(N);

  // ---- workspace layout (sizing pass, then the real one) ----
  struct Bufs {
    double2 *Bq, *bR, *bL, *yex, *Y;
    char *basis, *wbuf, *T, *S;
    double *part1, *part2, *dpart, *CD, *spart, *sums, *sumsb, *nb;
    double2 *alpha, *gamma, *sw, *coef, *x, *minor, *part, *H, *hcur, *ys, *acc, *xtmp;
    double *beta, *sv, *tnorm2, *qerr, *red, *apart, *npart, *tnpart, *dnorm;
    int *kstop, *status, *rhs_map, *ints, *kused, *pidx, *kv;
    int* expo;
    double2* probes;
    unsigned* bar;
  } B{};
  const bool probing = tol != nullptr;
  const bool debug = (l->debug_flags & OVS_DEBUG_CHECKS) != 0;  // progress alone checks nothing
  const bool monitor = debug && !arn && !two_pass;  // biorthogonality rows need the stored V
  const int P = (int)std::min<long>(kProbe, 12L * l->g.V);
  int wchunk = kIsignWaveChunk;  // waves per launch of the inner sign, chosen below
  auto layout = [&](Arena& a) {
    B.Bq = a.take<double2>((size_t)nr * N);
    if (m > 0) {
      B.bR = a.take<double2>((size_t)nr * N);
      B.bL = a.take<double2>((size_t)nr * N);
      B.yex = a.take<double2>((size_t)nr * N);
      B.dpart = a.take<double>((size_t)m * nr * defl_nchunk(N) * 4);
      B.CD = a.take<double>((size_t)m * nr * 4);
    }
    B.Y = a.take<double2>((size_t)nr * N);
    if (!grow) B.basis = a.take<char>((size_t)nslots * nr * N * es);
    if (!arn) B.wbuf = a.take<char>(3ul * nr * N * es);
    B.T = a.take<char>((size_t)nr * N * es);
    if (!arn) B.S = a.take<char>((size_t)nr * N * es);
    // the dual stencil's sums (of tiles or of their quarters, 96 bytes a tile at most)
    // are read before the result takes the same memory (192 bytes a site)
    B.part1 = reinterpret_cast<double*>(B.Y);
    B.part2 = a.take<double>((size_t)nr * nwg_u * 4);
    B.spart = a.take<double>((size_t)nr * nch_start * 3);
    B.sums = a.take<double>((size_t)nr * 3);
    B.sumsb = a.take<double>((size_t)nr * 3);
    B.nb = a.take<double>(nr);
    B.alpha = a.take<double2>((size_t)nr * K);
    B.beta = a.take<double>((size_t)nr * K);
    B.gamma = a.take<double2>((size_t)nr * K);
    B.sv = a.take<double>((size_t)nr * (K + 1));
    B.sw = a.take<double2>((size_t)nr * (K + 1));
    B.tnorm2 = a.take<double>((size_t)nr * K);
    B.kstop = a.take<int>(nr);
    B.status = a.take<int>(nr);
    B.rhs_map = a.take<int>(nr);
    B.ints = a.take<int>(4);
    if (use_persist) B.bar = a.take<unsigned>(kPersistBarWords);
    B.kused = a.take<int>(nr);
    B.x = a.take<double2>((size_t)nr * K);
    B.qerr = a.take<double>(nr);
    B.coef = a.take<double2>((size_t)nr * K);
    if (probing) {
      B.pidx = a.take<int>(P);
      B.probes = a.take<double2>((size_t)nr * K * P);
    }
    if (!arn) {
      B.minor = a.take<double2>((size_t)nr * wchunk * K * 64);
      B.expo = a.take<int>((size_t)nr * wchunk * isign_expo_words(K) * 64);
      B.part = a.take<double2>((size_t)nr * nwave_max * 2 * K);
      B.dnorm = a.take<double>((size_t)nr * K);
      if (monitor) {
        B.red = a.take<double>((size_t)nr * K * 2);
        B.apart = a.take<double>((size_t)nr * K * nch_arn * 2);
      }
    } else {
      B.H = a.take<double2>((size_t)nr * K * K);
      B.hcur = a.take<double2>((size_t)nr * K);
      B.apart = a.take<double>((size_t)nr * K * nch_arn * 2);
      B.npart = a.take<double>((size_t)nr * nch_arn);
      B.tnpart = a.take<double>((size_t)nr * nch_arn);
      B.ys = a.take<double2>((size_t)nr * nq_chunk * K);
      B.acc = a.take<double2>((size_t)nr * 2 * K);
      B.xtmp = a.take<double2>((size_t)nr * K);
      B.kv = a.take<int>(nr);
    }
  };
  {
    auto bytes_for = [&](int chunk) {
      wchunk = chunk;
      Arena sizing{nullptr};
      layout(sizing);
      return sizing.off + 4096;
    };
    // what a call needs: with the narrow chunk, so that no part of a batch (a half,
    // the FP32 group) needs more than the batch; the wide one where there is room
    const size_t need = bytes_for(kIsignWaveChunk);
    if (ws_bytes) {
      *ws_bytes = need;
      return OVS_OK;
    }
    const size_t wide = arn ? need : bytes_for(isign_wave_chunk(nr));
    char* base;
    if (user_ws) {
      if (user_ws_bytes < need) return OVS_ERR_ARG;
      if (user_ws_bytes < wide) wchunk = kIsignWaveChunk;
      base = (char*)(((uintptr_t)user_ws + 255) & ~uintptr_t(255));
    } else {
      ovs_status st = ensure_ws(l, wide);
      if (st == OVS_ERR_ALLOC && wide > need) {
        wchunk = kIsignWaveChunk;
        st = ensure_ws(l, need);
      }
      if (st != OVS_OK) return st;
      base = (char*)l->ws;
    }
    Arena real{base};
    layout(real);
  }
  // growable basis (grow): capacity in vectors, the handle's cached buffer
  const size_t vec_bytes = (size_t)nr * N * es;
  int cap = 0;
  bool basis_moved = false;  // set when a graph captured the old address
  auto ensure_basis = [&](int need) -> ovs_status {
    need = std::min(need, K);
    if (!grow || need <= cap) return OVS_OK;
    const int held = (int)std::min<size_t>(l->bbuf_bytes / vec_bytes, (size_t)K);
    if (cap == 0 && held >= need) {  // the cached buffer of an earlier call
      cap = held;
      B.basis = (char*)l->bbuf;
      return OVS_OK;
    }
    int ncap = cap == 0 ? std::max(need, std::min(K, kBasisFirst)) : std::max(need, 2 * cap);
    ncap = std::min(ncap, K);
    std::lock_guard<std::mutex> lock(g_capture_mu);
    void* nb = nullptr;
    if (hipMalloc(&nb, (size_t)ncap * vec_bytes) != hipSuccess) {
      (void)hipGetLastError();
      return OVS_ERR_ALLOC;
    }
    if (cap > 0) {
      OVS_HIP(hipMemcpyAsync(nb, B.basis, (size_t)cap * vec_bytes, hipMemcpyDeviceToDevice,
                             l->stream));
      basis_moved = true;
    }
    OVS_HIP(hipStreamSynchronize(l->stream));
    if (l->bbuf) (void)hipFree(l->bbuf);
    l->bbuf = nb;
    l->bbuf_bytes = (size_t)ncap * vec_bytes;
    B.basis = (char*)nb;
    cap = ncap;
    return OVS_OK;
  };
  {
    ovs_status st = ensure_basis(kBasisFirst);
    if (st != OVS_OK) return st;
  }
  if (m == 0) {
    B.bR = B.Bq;
    B.bL = B.Bq;
    B.yex = nullptr;
  }

  StreamScope scope(l);
  hipStream_t s = l->stream;
  // stencil outputs write only s < V: their pad entries must start at zero
  launch_zero_pad(B.T, f32, 12L * nr, l->g, s);
  if (B.S) launch_zero_pad(B.S, f32, 12L * nr, l->g, s);
  hipEvent_t ev[5];
  for (auto& e : ev) OVS_HIP(hipEventCreate(&e));
  struct EvGuard {
    hipEvent_t* e;
    ~EvGuard() { for (int i = 0; i < 5; ++i) (void)hipEventDestroy(e[i]); }
  } evg{ev};
  const long bstride = (long)nr * N;  // elements between basis entries
  const Hop hA = make_hop(l->m_w, l->mu), hAd = make_hop(l->m_w, -l->mu);

  // ---- deflation and start vectors ----
  rg.phase("deflation");
  OVS_HIP(hipEventRecord(ev[0], s));
  launch_pack_f64((const double2*)b, B.Bq, nr, l->g, s);
  if (m > 0)
    launch_defl(defl->R, defl->L, B.Bq, defl->sgn, m, nr, N, B.dpart, B.CD, B.bR, B.bL, B.yex, s);
  launch_start(B.bR, B.bL, nr, N, B.spart, B.sums, B.basis, arn ? nullptr : B.wbuf, f32, s);
  if (m > 0) launch_start(B.Bq, B.Bq, nr, N, B.spart, B.sumsb, nullptr, nullptr, f32, s);
  OVS_HIP(hipGetLastError());
  std::vector<double> sums(nr * 3), sumsb(nr * 3);
  OVS_HIP(hipMemcpyAsync(sums.data(), B.sums, sizeof(double) * nr * 3, hipMemcpyDeviceToHost, s));
  if (m > 0)
    OVS_HIP(hipMemcpyAsync(sumsb.data(), B.sumsb, sizeof(double) * nr * 3, hipMemcpyDeviceToHost, s));
  rg.phase(arn ? "arnoldi" : "lanczos");
  OVS_HIP(hipEventRecord(ev[1], s));
  OVS_HIP(hipStreamSynchronize(s));
  if (m == 0) sumsb = sums;
  std::vector<double> nbh(nr), bnorm(nr);
  std::vector<int> hstatus(nr, 0), hkstop(nr, K);
  std::vector<char> done(nr, 0);
  std::vector<int> kused(nr, K);
  for (int r = 0; r < nr; ++r) {
    if (!std::isfinite(sums[3 * r]) || !std::isfinite(sumsb[3 * r])) return OVS_ERR_ARG;  // NaN/Inf in b
    nbh[r] = std::sqrt(sums[3 * r]);
    bnorm[r] = std::sqrt(sumsb[3 * r]);
    if (nbh[r] <= 1e-12 * bnorm[r]) {  // source in the deflation space (or zero): y = y_ex
      nbh[r] = 0.0;
      done[r] = 1;
      kused[r] = 0;
    } else if (sums[3 * r + 1] == 0.0 && sums[3 * r + 2] == 0.0) {
      done[r] = 1;
      kused[r] = 0;
      hstatus[r] = 2;
    }
  }
  OVS_HIP(hipMemcpyAsync(B.nb, nbh.data(), sizeof(double) * nr, hipMemcpyHostToDevice, s));

  // ---- coefficient arrays ----
  {
    std::vector<double> sv((size_t)nr * (K + 1), 0.0), sw((size_t)nr * (K + 1) * 2, 0.0);
    for (int r = 0; r < nr; ++r) {
      sv[(size_t)r * (K + 1)] = 1.0;
      sw[(size_t)r * (K + 1) * 2] = 1.0;
    }
    OVS_HIP(hipMemcpyAsync(B.sv, sv.data(), sv.size() * sizeof(double), hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemcpyAsync(B.sw, sw.data(), sw.size() * sizeof(double), hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemsetAsync(B.alpha, 0, sizeof(double2) * nr * K, s));
    OVS_HIP(hipMemsetAsync(B.beta, 0, sizeof(double) * nr * K, s));
    OVS_HIP(hipMemsetAsync(B.gamma, 0, sizeof(double2) * nr * K, s));
    OVS_HIP(hipMemsetAsync(B.tnorm2, 0, sizeof(double) * nr * K, s));
    OVS_HIP(hipMemcpyAsync(B.kstop, hkstop.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemcpyAsync(B.status, hstatus.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
    if (arn) OVS_HIP(hipMemsetAsync(B.H, 0, sizeof(double2) * nr * K * K, s));
  }
  CoefArrays co{B.alpha, B.beta, B.gamma, B.sv, B.sw, B.tnorm2, B.kstop, B.status, K};
  if (!arn) {
    co.dnorm = B.dnorm;
    co.inject_plus1 = l->debug_breakdown_at >= 0 ? l->debug_breakdown_at + 1 : 0;
    // all-ones bytes: NaN marks the beta steps that did not run
    OVS_HIP(hipMemsetAsync(B.dnorm, 0xFF, sizeof(double) * nr * K, s));
  }
  std::vector<double> biorth(nr, -1.0);
  // Biorthogonality row of w_i against the stored v_0..v_i (Section 4:
  // W^dagger V = I in exact arithmetic): max_m |w_i^dagger v_m - delta_mi|,
  // from the dot products V~_m^dagger W~_i and the scales sv, sw.
  auto biorth_row = [&](int i) -> ovs_status {
    const int nv = i + 1;
    launch_block_dots(f32, B.basis, bstride, B.wbuf + (size_t)(i % 3) * bstride * es, N, nv, nr,
                    B.apart, B.red, s);
    std::vector<double> red((size_t)nr * nv * 2), svh((size_t)nr * (K + 1)),
        swh((size_t)nr * (K + 1) * 2);
    std::vector<int> kst(nr);
    OVS_HIP(hipMemcpyAsync(kst.data(), B.kstop, sizeof(int) * nr, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(red.data(), B.red, red.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(svh.data(), B.sv, svh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(swh.data(), B.sw, swh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    OVS_HIP(hipStreamSynchronize(s));
    for (int r = 0; r < nr; ++r) {
      if (done[r] || i >= kst[r]) continue;  // w_i of this source was not formed
      const double swr = swh[((size_t)r * (K + 1) + i) * 2], swi = swh[((size_t)r * (K + 1) + i) * 2 + 1];
      double e = 0.0;
      for (int m = 0; m < nv; ++m) {
        // w_i^dagger v_m = conj(sw_i) sv_m conj(V~_m^dagger W~_i)
        const double dr = red[((size_t)r * nv + m) * 2], di = -red[((size_t)r * nv + m) * 2 + 1];
        const double svm = svh[(size_t)r * (K + 1) + m];
        double re = svm * (swr * dr + swi * di), im = svm * (swr * di - swi * dr);
        if (m == i) re -= 1.0;
        e = std::max(e, std::hypot(re, im));
      }
      biorth[r] = std::max(biorth[r], e);
    }
    return OVS_OK;
  };
  std::vector<double> ritz_re(nr, -1.0), inner_chk(nr, -1.0);
  // Dense check of the inner sign (debug): eigenvalues of G_k (or H_k) on the
  // host, the spectral sgn(G_k) e_1 of eq. (1.3) against the quadrature's x.
  auto debug_inner = [&](bool tri) -> ovs_status {
    std::vector<double> xh((size_t)nr * K * 2), ah, bh, gh, hh;
    OVS_HIP(hipMemcpyAsync(xh.data(), B.x, xh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    if (tri) {
      ah.resize((size_t)nr * K * 2);
      bh.resize((size_t)nr * K);
      gh.resize((size_t)nr * K * 2);
      OVS_HIP(hipMemcpyAsync(ah.data(), B.alpha, ah.size() * sizeof(double), hipMemcpyDeviceToHost, s));
      OVS_HIP(hipMemcpyAsync(bh.data(), B.beta, bh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
      OVS_HIP(hipMemcpyAsync(gh.data(), B.gamma, gh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    } else {
      hh.resize((size_t)nr * K * K * 2);
      OVS_HIP(hipMemcpyAsync(hh.data(), B.H, hh.size() * sizeof(double), hipMemcpyDeviceToHost, s));
    }
    OVS_HIP(hipStreamSynchronize(s));
    using cd = std::complex<double>;
    for (int r = 0; r < nr; ++r) {
      const int k = kused[r];
      if (k <= 0) continue;
      std::vector<cd> G((size_t)k * k, cd(0, 0)), lam(k), Vv((size_t)k * k);
      for (int c = 0; c < k; ++c)
        for (int rr = 0; rr < k; ++rr) {
          if (tri) {
            const size_t b0 = (size_t)r * K;
            if (rr == c) G[rr + (size_t)k * c] = cd(ah[(b0 + c) * 2], ah[(b0 + c) * 2 + 1]);
            else if (rr == c + 1) G[rr + (size_t)k * c] = cd(bh[b0 + c], 0.0);
            else if (rr + 1 == c) G[rr + (size_t)k * c] = cd(gh[(b0 + rr) * 2], gh[(b0 + rr) * 2 + 1]);
          } else {
            const size_t e = ((size_t)r * K + c) * K + rr;
            G[rr + (size_t)k * c] = cd(hh[e * 2], hh[e * 2 + 1]);
          }
        }
      if (dense::eig(k, G.data(), lam.data(), Vv.data()) != 0) continue;
      double mre = HUGE_VAL;
      for (int q = 0; q < k; ++q) mre = std::min(mre, std::abs(lam[q].real()) / std::abs(lam[q]));
      ritz_re[r] = mre;
      std::vector<cd> Vi(Vv);
      if (dense::inverse(k, Vi.data()) != 0) continue;
      double dn = 0.0, xn = 0.0;
      for (int rr = 0; rr < k; ++rr) {
        cd acc(0, 0);
        for (int q = 0; q < k; ++q)
          acc += Vv[rr + (size_t)k * q] * (lam[q].real() >= 0.0 ? 1.0 : -1.0) * Vi[q];  // row q, col 0
        const cd xg(xh[((size_t)r * K + rr) * 2], xh[((size_t)r * K + rr) * 2 + 1]);
        dn += std::norm(xg - acc);
        xn += std::norm(acc);
      }
      inner_chk[r] = xn > 0 ? std::sqrt(dn / xn) : 0.0;
    }
    return OVS_OK;
  };

  std::vector<double> est(nr, 0.0), qerr(nr, 0.0);
  // stall tracking (FP32 storage): best estimate so far, checks since it halved
  std::vector<double> best_est(nr, HUGE_VAL);
  std::vector<int> since_best(nr, 0);
  std::vector<char> stalled(nr, 0);
  InnerScratch isc{B.minor, B.expo, B.part, B.ys, B.acc, B.xtmp, B.kv, wchunk};
  const std::vector<double> qtarget = quad_targets(tol, nr);
  std::vector<double> errh;
  std::vector<IsignResult> ires;
  // sampled entries of the result, written by the device (pinned, behind the
  // exchange of the inner sign)
  const size_t pin_head = ((sizeof(IsignTask) + sizeof(IsignResult)) * (size_t)nr + 255) & ~size_t(255);
  double* yph = nullptr;
  {
    ovs_status st = ensure_pin(l, pin_head + (probing ? sizeof(double2) * (size_t)nr * P : 0));
    if (st != OVS_OK) return st;
    yph = (double*)((char*)l->pin + pin_head);
  }

  if (!arn) {
    // ---- two-sided Lanczos (Section 4) ----
    std::vector<int> amap;
    auto push_map = [&]() -> ovs_status {
      amap.clear();
      for (int r = 0; r < nr; ++r)
        if (!done[r]) amap.push_back(r);
      std::vector<int> full(nr, 0);
      std::copy(amap.begin(), amap.end(), full.begin());
      OVS_HIP(hipMemcpyAsync(B.rhs_map, full.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
      int na = (int)amap.size();
      OVS_HIP(hipMemcpyAsync(B.ints + 1, &na, sizeof(int), hipMemcpyHostToDevice, s));
      OVS_HIP(hipStreamSynchronize(s));  // host vector lifetime
      return OVS_OK;
    };
    // iteration counter and the tail kernel's ticket start at zero, and so do
    // the persistent launches' barrier words
    const int zeros[3] = {0, 0, 0};
    OVS_HIP(hipMemcpyAsync(B.ints, zeros, sizeof(int), hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemcpyAsync(B.ints + 2, zeros + 2, sizeof(int), hipMemcpyHostToDevice, s));
    if (use_persist) OVS_HIP(hipMemsetAsync(B.bar, 0, sizeof(unsigned) * kPersistBarWords, s));
    ovs_status st = push_map();
    if (st != OVS_OK) return st;
    std::vector<int> pidx_h;
    if (probing) {
      pidx_h = probe_positions(l->g, P);
      OVS_HIP(hipMemcpyAsync(B.pidx, pidx_h.data(), sizeof(int) * P, hipMemcpyHostToDevice, s));
      launch_probe_gather(f32, B.basis, bstride, N, two_pass, B.ints, true, B.pidx, P, K,
                          B.rhs_map, B.ints + 1, nr, B.probes, s);
      OVS_HIP(hipStreamSynchronize(s));  // pidx_h lifetime
    }
    const Tuning dt = get_dual_tuning(l, tune_key, nr);
    const int dual_b = std::min(dt.rhs_block, f32 ? 4 : 2);
    const bool quad = dt.hops;
    DualArgs da{l->links, B.basis, B.wbuf, bstride, two_pass, B.ints, B.T, B.S, B.part1,
                B.rhs_map, B.ints + 1, nr, dt.lds_kb, dt.order, dt.nt & 1, dual_pair_of(dt)};
    da.beta.partials = B.part2;
    da.beta.nparts = nwg_u;
    da.beta.co = co;
    da.beta.N = N;
    da.beta.idx = B.pidx;
    da.beta.P = P;
    da.beta.probes = probing ? B.probes : nullptr;
    // one full iteration is two launches: the dual stencil, with the beta step of
    // the iteration before (and its probe gather) beside it; the update, which
    // forms alpha.  The iteration index advances once per run of iterations
    // (enqueue_tail, with the last beta step); c: position in the run.  The last
    // iteration of a solve only forms alpha.
    auto enqueue_iter = [&](int c, bool full) -> ovs_status {
      da.off = c;
      da.beta.on = c > 0;
      OVS_HIP(launch_dual(f32, da, l->g, hA, hAd, dual_b, s));
      if (full)
        launch_update(f32, B.T, B.S, B.basis, bstride, B.wbuf, N, co, B.ints, c, B.rhs_map,
                      B.ints + 1, nr, B.part2, two_pass, B.part1, nwg_d, quad, (dt.nt >> 1) & 1, s);
      else
        launch_alpha(B.part1, nwg_d, quad, co, B.ints, c, B.rhs_map, B.ints + 1, nr, s);
      OVS_HIP(hipGetLastError());
      return OVS_OK;
    };
    auto enqueue_tail = [&](int n) -> ovs_status {
      launch_beta_tail(f32, B.part2, nwg_u, co, B.ints, n, B.rhs_map, B.ints + 1, nr, B.ints + 2,
                       B.basis, bstride, N, two_pass, B.pidx, P, probing ? B.probes : nullptr, s);
      OVS_HIP(hipGetLastError());
      return OVS_OK;
    };
    const int chunk = kCheckEvery;
    hipGraphExec_t gexec = nullptr;
    hipGraph_t graph = nullptr;
    struct GraphGuard {
      hipGraph_t* g;
      hipGraphExec_t* x;
      ~GraphGuard() {
        if (*x) (void)hipGraphExecDestroy(*x);
        if (*g) (void)hipGraphDestroy(*g);
      }
    } gg{&graph, &gexec};
    std::vector<std::vector<double>> xprev(nr);
    // per source: the quadrature step its next convergence check starts at
    std::vector<double> hcheck(nr, kHStart), hlev;
    int i = 0;
    while (i < K && !amap.empty()) {
      const int iend = (tol || monitor) ? std::min(K, (i / chunk + 1) * chunk) : K;
      // full iterations are those with i < K-1; the last one only forms alpha
      int nfull = std::min(iend, K - 1) - i;
      if (nfull < 0) nfull = 0;
      // iteration j writes basis vector j + 1
      st = ensure_basis(std::min(iend, K - 1) + 1);
      if (st != OVS_OK) return st;
      if (basis_moved) {  // the captured graph holds the old basis address
        da.basis = B.basis;
        if (gexec) (void)hipGraphExecDestroy(gexec);
        if (graph) (void)hipGraphDestroy(graph);
        gexec = nullptr;
        graph = nullptr;
        basis_moved = false;
      }
      int done_it = 0;
      while (use_persist && done_it < nfull) {
        const int n = std::min(chunk, nfull - done_it);
        PersistArgs pa{l->links, B.basis, B.wbuf, bstride, two_pass, B.ints, B.T, B.S, B.part1,
                       B.part2, B.rhs_map, B.ints + 1, nr, std::min(dual_b, f32 ? 2 : 1),
                       dt.tuned && dt.g == 5, dt.order, dt.nt & 1, (dt.nt >> 1) & 1, co, B.pidx, P,
                       probing ? B.probes : nullptr, n, B.bar};
        OVS_HIP(launch_persistent(f32, pa, l->g, hA, hAd, s));
        done_it += n;
      }
      if (use_graph && nfull >= chunk) {
        if (!gexec) {
          std::lock_guard<std::mutex> lock(g_capture_mu);  // see ensure_ws
          OVS_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
          for (int c = 0; c < chunk && st == OVS_OK; ++c) st = enqueue_iter(c, true);
          if (st == OVS_OK) st = enqueue_tail(chunk);
          hipError_t ce = hipStreamEndCapture(s, &graph);
          if (st != OVS_OK) return st;
          OVS_HIP(ce);
          OVS_HIP(hipGraphInstantiate(&gexec, graph, nullptr, nullptr, 0));
        }
        while (nfull - done_it >= chunk) {
          OVS_HIP(hipGraphLaunch(gexec, s));
          done_it += chunk;
        }
      }
      if (done_it < nfull) {
        const int n = nfull - done_it;
        for (int c = 0; c < n; ++c) {
          st = enqueue_iter(c, true);
          if (st != OVS_OK) return st;
        }
        st = enqueue_tail(n);
        if (st != OVS_OK) return st;
      }
      if (iend == K) {
        st = enqueue_iter(0, false);
        if (st != OVS_OK) return st;
      }
      i = iend;
      if (monitor) {
        st = biorth_row(std::min(i, K - 1));
        if (st != OVS_OK) return st;
      }
      if (tol && i < K) {
        // convergence check at k = i (the paper gives no stopping rule): the
        // relative change of y on the sampled entries since the previous check
        // against tol / 10
        std::vector<int> kcap(nr, 0);
        for (int r : amap) kcap[r] = i;
        hlev = hcheck;
        st = inner_sign_tri(l, B.alpha, B.beta, B.gamma, K, kcap, B.kstop, B.status, nr, isc, B.x,
                            B.kused, qtarget, ires, &hlev, [&]() -> ovs_status {
                              launch_probe_y(B.probes, B.x, B.sv, B.nb, B.kused, K, B.yex, N,
                                             B.pidx, P, (double2*)yph, nr, s);
                              OVS_HIP(hipGetLastError());
                              return OVS_OK;
                            });
        if (st != OVS_OK) return st;
        // a source that needed refinement starts its next check where it was
        // accepted; one accepted at its first step tries one step coarser (a
        // Ritz value near the imaginary axis may have moved away)
        for (int r : amap) {
          hkstop[r] = ires[r].kstop;
          if (ires[r].k > 0)
            hcheck[r] = hlev[r] < hcheck[r] ? hlev[r] : std::min(kHStart, 2.0 * hcheck[r]);
        }
        const size_t nact = amap.size();
        for (int r : amap) {
          const double* yr = &yph[(size_t)r * P * 2];
          std::vector<double>& yprev = xprev[r];
          double dn = 0.0, yn = 0.0;
          for (int q = 0; q < 2 * P; ++q) {
            yn += yr[q] * yr[q];
            if (!yprev.empty()) dn += (yr[q] - yprev[q]) * (yr[q] - yprev[q]);
          }
          const bool had_prev = !yprev.empty();
          est[r] = (had_prev && yn > 0) ? std::sqrt(dn / yn) : 1.0;
          yprev.assign(yr, yr + 2 * P);
          if (hkstop[r] <= i || (had_prev && est[r] <= 0.1 * tol[r])) {
            done[r] = 1;
            kused[r] = ires[r].k;
          } else if (f32 && had_prev) {
            // FP32 rounding of the stored vectors can stall one source's
            // recurrence: an estimate that has not halved in kStallChecks
            // checks stops the source here, to be solved again with FP64
            // storage by ovs_sign_apply
            if (est[r] < 0.5 * best_est[r]) {
              best_est[r] = est[r];
              since_best[r] = 0;
            } else if (++since_best[r] >= kStallChecks) {
              done[r] = 1;
              kused[r] = ires[r].k;
              stalled[r] = 1;
            }
          }
        }
        size_t left = 0;
        for (int r = 0; r < nr; ++r) left += !done[r];
        if (left != nact) {
          st = push_map();
          if (st != OVS_OK) return st;
        }
      }
    }
    if (use_persist) {
      unsigned berr = 0;
      OVS_HIP(hipMemcpyAsync(&berr, B.bar + kPersistBarErr, sizeof(unsigned),
                             hipMemcpyDeviceToHost, s));
      OVS_HIP(hipStreamSynchronize(s));
      if (berr) {
        ovs::record_error("persistent Lanczos: a grid barrier wait ran out of polls", __LINE__,
                          hipErrorLaunchFailure);
        return OVS_ERR_HIP;
      }
    }
    rg.phase("inner_sign");
    OVS_HIP(hipEventRecord(ev[2], s));
    // the size of each source: where it stopped, or all steps (less after a breakdown)
    std::vector<int> kcap(nr);
    for (int r = 0; r < nr; ++r) kcap[r] = done[r] ? kused[r] : K;
    st = inner_sign_tri(l, B.alpha, B.beta, B.gamma, K, kcap, B.kstop, B.status, nr, isc, B.x,
                        B.kused, qtarget, ires);
    if (st != OVS_OK) return st;
    for (int r = 0; r < nr; ++r) {
      hkstop[r] = ires[r].kstop;
      hstatus[r] = ires[r].status;
      kused[r] = ires[r].k;
      qerr[r] = ires[r].err;
    }
    if (debug) {
      st = debug_inner(true);
      if (st != OVS_OK) return st;
    }
    rg.phase("combine");
    OVS_HIP(hipEventRecord(ev[3], s));
    launch_make_coef(B.x, B.sv, B.nb, K, nr, B.coef, s);
    if (!two_pass) {
      launch_combine(f32, B.basis, bstride, N, B.coef, K, B.kused, B.yex, B.Y, nr, s);
    } else {
      // second pass: regenerate v_1..v_k and accumulate (end of Section 5)
      launch_start(B.bR, B.bL, nr, N, B.spart, B.sums, B.basis, nullptr, f32, s);
      if (B.yex)
        OVS_HIP(hipMemcpyAsync(B.Y, B.yex, sizeof(double2) * nr * N, hipMemcpyDeviceToDevice, s));
      else
        OVS_HIP(hipMemsetAsync(B.Y, 0, sizeof(double2) * nr * N, s));
      const int kmx = *std::max_element(kused.begin(), kused.end());
      Tuning tn = get_tuning(l, tune_key, nr);
      for (int it = 0; it < kmx; ++it) {
        if (it + 1 < kmx)
          OVS_HIP(launch_wilson(f32, l->links, B.basis + (size_t)(it % 3) * bstride * es, B.T, nr,
                                l->g, hA, false, true, tn, s));
        launch_replay(f32, B.T, B.basis, bstride, N, co, it, B.coef, B.kused, B.Y, nr, s);
      }
    }
    OVS_HIP(hipGetLastError());
    // keep host copies of the coefficients
    l->last_nrhs = nr;
    l->last_kmax = K;
    l->last_alpha.resize((size_t)nr * K * 2);
    l->last_beta.resize((size_t)nr * K);
    l->last_gamma.resize((size_t)nr * K * 2);
    l->last_x.resize((size_t)nr * K * 2);
    OVS_HIP(hipMemcpyAsync(l->last_alpha.data(), B.alpha, sizeof(double2) * nr * K, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(l->last_beta.data(), B.beta, sizeof(double) * nr * K, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(l->last_gamma.data(), B.gamma, sizeof(double2) * nr * K, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(l->last_x.data(), B.x, sizeof(double2) * nr * K, hipMemcpyDeviceToHost, s));
  } else {
    // ---- Arnoldi with classical Gram-Schmidt applied twice (Section 2) ----
    Tuning tn = get_tuning(l, tune_key, nr);
    // convergence checks as for 2sL: every kCheckEvery steps, x_j = sgn(H_j) e_1
    // and y on the sampled entries; a converged source keeps its k (its later
    // columns are computed but not used)
    std::vector<int> pidx_h;
    std::vector<std::vector<double>> yprev(nr);
    std::vector<int> ks(nr, 0);
    if (probing) {
      std::vector<int> ident(nr);
      for (int r = 0; r < nr; ++r) ident[r] = r;
      const int hints[2] = {0, nr};
      pidx_h = probe_positions(l->g, P);
      OVS_HIP(hipMemcpyAsync(B.rhs_map, ident.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
      OVS_HIP(hipMemcpyAsync(B.ints, hints, sizeof(hints), hipMemcpyHostToDevice, s));
      OVS_HIP(hipMemcpyAsync(B.pidx, pidx_h.data(), sizeof(int) * P, hipMemcpyHostToDevice, s));
      launch_probe_gather(f32, B.basis, bstride, N, false, B.ints, true, B.pidx, P, K, B.rhs_map,
                          B.ints + 1, nr, B.probes, s);
      OVS_HIP(hipStreamSynchronize(s));  // host vector lifetimes
    }
    for (int j = 0; j < K; ++j) {
      OVS_HIP(launch_wilson(f32, l->links, B.basis + (size_t)j * bstride * es, B.T, nr, l->g, hA,
                            false, true, tn, s));
      for (int pass = 0; pass < 2; ++pass) {
        launch_arn_dots(f32, B.basis, bstride, B.T, N, j + 1, nr, B.apart,
                        pass == 0 ? B.tnpart : nullptr, s);
        launch_arn_accum(B.apart, N, j + 1, K, j, pass == 0, B.H, B.hcur, nr, s);
        launch_arn_axpy(f32, B.basis, bstride, B.T, N, j + 1, B.hcur, K, nr,
                        pass == 1 ? B.npart : nullptr, s);
      }
      if (j < K - 1) {
        launch_arn_next(f32, B.T, B.basis + (size_t)(j + 1) * bstride * es, N, B.npart, B.tnpart,
                        B.H, K, j, B.kstop, B.status, nr, s);
        if (probing) {
          // sampled entries of v_{j+2} (B.ints[0] = j, so the gather takes j + 1)
          launch_probe_gather(f32, B.basis, bstride, N, false, B.ints, false, B.pidx, P, K,
                              B.rhs_map, B.ints + 1, nr, B.probes, s);
          launch_advance(B.ints, s);
        }
      }
      OVS_HIP(hipGetLastError());
      const int kj = j + 1;
      if (probing && kj % kCheckEvery == 0 && kj < K) {
        OVS_HIP(hipMemcpyAsync(hkstop.data(), B.kstop, sizeof(int) * nr, hipMemcpyDeviceToHost, s));
        OVS_HIP(hipStreamSynchronize(s));
        int nact = 0;
        for (int r = 0; r < nr; ++r) {
          ks[r] = done[r] ? 0 : std::min(kj, hkstop[r]);
          nact += done[r] ? 0 : 1;
        }
        if (nact == 0) break;
        OVS_HIP(hipMemcpyAsync(B.kused, ks.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
        ovs_status st = inner_sign_hess(l, B.H, K, ks, nr, isc, B.x, B.qerr, qtarget, errh);
        if (st != OVS_OK) return st;
        launch_probe_y(B.probes, B.x, nullptr, B.nb, B.kused, K, B.yex, N, B.pidx, P, (double2*)yph,
                       nr, s);
        OVS_HIP(hipGetLastError());
        OVS_HIP(hipStreamSynchronize(s));
        bool all_done = true;
        for (int r = 0; r < nr; ++r) {
          if (done[r]) continue;
          const double* yr = &yph[(size_t)r * P * 2];
          double dn = 0.0, yn = 0.0;
          for (int q = 0; q < 2 * P; ++q) {
            yn += yr[q] * yr[q];
            if (!yprev[r].empty()) dn += (yr[q] - yprev[r][q]) * (yr[q] - yprev[r][q]);
          }
          const bool had_prev = !yprev[r].empty();
          est[r] = (had_prev && yn > 0) ? std::sqrt(dn / yn) : 1.0;
          yprev[r].assign(yr, yr + 2 * P);
          if (hkstop[r] <= kj || (had_prev && est[r] <= 0.1 * tol[r])) {
            done[r] = 1;
            kused[r] = ks[r];
          } else {
            all_done = false;
          }
        }
        if (all_done) break;
      }
    }
    rg.phase("inner_sign");
    OVS_HIP(hipEventRecord(ev[2], s));
    OVS_HIP(hipMemcpyAsync(hkstop.data(), B.kstop, sizeof(int) * nr, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipMemcpyAsync(hstatus.data(), B.status, sizeof(int) * nr, hipMemcpyDeviceToHost, s));
    OVS_HIP(hipStreamSynchronize(s));
    for (int r = 0; r < nr; ++r) {
      if (!done[r]) kused[r] = std::min(K, hkstop[r]);
      else if (kused[r] > 0) kused[r] = std::min(kused[r], hkstop[r]);
    }
    OVS_HIP(hipMemcpyAsync(B.kused, kused.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
    ovs_status st = inner_sign_hess(l, B.H, K, kused, nr, isc, B.x, B.qerr, qtarget, errh);
    if (st != OVS_OK) return st;
    qerr = errh;
    if (debug) {
      st = debug_inner(false);
      if (st != OVS_OK) return st;
    }
    rg.phase("combine");
    OVS_HIP(hipEventRecord(ev[3], s));
    launch_make_coef(B.x, nullptr, B.nb, K, nr, B.coef, s);
    launch_combine(f32, B.basis, bstride, N, B.coef, K, B.kused, B.yex, B.Y, nr, s);
    OVS_HIP(hipGetLastError());
  }
  if (flags & OVS_FLAG_OVERLAP) launch_overlap(B.Bq, B.Y, (long)nr * N, l->g.Vs, s);
  launch_unpack_f64(B.Y, (double2*)y, nr, l->g, s);
  OVS_HIP(hipEventRecord(ev[4], s));
  OVS_HIP(hipGetLastError());
  OVS_HIP(hipStreamSynchronize(s));
  float t01 = 0, t12 = 0, t23 = 0, t34 = 0;
  (void)hipEventElapsedTime(&t01, ev[0], ev[1]);
  (void)hipEventElapsedTime(&t12, ev[1], ev[2]);
  (void)hipEventElapsedTime(&t23, ev[2], ev[3]);
  (void)hipEventElapsedTime(&t34, ev[3], ev[4]);
  std::vector<double> mind(nr, -1.0);
  if (!arn) {
    std::vector<double> dn((size_t)nr * K);
    // on the handle's (non-blocking) stream: a synchronous copy on the legacy
    // stream would have to wait for every blocking stream, and is refused
    // while the other half of a split batch captures its graph
    OVS_HIP(hipMemcpyAsync(dn.data(), B.dnorm, dn.size() * sizeof(double), hipMemcpyDeviceToHost,
                           s));
    OVS_HIP(hipStreamSynchronize(s));
    for (int r = 0; r < nr; ++r) {
      double mn = HUGE_VAL;
      for (int i = 0; i < K; ++i) {
        const double d = dn[(size_t)r * K + i];
        if (!std::isnan(d)) mn = std::min(mn, d);
      }
      if (mn != HUGE_VAL) mind[r] = mn;
    }
  }
  ovs_status worst = OVS_OK;
  for (int r = 0; r < nr; ++r) {
    int rs = OVS_OK;
    if (hstatus[r] == 2) rs = OVS_WARN_BREAKDOWN;
    else if (kused[r] > 0 && !(qerr[r] <= qtarget[r])) rs = OVS_WARN_SIGN_AMBIGUOUS;
    else if (debug && ritz_re[r] >= 0.0 && ritz_re[r] <= 1e-12) rs = OVS_WARN_SIGN_AMBIGUOUS;
    else if (tol && (!done[r] || stalled[r]) && hstatus[r] == 0) rs = OVS_WARN_NOT_CONVERGED;
    if (rs > worst) worst = rs;
    if (info) {
      info[r].fp64 = f32 ? 0 : 1;
      info[r].escalated = stalled[r] ? 1 : 0;  // marks "to escalate" until ovs_sign_apply does
      info[r].k_used = kused[r];
      info[r].status = rs;
      info[r].est_rel_err = est[r];
      info[r].quad_err = qerr[r];
      info[r].n_b = nbh[r];
      info[r].t_defl_ms = t01;
      info[r].t_krylov_ms = t12;
      info[r].t_inner_ms = t23;
      info[r].t_combine_ms = t34;
      info[r].min_abs_delta = mind[r];
      info[r].biorth_err = biorth[r];
      info[r].ritz_min_re = ritz_re[r];
      info[r].inner_check_err = inner_chk[r];
    }
  }
  return worst;
}

// Batches of kSplitMin or more sources run as two contiguous halves at the
// same time: the first on the handle's stream, the second on a worker handle
// (its own stream; the same links, parameters and tuning) from a second host
// thread.  The latency-bound dual stencil and the per-iteration scalar steps
// of one half overlap the bandwidth-bound update of the other (+10% solves/s
// measured at 16^3 x 32 with 12 sources).  Per source the arithmetic is that
// of the whole batch (both halves use the whole batch's tuned kernels).

static ovs_status worker_ready(ovs_lattice_s* l) {
  if (!l->worker) {
    ovs_lattice_s* w = new (std::nothrow) ovs_lattice_s();
    if (!w) return OVS_ERR_ALLOC;
    w->g = l->g;
    for (int i = 0; i < 4; ++i) w->bc[i] = l->bc[i];
    w->prec = l->prec;
    w->device = l->device;
    w->lds_max_kb = l->lds_max_kb;
    w->parent = l;
    if (hipStreamCreateWithFlags(&w->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&w->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&w->ev_out, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      delete w;
      return OVS_ERR_HIP;
    }
    l->worker = w;
  }
  if (!l->ev_fork && hipEventCreateWithFlags(&l->ev_fork, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    l->ev_fork = nullptr;
    return OVS_ERR_HIP;
  }
  ovs_lattice_s* w = l->worker;
  w->user_stream = l->user_stream;
  w->links = l->links;
  w->links64 = l->links64;
  w->m_w = l->m_w;
  w->mu = l->mu;
  w->links_set = l->links_set;
  w->params_set = l->params_set;
  w->tuning = l->tuning;
  w->dual_tuning = l->dual_tuning;
  w->debug_flags = l->debug_flags;
  w->debug_breakdown_at = l->debug_breakdown_at;
  return OVS_OK;
}

// ws, ws_bytes: the caller's workspace (NULL: the handles' cached ones); a
// split batch lays its halves out one after the other in it.
static ovs_status run_batch(ovs_lattice l, ovs_deflation defl, int32_t n_defl, const void* b,
                            void* y, int32_t nrhs, int32_t k_max, const double* tol,
                            ovs_method method, int32_t flags, ovs_rhs_info* info,
                            void* ws = nullptr, size_t ws_bytes = 0) {
  if (nrhs < kSplitMin || (flags & (OVS_FLAG_NO_SPLIT | OVS_FLAG_PERSISTENT)))
    return sign_apply_impl(l, defl, n_defl, b, y, nrhs, k_max, tol, method, flags, info, nrhs,
                           nullptr, ws, ws_bytes);
  if (!ready(l)) return OVS_ERR_STATE;
  ovs_status st = worker_ready(l);
  if (st != OVS_OK) return st;
  const int n1 = nrhs / 2, n2 = nrhs - n1;
  void* ws2 = nullptr;
  size_t ws1_bytes = 0, ws2_bytes = 0;
  if (ws) {
    const std::vector<double> tols(nrhs, 1.0);
    st = sign_apply_impl(l, defl, n_defl, nullptr, nullptr, n1, k_max, tols.data(), method,
                         flags, nullptr, nrhs, &ws1_bytes);
    if (st != OVS_OK) return st;
    if (ws1_bytes > ws_bytes) return OVS_ERR_ARG;
    ws2 = (char*)ws + ws1_bytes;
    ws2_bytes = ws_bytes - ws1_bytes;
  }
  const size_t fb = 12ul * l->g.V * sizeof(double2);
  // the second half reads b on the worker stream: order it after the caller's
  // stream (the worker's StreamScope) and after everything already enqueued
  // on this handle's stream (the gather of solve_subset writes b there)
  OVS_HIP(hipEventRecord(l->ev_fork, l->stream));
  OVS_HIP(hipStreamWaitEvent(l->worker->stream, l->ev_fork, 0));
  ovs_status st2 = OVS_OK;
  std::string err2;
  std::thread second([&] {
    if (hipSetDevice(l->device) != hipSuccess) {
      st2 = OVS_ERR_HIP;
      return;
    }
    st2 = sign_apply_impl(l->worker, defl, n_defl, (const char*)b + n1 * fb, (char*)y + n1 * fb,
                          n2, k_max, tol ? tol + n1 : nullptr, method, flags,
                          info ? info + n1 : nullptr, nrhs, nullptr, ws2, ws2_bytes);
    if (st2 < 0) err2 = g_last_error;
  });
  const ovs_status st1 = sign_apply_impl(l, defl, n_defl, b, y, n1, k_max, tol, method, flags,
                                         info, nrhs, nullptr, ws, ws1_bytes);
  second.join();
  if (st2 < 0 && st1 >= 0) snprintf(g_last_error, sizeof(g_last_error), "%s", err2.c_str());
  if (st1 < 0) return st1;
  if (st2 < 0) return st2;
  return std::max(st1, st2);
}

// FP32 storage limits the attainable relative error to a few 1e-8 (measured
// with the oracle at 4^4).  Sources asking for less than kF32Floor run in
// FP64 on the shadow handle: the same driver on the FP64 copy of the links,
// on the same stream.  Each group is gathered into contiguous buffers.
constexpr double kF32Floor = 1e-6;

static ovs_status shadow_ready(ovs_lattice_s* l) {
  if (!l->links64) return OVS_ERR_STATE;
  if (!l->shadow64) {
    ovs_lattice_s* sh = new (std::nothrow) ovs_lattice_s();
    if (!sh) return OVS_ERR_ALLOC;
    sh->g = l->g;
    for (int i = 0; i < 4; ++i) sh->bc[i] = l->bc[i];
    sh->prec = OVS_F64;
    sh->user_stream = l->stream;
    sh->stream = l->stream;
    sh->device = l->device;
    sh->lds_max_kb = l->lds_max_kb;
    sh->parent = l;
    if (hipEventCreateWithFlags(&sh->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&sh->ev_out, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      delete sh;
      return OVS_ERR_HIP;
    }
    l->shadow64 = sh;
  }
  ovs_lattice_s* sh = l->shadow64;
  sh->links = l->links64;
  sh->m_w = l->m_w;
  sh->mu = l->mu;
  sh->links_set = l->links_set;
  sh->params_set = l->params_set;
  sh->debug_flags = l->debug_flags;
  sh->debug_breakdown_at = l->debug_breakdown_at;
  return OVS_OK;
}

// Solves the sources idx (ascending) of (b, y) with FP32 storage through
// run_batch, or with FP64 storage on the FP64 shadow handle; through the
// gather buffer unless idx is the whole batch.  Records go to inf[idx[j]].
static ovs_status solve_subset(ovs_lattice l, bool fp64, ovs_deflation defl, int32_t n_defl,
                               const void* b, void* y, int32_t nrhs, const std::vector<int>& idx,
                               int32_t k_max, const double* tol, ovs_method method,
                               int32_t flags, ovs_rhs_info* inf, void* ws = nullptr,
                               size_t ws_bytes = 0) {
  const int n = (int)idx.size();
  std::vector<double> t(n);
  for (int j = 0; j < n; ++j) t[j] = tol[idx[j]];
  std::vector<ovs_rhs_info> rec(n);
  ovs_status st;
  if (n == nrhs) {
    st = fp64 ? sign_apply_impl(l->shadow64, defl, n_defl, b, y, n, k_max, t.data(), method,
                                flags, rec.data(), n)
              : run_batch(l, defl, n_defl, b, y, n, k_max, t.data(), method, flags, rec.data(), ws,
                          ws_bytes);
  } else {
    const size_t fb = 12ul * l->g.V * sizeof(double2);
    const size_t need = 2 * (size_t)n * fb;
    if (l->split_bytes < need) {
      OVS_HIP(hipStreamSynchronize(l->stream));
      if (l->split_buf) (void)hipFree(l->split_buf);
      l->split_buf = nullptr;
      l->split_bytes = 0;
      if (hipMalloc(&l->split_buf, need) != hipSuccess) {
        (void)hipGetLastError();
        return OVS_ERR_ALLOC;
      }
      l->split_bytes = need;
    }
    char* bb = (char*)l->split_buf;
    char* yy = bb + n * fb;
    for (int j = 0; j < n; ++j)
      OVS_HIP(hipMemcpyAsync(bb + j * fb, (const char*)b + idx[j] * fb, fb,
                             hipMemcpyDeviceToDevice, l->stream));
    st = fp64 ? sign_apply_impl(l->shadow64, defl, n_defl, bb, yy, n, k_max, t.data(), method,
                                flags, rec.data(), n)
              : run_batch(l, defl, n_defl, bb, yy, n, k_max, t.data(), method, flags, rec.data(), ws,
                          ws_bytes);
    if (st < 0) return st;
    for (int j = 0; j < n; ++j)
      OVS_HIP(hipMemcpyAsync((char*)y + idx[j] * fb, yy + j * fb, fb, hipMemcpyDeviceToDevice,
                             l->stream));
    OVS_HIP(hipStreamSynchronize(l->stream));
  }
  if (st < 0) return st;
  for (int j = 0; j < n; ++j) inf[idx[j]] = rec[j];
  return st;
}

ovs_status ovs_workspace_size(ovs_lattice l, ovs_deflation defl, int32_t n_defl, int32_t nrhs,
                              int32_t k_max, ovs_method method, int32_t flags, size_t* bytes) {
  if (!l || !bytes || l->parent) return OVS_ERR_ARG;
  *bytes = 0;
  const bool split = nrhs >= kSplitMin && !(flags & (OVS_FLAG_NO_SPLIT | OVS_FLAG_PERSISTENT));
  const int n1 = split ? nrhs / 2 : nrhs, n2 = nrhs - n1;
  size_t w1 = 0, w2 = 0;
  const std::vector<double> tols(nrhs > 0 ? nrhs : 1, 1.0);  // with convergence checks
  ovs_status st = sign_apply_impl(l, defl, n_defl, nullptr, nullptr, n1, k_max, tols.data(),
                                  method, flags, nullptr, nrhs, &w1);
  if (st == OVS_OK && split)
    st = sign_apply_impl(l, defl, n_defl, nullptr, nullptr, n2, k_max, tols.data(), method,
                         flags, nullptr, nrhs, &w2);
  if (st != OVS_OK) return st;
  *bytes = w1 + w2;
  return OVS_OK;
}

ovs_status ovs_sign_apply(ovs_lattice l, ovs_deflation defl, int32_t n_defl, const void* b,
                          void* y, int32_t nrhs, int32_t k_max, const double* tol,
                          ovs_method method, int32_t flags, void* workspace, size_t ws_bytes,
                          ovs_rhs_info* info) {
  if (!l || !b || !y || b == y || nrhs < 1 || nrhs > kMaxNrhs || l->parent) return OVS_ERR_ARG;
  if (!workspace) ws_bytes = 0;
  if (!tol || l->prec != OVS_F32_STORE)
    return run_batch(l, defl, n_defl, b, y, nrhs, k_max, tol, method, flags, info, workspace,
                     ws_bytes);
  // FP32-storage lattice with targets: the FP64 group (targets below the FP32
  // floor), the FP32 group, then the FP32 sources that stalled, again with
  // FP64 storage
  std::vector<int> lo, hi;
  for (int r = 0; r < nrhs; ++r) {
    if (!(tol[r] > 0.0)) return OVS_ERR_ARG;
    (tol[r] < kF32Floor ? lo : hi).push_back(r);
  }
  if (!ready(l)) return OVS_ERR_STATE;
  std::vector<ovs_rhs_info> inf(nrhs);
  StreamScope sc(l);
  ovs_status st = OVS_OK;
  if (!lo.empty()) {
    st = shadow_ready(l);
    if (st == OVS_OK)
      st = solve_subset(l, true, defl, n_defl, b, y, nrhs, lo, k_max, tol, method, flags,
                        inf.data());
    if (st < 0) return st;
  }
  if (!hi.empty()) {
    st = solve_subset(l, false, defl, n_defl, b, y, nrhs, hi, k_max, tol, method, flags,
                      inf.data(), workspace, ws_bytes);
    if (st < 0) return st;
    std::vector<int> esc;
    for (int r : hi)
      if (inf[r].escalated) esc.push_back(r);
    if (!esc.empty()) {
      st = shadow_ready(l);
      if (st == OVS_OK)
        st = solve_subset(l, true, defl, n_defl, b, y, nrhs, esc, k_max, tol, method, flags,
                          inf.data());
      if (st < 0) return st;
      for (int r : esc) inf[r].escalated = 1;
    }
  }
  ovs_status worst = OVS_OK;
  for (int r = 0; r < nrhs; ++r) worst = std::max(worst, (ovs_status)inf[r].status);
  if (info) std::copy(inf.begin(), inf.end(), info);
  return worst;
}

ovs_status ovs_workspace_held(ovs_lattice l, size_t* bytes) {
  if (!l || !bytes || l->parent) return OVS_ERR_ARG;
  size_t b = 0;
  for (const ovs_lattice_s* h : {(const ovs_lattice_s*)l, (const ovs_lattice_s*)l->worker,
                                 (const ovs_lattice_s*)l->shadow64})
    if (h) b += h->ws_bytes + h->bbuf_bytes + h->split_bytes;
  *bytes = b;
  return OVS_OK;
}

ovs_status ovs_last_coefficients(ovs_lattice l, double* alpha, double* beta, double* gamma,
                                 double* x) {
  if (!l) return OVS_ERR_ARG;
  if (l->last_nrhs == 0) return OVS_ERR_STATE;
  if (alpha) std::memcpy(alpha, l->last_alpha.data(), l->last_alpha.size() * sizeof(double));
  if (beta) std::memcpy(beta, l->last_beta.data(), l->last_beta.size() * sizeof(double));
  if (gamma) std::memcpy(gamma, l->last_gamma.data(), l->last_gamma.size() * sizeof(double));
  if (x) std::memcpy(x, l->last_x.data(), l->last_x.size() * sizeof(double));
  return OVS_OK;
}

static ovs_status inner_sign_entry(ovs_lattice l, bool tri, int batch, int k, const double* diag,
                                   const double* sub, const double* super, const double* Hh,
                                   double* x, double* err) {
  if (!l || batch < 1 || k < 1 || !x) return OVS_ERR_ARG;
  if (tri && (!diag || !sub || !super)) return OVS_ERR_ARG;
  if (!tri && (!Hh || k > kHessMaxK)) return OVS_ERR_ARG;
  StreamScope scope(l);
  hipStream_t s = l->stream;
  const int nwave = isign_tri_nwave(max_nodes());
  const int nq = std::min(kIsignHessChunk, 2 * max_nodes());
  auto lay = [&](Arena& a, double2*& al, double*& be, double2*& ga, double2*& H, InnerScratch& sc,
                 double2*& xd, double*& ed) {
    if (tri) {
      al = a.take<double2>((size_t)batch * k);
      be = a.take<double>((size_t)batch * k);
      ga = a.take<double2>((size_t)batch * k);
      sc.minor = a.take<double2>((size_t)batch * sc.chunk * k * 64);
      sc.expo = a.take<int>((size_t)batch * sc.chunk * isign_expo_words(k) * 64);
      sc.part = a.take<double2>((size_t)batch * nwave * 2 * k);
    } else {
      H = a.take<double2>((size_t)batch * k * k);
      sc.ys = a.take<double2>((size_t)batch * nq * k);
      sc.acc = a.take<double2>((size_t)batch * 2 * k);
    }
    xd = a.take<double2>((size_t)batch * k);
    ed = a.take<double>(batch);
    sc.xtmp = a.take<double2>((size_t)batch * k);
    sc.kv = a.take<int>(batch);
  };
  double2 *al = nullptr, *ga = nullptr, *H = nullptr, *xd = nullptr;
  double *be = nullptr, *ed = nullptr;
  InnerScratch sc;
  auto reserve = [&](int chunk) {
    sc.chunk = chunk;
    Arena sizing{nullptr};
    lay(sizing, al, be, ga, H, sc, xd, ed);
    return ensure_ws(l, sizing.off + 4096);
  };
  ovs_status st = reserve(isign_wave_chunk(batch));
  if (st == OVS_ERR_ALLOC) st = reserve(kIsignWaveChunk);
  if (st != OVS_OK) return st;
  Arena a{(char*)l->ws};
  lay(a, al, be, ga, H, sc, xd, ed);
  std::vector<int> kh(batch, k);
  if (tri) {
    std::vector<double> bre((size_t)batch * k);
    for (size_t q = 0; q < bre.size(); ++q) {
      if (sub[2 * q + 1] != 0.0) return OVS_ERR_ARG;  // beta is real in the 2sL reading
      bre[q] = sub[2 * q];
    }
    OVS_HIP(hipMemcpyAsync(al, diag, sizeof(double2) * batch * k, hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemcpyAsync(be, bre.data(), sizeof(double) * batch * k, hipMemcpyHostToDevice, s));
    OVS_HIP(hipMemcpyAsync(ga, super, sizeof(double2) * batch * k, hipMemcpyHostToDevice, s));
    OVS_HIP(hipStreamSynchronize(s));
  } else {
    OVS_HIP(hipMemcpyAsync(H, Hh, sizeof(double2) * batch * k * k, hipMemcpyHostToDevice, s));
  }
  std::vector<double> eh;
  const std::vector<double> target = quad_targets(nullptr, batch);
  if (tri) {
    std::vector<IsignResult> res;
    st = inner_sign_tri(l, al, be, ga, k, kh, nullptr, nullptr, batch, sc, xd, nullptr, target, res);
    for (const IsignResult& q : res) eh.push_back(q.err);
  } else {
    st = inner_sign_hess(l, H, k, kh, batch, sc, xd, ed, target, eh);
  }
  if (st != OVS_OK) return st;
  OVS_HIP(hipMemcpyAsync(x, xd, sizeof(double2) * batch * k, hipMemcpyDeviceToHost, s));
  OVS_HIP(hipStreamSynchronize(s));
  if (err) std::memcpy(err, eh.data(), sizeof(double) * batch);
  for (int r = 0; r < batch; ++r)
    if (!(eh[r] <= target[r])) return OVS_WARN_SIGN_AMBIGUOUS;
  return OVS_OK;
}

ovs_status ovs_small_eig(int32_t n, const double* A, double* lambda, double* V) {
  if (n < 1 || n > 4096 || !A || !lambda || !V) return OVS_ERR_ARG;
  const int r = dense::eig(n, reinterpret_cast<const std::complex<double>*>(A),
                           reinterpret_cast<std::complex<double>*>(lambda),
                           reinterpret_cast<std::complex<double>*>(V));
  return r == 0 ? OVS_OK : OVS_ERR_ARG;
}

ovs_status ovs_inner_sign_tridiag(ovs_lattice l, int32_t batch, int32_t k, const double* diag,
                                  const double* sub, const double* super, double* x, double* err) {
  return inner_sign_entry(l, true, batch, k, diag, sub, super, nullptr, x, err);
}

ovs_status ovs_inner_sign_hessenberg(ovs_lattice l, int32_t batch, int32_t k, const double* H,
                                     double* x, double* err) {
  return inner_sign_entry(l, false, batch, k, nullptr, nullptr, nullptr, H, x, err);
}

}  // extern "C"
