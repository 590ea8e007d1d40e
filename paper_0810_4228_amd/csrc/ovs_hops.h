// Stencil with one wave per hop, for launches too small to fill the chip with
// one thread per site.
//
// A workgroup of eight waves takes 64 sites (a lane each) of one source and one
// operator; wave 2 nu + d computes the hop of direction nu (d = 0: from s - nu,
// 1: from s + nu): link times projected neighbour spinor, six colour-spin
// entries, to LDS.  Waves 0 to 5 then form one component pair each of the
// result from the eight hops in the order of the one-thread-per-site kernels
// (each accumulation is the same fused multiply-add), so the results are equal
// bit for bit.
//
// Bound by latency: one batch of loads instead of eight in a row, and an eighth
// of the arithmetic per lane.  The price is that nothing is shared between the
// operators or sources, and 48 KiB of LDS in FP64 that take 144 KiB of traffic (six
// entries of eight hops written, twelve components of eight hops read): larger
// grids, whose other waves hide the latency, are faster with one thread per site.
#pragma once

#include "ovs_common.h"
#include "ovs_device.h"
#include "ovs_spin.h"

namespace ovs {

// s + nu (FWD) or s - nu with periodic wrap.
template <int NU, bool FWD>
__device__ __forceinline__ int neighbour(int s, const Geometry& g) {
  const int stride = NU == 0 ? 1 : NU == 1 ? g.lx : NU == 2 ? g.lx * g.ly : g.lx * g.ly * g.lz;
  const int ext = NU == 0 ? g.lx : NU == 1 ? g.ly : NU == 2 ? g.lz : g.lt;
  const int q = s / stride;
  const int c = NU == 3 ? q : q % ext;
  if (FWD) return c == ext - 1 ? s - (ext - 1) * stride : s + stride;
  return c == 0 ? s + (ext - 1) * stride : s - stride;
}

// A source field in the library's layout, or a canonical FP64 one ([V][12],
// rounded to storage precision as it is read).
template <typename R, bool CANON> struct HopField;
template <typename R> struct HopField<R, false> {
  typename Vec2<R>::T* f;
  static constexpr bool kFormed = false;
  __device__ void load(int Vs, int s, bool g5, Cx<R> (&p)[12]) const {
    load_spinor_u(f, Vs, s, g5, p);
  }
  __device__ void load_pair(int Vs, int s, int q, Cx<R>& a, Cx<R>& b) const {
    ld_pair(pair_at(f + (long)q * 2 * Vs, s), a, b);
  }
  __device__ void store_pair(int Vs, int s, int q, Cx<R> a, Cx<R> b) const {
    st_pair(pair_at(f + (long)q * 2 * Vs, s), a, b);
  }
};
template <typename R> struct HopField<R, true> {
  double2* f;
  __device__ static Cx<R> conv(double2 v) { return {(R)v.x, (R)v.y}; }
  static constexpr bool kFormed = false;
  __device__ void load(int, int s, bool g5, Cx<R> (&p)[12]) const {
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      p[c] = conv(f[12L * s + c]);
      if (g5 && c >= 6) p[c] = -p[c];
    }
  }
  __device__ void load_pair(int, int s, int q, Cx<R>& a, Cx<R>& b) const {
    a = conv(f[12L * s + 2 * q]);
    b = conv(f[12L * s + 2 * q + 1]);
  }
  __device__ void store_pair(int, int s, int q, Cx<R> a, Cx<R> b) const {
    f[12L * s + 2 * q] = make_double2((double)a.re, (double)a.im);
    f[12L * s + 2 * q + 1] = make_double2((double)b.re, (double)b.im);
  }
};

// The direction p' = r + beta p of a conjugate gradient step, formed where it is
// read (every workgroup forms beta itself) and stored to `next` once per site.
// beta = rr' / rr, rr' the sum of the nch <= 256 partials (of the residual's
// norm, in the order of a 256-thread reduction); workgroup 0 stores rr'.
struct HopDirection {
  static constexpr bool kFormed = true;
  const double2 *r, *p;
  double2* next;
  const double *rr, *part;
  double* rr_next;
  int nch;
  bool first;   // the workgroup that stores rr'
  double* lds;  // 5 entries
  mutable double beta;
  __device__ void head() const {
    const double old = *rr;
    double v[1] = {0.0};
    if ((int)threadIdx.x < nch) v[0] += part[threadIdx.x];
    block_sum<1>(v, lds, 4);
    if (threadIdx.x == 0) {
      lds[4] = old > 0.0 ? v[0] / old : 0.0;
      if (first) *rr_next = v[0];
    }
    __syncthreads();
    beta = lds[4];
  }
  struct Spinor {
    Cx<double> r[12], p[12];
  };
  struct Pair {
    Cx<double> r[2], p[2];
  };
  __device__ Cx<double> step(Cx<double> rv, Cx<double> pv) const {
    return {rv.re + beta * pv.re, rv.im + beta * pv.im};
  }
  __device__ void load(int Vs, int s, Spinor& v) const {
    load_spinor_u(r, Vs, s, false, v.r);
    load_spinor_u(p, Vs, s, false, v.p);
  }
  __device__ void form(const Spinor& v, Cx<double> (&o)[12]) const {
#pragma unroll
    for (int c = 0; c < 12; ++c) o[c] = step(v.r[c], v.p[c]);
  }
  __device__ void load(int Vs, int s, int q, Pair& v) const {
    ld_pair(pair_at(r + (long)q * 2 * Vs, s), v.r[0], v.r[1]);
    ld_pair(pair_at(p + (long)q * 2 * Vs, s), v.p[0], v.p[1]);
  }
  __device__ void form(const Pair& v, int Vs, int s, int q, bool live, Cx<double>& a,
                       Cx<double>& b) const {
    a = step(v.r[0], v.p[0]);
    b = step(v.r[1], v.p[1]);
    if (live) st_pair(pair_at(next + (long)q * 2 * Vs, s), a, b);
  }
};

// The half spinor of the hop (NU, FWD): U (1 + g_nu) psi(s - nu) or U^dagger
// (1 - g_nu) psi(s + nu), before expansion.
template <typename R, int NU, bool FWD>
__device__ __forceinline__ void hop_half(const Cx<R> (&u)[9], const Cx<R> (&psi)[12],
                                         Cx<R> (&uh)[6]) {
  Cx<R> h[6];
  project<R, NU, FWD ? -1 : +1>(psi, h);
  link_mul<R, FWD>(u, h, uh);
}
template <typename R, int NU, bool FWD, typename In>
__device__ __forceinline__ void hop_half_at(const typename Vec2<R>::T* __restrict__ links,
                                            const In& in, const Geometry& g, int s, bool g5in,
                                            Cx<R> (&uh)[6]) {
  const int n = neighbour<NU, FWD>(s, g);
  Cx<R> u[9], psi[12];
  load_link_u(links, g.Vs, NU, FWD ? s : n, u);
  in.load(g.Vs, n, g5in, psi);
  hop_half<R, NU, FWD>(u, psi, uh);
}

// acc += the share of component C (3 spin + colour) in the expansion of the hop
// (NU, S) with half spinor h[i * 64], as expand_acc adds it.
template <typename R, int NU, int S, int C>
__device__ __forceinline__ void expand_one(Cx<R>& acc, const typename Vec2<R>::T* h, R coef) {
  constexpr int spin = C / 3, col = C % 3;
  const R cs = (S > 0) ? coef : -coef;
  auto at = [&](int i) {
    const typename Vec2<R>::T v = h[i * 64];
    return Cx<R>{v.x, v.y};
  };
  if constexpr (spin == 0) acc_add(acc, coef, at(col));
  else if constexpr (spin == 1) acc_add(acc, coef, at(3 + col));
  else if constexpr (NU == 0) acc_add(acc, cs, mul_i(at(spin == 2 ? 3 + col : col)));
  else if constexpr (NU == 1) acc_add(acc, spin == 2 ? cs : -cs, at(spin == 2 ? 3 + col : col));
  else if constexpr (NU == 2) acc_add(acc, spin == 2 ? cs : -cs, mul_i(at(spin == 2 ? col : 3 + col)));
  else acc_add(acc, cs, at(spin == 2 ? col : 3 + col));
}

// Component C of the hop sum, the eight hops in order; hops: [8][6][64] at the lane.
template <typename R, int C>
__device__ __forceinline__ Cx<R> hop_sum(const typename Vec2<R>::T* hops, const HopR<R>& hc) {
  Cx<R> acc = {R(0), R(0)};
  constexpr int H = 6 * 64;
  expand_one<R, 0, +1, C>(acc, hops + 0 * H, hc.fwd[0]);
  expand_one<R, 0, -1, C>(acc, hops + 1 * H, hc.bwd[0]);
  expand_one<R, 1, +1, C>(acc, hops + 2 * H, hc.fwd[1]);
  expand_one<R, 1, -1, C>(acc, hops + 3 * H, hc.bwd[1]);
  expand_one<R, 2, +1, C>(acc, hops + 4 * H, hc.fwd[2]);
  expand_one<R, 2, -1, C>(acc, hops + 5 * H, hc.bwd[2]);
  expand_one<R, 3, +1, C>(acc, hops + 6 * H, hc.fwd[3]);
  expand_one<R, 3, -1, C>(acc, hops + 7 * H, hc.bwd[3]);
  return acc;
}

// The workgroup's 64 sites from site0 on (sites from g.V on are skipped; every
// wave reaches the barriers).  part != nullptr: also the sums over the 64 sites
// of conj(w) out (complex) and |out|^2 into part[0..3), w the source field at
// `w` (library layout), summed per site over the components and then over the
// lanes as the one-thread-per-site kernels do.
template <typename R, bool PART, typename In, typename Out>
__device__ __forceinline__ void hops_body(const typename Vec2<R>::T* __restrict__ links,
                                          const In& in, const Out& out, const Geometry& g,
                                          const HopR<R>& hc, int site0, bool g5in, bool g5out,
                                          const typename Vec2<R>::T* __restrict__ w,
                                          double* __restrict__ part) {
  using T2 = typename Vec2<R>::T;
  __shared__ T2 hops[8 * 6 * 64];
  __shared__ double prod[PART ? 12 * 3 * 64 : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int s = site0 + lane;
  const bool live = s < g.V;
  const int q = wave;  // the component pair formed after the barrier (waves 0 to 5)
  Cx<R> p0 = {R(0), R(0)}, p1 = p0, w0 = p0, w1 = p0;
  Cx<R> uh[6];
  if constexpr (In::kFormed) {
    // all loads, the input's head meanwhile, then the arithmetic (lanes past the
    // end load the last site); takes 161 registers against 96 with each wave's
    // loads in its own case, so for the small grids of latency-bound launches only
    const int sl = live ? s : g.V - 1;
    int n;
    switch (wave) {
      case 0: n = neighbour<0, false>(sl, g); break;
      case 1: n = neighbour<0, true>(sl, g); break;
      case 2: n = neighbour<1, false>(sl, g); break;
      case 3: n = neighbour<1, true>(sl, g); break;
      case 4: n = neighbour<2, false>(sl, g); break;
      case 5: n = neighbour<2, true>(sl, g); break;
      case 6: n = neighbour<3, false>(sl, g); break;
      default: n = neighbour<3, true>(sl, g); break;
    }
    Cx<R> u[9], psi[12];
    typename In::Spinor nb;
    typename In::Pair own;
    load_link_u(links, g.Vs, wave >> 1, (wave & 1) ? sl : n, u);
    in.load(g.Vs, n, nb);
    if (q < 6) in.load(g.Vs, sl, q, own);
    in.head();
    if (q < 6) in.form(own, g.Vs, sl, q, live, p0, p1);
    in.form(nb, psi);
    switch (wave) {
      case 0: hop_half<R, 0, false>(u, psi, uh); break;
      case 1: hop_half<R, 0, true>(u, psi, uh); break;
      case 2: hop_half<R, 1, false>(u, psi, uh); break;
      case 3: hop_half<R, 1, true>(u, psi, uh); break;
      case 4: hop_half<R, 2, false>(u, psi, uh); break;
      case 5: hop_half<R, 2, true>(u, psi, uh); break;
      case 6: hop_half<R, 3, false>(u, psi, uh); break;
      default: hop_half<R, 3, true>(u, psi, uh); break;
    }
  } else if (live) {
    if (q < 6) {
      in.load_pair(g.Vs, s, q, p0, p1);
      if (PART && part) ld_pair(pair_at(w + (long)q * 2 * g.Vs, s), w0, w1);
    }
    switch (wave) {
      case 0: hop_half_at<R, 0, false>(links, in, g, s, g5in, uh); break;
      case 1: hop_half_at<R, 0, true>(links, in, g, s, g5in, uh); break;
      case 2: hop_half_at<R, 1, false>(links, in, g, s, g5in, uh); break;
      case 3: hop_half_at<R, 1, true>(links, in, g, s, g5in, uh); break;
      case 4: hop_half_at<R, 2, false>(links, in, g, s, g5in, uh); break;
      case 5: hop_half_at<R, 2, true>(links, in, g, s, g5in, uh); break;
      case 6: hop_half_at<R, 3, false>(links, in, g, s, g5in, uh); break;
      default: hop_half_at<R, 3, true>(links, in, g, s, g5in, uh); break;
    }
  }
  if (live) {
#pragma unroll
    for (int i = 0; i < 6; ++i) hops[(wave * 6 + i) * 64 + lane] = T2{uh[i].re, uh[i].im};
  }
  __syncthreads();
  if (q < 6) {
    Cx<R> a0 = {R(0), R(0)}, a1 = a0;
    if (live) {
      const T2* h = hops + lane;
      switch (q) {
        case 0: a0 = hop_sum<R, 0>(h, hc); a1 = hop_sum<R, 1>(h, hc); break;
        case 1: a0 = hop_sum<R, 2>(h, hc); a1 = hop_sum<R, 3>(h, hc); break;
        case 2: a0 = hop_sum<R, 4>(h, hc); a1 = hop_sum<R, 5>(h, hc); break;
        case 3: a0 = hop_sum<R, 6>(h, hc); a1 = hop_sum<R, 7>(h, hc); break;
        case 4: a0 = hop_sum<R, 8>(h, hc); a1 = hop_sum<R, 9>(h, hc); break;
        default: a0 = hop_sum<R, 10>(h, hc); a1 = hop_sum<R, 11>(h, hc); break;
      }
      if (g5in && q >= 3) {
        p0 = -p0;
        p1 = -p1;
      }
      a0 = p0 - a0;
      a1 = p1 - a1;
      if (g5out && q >= 3) {
        a0 = -a0;
        a1 = -a1;
      }
      out.store_pair(g.Vs, s, q, a0, a1);
    }
    if (PART && part) {
      auto put = [&](int c, Cx<R> o, Cx<R> wv) {
        const Cx<double> t64 = {(double)o.re, (double)o.im};
        const Cx<double> w64 = {(double)wv.re, (double)wv.im};
        const Cx<double> d = cmulc(w64, t64);
        prod[(c * 3 + 0) * 64 + lane] = d.re;
        prod[(c * 3 + 1) * 64 + lane] = d.im;
        prod[(c * 3 + 2) * 64 + lane] = cnorm2(t64);
      };
      put(2 * q, a0, w0);
      put(2 * q + 1, a1, w1);
    }
  }
  if (PART && part) {
    __syncthreads();
    if (wave < 3) {
      double v = 0.0;
#pragma unroll
      for (int c = 0; c < 12; ++c) v += prod[(c * 3 + wave) * 64 + lane];
      v = wave_sum(v);
      if (lane == 0) part[wave] = v;
    }
  }
}

}  // namespace ovs
