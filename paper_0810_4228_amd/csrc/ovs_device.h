// Device-side helpers: complex arithmetic in registers, storage conversion,
// lattice neighbours and deterministic workgroup reductions.
#pragma once

#include <hip/hip_runtime.h>

namespace ovs {

template <typename R> struct Vec2;
template <> struct Vec2<double> { using T = double2; };
template <> struct Vec2<float> { using T = float2; };

template <typename R>
struct Cx {
  R re, im;
};

template <typename R>
__device__ __forceinline__ Cx<R> cx(R a, R b) { return Cx<R>{a, b}; }

template <typename R>
__device__ __forceinline__ Cx<R> operator+(Cx<R> a, Cx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <typename R>
__device__ __forceinline__ Cx<R> operator-(Cx<R> a, Cx<R> b) { return {a.re - b.re, a.im - b.im}; }
template <typename R>
__device__ __forceinline__ Cx<R> operator-(Cx<R> a) { return {-a.re, -a.im}; }
// i * a
template <typename R>
__device__ __forceinline__ Cx<R> mul_i(Cx<R> a) { return {-a.im, a.re}; }
template <typename R>
__device__ __forceinline__ Cx<R> scale(R s, Cx<R> a) { return {s * a.re, s * a.im}; }
// a * b
template <typename R>
__device__ __forceinline__ Cx<R> cmul(Cx<R> a, Cx<R> b) {
  return {fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re)};
}
// conj(a) * b
template <typename R>
__device__ __forceinline__ Cx<R> cmulc(Cx<R> a, Cx<R> b) {
  return {fma(a.re, b.re, a.im * b.im), fma(a.re, b.im, -(a.im * b.re))};
}
// acc + a * b
template <typename R>
__device__ __forceinline__ Cx<R> cfma(Cx<R> a, Cx<R> b, Cx<R> acc) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(-a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(a.im, b.re, acc.im);
  return acc;
}
// acc + conj(a) * b
template <typename R>
__device__ __forceinline__ Cx<R> cfmac(Cx<R> a, Cx<R> b, Cx<R> acc) {
  acc.re = fma(a.re, b.re, acc.re);
  acc.re = fma(a.im, b.im, acc.re);
  acc.im = fma(a.re, b.im, acc.im);
  acc.im = fma(-a.im, b.re, acc.im);
  return acc;
}
template <typename R>
__device__ __forceinline__ R cnorm2(Cx<R> a) { return fma(a.re, a.re, a.im * a.im); }

__device__ __forceinline__ Cx<double> ld(const double2* p) {
  double2 v = *p;
  return {v.x, v.y};
}
__device__ __forceinline__ Cx<float> ld(const float2* p) {
  float2 v = *p;
  return {v.x, v.y};
}
__device__ __forceinline__ void st(double2* p, Cx<double> a) { *p = make_double2(a.re, a.im); }
__device__ __forceinline__ void st(float2* p, Cx<float> a) { *p = make_float2(a.re, a.im); }
// FP64 view of a stored value
__device__ __forceinline__ Cx<double> ld64(const double2* p) { return ld(p); }
__device__ __forceinline__ Cx<double> ld64(const float2* p) {
  float2 v = *p;
  return {(double)v.x, (double)v.y};
}
// store an FP64 value in storage precision (round to nearest)
__device__ __forceinline__ void st64(double2* p, Cx<double> a) { *p = make_double2(a.re, a.im); }
__device__ __forceinline__ void st64(float2* p, Cx<double> a) {
  *p = make_float2((float)a.re, (float)a.im);
}
// streaming (non-temporal) stores of an FP64 value in storage precision
__device__ __forceinline__ void st64_nt(double2* p, Cx<double> a) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  v2 v = {a.re, a.im};
  __builtin_nontemporal_store(v, reinterpret_cast<v2*>(p));
}
__device__ __forceinline__ void st64_nt(float2* p, Cx<double> a) {
  typedef float v2 __attribute__((ext_vector_type(2)));
  v2 v = {(float)a.re, (float)a.im};
  __builtin_nontemporal_store(v, reinterpret_cast<v2*>(p));
}
// the stored value as seen after rounding to storage precision
__device__ __forceinline__ Cx<double> round_to(const double2*, Cx<double> a) { return a; }
__device__ __forceinline__ Cx<double> round_to(const float2*, Cx<double> a) {
  return {(double)(float)a.re, (double)(float)a.im};
}

// Two adjacent complex values (a component pair of the field layout) in one
// access: a 16-byte load or store in FP32, two in FP64.
__device__ __forceinline__ void ld_pair(const float2* p, Cx<float>& a, Cx<float>& b) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  a = {v.x, v.y};
  b = {v.z, v.w};
}
__device__ __forceinline__ void ld_pair(const double2* p, Cx<double>& a, Cx<double>& b) {
  a = ld(p);
  b = ld(p + 1);
}
__device__ __forceinline__ void st_pair(float2* p, Cx<float> a, Cx<float> b) {
  *reinterpret_cast<float4*>(p) = make_float4(a.re, a.im, b.re, b.im);
}
__device__ __forceinline__ void st_pair(double2* p, Cx<double> a, Cx<double> b) {
  st(p, a);
  st(p + 1, b);
}
__device__ __forceinline__ void st_pair_nt(float2* p, Cx<float> a, Cx<float> b) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  v4 v = {a.re, a.im, b.re, b.im};
  __builtin_nontemporal_store(v, reinterpret_cast<v4*>(p));
}
__device__ __forceinline__ void st_pair_nt(double2* p, Cx<double> a, Cx<double> b) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  v2 va = {a.re, a.im}, vb = {b.re, b.im};
  __builtin_nontemporal_store(va, reinterpret_cast<v2*>(p));
  __builtin_nontemporal_store(vb, reinterpret_cast<v2*>(p + 1));
}

// A pair of stored values as FP64, and a pair stored in storage precision
// (streaming), for the elementwise kernels.
__device__ __forceinline__ void ld_pair64(const float2* p, Cx<double>& a, Cx<double>& b) {
  Cx<float> x, y;
  ld_pair(p, x, y);
  a = {(double)x.re, (double)x.im};
  b = {(double)y.re, (double)y.im};
}
__device__ __forceinline__ void ld_pair64(const double2* p, Cx<double>& a, Cx<double>& b) {
  ld_pair(p, a, b);
}
__device__ __forceinline__ void st_pair64(float2* p, Cx<double> a, Cx<double> b) {
  st_pair(p, Cx<float>{(float)a.re, (float)a.im}, Cx<float>{(float)b.re, (float)b.im});
}
__device__ __forceinline__ void st_pair64(double2* p, Cx<double> a, Cx<double> b) {
  st_pair(p, a, b);
}
__device__ __forceinline__ void st_pair64_nt(float2* p, Cx<double> a, Cx<double> b) {
  st_pair_nt(p, Cx<float>{(float)a.re, (float)a.im}, Cx<float>{(float)b.re, (float)b.im});
}
__device__ __forceinline__ void st_pair64_nt(double2* p, Cx<double> a, Cx<double> b) {
  st_pair_nt(p, a, b);
}

__device__ __forceinline__ Cx<double> cconj(Cx<double> a) { return {a.re, -a.im}; }
__device__ __forceinline__ Cx<double> c64(double2 v) { return {v.x, v.y}; }
__device__ __forceinline__ double2 d2(Cx<double> a) { return make_double2(a.re, a.im); }
__device__ __forceinline__ Cx<double> cdiv(Cx<double> a, Cx<double> b) {
  // Smith's algorithm for a / b
  if (fabs(b.re) >= fabs(b.im)) {
    double r = b.im / b.re, den = b.re + b.im * r;
    return {(a.re + a.im * r) / den, (a.im - a.re * r) / den};
  } else {
    double r = b.re / b.im, den = b.re * r + b.im;
    return {(a.re * r + a.im) / den, (a.im * r - a.re) / den};
  }
}
__device__ __forceinline__ double cabs1(Cx<double> a) { return hypot(a.re, a.im); }

// 1 / d to within an ulp by two Newton steps, and n / d from it with one
// residual correction: the quotient an IEEE division returns (whose expansion
// is these steps between scalings by powers of two) while no intermediate
// leaves the normal range.
__device__ __forceinline__ double newton_rcp(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(y, fma(-d, y, 1.0), y);
  return fma(y, fma(-d, y, 1.0), y);
}
__device__ __forceinline__ double quotient(double n, double d, double y) {
  const double q = n * y;
  return fma(fma(-d, q, n), y, q);
}

// c ? a : b by components (a select of whole structures can go through scratch)
__device__ __forceinline__ Cx<double> csel(bool c, Cx<double> a, Cx<double> b) {
  return {c ? a.re : b.re, c ? a.im : b.im};
}

// The pivot decision and multiplier of a tridiagonal elimination step with the
// real subdiagonal entry b and the pivot candidate c: sw = |b| > |c| as hypot
// compares them, m = sw ? c / b : b / c as cdiv forms them (Smith's algorithm;
// by a real divisor two plain quotients).  Squares where they are apart by more
// than their rounding and every quotient is in the normal range, selects instead
// of branches; hypot and IEEE divisions for the rest (skipped when no lane needs
// them).
__device__ __forceinline__ Cx<double> pivot_quotient(double b, Cx<double> c, bool& sw) {
  const double b2 = b * b, c2 = fma(c.re, c.re, c.im * c.im);
  const double top = fmax(b2, c2), low = fmin(b2, c2);
  sw = b2 > c2;
  const bool big = fabs(c.re) >= fabs(c.im);
  const double hi = big ? c.re : c.im, lo = big ? c.im : c.re;
  double rr = quotient(lo, hi, newton_rcp(hi));
  const bool plain = (top > low * 1.0000000001) & (top < 1e280) & (c2 > 1e-280);
  if (!plain) {
    sw = fabs(b) > cabs1(c);
    rr = lo / hi;
  }
  const double den = sw ? b : hi + lo * rr;
  const double br = b * rr;
  const double nre = sw ? c.re : (big ? b : br);
  const double nim = sw ? c.im : (big ? -br : -b);
  const double y = newton_rcp(den);
  Cx<double> m = {quotient(nre, den, y), quotient(nim, den, y)};
  if (!plain) m = {nre / den, nim / den};
  return m;
}

// cdiv(a, b) with the quotients formed as above while all of them are in the
// normal range, cdiv itself for the rest.
__device__ __forceinline__ Cx<double> cdiv_fast(Cx<double> a, Cx<double> b) {
  const double b2 = fma(b.re, b.re, b.im * b.im), na = fabs(a.re) + fabs(a.im);
  const bool big = fabs(b.re) >= fabs(b.im);
  const double hi = big ? b.re : b.im, lo = big ? b.im : b.re;
  const double r = quotient(lo, hi, newton_rcp(hi));
  const double den = hi + lo * r;
  const double y = newton_rcp(den);
  const double nre = big ? a.re + a.im * r : a.re * r + a.im;
  const double nim = big ? a.im - a.re * r : a.im * r - a.re;
  Cx<double> q = {quotient(nre, den, y), quotient(nim, den, y)};
  const bool plain =
      (b2 > 1e-280) & (b2 < 1e280) & (((na > 1e-150) & (na < 1e150)) | (na == 0.0));
  if (!plain) q = cdiv(a, b);
  return q;
}

// The value that lane l (uniform) of the wave holds.
__device__ __forceinline__ double lane_value(double v, int l) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
  return __hiloint2double(hi, lo);
}


// ---- XCD-aware workgroup -> (site tile, source block) map -----------------
// Workgroups are handed to the 8 XCDs round robin (bid % 8).  The map gives
// each XCD a contiguous range of tiles so that neighbour sites read by a tile
// were loaded into the same XCD's L2 by nearby tiles.  On "planar" lattices
// (the tile size divides Lx*Ly) the XCD ranges are chunks of time slices and
// the tiles inside a chunk are ordered plane-tile, then t, then z, so the
// x/y/z/t neighbours of a tile are at most (tiles per plane)*(t per chunk)
// tiles away.  The source blocks of one tile are adjacent, so its links are
// reused from L2 across blocks.
struct TileMap {
  int ntiles;      // site tiles of `wg` sites
  int nrb;         // source blocks
  int per_xcd;     // workgroups per XCD (grid = 8 * per_xcd)
  int planar;      // tile size divides Lx*Ly
  int ppt;         // tiles per xy plane (planar)
  int tchunk;      // time slices per XCD chunk (planar)
  int wg;          // sites per tile
  int plane;       // Lx*Ly
  int lz;
  int rb_slow;     // source block is the slowest index
  int group;       // > 0: each XCD sweeps its time chunk once per window of
                   // `group` source blocks (adjacent within the window)
  int tiles_xcd;   // tiles of one XCD's time chunk (group > 0)
};

// Tile map of a launch with nrb source blocks and wg-site tiles (stencil.hip).
// order 0: source blocks of a tile adjacent; 1: source block slowest; 2 to 7:
// per XCD time chunk, windows of 1, 2, 3, 4, 6 or all source blocks (planar
// lattices with Lt a multiple of 8; otherwise as order 0).
TileMap make_tile_map(const Geometry& g, int wg, int nrb, int order);

// First site of tile tq.
__device__ __forceinline__ int tile_site(int tq, const TileMap& m) {
  if (!m.planar) return tq * m.wg;
  const int p = tq % m.ppt;
  int r = tq / m.ppt;
  const int tin = r % m.tchunk;
  r /= m.tchunk;
  const int z = r % m.lz;
  const int tc = r / m.lz;
  return p * m.wg + m.plane * (z + m.lz * (tc * m.tchunk + tin));
}

__device__ __forceinline__ bool map_tile(int bid, const TileMap& m, int& site0, int& rb, int& tile) {
  int tq;
  if (m.group > 0) {
    // XCD x owns time chunk x; it sweeps the chunk's tiles (plane tile, t, z)
    // once per window of `group` source blocks, so the sites, links and z / t
    // neighbours a window touches stay within that XCD's L2
    const int local = bid >> 3;
    const int span = m.tiles_xcd * m.group;
    const int grp = local / span, rem = local - grp * span;
    const int tl = rem / m.group;
    rb = grp * m.group + (rem - tl * m.group);
    if (rb >= m.nrb) return false;
    tq = (bid & 7) * m.tiles_xcd + tl;
  } else {
    const int q = (bid & 7) * m.per_xcd + (bid >> 3);
    if (q >= m.ntiles * m.nrb) return false;
    rb = m.rb_slow ? q / m.ntiles : q % m.nrb;
    tq = m.rb_slow ? q % m.ntiles : q / m.nrb;
  }
  tile = tq;
  site0 = tile_site(tq, m);
  return true;
}

// ---- deterministic reductions over one workgroup ------------------------
// Wave64 tree, then a fixed-order pass over the waves in LDS.

// The value of lane l + OFF, for the lanes l < OFF (OFF 1, 2, 4, 8: row shifts
// within 16 lanes; 16, 32: row swaps): register moves, no LDS crossbar.
template <int OFF>
__device__ __forceinline__ double lane_down(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  if constexpr (OFF == 32) {
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double(b[1], a[1]);
  } else if constexpr (OFF == 16) {
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double(b[1], a[1]);
  } else {
    constexpr int kRowShl = 0x100 + OFF;
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, kRowShl, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, lo, kRowShl, 0xf, 0xf, true));
  }
}
// Sum over the 64 lanes, valid in lane 0: the tree of halves (lane + 32, + 16,
// ... + 1).  Bound by the latency of its six steps: register moves instead of
// shuffles through LDS.
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_down<32>(v);
  v += lane_down<16>(v);
  v += lane_down<8>(v);
  v += lane_down<4>(v);
  v += lane_down<2>(v);
  v += lane_down<1>(v);
  return v;
}

// Two values on their way down the tree of halves at once: lanes without bit OFF
// return a + a(lane + OFF), the others b + b(lane - OFF), the sums that wave_sum
// forms at this step.
template <int OFF>
__device__ __forceinline__ double lane_merge(double a, double b) {
  static_assert(OFF == 32 || OFF == 16 || OFF == 8 || OFF == 4 || OFF == 2);
  if constexpr (OFF >= 16) {
    auto swap = [](int x, int y) {
      if constexpr (OFF == 32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
      else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto l = swap(__double2loint(a), __double2loint(b));
    const auto h = swap(__double2hiint(a), __double2hiint(b));
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
  } else {
    const bool up = threadIdx.x & OFF;
    const double keep = up ? b : a, give = up ? a : b;
    auto swap = [](int x) {  // lane ^ OFF
      if constexpr (OFF == 8) return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true);
      else if constexpr (OFF == 2) return __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, true);
      else
        return __builtin_amdgcn_update_dpp(
            0, __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
    };
    return keep + __hiloint2double(swap(__double2hiint(give)), swap(__double2loint(give)));
  }
}
template <int NV, int OFF>
__device__ __forceinline__ double wave_sums_from(double (&v)[NV]) {
  if constexpr (NV == 1) {
    double s = v[0];
    if constexpr (OFF >= 32) s += lane_down<32>(s);
    if constexpr (OFF >= 16) s += lane_down<16>(s);
    if constexpr (OFF >= 8) s += lane_down<8>(s);
    if constexpr (OFF >= 4) s += lane_down<4>(s);
    if constexpr (OFF >= 2) s += lane_down<2>(s);
    if constexpr (OFF >= 1) s += lane_down<1>(s);
    return s;
  } else {
    double w[NV / 2];
#pragma unroll
    for (int j = 0; j < NV / 2; ++j) w[j] = lane_merge<OFF>(v[j], v[j + NV / 2]);
    return wave_sums_from<NV / 2, OFF / 2>(w);
  }
}
// Sums over the workgroup of NV (8, 16 or 32) values per thread, of value j in
// thread j: block_sum's sums with a thread for each last one.  All threads call
// it; lds holds NV doubles a wave.
template <int NV>
__device__ __forceinline__ double block_sums(double (&v)[NV], double* lds) {
  static_assert(NV == 8 || NV == 16 || NV == 32);
  constexpr int L = 64 / NV;  // lanes that end up with one value
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double s = wave_sums_from<NV, 32>(v);
  if (lane % L == 0) lds[wave * NV + lane / L] = s;
  __syncthreads();
  double a = 0.0;
  if ((int)threadIdx.x < NV) {
    a = lds[threadIdx.x];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) a += lds[w * NV + threadIdx.x];
  }
  __syncthreads();
  return a;
}

// Sums `n` values per thread over the first nw waves of the workgroup (all its
// threads call it); result valid in thread 0.  lds must hold nw * n doubles.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds, int nw) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // NV values (padded to a power of two P) share one tree, P + 5 - log2 P additions
  // a lane instead of 6 NV, with the same sums (16^3 x 32 x 12 solve 208.8 -> 204.3
  // ms, 8^4 gradient 12.75 -> 12.24 ms)
  constexpr int P = NV == 1 ? 1 : NV <= 2 ? 2 : NV <= 4 ? 4 : NV <= 8 ? 8 : NV <= 16 ? 16 : 32;
  static_assert(NV <= 32);
  double p[P];
#pragma unroll
  for (int j = 0; j < P; ++j) p[j] = j < NV ? v[j] : 0.0;
  const double s = wave_sums_from<P, 32>(p);
  constexpr int L = 64 / P;
  if (lane % L == 0 && lane / L < NV && wave < nw) lds[wave * NV + lane / L] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      double a = lds[j];
      for (int w = 1; w < nw; ++w) a += lds[w * NV + j];
      v[j] = a;
    }
  }
  __syncthreads();
}
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
  block_sum<NV>(v, lds, blockDim.x >> 6);
}

// partials[b] = workgroup b's share (of nb) of the sum of |T[e]|^2, e < N, by its
// first 256 threads.
template <typename T2>
__device__ __forceinline__ void norm2_part(const T2* __restrict__ T, long N, int b, int nb,
                                           double* __restrict__ partials) {
  __shared__ double lds[4];
  double v[1] = {0.0};
  if (threadIdx.x < 256)
    for (long e = b * 256L + threadIdx.x; e < N; e += nb * 256L) v[0] += cnorm2(ld64(T + e));
  block_sum<1>(v, lds, 4);
  if (threadIdx.x == 0) partials[b] = v[0];
}

// Two adjacent stored values as they come from memory, for loads issued ahead of
// their use (a conversion at the load would wait for it).
template <typename T2> struct RawPair;
template <> struct RawPair<float2> {
  float4 v;
  __device__ void load(const float2* p) { v = *reinterpret_cast<const float4*>(p); }
  __device__ Cx<double> first() const { return {(double)v.x, (double)v.y}; }
  __device__ Cx<double> second() const { return {(double)v.z, (double)v.w}; }
};
template <> struct RawPair<double2> {
  double2 a, b;
  __device__ void load(const double2* p) {
    a = p[0];
    b = p[1];
  }
  __device__ Cx<double> first() const { return {a.x, a.y}; }
  __device__ Cx<double> second() const { return {b.x, b.y}; }
};

}  // namespace ovs
