// HIP kernels for CDNA4 (gfx950): the honeycomb fermion operator of eq. (ferm_op),
// its adjoint, the normal operator M M^dagger + mu^2 (Sec. 3, Sec. 5.1), the fused
// conjugate-gradient iteration in FP64 and complex64, the Krylov helpers of the
// flexible GMRES of Appendix A, and the pseudofermion force of eqs. (p_dot), (eta_xi).
//
// Design (memory-bound stencil, no dense contraction, so no MFMA):
// * one thread per site, kSitesPerThread sites per thread, site-major layout with
//   j fastest so every neighbour stream is a coalesced, shifted copy of the own stream;
//   the neighbour index is computed from the site coordinates, never stored;
// * workgroup ids are remapped so that each XCD walks a contiguous range of tiles and
//   the t +- 1 and i +- 1 neighbours of a tile are mostly in the same XCD's L2;
// * the CG iteration is two kernels: (1) p = r + beta p on the fly, u = M^dagger p,
//   <p, A p> = |u|^2 + mu^2 |p|^2; (2) q = M u + mu^2 p, x += alpha p, r -= alpha q,
//   |r|^2.  Scalars alpha, beta and the convergence test never leave the device;
// * reductions are deterministic and use no atomics: each workgroup stores one
//   partial per tile (wave64 butterfly + fixed LDS combine), and every workgroup of
//   the consuming kernel sums all partials of its system in the same fixed order,
//   so all of them hold bit-identical alpha and beta.  A system's results depend
//   only on its own shape, never on the other systems of the launch.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "hub_device.h"

namespace hub {
namespace {

// Loads in flight per thread in the stencil kernels: site pairs of the complex64
// pair path, and sites of the generic path in FP64 and complex64.  With 8 sites
// per thread (tiles of at most 2048 sites) a 102x102x64 system is 768 workgroups,
// resident in one round at the register use these give; more loads per round would
// cost occupancy, fewer (one pair per round: 7 waves per SIMD) made the solve slower.
#ifndef HUB_PAIRS_PER_ROUND
#define HUB_PAIRS_PER_ROUND 2
#endif
#ifndef HUB_SPT64
#define HUB_SPT64 (HUB_SITES_PER_THREAD < 2 ? HUB_SITES_PER_THREAD : 2)
#endif
#ifndef HUB_SPT32
#define HUB_SPT32 (HUB_SITES_PER_THREAD < 2 ? HUB_SITES_PER_THREAD : 2)
#endif
template <typename R> struct Spt;
template <> struct Spt<double> { static constexpr int v = HUB_SPT64; };
template <> struct Spt<float> { static constexpr int v = HUB_SPT32; };

// cos x and sin x in FP64 for the public operator kernels (the phase of each site from
// phi): Cody-Waite reduction r = x - q pi/2 with q the integer nearest 2x/pi and pi/2
// split into the nearest double and its remainder (each product inside one FMA, so r is
// exact to an ulp for |q| < 2^20), then the Taylor series of cos r and sin r through
// degree 18 and 17 on |r| <= pi/4 (first omitted terms below 5e-17) and a turn by q
// quarter turns.  Error against e^{ix}: under 2e-16, without the library routine's
// branch for huge arguments.
__device__ __forceinline__ void cis64(double x, double& c, double& s) {
  const double q = rint(x * 0.6366197723675814);
  double r = fma(-q, 1.5707963267948966, x);
  r = fma(-q, 6.123233995736766e-17, r);
  const double r2 = r * r;
  double ps = 2.8114572543455206e-15;         // 1/17!
  ps = fma(ps, r2, -7.647163731819816e-13);   // -1/15!
  ps = fma(ps, r2, 1.6059043836821613e-10);   // 1/13!
  ps = fma(ps, r2, -2.505210838544172e-08);   // -1/11!
  ps = fma(ps, r2, 2.7557319223985893e-06);   // 1/9!
  ps = fma(ps, r2, -0.0001984126984126984);   // -1/7!
  ps = fma(ps, r2, 0.008333333333333333);     // 1/5!
  ps = fma(ps, r2, -0.16666666666666666);     // -1/3!
  const double sr = fma(ps * r2, r, r);
  double pc = 1.5619206968586225e-16;         // 1/18!
  pc = fma(pc, r2, -4.779477332387385e-14);   // -1/16!
  pc = fma(pc, r2, 1.1470745597729725e-11);   // 1/14!
  pc = fma(pc, r2, -2.08767569878681e-09);    // -1/12!
  pc = fma(pc, r2, 2.755731922398589e-07);    // 1/10!
  pc = fma(pc, r2, -2.48015873015873e-05);    // -1/8!
  pc = fma(pc, r2, 0.001388888888888889);     // 1/6!
  pc = fma(pc, r2, -0.041666666666666664);    // -1/4!
  pc = fma(pc, r2, 0.5);                      // 1/2!
  const double cr = fma(-pc, r2, 1.0);
  const int k = (int)q & 3;
  c = (k == 0) ? cr : (k == 1) ? -sr : (k == 2) ? -cr : sr;
  s = (k == 0) ? sr : (k == 1) ? cr : (k == 2) ? -sr : -cr;
}


// Workgroups are dispatched round-robin over the XCDs; give XCD x the x-th
// contiguous chunk of logical tiles.
__device__ __forceinline__ int xcd_remap(int b, int G) {
  const int per = G / kNumXcd, rem = G % kNumXcd;
  const int x = b % kNumXcd, k = b / kNumXcd;
  return (x < rem) ? x * (per + 1) + k : rem * (per + 1) + (x - rem) * per + k;
}

// The phase e^{i phi} a stencil needs, from one of three sources:
//  * AnglePhi - phi itself (FP64); cos and sin from cis64 per site (the public
//               operator kernels, whose input is phi);
//  * PhasePhi - (cos phi, sin phi) precomputed once per solve (the FP64 solver
//               kernels: a 16-byte load replaces a sincos per site);
//  * Angle32  - phi reduced to [-pi, pi] and rounded to float once per solve, cos and
//               sin from cis32 (the complex64 solver kernels: a 4-byte load and a few
//               FMAs, against 8 bytes for a precomputed complex64 phase).
// load(k) returns the raw value of site k, cs() turns it into (cos, sin); load2 / cs2
// do the same for the two sites k, k+1 (k even) of the complex64 pair path.
template <typename R> struct AnglePhi;
template <> struct AnglePhi<double> {
  Real<double> a;
  using Raw = double;
  __device__ __forceinline__ explicit AnglePhi(const void* q) : a(q) {}
  __device__ __forceinline__ Raw load(int k) const { return a[k]; }
  __device__ __forceinline__ void cs(Raw v, double& c, double& s) const { cis64(v, c, s); }
};
struct Angle32 {
  Real<float> a;
  using Raw = float;
  using Raw2 = hub_f2v;
  __device__ __forceinline__ explicit Angle32(const void* q) : a(q) {}
  __device__ __forceinline__ Raw load(int k) const { return a[k]; }
  __device__ __forceinline__ void cs(Raw v, float& c, float& s) const { cis32(v, c, s); }
  __device__ __forceinline__ Raw2 load2(int k) const { return a.pair(k); }
  __device__ __forceinline__ void cs2(Raw2 v, int h, float& c, float& s) const { cis32(h ? v.y : v.x, c, s); }
};
template <typename R> struct PhasePhi {
  using C = typename V2<R>::T;
  Vec<C> p;
  using Raw = C;
  using Raw2 = C64x2;
  __device__ __forceinline__ explicit PhasePhi(const void* q) : p(q) {}
  __device__ __forceinline__ Raw load(int k) const { return p[k]; }
  __device__ __forceinline__ void cs(Raw v, R& c, R& s) const {
    c = v.x;
    s = v.y;
  }
  __device__ __forceinline__ Raw2 load2(int k) const { return p.pair(k); }
  __device__ __forceinline__ void cs2(Raw2 v, int h, float& c, float& s) const {
    c = h ? v.b.x : v.a.x;
    s = h ? v.b.y : v.a.y;
  }
};

// The stencil of M (DAG = false) or M^dagger (DAG = true) at site n (eq. (ferm_op) and its
// conjugate transpose):
//   M,  A row: -x(n) + s (e^{ i phi(n)}  - m) x(t-1) - kappa sum_bonds x_B
//   M,  B row: +x(n) - s (e^{-i phi(n)}  - m) x(t+1) - kappa sum_bonds x_A
//   M+, A row: -x(n) + s (e^{-i phi(tn)} - m) x(t+1) - kappa sum_bonds x_B
//   M+, B row: +x(n) - s (e^{ i phi(tn)} - m) x(t-1) - kappa sum_bonds x_A
// with s = -1 on a hop across the antiperiodic temporal boundary.
//
// Index part of the stencil at site n: own site, temporal
// neighbour, three bonds, the phi index and the row's signs.
struct SiteIdx {
  int n, tn, h0, h1, h2, pn;
  bool isA;
  bool wrap;
};

// The same from the coordinates of site n: cell (i, j) and plane q2 = 2 t + s.
template <bool DAG>
__device__ __forceinline__ SiteIdx site_index_at(const Geom& g, int n, int i, int j, uint32_t q2) {
  SiteIdx s;
  s.isA = (q2 & 1u) == 0;
  const int t = (int)(q2 >> 1);
  const int P2 = 2 * g.P;
  if (s.isA == DAG) {
    s.wrap = t == g.Nt - 1;
    s.tn = s.wrap ? n - (g.Nt - 1) * P2 : n + P2;
  } else {
    s.wrap = t == 0;
    s.tn = s.wrap ? n + (g.Nt - 1) * P2 : n - P2;
  }
  if (s.isA) {
    const int b = n + g.P;
    s.h0 = b;
    s.h1 = (i > 0) ? b - g.L2 : b + (g.L1 - 1) * g.L2;
    s.h2 = (j > 0) ? b - 1 : b + g.L2 - 1;
  } else {
    const int a = n - g.P;
    s.h0 = a;
    s.h1 = (i < g.L1 - 1) ? a + g.L2 : a - (g.L1 - 1) * g.L2;
    s.h2 = (j < g.L2 - 1) ? a + 1 : a - (g.L2 - 1);
  }
  s.n = n;
  s.pn = DAG ? s.tn : n;
  return s;
}

template <bool DAG>
__device__ __forceinline__ SiteIdx site_index(const Geom& g, int n) {
  const uint32_t q1 = fdiv((uint32_t)n, g.dL2);
  const int j = n - (int)q1 * g.L2;
  const uint32_t q2 = fdiv(q1, g.dL1);
  const int i = (int)q1 - (int)q2 * g.L1;
  return site_index_at<DAG>(g, n, i, j, q2);
}

template <typename R, bool DAG, typename C>
__device__ __forceinline__ C stencil_combine(const Geom& g, const SiteIdx& st, R c, R s, C xs, C xt, C x0, C x1,
                                             C x2) {
  const R sgn = st.wrap ? R(-1) : R(1);
  const R es = (st.isA != DAG) ? s : -s;
  const R cr = sgn * (c - (R)g.ms), ci = sgn * es;
  // the product written out: left to the compiler, the rounded half differs from kernel to kernel
  const R tr = fma(cr, xt.x, -(ci * xt.y)), ti = fma(cr, xt.y, ci * xt.x);
  const R sig = st.isA ? R(-1) : R(1);
  const R kap = (R)g.kappa;
  C y;
  y.x = sig * (xs.x - tr) - kap * (x0.x + x1.x + x2.x);
  y.y = sig * (xs.y - ti) - kap * (x0.y + x1.y + x2.y);
  return y;
}

// Apply the stencil to the kSitesPerThread sites of this thread in a tile, SPT
// sites at a time: all index arithmetic first, then every load of the SPT sites
// (raw stencil inputs `ld`, phi and the epilogue's own operands `pre`), then, in
// the first round only, `mid()` (which may compute scalars from partial sums and
// returns false to skip the rest), then `cook(raw)` turns raw loads into stencil
// inputs, the arithmetic, and `post(n, y, self, pre_value)`.  Issuing the loads
// of several sites before the first wait keeps enough bytes in flight to cover
// HBM latency, and the partial-sum prologue of `mid` overlaps those loads.  The
// thread's sites are base + m*kBlock below `end` (the end of its tile); lanes past
// it load a valid site and skip `post`.
template <typename R, bool DAG, int SPT, int TOTAL = kSitesPerThread, typename Phi, typename Load, typename Cook,
          typename Pre, typename Mid, typename Post>
__device__ __forceinline__ void stencil_sites(const Geom& g, const Phi& phi, int base, int end, Load ld, Cook cook,
                                              Pre pre, Mid mid, Post post) {
  using C = typename V2<R>::T;
  using RW = decltype(ld(0));
  using PV = decltype(pre(0));
  static_assert(TOTAL % SPT == 0, "SPT must divide TOTAL");
#pragma unroll
  for (int r0 = 0; r0 < TOTAL; r0 += SPT) {
    SiteIdx st[SPT];
    bool ok[SPT];
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      int n = base + (r0 + m) * kBlock;
      ok[m] = n < end;
      n = ok[m] ? n : end - 1;
      st[m] = site_index<DAG>(g, n);
    }
    RW xs[SPT], xt[SPT], x0[SPT], x1[SPT], x2[SPT];
    typename Phi::Raw ph[SPT];
    PV pv[SPT];
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      xs[m] = ld(st[m].n);
      xt[m] = ld(st[m].tn);
      x0[m] = ld(st[m].h0);
      x1[m] = ld(st[m].h1);
      x2[m] = ld(st[m].h2);
      ph[m] = phi.load(st[m].pn);
      pv[m] = pre(st[m].n);
    }
    if (r0 == 0 && !mid()) return;
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      const C s0 = cook(xs[m]);
      R c, s;
      phi.cs(ph[m], c, s);
      const C y = stencil_combine<R, DAG>(g, st[m], c, s, s0, cook(xt[m]), cook(x0[m]), cook(x1[m]),
                                          cook(x2[m]));
      if (ok[m]) post(st[m].n, y, s0, pv[m]);
    }
  }
}

struct NoMid {
  __device__ __forceinline__ bool operator()() const { return true; }
};
struct Same {
  template <typename T>
  __device__ __forceinline__ T operator()(T v) const {
    return v;
  }
};

struct NoPre {
  int dummy;
};

// ---------------------------------------------------------------------------
// Complex64 stencil on site pairs (j, j+1), j even, for lattices with even L2.
// A pair never straddles a row, so the own values, the temporal neighbours, the
// sublattice partners and the i-neighbour row are 16-byte loads of two sites; of
// the j-bonds one is the partner load's other half and one is an extra 8-byte
// load.  This halves the memory instructions per site of the complex64 kernels.
// ---------------------------------------------------------------------------
struct PairIdx {
  int n, tn, h0, h1, hx;
  bool isA, wrap;
};

// Index part of the stencil on the pair (n, n + 1), n even, from the coordinates of
// site n: cell (i, j) and plane q2 = 2 t + s.
template <bool DAG>
__device__ __forceinline__ PairIdx pair_index_at(const Geom& g, int n, int i, int j, uint32_t q2) {
  PairIdx s;
  s.isA = (q2 & 1u) == 0;
  const int t = (int)(q2 >> 1);
  const int P2 = 2 * g.P;
  if (s.isA == DAG) {
    s.wrap = t == g.Nt - 1;
    s.tn = s.wrap ? n - (g.Nt - 1) * P2 : n + P2;
  } else {
    s.wrap = t == 0;
    s.tn = s.wrap ? n + (g.Nt - 1) * P2 : n - P2;
  }
  if (s.isA) {
    const int b = n + g.P;
    s.h0 = b;
    s.h1 = (i > 0) ? b - g.L2 : b + (g.L1 - 1) * g.L2;
    s.hx = (j > 0) ? b - 1 : b + g.L2 - 1;  // B(i, j-1)
  } else {
    const int a = n - g.P;
    s.h0 = a;
    s.h1 = (i < g.L1 - 1) ? a + g.L2 : a - (g.L1 - 1) * g.L2;
    s.hx = (j + 2 < g.L2) ? a + 2 : a + 2 - g.L2;  // A(i, j+2)
  }
  s.n = n;
  return s;
}

template <bool DAG>
__device__ __forceinline__ PairIdx pair_index(const Geom& g, int n) {
  const uint32_t q1 = fdiv((uint32_t)n, g.dL2);
  const int j = n - (int)q1 * g.L2;
  const uint32_t q2 = fdiv(q1, g.dL1);
  const int i = (int)q1 - (int)q2 * g.L1;
  return pair_index_at<DAG>(g, n, i, j, q2);
}

// The stencil on one site pair: own values xs, temporal neighbours xt, the partner
// pair x0, the i-neighbour pair x1 and the extra j-neighbour xe; csf(h, c, s) gives the
// phase (cos, sin) of row h of the pair, evaluated as the row is reached.
template <bool DAG, typename CsF>
__device__ __forceinline__ C64x2 pair_stencil(const Geom& g, const PairIdx& sm, CsF csf, C64x2 xs, C64x2 xt,
                                              C64x2 x0, C64x2 x1, float2 xe) {
  // bond sums of the two sites
  float2 b0, b1;
  if (sm.isA) {
    b0.x = x0.a.x + x1.a.x + xe.x;
    b0.y = x0.a.y + x1.a.y + xe.y;
    b1.x = x0.b.x + x1.b.x + x0.a.x;
    b1.y = x0.b.y + x1.b.y + x0.a.y;
  } else {
    b0.x = x0.a.x + x1.a.x + x0.b.x;
    b0.y = x0.a.y + x1.a.y + x0.b.y;
    b1.x = x0.b.x + x1.b.x + xe.x;
    b1.y = x0.b.y + x1.b.y + xe.y;
  }
  const float sgn = sm.wrap ? -1.0f : 1.0f;
  const float sig = sm.isA ? -1.0f : 1.0f;
  const float kap = (float)g.kappa, mst = (float)g.ms;
  const bool plus = (sm.isA != DAG);
  C64x2 y;
  {
    float c0, s0;
    csf(0, c0, s0);
    const float es = plus ? s0 : -s0;
    const float cr = sgn * (c0 - mst), ci = sgn * es;
    const float tr = cr * xt.a.x - ci * xt.a.y, ti = cr * xt.a.y + ci * xt.a.x;
    y.a.x = sig * (xs.a.x - tr) - kap * b0.x;
    y.a.y = sig * (xs.a.y - ti) - kap * b0.y;
  }
  {
    float c1, s1;
    csf(1, c1, s1);
    const float es = plus ? s1 : -s1;
    const float cr = sgn * (c1 - mst), ci = sgn * es;
    const float tr = cr * xt.b.x - ci * xt.b.y, ti = cr * xt.b.y + ci * xt.b.x;
    y.b.x = sig * (xs.b.x - tr) - kap * b1.x;
    y.b.y = sig * (xs.b.y - ti) - kap * b1.y;
  }
  return y;
}

// Apply M (DAG = false) or M^dagger to the TOTAL/2 site pairs of this thread in the
// tile of sites [lo, end) (lo even, at most kBlock * TOTAL sites): the pairs starting
// at lo + 2*(threadIdx.x + m*kBlock) below end.  ld2(k) loads the raw
// input at k, k+1 and ld1(k) at k; after `mid()` (see stencil_sites), cook2 / cook1
// turn them into C64x2 / float2 inputs; post(n, y, self, pre) per pair.
template <bool DAG, int TOTAL = kSitesPerThread, typename Phi, typename Ld2, typename Ld1, typename Cook2,
          typename Cook1, typename Pre, typename Mid, typename Post>
__device__ __forceinline__ void stencil_pairs(const Geom& g, const Phi& phi, int lo, int end, Ld2 ld2, Ld1 ld1,
                                              Cook2 cook2, Cook1 cook1, Pre pre, Mid mid, Post post) {
  using PV = decltype(pre(0));
  using R2 = decltype(ld2(0));
  using R1 = decltype(ld1(0));
  constexpr int NPT = TOTAL / 2;  // pairs per thread
  constexpr int NP = HUB_PAIRS_PER_ROUND < NPT ? HUB_PAIRS_PER_ROUND : NPT;  // pairs in flight per round
  static_assert(NPT % NP == 0, "rounds must divide the pairs");
#pragma unroll
  for (int q0 = 0; q0 < NPT; q0 += NP) {
  PairIdx st[NP];
  bool ok[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    int n = lo + 2 * (threadIdx.x + (q0 + m) * kBlock);
    ok[m] = n < end;
    n = ok[m] ? n : end - 2;
    st[m] = pair_index<DAG>(g, n);
  }
  R2 rs[NP], rt[NP], r0[NP], r1[NP];
  R1 re[NP];
  typename Phi::Raw2 ph[NP];
  PV pv[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    rs[m] = ld2(st[m].n);
    rt[m] = ld2(st[m].tn);
    r0[m] = ld2(st[m].h0);
    r1[m] = ld2(st[m].h1);
    re[m] = ld1(st[m].hx);
    ph[m] = phi.load2(DAG ? st[m].tn : st[m].n);
    pv[m] = pre(st[m].n);
  }
  if (q0 == 0 && !mid()) return;
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    const PairIdx& sm = st[m];
    const C64x2 xs = cook2(rs[m]), xt = cook2(rt[m]), x0 = cook2(r0[m]), x1 = cook2(r1[m]);
    const float2 xe = cook1(re[m]);
    // the arithmetic of pair_stencil, written out here: through the helper the compiler
    // schedules this loop with 10 more registers per thread
    float2 b0, b1;
    if (sm.isA) {
      b0.x = x0.a.x + x1.a.x + xe.x;
      b0.y = x0.a.y + x1.a.y + xe.y;
      b1.x = x0.b.x + x1.b.x + x0.a.x;
      b1.y = x0.b.y + x1.b.y + x0.a.y;
    } else {
      b0.x = x0.a.x + x1.a.x + x0.b.x;
      b0.y = x0.a.y + x1.a.y + x0.b.y;
      b1.x = x0.b.x + x1.b.x + xe.x;
      b1.y = x0.b.y + x1.b.y + xe.y;
    }
    const float sgn = sm.wrap ? -1.0f : 1.0f;
    const float sig = sm.isA ? -1.0f : 1.0f;
    const float kap = (float)g.kappa, mst = (float)g.ms;
    const bool plus = (sm.isA != DAG);
    C64x2 y;
    {
      float c, s;
      phi.cs2(ph[m], 0, c, s);
      const float es = plus ? s : -s;
      const float cr = sgn * (c - mst), ci = sgn * es;
      const float tr = cr * xt.a.x - ci * xt.a.y, ti = cr * xt.a.y + ci * xt.a.x;
      y.a.x = sig * (xs.a.x - tr) - kap * b0.x;
      y.a.y = sig * (xs.a.y - ti) - kap * b0.y;
    }
    {
      float c, s;
      phi.cs2(ph[m], 1, c, s);
      const float es = plus ? s : -s;
      const float cr = sgn * (c - mst), ci = sgn * es;
      const float tr = cr * xt.b.x - ci * xt.b.y, ti = cr * xt.b.y + ci * xt.b.x;
      y.b.x = sig * (xs.b.x - tr) - kap * b1.x;
      y.b.y = sig * (xs.b.y - ti) - kap * b1.y;
    }
    if (ok[m]) post(sm.n, y, xs, pv[m]);
  }
  }
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Deterministic sum over the 256 threads; every thread gets the same value.
template <typename T>
__device__ __forceinline__ T block_sum(T v) {
  __shared__ T lds[kBlock / 64];
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Sum of `cnt` partials spaced `stride` apart, fixed order, same value in every thread.
__device__ __forceinline__ double sum_partials(const double* part, int cnt, int stride) {
  const Real<double> p(part);
  double acc = 0.0;
  for (int k = threadIdx.x; k < cnt; k += kBlock) acc += p[k * stride];
  return block_sum(acc);
}

template <typename LL>
__device__ __forceinline__ int find_sys(const LL& L, int lt) {
  int lo = 0, hi = L.nsys - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (L.tile_begin[mid] <= lt) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The phase source of the solver kernels in precision R.
template <typename R> struct SolverPhase;
template <> struct SolverPhase<double> { using T = PhasePhi<double>; };
template <> struct SolverPhase<float> { using T = Angle32; };
template <typename R> __device__ __forceinline__ typename SolverPhase<R>::T phase_of(const SysDesc* d);
template <> __device__ __forceinline__ PhasePhi<double> phase_of<double>(const SysDesc* d) {
  return PhasePhi<double>(d->ph64);
}
template <> __device__ __forceinline__ Angle32 phase_of<float>(const SysDesc* d) { return Angle32(d->ph32); }

// ---------------------------------------------------------------------------
// Public operator kernels (shared phi, batch of vectors, no descriptors).  They
// have no reduction partials, so they use smaller tiles (two sites per thread,
// both loaded together): more waves in flight than the CG kernels' tiles.  A
// workgroup applies the operator to a group of `per` consecutive vectors of the
// batch: the site indices, phi and its phase are loaded and evaluated once per site
// for the whole group (the launcher makes the group the whole batch whenever the
// lattice alone gives enough workgroups).
// ---------------------------------------------------------------------------
constexpr int kPubSites = 2;
constexpr int kPubTile = kBlock * kPubSites;

// Store of an operator result.  NT = true: a non-temporal store, for outputs handed
// back to the caller (the result is not read again by this launch or the next one;
// at 102x102x64 the public FP64 apply takes 8.1-8.6 us instead of 10.2 us with its
// working set in the infinity cache and 13.7-14.2 us instead of 15.3 us with buffers
// rotated past it).  NT = false: a plain store, for results a following kernel of the
// library reads at once (xi for the force, the first pass of the normal operator),
// which a non-temporal store would send past the infinity cache.
template <bool NT>
__device__ __forceinline__ void store_out(double2* p, double2 v) {
  if constexpr (NT) {
    hub_d2v w;
    w.x = v.x;
    w.y = v.y;
    __builtin_nontemporal_store(w, (hub_d2v*)p);
  } else {
    *p = v;
  }
}

// One vector per workgroup: all loads of a round in flight together, then the phase.
template <bool DAG, bool NT>
__global__ __launch_bounds__(kBlock) void k_apply(Geom g, const double* __restrict__ phi,
                                                  const double2* __restrict__ x, double2* __restrict__ y,
                                                  int ntiles) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int b = l / ntiles, tile = l - b * ntiles;
  const double2* __restrict__ xb = x + (size_t)b * g.n;
  double2* __restrict__ yb = y + (size_t)b * g.n;
  const int base = tile * kPubTile + threadIdx.x;
  auto ld = [=](int k) { return xb[k]; };
  auto pre = [](int) { return NoPre{}; };
  auto post = [=](int n, double2 v, double2, NoPre) { store_out<NT>(yb + n, v); };
  stencil_sites<double, DAG, kPubSites, kPubSites>(g, AnglePhi<double>(phi), base, g.n, ld, Same{}, pre, NoMid{},
                                                   post);
}

// A group of `per` vectors per workgroup (separate kernel, so that the one-vector
// kernel keeps its register budget).
template <bool DAG, bool NT>
__global__ __launch_bounds__(kBlock) void k_apply_grp(Geom g, const double* __restrict__ phi,
                                                      const double2* __restrict__ x, double2* __restrict__ y,
                                                      int ntiles, int per, int batch) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int grp = l / ntiles, tile = l - grp * ntiles;
  const int b0 = grp * per, b1 = min(batch, b0 + per);
  const int base = tile * kPubTile + threadIdx.x;
  SiteIdx st[kPubSites];
  bool ok[kPubSites];
  double ph[kPubSites], c[kPubSites], s[kPubSites];
#pragma unroll
  for (int m = 0; m < kPubSites; ++m) {
    int n = base + m * kBlock;
    ok[m] = n < g.n;
    n = ok[m] ? n : g.n - 1;
    st[m] = site_index<DAG>(g, n);
    ph[m] = phi[st[m].pn];
  }
  for (int b = b0; b < b1; ++b) {
    const double2* __restrict__ xb = x + (size_t)b * g.n;
    double2* __restrict__ yb = y + (size_t)b * g.n;
    double2 xs[kPubSites], xt[kPubSites], x0[kPubSites], x1[kPubSites], x2[kPubSites];
#pragma unroll
    for (int m = 0; m < kPubSites; ++m) {
      xs[m] = xb[st[m].n];
      xt[m] = xb[st[m].tn];
      x0[m] = xb[st[m].h0];
      x1[m] = xb[st[m].h1];
      x2[m] = xb[st[m].h2];
    }
    if (b == b0) {
#pragma unroll
      for (int m = 0; m < kPubSites; ++m) cis64(ph[m], c[m], s[m]);
    }
#pragma unroll
    for (int m = 0; m < kPubSites; ++m) {
      const double2 v = stencil_combine<double, DAG>(g, st[m], c[m], s[m], xs[m], xt[m], x0[m], x1[m], x2[m]);
      if (ok[m]) store_out<NT>(yb + st[m].n, v);
    }
  }
}

struct Mu2Arr { double v[kMaxSys]; };

// y_b = M u_b + mu2_b x_b: the second pass of the public normal operator (u = M^dagger x),
// one vector per workgroup.
__global__ __launch_bounds__(kBlock) void k_normal2_pub(Geom g, const double* __restrict__ phi, Mu2Arr mu2,
                                                        const double2* __restrict__ u,
                                                        const double2* __restrict__ x, double2* __restrict__ y,
                                                        int ntiles) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int b = l / ntiles, tile = l - b * ntiles;
  const size_t off = (size_t)b * g.n;
  const double m2 = mu2.v[b];
  const int base = tile * kPubTile + threadIdx.x;
  auto ld = [=](int k) { return u[off + k]; };
  auto pre = [=](int n) { return x[off + n]; };
  auto post = [=](int n, double2 q, double2, double2 xv) {
    q.x += m2 * xv.x;
    q.y += m2 * xv.y;
    y[off + n] = q;
  };
  stencil_sites<double, false, kPubSites, kPubSites>(g, AnglePhi<double>(phi), base, g.n, ld, Same{}, pre, NoMid{},
                                                     post);
}

// The public normal operator on a batch that shares phi: y_b = (M M^dagger + mu2_b) x_b for a
// group of `per` vectors per workgroup, in one pass after k_phase_pub.  A site's thread
// evaluates u = M^dagger x at the five sites that M reads, from 15 values of x (the
// cancelled 12-point form reads 12 but rounds worse: 1.5e-16 against 0.9e-16 of |y|).  That
// reads x and writes y, where a pass for u and one for y also write u, read it back, read x
// again and evaluate each phase twice; the neighbours come from the caches.  Two vectors at
// 102x102x64 with buffers rotated: 47.6 -> 38.8 us (31 and 7.5 us in the two kernels; 96 MB moved, and
// the L1 loads of the neighbours, 35 of 16 bytes per site, take 19 us of the 31 by
// themselves); resident 42.2 -> 41.6, four vectors 79.9 -> 60.9.
__global__ __launch_bounds__(kBlock) void k_normal_pub(Geom g, const double2* __restrict__ ph64, Mu2Arr mu2,
                                                       const double2* __restrict__ x, double2* __restrict__ y,
                                                       int ntiles, int per, int batch) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int grp = l / ntiles, tile = l - grp * ntiles;
  const int v0 = grp * per, v1 = min(batch, v0 + per);
  const int n = tile * kBlock + threadIdx.x;
  if (n >= g.n) return;
  const uint32_t q1 = fdiv((uint32_t)n, g.dL2), q2 = fdiv(q1, g.dL1);
  const int j = n - (int)q1 * g.L2, i = (int)q1 - (int)q2 * g.L1, t = (int)(q2 >> 1), L2 = g.L2, P = g.P;
  const bool isA = (q2 & 1u) == 0;
  const bool first = t == 0, last = t == g.Nt - 1;
  const int tp = last ? 0 : t + 1, tm = first ? g.Nt - 1 : t - 1;
  const int ip = i + 1 == g.L1 ? 0 : i + 1, im = i == 0 ? g.L1 - 1 : i - 1;
  const int jp = j + 1 == L2 ? 0 : j + 1, jm = j == 0 ? L2 - 1 : j - 1;
  // bonds go to (i, j), (i1, j), (i, j1) of the other sublattice and back to (i, j), (i0, j),
  // (i, j0); M reads slice tb of the own sublattice, M^dagger slice tf
  const int i1 = isA ? im : ip, i0 = isA ? ip : im, j1 = isA ? jm : jp, j0 = isA ? jp : jm;
  const int tb = isA ? tm : tp, tf = isA ? tp : tm;
  const int c = i * L2 + j, c1 = i1 * L2 + j, c2 = i * L2 + j1;
  const int own = n - c, ownb = (2 * tb + (isA ? 0 : 1)) * P, ownf = (2 * tf + (isA ? 0 : 1)) * P;
  const int opp = isA ? own + P : own - P, oppb = isA ? ownb + P : ownb - P;
  SiteIdx f, b, o;  // u(t) and u(tb) of the own sublattice, u(t) of the other
  f.isA = b.isA = isA;
  o.isA = !isA;
  f.wrap = isA ? last : first;
  b.wrap = o.wrap = isA ? first : last;
  const Vec<double2> ph(ph64);
  const double2 e = ph[n], ef = ph[ownf + c], e0 = ph[oppb + c], e1 = ph[oppb + c1], e2 = ph[oppb + c2];
  for (int v = v0; v < v1; ++v) {
    const Vec<double2> xv(x + (size_t)v * g.n);
    const double2 xs = xv[n], xf = xv[ownf + c], xb = xv[ownb + c];
    const double2 p0 = xv[opp + c], p1 = xv[opp + c1], p2 = xv[opp + c2];
    const double2 r0 = xv[oppb + c], r1 = xv[oppb + c1], r2 = xv[oppb + c2];
    const double2 s1 = xv[own + i0 * L2 + j], s2 = xv[own + i * L2 + j0], s3 = xv[own + c1], s4 = xv[own + i1 * L2 + j0],
                  s5 = xv[own + c2], s6 = xv[own + i0 * L2 + j1];
    const double2 uf = stencil_combine<double, true>(g, f, ef.x, ef.y, xs, xf, p0, p1, p2);
    const double2 ub = stencil_combine<double, true>(g, b, e.x, e.y, xb, xs, r0, r1, r2);
    const double2 u0 = stencil_combine<double, true>(g, o, e0.x, e0.y, p0, r0, xs, s1, s2);
    const double2 u1 = stencil_combine<double, true>(g, o, e1.x, e1.y, p1, r1, s3, xs, s4);
    const double2 u2 = stencil_combine<double, true>(g, o, e2.x, e2.y, p2, r2, s5, s6, xs);
    double2 q = stencil_combine<double, false>(g, b, e.x, e.y, uf, ub, u0, u1, u2);
    q.x += mu2.v[v] * xs.x;
    q.y += mu2.v[v] * xs.y;
    store_out<true>(y + (size_t)v * g.n + n, q);
  }
}

// Vectors per workgroup of the public batched kernels: the whole batch when the
// lattice alone gives about 1024 workgroups or more, else fewer so that the launch
// still has that many.
static int pub_group(int ntiles, int batch) {
  const long want = 1024;
  const long per = (long)ntiles * batch / want;
  return (int)std::max<long>(1, std::min<long>(batch, per));
}

// dS/dphi at every site: A: 2 Im[conj(eta(t)) s e^{i phi} z(t-1)],
//                        B: 2 Im[conj(eta(t)) s e^{-i phi} z(t+1)],
// with z = xi; the derivative of M does not depend on the staggered mass.
__global__ __launch_bounds__(kBlock) void k_force(Geom g, const double* __restrict__ phi,
                                                  const double2* __restrict__ eta,
                                                  const double2* __restrict__ xi,
                                                  double scale, int accumulate, double* __restrict__ out,
                                                  int ntiles) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int b = l / ntiles, tile = l - b * ntiles;
  const size_t off = (size_t)b * g.n;
  const int base = tile * kTile + threadIdx.x;
  const int P2 = 2 * g.P;
#pragma unroll
  for (int m = 0; m < kSitesPerThread; ++m) {
    const int n = base + m * kBlock;
    if (n < g.n) {
      const uint32_t q2 = fdiv(fdiv((uint32_t)n, g.dL2), g.dL1);
      const bool isA = (q2 & 1u) == 0;
      const int t = (int)(q2 >> 1);
      int tn;
      double sgn;
      if (isA) {
        const bool wrap = t == 0;
        tn = wrap ? n + (g.Nt - 1) * P2 : n - P2;
        sgn = wrap ? -1.0 : 1.0;
      } else {
        const bool wrap = t == g.Nt - 1;
        tn = wrap ? n - (g.Nt - 1) * P2 : n + P2;
        sgn = wrap ? -1.0 : 1.0;
      }
      double c, s;
      cis64(phi[n], c, s);
      if (!isA) s = -s;
      const double2 e = eta[off + n];
      const double2 z = xi[off + tn];
      // w = sgn (c + i s) z ; F = 2 Im(conj(e) w)
      const double wr = sgn * (c * z.x - s * z.y), wi = sgn * (c * z.y + s * z.x);
      const double F = 2.0 * (e.x * wi - e.y * wr);
      double* o = out + off + n;
      *o = accumulate ? *o + scale * F : scale * F;
    }
  }
}

// The same for a group of `per` vectors per workgroup: the temporal neighbour and
// the phase of each site are evaluated once for the group.
__global__ __launch_bounds__(kBlock) void k_force_grp(Geom g, const double* __restrict__ phi,
                                                      const double2* __restrict__ eta,
                                                      const double2* __restrict__ xi,
                                                      double scale, int accumulate, double* __restrict__ out,
                                                      int ntiles, int per, int batch) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int grp = l / ntiles, tile = l - grp * ntiles;
  const int b0 = grp * per, b1 = min(batch, b0 + per);
  const int base = tile * kTile + threadIdx.x;
  const int P2 = 2 * g.P;
  // per site: the temporal neighbour and s e^{+-i phi}, shared by the vectors of the group
  int tn[kSitesPerThread];
  double ec[kSitesPerThread], es[kSitesPerThread];
#pragma unroll
  for (int m = 0; m < kSitesPerThread; ++m) {
    const int n = min(base + m * kBlock, g.n - 1);
    const uint32_t q2 = fdiv(fdiv((uint32_t)n, g.dL2), g.dL1);
    const bool isA = (q2 & 1u) == 0;
    const int t = (int)(q2 >> 1);
    double sgn;
    if (isA) {
      const bool wrap = t == 0;
      tn[m] = wrap ? n + (g.Nt - 1) * P2 : n - P2;
      sgn = wrap ? -1.0 : 1.0;
    } else {
      const bool wrap = t == g.Nt - 1;
      tn[m] = wrap ? n - (g.Nt - 1) * P2 : n + P2;
      sgn = wrap ? -1.0 : 1.0;
    }
    double c, s;
    cis64(phi[n], c, s);
    ec[m] = sgn * c;
    es[m] = sgn * (isA ? s : -s);
  }
  for (int b = b0; b < b1; ++b) {
    const size_t off = (size_t)b * g.n;
#pragma unroll
    for (int m = 0; m < kSitesPerThread; ++m) {
      const int n = base + m * kBlock;
      if (n < g.n) {
        const double2 e = eta[off + n];
        const double2 z = xi[off + tn[m]];
        // w = s e^{+-i phi} z ; F = 2 Im(conj(e) w)
        const double wr = ec[m] * z.x - es[m] * z.y, wi = ec[m] * z.y + es[m] * z.x;
        const double F = 2.0 * (e.x * wi - e.y * wr);
        double* o = out + off + n;
        *o = accumulate ? *o + scale * F : scale * F;
      }
    }
  }
}

// y = M x or M^dagger x of several jobs (fields, vectors and masses of their own).  One
// launch for all of them: a job of 256 to 4608 unknowns is a few microseconds of latency
// by itself, so a launch per job leaves the device idle but for one workgroup (with
// k_terms and k_phase_jobs: 32 chains of 2x1x64 through a trajectory 30.3 -> 14.1 ms).
template <bool DAG>
__global__ __launch_bounds__(kBlock) void k_apply_jobs(Geom g, ApplyJobs J, int ntiles) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int q = l / ntiles, tile = l - q * ntiles;
  const double2* __restrict__ x = J.j[q].x;
  double2* __restrict__ y = J.j[q].y;
  g.ms = J.j[q].ms;
  const int base = tile * kPubTile + threadIdx.x;
  auto ld = [=](int k) { return x[k]; };
  auto pre = [](int) { return NoPre{}; };
  auto post = [=](int n, double2 v, double2, NoPre) { y[n] = v; };
  stencil_sites<double, DAG, kPubSites, kPubSites>(g, AnglePhi<double>(J.j[q].phi), base, g.n, ld, Same{}, pre,
                                                   NoMid{}, post);
}

// The actions and the summed force of a kick group in one pass (TermJobs): a workgroup
// owns kBlock sites of one chain and goes through its terms in order.  The force at site m
// needs xi = M^dagger eta at one site only, its temporal neighbour n in the direction in
// which M hops, and no other site needs that value: the thread of n evaluates xi(n), whose
// temporal neighbour is m again with the phase of m, and writes dS(m).  So xi is never
// stored, each site's phase is evaluated once for all terms, and dS is written once.
// Memory per site and term: eta, rhs and sub once (16 B each, the hops from the caches).
// FORCE = false: the actions only.  Ratio terms take xi - sub (eq. (f_chi_i)).
template <bool FORCE>
__global__ __launch_bounds__(kBlock) void k_terms(Geom g, TermJobs J, int ntiles, double* __restrict__ part,
                                                  double* __restrict__ result) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int ch = l / ntiles, tile = l - ch * ntiles;
  const int n0 = tile * kBlock + threadIdx.x;
  const bool ok = n0 < g.n;
  SiteIdx st;
  st.n = ok ? n0 : g.n - 1;
  double c = 0.0, s = 0.0, sum = 0.0;
  double* __restrict__ dS = J.chain[ch].dS;
  if (FORCE) {
    st = site_index<true>(g, st.n);
    cis64(J.chain[ch].phi[st.pn], c, s);
    if (J.accumulate) sum = dS[st.tn];
  }
  const double sgn = st.wrap ? -1.0 : 1.0;
  const double ec = sgn * c, es = sgn * (st.isA ? s : -s);
  for (int k = 0; k < J.nterm; ++k) {
    const TermJob& T = J.term[ch * J.nterm + k];
    const double2* __restrict__ eta = T.eta;
    const double2 e0 = eta[st.n], b = T.rhs[st.n];
    if (FORCE) {
      const double2 e = eta[st.tn];
      const double2 x0 = eta[st.h0], x1 = eta[st.h1], x2 = eta[st.h2];
      double2 v;
      v.x = v.y = 0.0;
      if (T.sub) v = T.sub[st.n];
      g.ms = T.ms;
      double2 z = stencil_combine<double, true>(g, st, c, s, e0, e, x0, x1, x2);
      z.x -= v.x;
      z.y -= v.y;
      // w = s e^{+-i phi} z ; F = 2 Im(conj(e) w)
      const double wr = fma(ec, z.x, -(es * z.y)), wi = fma(ec, z.y, es * z.x);
      const double F = 2.0 * fma(e.x, wi, -(e.y * wr));
      sum = (k > 0 || J.accumulate) ? sum + J.scale[k] * F : J.scale[k] * F;
    }
    const double d = ok ? b.x * e0.x + b.y * e0.y : 0.0;
    const double tot = block_sum(d);
    const int q = ch * J.nterm + k;
    if (threadIdx.x == 0) {
      if (ntiles == 1)
        result[q] = tot;
      else
        part[(size_t)q * ntiles + tile] = tot;
    }
  }
  if (FORCE && ok) dS[st.tn] = sum;
}

// Sum over the vectors of a batch: out (+)= sum_b scale_b F_b with F_b the force of
// k_force.  phi, its phase and the temporal neighbour are evaluated once per site; per
// site and vector only eta and xi (at the neighbour) are read, and out is written once.
__global__ __launch_bounds__(kBlock) void k_force_sum(Geom g, const double* __restrict__ phi,
                                                      const double2* __restrict__ eta,
                                                      const double2* __restrict__ xi, Mu2Arr scale,
                                                      int accumulate, double* __restrict__ out, int batch) {
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int base = tile * kTile + threadIdx.x;
  const int P2 = 2 * g.P;
#pragma unroll 2
  for (int m = 0; m < kSitesPerThread; ++m) {
    const int n = base + m * kBlock;
    if (n >= g.n) break;
    const uint32_t q2 = fdiv(fdiv((uint32_t)n, g.dL2), g.dL1);
    const bool isA = (q2 & 1u) == 0;
    const int t = (int)(q2 >> 1);
    int tn;
    double sgn;
    if (isA) {
      const bool wrap = t == 0;
      tn = wrap ? n + (g.Nt - 1) * P2 : n - P2;
      sgn = wrap ? -1.0 : 1.0;
    } else {
      const bool wrap = t == g.Nt - 1;
      tn = wrap ? n - (g.Nt - 1) * P2 : n + P2;
      sgn = wrap ? -1.0 : 1.0;
    }
    double c, s;
    cis64(phi[n], c, s);
    const double ec = sgn * c, es = sgn * (isA ? s : -s);
    double F = 0.0;
    for (int b = 0; b < batch; ++b) {
      const size_t off = (size_t)b * g.n;
      const double2 e = eta[off + n];
      const double2 z = xi[off + tn];
      // w = s e^{+-i phi} z ; F_b = 2 Im(conj(e) w)
      const double wr = ec * z.x - es * z.y, wi = ec * z.y + es * z.x;
      F = fma(scale.v[b], 2.0 * (e.x * wi - e.y * wr), F);
    }
    out[n] = accumulate ? out[n] + F : F;
  }
}

// Measurement only: the bytes of one FP64 apply (x and phi read, y written per site)
// with no stencil and no phase, two sites per thread, the apply's grid and workgroup
// order.  NTL: non-temporal loads; NTS: non-temporal stores.
template <bool NTL, bool NTS>
__global__ __launch_bounds__(kBlock) void k_stream_bytes(const double* __restrict__ phi,
                                                         const double2* __restrict__ x, double2* __restrict__ y,
                                                         int n) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int base = l * kPubTile + threadIdx.x;
  double2 v[kPubSites];
  double p[kPubSites];
#pragma unroll
  for (int m = 0; m < kPubSites; ++m) {
    const int k = min(base + m * kBlock, n - 1);
    if constexpr (NTL) {
      const hub_d2v w = __builtin_nontemporal_load((const hub_d2v*)(x + k));
      v[m].x = w.x;
      v[m].y = w.y;
      p[m] = __builtin_nontemporal_load(phi + k);
    } else {
      v[m] = x[k];
      p[m] = phi[k];
    }
  }
#pragma unroll
  for (int m = 0; m < kPubSites; ++m) {
    const int k = base + m * kBlock;
    double2 o;
    o.x = v[m].x * p[m];
    o.y = v[m].y + p[m];
    if (k < n) store_out<NTS>(y + k, o);
  }
}

// Per-tile partials of Re sum conj(a_b) b_b.
__global__ __launch_bounds__(kBlock) void k_dot_re(Geom g, const double2* __restrict__ a,
                                                   const double2* __restrict__ bb, int ntiles,
                                                   double* __restrict__ part) {
  const int l = xcd_remap(blockIdx.x, gridDim.x);
  const int b = l / ntiles, tile = l - b * ntiles;
  const size_t off = (size_t)b * g.n;
  const int base = tile * kTile + threadIdx.x;
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < kSitesPerThread; ++m) {
    const int n = base + m * kBlock;
    if (n < g.n) {
      const double2 u = a[off + n], v = bb[off + n];
      acc += u.x * v.x + u.y * v.y;
    }
  }
  const double tot = block_sum(acc);
  if (threadIdx.x == 0) part[(size_t)b * ntiles + tile] = tot;
}

// result[b] = fixed-order sum of the partials of system b (one workgroup each).
__global__ __launch_bounds__(kBlock) void k_dot_finish(const double* __restrict__ part, int ntiles,
                                                       double* __restrict__ result) {
  const double s = sum_partials(part + (size_t)blockIdx.x * ntiles, ntiles, 1);
  if (threadIdx.x == 0) result[blockIdx.x] = s;
}

// (cos phi, sin phi) per site in FP64 and, when p32 is given, phi - 2 pi k (k the
// integer nearest phi / 2 pi, in FP64) rounded to float.
__device__ __forceinline__ void phase_site(const double* __restrict__ phi, double2* __restrict__ p64,
                                           float* __restrict__ p32, int i) {
  const double a = phi[i];
  double c, s;
  sincos(a, &s, &c);
  double2 v;
  v.x = c;
  v.y = s;
  p64[i] = v;
  const float a32 = (float)fma(-rint(a * 0.15915494309189535), 6.283185307179586, a);
  if (p32) p32[i] = a32;
}

__global__ __launch_bounds__(kBlock) void k_phase(const double* __restrict__ phi, double2* __restrict__ p64,
                                                  float* __restrict__ p32, int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) phase_site(phi, p64, p32, i);
}

// The phase as the public operators evaluate it.
__global__ __launch_bounds__(kBlock) void k_phase_pub(const double* __restrict__ phi, double2* __restrict__ p64,
                                                      int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double2 v;
  cis64(phi[i], v.x, v.y);
  p64[i] = v;
}

// The same for the fields of a batch, one field per grid row.
__global__ __launch_bounds__(kBlock) void k_phase_jobs(PhaseJobs J, int n) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const PhaseJob& j = J.j[blockIdx.y];
  if (i < n) phase_site(j.phi, j.p64, j.p32, i);
}

// Molecular dynamics (Sec. 5.2): phi += eps pi (T_pi), and the momentum kick
// pi -= G + cg phi, where G holds the summed pseudofermion force contributions
// sum_k eps_k dS_k/dphi and cg = eps/U~ is the gauge force's share.
__global__ __launch_bounds__(kBlock) void k_md_drift(double* __restrict__ phi, const double* __restrict__ pi,
                                                     double eps, int n) {
  const int i = xcd_remap(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i < n) phi[i] += eps * pi[i];
}

__global__ __launch_bounds__(kBlock) void k_md_kick(double* __restrict__ pi, const double* __restrict__ phi,
                                                    const double* __restrict__ G, double cg, int n) {
  const int i = xcd_remap(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
  if (i < n) pi[i] -= (G ? G[i] : 0.0) + cg * phi[i];
}

// ---------------------------------------------------------------------------
// Batched solver kernels (descriptor + launch list).
// ---------------------------------------------------------------------------
// Sites [lo, hi) of solver tile `tile` (block tile % nb of segment tile / nb).
struct TileRange {
  int lo, hi;
};
__device__ __forceinline__ TileRange tile_range(int tile, int nb, int bsz, int seg) {
  const int sg = tile / nb;
  TileRange r;
  r.lo = sg * seg + (tile - sg * nb) * bsz;
  r.hi = min(r.lo + bsz, (sg + 1) * seg);
  return r;
}

// Prologue of the batched solver kernels: the system and tile of this workgroup.
// The tile holds the sites [t_lo, t_hi) (block tile % tnb of segment tile / tnb, at
// most TILE sites: every kernel of a system uses the tile size of its class); the
// thread's sites are base + m*kBlock below t_hi.
#define HUB_PROLOGUE_T(TILE)                                            \
  const int lt = xcd_remap(blockIdx.x, gridDim.x);                      \
  const int kk = find_sys(L, lt);                                       \
  const SysDesc* __restrict__ d = sys + L.sys[kk];                      \
  const int tile = lt - L.tile_begin[kk];                               \
  Scal* sc = L.scal + L.sys[kk];                                        \
  const Geom g = d->g;                                                  \
  const TileRange t_r = tile_range(tile, d->tnb, d->tbsz, d->tseg);     \
  const int t_lo = t_r.lo, t_hi = t_r.hi;                               \
  const int base = t_lo + threadIdx.x;                                  \
  (void)t_hi;                                                           \
  (void)g;                                                              \
  static_assert((TILE) > 0, "tile size");

// CG stage 1 of iteration it = L.it[kk]:
//   |r_it|^2 from the stage-2 partials of iteration it-1 (it > 0) and the stopping
//   test; p_new = r + beta p_old with beta = |r_it|^2 / |r_{it-1}|^2 (p_new = r at
//   it = 0), u = M^dagger p_new, partial of |u|^2 + mu^2 |p_new|^2 = <p, A p>.
// The loads of r and p_old are issued before the partial sums are read.
// The solution advances every second iteration (see k_cg2): a stage 1 that stops at
// an odd it adds the pending alpha_{it-1} p_{it-1} (p_old here) to x.  It marks the
// stop with active = 2 rather than 0 so that every workgroup of this launch still
// takes the stopping path; the next stage 2 sets 0.
template <typename C>
struct RP {
  C r, p;
};

template <typename R, typename LL, int SPT>
__global__ __launch_bounds__(kBlock) void k_cg1(const SysDesc* __restrict__ sys, LL L, int sR, int sP, int sU) {
  using C = typename V2<R>::T;
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  if (!load_active(sc)) return;
  const int it = L.it[kk];
  const R mu2 = (R)d->mu2;
  const Vec<C> r(d->vec[sR]), po(d->vec[sP + (it & 1)]), pn(d->vec[sP + 1 - (it & 1)]), u(d->vec[sU]);
  const auto phi = phase_of<R>(d);
  R beta = 0;
  bool stopped = false;  // same value in every thread of every workgroup of the system
  // |r_it|^2, the stopping test and beta, once the stencil loads are in flight
  auto mid = [&]() -> bool {
    if (it == 0) return true;
    const double rr = sum_partials(d->part2, d->ntiles, 1);
    const double rr_prev = sc->rrv[(it - 1) & 1];
    const bool first = (tile == 0 && threadIdx.x == 0);
    if (!(rr > sc->stop2) || it >= sc->maxit) {
      if (first) {
        sc->rrv[it & 1] = rr;
        sc->iters = it;
        store_active(sc, 2);
      }
      stopped = true;
      return false;
    }
    if (first) sc->rrv[it & 1] = rr;
    beta = (R)(rr / rr_prev);
    return true;
  };
  R acc = 0;
  bool done = false;
  if constexpr (sizeof(R) == 4) {
    if ((g.L2 & 1) == 0) {
      auto pre2 = [](int) { return NoPre{}; };
      auto post2 = [&](int n, C64x2 uu, C64x2 p, NoPre) {
        pn.set_pair(n, p);
        u.set_pair(n, uu);
        acc += norm2<R>(uu.a) + norm2<R>(uu.b) + mu2 * (norm2<R>(p.a) + norm2<R>(p.b));
      };
      if (it == 0) {
        auto ld2 = [=](int k) { return r.pair(k); };
        auto ld1 = [=](int k) { return r[k]; };
        stencil_pairs<true, SPT>(g, phi, t_lo, t_hi, ld2, ld1, Same{}, Same{}, pre2, NoMid{}, post2);
      } else {
        auto ld2 = [=](int k) { return RP<C64x2>{r.pair(k), po.pair(k)}; };
        auto ld1 = [=](int k) { return RP<C>{r[k], po[k]}; };
        auto cook2 = [&](RP<C64x2> v) {
          C64x2 o;
          o.a.x = v.r.a.x + beta * v.p.a.x;
          o.a.y = v.r.a.y + beta * v.p.a.y;
          o.b.x = v.r.b.x + beta * v.p.b.x;
          o.b.y = v.r.b.y + beta * v.p.b.y;
          return o;
        };
        auto cook1 = [&](RP<C> v) {
          C o;
          o.x = v.r.x + beta * v.p.x;
          o.y = v.r.y + beta * v.p.y;
          return o;
        };
        stencil_pairs<true, SPT>(g, phi, t_lo, t_hi, ld2, ld1, cook2, cook1, pre2, mid, post2);
      }
      done = true;
    }
  }
  if (!done) {
    auto pre = [](int) { return NoPre{}; };
    auto post = [&](int n, C uu, C p, NoPre) {
      pn.set(n, p);
      u.set(n, uu);
      acc += norm2<R>(uu) + mu2 * norm2<R>(p);
    };
    if (it == 0) {
      auto ld = [=](int k) { return r[k]; };
      stencil_sites<R, true, Spt<R>::v, SPT>(g, phi, base, t_hi, ld, Same{}, pre, NoMid{}, post);
    } else {
      auto ld = [=](int k) { return RP<C>{r[k], po[k]}; };
      auto cook = [&](RP<C> v) {
        C o;
        o.x = v.r.x + beta * v.p.x;
        o.y = v.r.y + beta * v.p.y;
        return o;
      };
      stencil_sites<R, true, Spt<R>::v, SPT>(g, phi, base, t_hi, ld, cook, pre, mid, post);
    }
  }
  // a system that met its stopping test in `mid` writes no partial (none is read)
  if (stopped) {
    if (it & 1) {
      const R a = (R)sc->alpha[(it - 1) & 1];
      const Vec<C> x(d->vec[L.pi[kk]]);
      for (int k = base; k < t_hi; k += kBlock) {
        const C pv = po[k];
        C xv = x[k];
        xv.x = fma(a, pv.x, xv.x);
        xv.y = fma(a, pv.y, xv.y);
        x.set(k, xv);
      }
    }
    return;
  }
  const double tot = (double)block_sum(acc);
  if (threadIdx.x == 0) Real<double>(d->part1).set(tile, tot);
}

// CG stage 2 of iteration it: alpha = |r_it|^2 / <p, A p> (stage-1 partials),
// q = M u + mu^2 p, r -= alpha q, partial of |r_{it+1}|^2, and the solution every
// second iteration: x += alpha_{it-1} p_{it-1} + alpha_it p_it at odd it (p_{it-1}
// is still in the other slot of the pair), which saves a read and a write of x per
// two iterations for one read of p_{it-1}.  The solution slot of system k is L.pi[k].
// Loads are issued before alpha is read.  A system whose stage 1 stopped (active 2)
// does nothing here; workgroup 0 marks it stopped for good.
template <typename C, bool UPD>
struct Own {
  C p, r, x, q;  // x, q (p_{it-1}) loaded only when UPD
};
template <typename R, typename LL, int SPT>
__global__ __launch_bounds__(kBlock) void k_cg2(const SysDesc* __restrict__ sys, LL L, int sR, int sP, int sU) {
  using C = typename V2<R>::T;
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  const int act = load_active(sc);
  if (act != 1) {
    if (act == 2 && tile == 0 && threadIdx.x == 0) store_active(sc, 0);
    return;
  }
  const int it = L.it[kk];
  R alpha = 0, alpha_prev = 0;
  auto mid = [&]() -> bool {
    const double pq = sum_partials(d->part1, d->ntiles, 1);
    const double a = sc->rrv[it & 1] / pq;
    if (tile == 0 && threadIdx.x == 0) sc->alpha[it & 1] = a;
    alpha = (R)a;
    if (it & 1) alpha_prev = (R)sc->alpha[(it - 1) & 1];
    return true;
  };
  const R mu2 = (R)d->mu2;
  const Vec<C> p(d->vec[sP + 1 - (it & 1)]), pp(d->vec[sP + (it & 1)]), u(d->vec[sU]), x(d->vec[L.pi[kk]]),
      r(d->vec[sR]);
  const auto phi = phase_of<R>(d);
  R acc = 0;
  auto run = [&](auto upd) {
    constexpr bool U = decltype(upd)::value;
    if constexpr (sizeof(R) == 4) {
      if ((g.L2 & 1) == 0) {
        auto ld2 = [=](int k) { return u.pair(k); };
        auto ld1 = [=](int k) { return u[k]; };
        auto pre2 = [=](int n) {
          Own<C64x2, U> o;
          o.p = p.pair(n);
          o.r = r.pair(n);
          if constexpr (U) {
            o.x = x.pair(n);
            o.q = pp.pair(n);
          }
          return o;
        };
        auto post2 = [&](int n, C64x2 q, C64x2, Own<C64x2, U> o) {
          C64x2 rv;
          rv.a.x = o.r.a.x - alpha * fma(mu2, o.p.a.x, q.a.x);
          rv.a.y = o.r.a.y - alpha * fma(mu2, o.p.a.y, q.a.y);
          rv.b.x = o.r.b.x - alpha * fma(mu2, o.p.b.x, q.b.x);
          rv.b.y = o.r.b.y - alpha * fma(mu2, o.p.b.y, q.b.y);
          r.set_pair(n, rv);
          if constexpr (U) {
            C64x2 xv;
            xv.a.x = fma(alpha, o.p.a.x, fma(alpha_prev, o.q.a.x, o.x.a.x));
            xv.a.y = fma(alpha, o.p.a.y, fma(alpha_prev, o.q.a.y, o.x.a.y));
            xv.b.x = fma(alpha, o.p.b.x, fma(alpha_prev, o.q.b.x, o.x.b.x));
            xv.b.y = fma(alpha, o.p.b.y, fma(alpha_prev, o.q.b.y, o.x.b.y));
            x.set_pair(n, xv);
          }
          acc += norm2<R>(rv.a) + norm2<R>(rv.b);
        };
        stencil_pairs<false, SPT>(g, phi, t_lo, t_hi, ld2, ld1, Same{}, Same{}, pre2, mid, post2);
        return;
      }
    }
    auto ld = [=](int k) { return u[k]; };
    auto pre = [=](int n) {
      Own<C, U> o;
      o.p = p[n];
      o.r = r[n];
      if constexpr (U) {
        o.x = x[n];
        o.q = pp[n];
      }
      return o;
    };
    auto post = [&](int n, C q, C, Own<C, U> o) {
      C rv;
      rv.x = o.r.x - alpha * fma(mu2, o.p.x, q.x);
      rv.y = o.r.y - alpha * fma(mu2, o.p.y, q.y);
      r.set(n, rv);
      if constexpr (U) {
        C xv;
        xv.x = fma(alpha, o.p.x, fma(alpha_prev, o.q.x, o.x.x));
        xv.y = fma(alpha, o.p.y, fma(alpha_prev, o.q.y, o.x.y));
        x.set(n, xv);
      }
      acc += norm2<R>(rv);
    };
    stencil_sites<R, false, Spt<R>::v, SPT>(g, phi, base, t_hi, ld, Same{}, pre, mid, post);
  };
  if (it & 1)
    run(std::true_type{});
  else
    run(std::false_type{});
  const double tot = (double)block_sum(acc);
  if (threadIdx.x == 0) Real<double>(d->part2).set(tile, tot);
}

// ---------------------------------------------------------------------------
// Multi-shift CG (FP64).  Base CG on A_0 as k_cg1 / k_cg2; every shifted system s
// follows with x_s += alpha^s_k p^s_k, p^s_{k+1} = zeta^s_{k+1} r_{k+1} + beta^s_k p^s_k,
//   zeta^s_{k+1} = zeta_k zeta_{k-1} alpha_{k-1} /
//                  (alpha_k beta_{k-1} (zeta_{k-1} - zeta_k) + zeta_{k-1} alpha_{k-1} (1 + sigma_s alpha_k)),
//   alpha^s_k = alpha_k zeta_{k+1} / zeta_k,  beta^s_k = beta_k (zeta_{k+1} / zeta_k)^2,
// until its residual |zeta^s| |r| meets the tolerance.  Every workgroup evaluates the
// scalar recurrences in the same order (one thread per shift), so they agree.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_ms_start(const MsDesc* __restrict__ d) {
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const TileRange tr = tile_range(tile, d->tnb, d->tbsz, d->tseg);
  const int base = tr.lo + threadIdx.x;
  double acc = 0.0;
  const double2 z = {0.0, 0.0};
  for (int m = 0; m < kSitesPerThread; ++m) {
    const int n = base + m * kBlock;
    if (n >= tr.hi) break;
    const double2 v = d->b[n];
    d->r[n] = v;
    d->x[n] = z;
    for (int s = 0; s < d->ns; ++s) {
      d->xs[s][n] = z;
      d->ps[s][n] = v;
    }
    acc += v.x * v.x + v.y * v.y;
  }
  const double tot = block_sum(acc);
  if (threadIdx.x == 0) d->part2[tile] = tot;
}

__global__ __launch_bounds__(kBlock) void k_ms_setup(const MsDesc* __restrict__ d) {
  const double rr = sum_partials(d->part2, d->ntiles, 1);
  if (threadIdx.x == 0) {
    MsScal* sc = d->sc;
    sc->rrv[0] = rr;
    sc->rrv[1] = rr;
    sc->alpha[0] = 1.0;
    sc->alpha[1] = 1.0;
    sc->beta[0] = 0.0;
    sc->beta[1] = 0.0;
    sc->stop2 = d->tol2 * rr;
    for (int s = 0; s < kMsMax; ++s) {
      sc->zeta[s][0] = sc->zeta[s][1] = sc->zeta[s][2] = 1.0;
      sc->frozen[s][0] = sc->frozen[s][1] = 0;
    }
    sc->iters = 0;
    sc->maxit = d->maxit;
    sc->stop = 0;
    __hip_atomic_store(&sc->active, rr > 0.0 ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ int ms_load_active(MsScal* sc) {
  return __hip_atomic_load(&sc->active, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Stage 1 of iteration it: |r_it|^2, beta_{it-1}, the shifted scalars of step it-1 and
// the stopping test; p_it = r_it + beta p_{it-1}, u = M^dagger p_it, partial <p, A_0 p>;
// then the shifted vector updates of step it-1 (also in the iteration that stops).
__global__ __launch_bounds__(kBlock) void k_ms1(const MsDesc* __restrict__ d, int it) {
  MsScal* sc = d->sc;
  if (!ms_load_active(sc)) return;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const Geom g = d->g;
  const TileRange tr = tile_range(tile, d->tnb, d->tbsz, d->tseg);
  const int base = tr.lo + threadIdx.x;
  const double mu2 = d->mu2;
  const int ns = d->ns;
  const Vec<double2> r(d->r), po(d->p[it & 1]), pn(d->p[1 - (it & 1)]), u(d->u);
  const PhasePhi<double> phi(d->ph64);
  __shared__ double s_as[kMsMax], s_bs[kMsMax], s_zn[kMsMax];
  __shared__ int s_live[kMsMax];
  double beta = 0.0;
  bool stopped = false;
  auto mid = [&]() -> bool {
    const double rr = sum_partials(d->part2, d->ntiles, 1);
    const double rr_prev = sc->rrv[(it - 1) & 1];
    beta = rr / rr_prev;
    const int k = it - 1;
    const double a_k = sc->alpha[k & 1], a_km = sc->alpha[(k + 1) & 1], b_km = sc->beta[(k + 1) & 1];
    if ((int)threadIdx.x < ns) {
      const int s = threadIdx.x;
      const bool live = sc->frozen[s][k & 1] == 0;
      const double zk = sc->zeta[s][k % 3], zkm = sc->zeta[s][(k + 2) % 3];
      double zn = zk, as = 0.0, bs = 1.0;
      if (live) {
        zn = zk * zkm * a_km / (a_k * b_km * (zkm - zk) + zkm * a_km * (1.0 + d->sigma[s] * a_k));
        as = a_k * zn / zk;
        bs = beta * (zn / zk) * (zn / zk);
      }
      s_as[s] = as;
      s_bs[s] = bs;
      s_zn[s] = zn;
      s_live[s] = live ? 1 : 0;
      if (tile == 0) {
        sc->zeta[s][(k + 1) % 3] = zn;
        sc->frozen[s][(k + 1) & 1] = (!live || zn * zn * rr <= sc->stop2) ? 1 : 0;
      }
    }
    __syncthreads();
    const bool first = (tile == 0 && threadIdx.x == 0);
    if (first) {
      sc->rrv[it & 1] = rr;
      sc->beta[k & 1] = beta;
      d->hist[2 * k + 1] = beta;
    }
    if (!(rr > sc->stop2) || it >= sc->maxit) {
      // every workgroup of this launch still runs (active stays set until the next
      // stage 2), so all of them apply the last shifted updates below
      if (first) {
        sc->iters = it;
        sc->stop = 1;
      }
      stopped = true;
      return false;
    }
    return true;
  };
  double acc = 0.0;
  auto pre = [](int) { return NoPre{}; };
  auto post = [&](int n, double2 uu, double2 p, NoPre) {
    pn.set(n, p);
    u.set(n, uu);
    acc += norm2<double>(uu) + mu2 * norm2<double>(p);
  };
  if (it == 0) {
    auto ld = [=](int k) { return r[k]; };
    stencil_sites<double, true, HUB_SPT64>(g, phi, base, tr.hi, ld, Same{}, pre, NoMid{}, post);
  } else {
    auto ld = [=](int k) { return RP<double2>{r[k], po[k]}; };
    auto cook = [&](RP<double2> v) {
      double2 o;
      o.x = v.r.x + beta * v.p.x;
      o.y = v.r.y + beta * v.p.y;
      return o;
    };
    stencil_sites<double, true, HUB_SPT64>(g, phi, base, tr.hi, ld, cook, pre, mid, post);
    // shifted systems, step it-1 -> it
    for (int m = 0; m < kSitesPerThread; ++m) {
      const int n = base + m * kBlock;
      if (n >= tr.hi) break;
      const double2 rv = r[n];
      for (int s = 0; s < ns; ++s) {
        if (!s_live[s]) continue;
        const Vec<double2> xs(d->xs[s]), ps(d->ps[s]);
        const double2 pv = ps[n];
        double2 xv = xs[n];
        xv.x += s_as[s] * pv.x;
        xv.y += s_as[s] * pv.y;
        double2 q;
        q.x = s_zn[s] * rv.x + s_bs[s] * pv.x;
        q.y = s_zn[s] * rv.y + s_bs[s] * pv.y;
        xs.set(n, xv);
        ps.set(n, q);
      }
    }
  }
  if (stopped) return;
  const double tot = block_sum(acc);
  if (threadIdx.x == 0) Real<double>(d->part1).set(tile, tot);
}

// Stage 2 of iteration it: alpha_it = |r_it|^2 / <p, A_0 p>, q = M u + mu2 p,
// x += alpha p, r -= alpha q, partial |r_{it+1}|^2.
__global__ __launch_bounds__(kBlock) void k_ms2(const MsDesc* __restrict__ d, int it) {
  MsScal* sc = d->sc;
  if (!ms_load_active(sc)) return;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  if (sc->stop) {
    if (tile == 0 && threadIdx.x == 0)
      __hip_atomic_store(&sc->active, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  const Geom g = d->g;
  const TileRange tr = tile_range(tile, d->tnb, d->tbsz, d->tseg);
  const int base = tr.lo + threadIdx.x;
  const double mu2 = d->mu2;
  double alpha = 0.0;
  auto mid = [&]() -> bool {
    const double pq = sum_partials(d->part1, d->ntiles, 1);
    alpha = sc->rrv[it & 1] / pq;
    if (tile == 0 && threadIdx.x == 0) {
      sc->alpha[it & 1] = alpha;
      d->hist[2 * it] = alpha;
    }
    return true;
  };
  const Vec<double2> p(d->p[1 - (it & 1)]), u(d->u), x(d->x), r(d->r);
  const PhasePhi<double> phi(d->ph64);
  struct Own {
    double2 p, x, r;
  };
  double acc = 0.0;
  auto ld = [=](int k) { return u[k]; };
  auto pre = [=](int n) { return Own{p[n], x[n], r[n]}; };
  auto post = [&](int n, double2 q, double2, Own o) {
    q.x += mu2 * o.p.x;
    q.y += mu2 * o.p.y;
    double2 xv = o.x, rv = o.r;
    xv.x += alpha * o.p.x;
    xv.y += alpha * o.p.y;
    rv.x -= alpha * q.x;
    rv.y -= alpha * q.y;
    x.set(n, xv);
    r.set(n, rv);
    acc += norm2<double>(rv);
  };
  stencil_sites<double, false, HUB_SPT64>(g, phi, base, tr.hi, ld, Same{}, pre, mid, post);
  const double tot = block_sum(acc);
  if (threadIdx.x == 0) Real<double>(d->part2).set(tile, tot);
}

__device__ __forceinline__ double2 to_c128(float2 v) {
  double2 o;
  o.x = v.x;
  o.y = v.y;
  return o;
}

// Scal records to host-coherent memory in 8-byte words, every store arrived there before the
// flag is written.
__device__ __forceinline__ void publish(const Publish& pub) {
  const unsigned long long* src = reinterpret_cast<const unsigned long long*>(pub.d);
  unsigned long long* dst = reinterpret_cast<unsigned long long*>(pub.h);
  const int nw = pub.cnt * (int)(sizeof(Scal) / 8);
  for (int k = threadIdx.x; k < nw; k += kBlock)
    __hip_atomic_store(dst + k, __hip_atomic_load(src + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  drain();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(pub.flag, pub.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// True in the workgroup that counts to n; the counter is zero again then.
__device__ __forceinline__ bool count_last(unsigned* c, unsigned n) {
  __shared__ int last;
  if (threadIdx.x == 0) {
    last = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return last != 0;
}

// The same over n workgroups, this one being number k of them, on the counters c + 0,
// kCounterStride, ..: increments of one word take about 25 ns each, one after the other, so
// more than kCounterFan workgroups count in kCounterFan groups first.
__device__ __forceinline__ bool count_last_of(unsigned* c, unsigned k, unsigned n) {
  if (n <= kCounterFan) return count_last(c, n);
  const unsigned g = k % kCounterFan;
  if (!count_last(c + (1 + g) * kCounterStride, n / kCounterFan + (g < n % kCounterFan ? 1 : 0))) return false;
  __syncthreads();
  return count_last(c, kCounterFan);
}

// The end of a reducing kernel: thread q < nv holds value q of this tile.  The values go out
// as the tile's partials; the workgroup of the system's last tile sums them over the tiles
// in a fixed order (16 loads per thread in flight, the values of a tile side by side) into
// red[off(q)]; the workgroup of the last system publishes.  A kernel that does this by itself
// saves the launch of a reduction and of a publication, 4 to 6 us each with its gap, for
// 1 to 2 us of waiting in one workgroup.
template <int W, typename Off, typename Done>
__device__ __forceinline__ void close_tile(const LaunchList& L, int kk, const SysDesc* d, int tile, double val, int nv,
                                           Off off, Done done, const Publish& pub) {
  static_assert(W <= 64 && kBlock % W == 0, "values side by side");
  constexpr int G = kBlock / W, U = 16;
  double* part = d->part;
  const int nt = d->ntiles;
  unsigned* cnt = reinterpret_cast<unsigned*>(L.scal + kMaxSys);
  Scal* sc = L.scal + L.sys[kk];
  // the values lie in one wave, which waits for its stores before its first thread counts
  if ((int)threadIdx.x < nv) put_agent(part + (size_t)tile * kMaxRed + threadIdx.x, val);
  drain();
  if (!count_last_of(cnt + L.sys[kk] * kCountersPerSys, (unsigned)tile, (unsigned)nt)) return;
  __shared__ double lds[kBlock];
  const int q = threadIdx.x % W, grp = threadIdx.x / W;
  const double* pq = part + (q < nv ? q : 0);
  double acc = 0.0;
  for (int k = grp; k < nt; k += G * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = get_agent(pq + (size_t)min(k + u * G, nt - 1) * kMaxRed);
#pragma unroll
    for (int u = 0; u < U; ++u) acc += k + u * G < nt ? v[u] : 0.0;
  }
  double s;
  if (W == 1) {
    s = block_sum(acc);
  } else {
    lds[threadIdx.x] = acc;
    __syncthreads();
    s = lds[q];
#pragma unroll
    for (int i = 1; i < G; ++i) s += lds[i * W + q];
    __syncthreads();
    if ((int)threadIdx.x < nv) lds[threadIdx.x] = s;
    __syncthreads();
  }
  if ((int)threadIdx.x < nv) {
    put_agent(sc->red + off(q), s);
    done(sc, q, s, nv > 1 ? lds[1] : 0.0);
  }
  if (!pub.flag) return;
  drain();
  if (count_last(cnt + kMaxSys * kCountersPerSys, (unsigned)L.nsys)) publish(pub);
}

// Start of a CG on |r|^2 = rr.
__device__ __forceinline__ void cg_setup(Scal* sc, double rr, double stop2, int maxit) {
  sc->rrv[0] = rr;
  sc->stop2 = stop2;
  sc->maxit = maxit;
  sc->iters = 0;
  sc->git = 0;
  sc->gang = 0;
  store_active(sc, rr > stop2 ? 1 : 0);
}

// ---------------------------------------------------------------------------
// The normal operator A = M M^dagger + mu2 in one pass.  From eq. (ferm_op), with
// c_A(t) = s(t) (e^{i phi_A(t)} - m) and c_B(t) = s'(t) (e^{-i phi_B(t)} - m) (s = -1
// on the A hop out of t = 0, s' = -1 on the B hop out of t = N_t - 1), the same-slice
// A-B terms of M M^dagger cancel and each row has 12 entries:
//   A(t): (1 + |c_A(t)|^2 + 3 kappa^2 + mu2) x - c_A(t) x_A(t-1) - conj(c_A(t+1)) x_A(t+1)
//         + kappa^2 sum_6 x_A(t) - kappa sum_b (c_A(t) - conj(c_B(t-1)[b])) x_B(t-1)[b]
//   B(t): (1 + |c_B(t)|^2 + 3 kappa^2 + mu2) x - c_B(t) x_B(t+1) - conj(c_B(t-1)) x_B(t-1)
//         + kappa^2 sum_6 x_B(t) - kappa sum_a (conj(c_A(t+1)[a]) - c_B(t)) x_A(t+1)[a]
// where sum_6 runs over the second neighbours (i, j) + {(1,0), (0,1), (-1,0), (-1,1),
// (0,-1), (1,-1)} (the A-B-A and B-A-B paths; wrapped offsets that coincide add,
// exactly as the paths do) and b / a over the three bonds of the site (at slice
// t-1 for A rows, t+1 for B rows).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  double2 r;
  r.x = a.x * b.x - a.y * b.y;
  r.y = a.x * b.y + a.y * b.x;
  return r;
}
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {  // conj(a) b
  double2 r;
  r.x = a.x * b.x + a.y * b.y;
  r.y = a.x * b.y - a.y * b.x;
  return r;
}

template <typename Load>
__device__ __forceinline__ double2 normal12(const Geom& g, const PhasePhi<double>& ph, int n, double mu2, Load ld) {
  const uint32_t q1 = fdiv((uint32_t)n, g.dL2);
  const int j = n - (int)q1 * g.L2;
  const uint32_t q2 = fdiv(q1, g.dL1);
  const int i = (int)q1 - (int)q2 * g.L1;
  const bool isA = (q2 & 1u) == 0;
  const int t = (int)(q2 >> 1);
  const int P = g.P, L1 = g.L1, L2 = g.L2;
  const int tp = (t + 1 == g.Nt) ? 0 : t + 1, tm = (t == 0) ? g.Nt - 1 : t - 1;
  const int ip = (i + 1 == L1) ? 0 : i + 1, im = (i == 0) ? L1 - 1 : i - 1;
  const int jp = (j + 1 == L2) ? 0 : j + 1, jm = (j == 0) ? L2 - 1 : j - 1;
  const int r0 = i * L2, rp = ip * L2, rm = im * L2;
  const int own = n;
  const int pA = 2 * t * P, pB = pA + P;                // planes of slice t
  const int here = isA ? pA : pB;
  // same sublattice at t-1, t+1
  const int nm = (isA ? 2 * tm * P : 2 * tm * P + P) + r0 + j;
  const int np = (isA ? 2 * tp * P : 2 * tp * P + P) + r0 + j;
  // opposite sublattice: A rows take B at t-1 (bonds (i,j), (i-1,j), (i,j-1));
  // B rows take A at t+1 (bonds (i,j), (i+1,j), (i,j+1))
  const int ob = isA ? 2 * tm * P + P : 2 * tp * P;
  const int b0 = ob + r0 + j;
  const int b1 = isA ? ob + rm + j : ob + rp + j;
  const int b2 = isA ? ob + r0 + jm : ob + r0 + jp;
  const double2 xs = ld(own), xm = ld(nm), xp = ld(np);
  const double2 s0 = ld(here + rp + j), s1 = ld(here + r0 + jp), s2 = ld(here + rm + j);
  const double2 s3 = ld(here + rm + jp), s4 = ld(here + r0 + jm), s5 = ld(here + rp + jm);
  const double2 y0 = ld(b0), y1 = ld(b1), y2 = ld(b2);
  const double2 e_own = ph.p[own];
  const double2 e_t = ph.p[isA ? np : nm];  // A: c_A(t+1); B: c_B(t-1)
  const double2 e0 = ph.p[b0], e1 = ph.p[b1], e2 = ph.p[b2];
  const double m = g.ms, kap = g.kappa;
  // signs of the hops: A hop out of slice u carries -1 iff u = 0; B hop iff u = N_t - 1
  const double sA_t = (t == 0) ? -1.0 : 1.0, sA_tp = (t == g.Nt - 1) ? -1.0 : 1.0;
  const double sB_t = (t == g.Nt - 1) ? -1.0 : 1.0, sB_tm = (t == 0) ? -1.0 : 1.0;
  auto cA = [&](double2 e, double sg) { double2 c; c.x = sg * (e.x - m); c.y = sg * e.y; return c; };
  auto cB = [&](double2 e, double sg) { double2 c; c.x = sg * (e.x - m); c.y = -sg * e.y; return c; };
  double2 c_own, c_t, k0, k1, k2;
  if (isA) {
    c_own = cA(e_own, sA_t);                 // c_A(t)
    c_t = cA(e_t, sA_tp);                    // c_A(t+1)
    const double2 d0 = cB(e0, sB_tm), d1 = cB(e1, sB_tm), d2 = cB(e2, sB_tm);  // c_B(t-1)[b]
    k0.x = c_own.x - d0.x; k0.y = c_own.y + d0.y;   // c_A(t) - conj(c_B)
    k1.x = c_own.x - d1.x; k1.y = c_own.y + d1.y;
    k2.x = c_own.x - d2.x; k2.y = c_own.y + d2.y;
  } else {
    c_own = cB(e_own, sB_t);                 // c_B(t)
    c_t = cB(e_t, sB_tm);                    // c_B(t-1)
    const double2 d0 = cA(e0, sA_tp), d1 = cA(e1, sA_tp), d2 = cA(e2, sA_tp);  // c_A(t+1)[a]
    k0.x = d0.x - c_own.x; k0.y = -d0.y - c_own.y;  // conj(c_A) - c_B(t)
    k1.x = d1.x - c_own.x; k1.y = -d1.y - c_own.y;
    k2.x = d2.x - c_own.x; k2.y = -d2.y - c_own.y;
  }
  const double diag = 1.0 + c_own.x * c_own.x + c_own.y * c_own.y + 3.0 * kap * kap + mu2;
  // temporal: A: - c_A(t) x(t-1) - conj(c_A(t+1)) x(t+1);  B: - c_B(t) x(t+1) - conj(c_B(t-1)) x(t-1)
  const double2 ta = cmul(c_own, isA ? xm : xp);
  const double2 tb = cmulc(c_t, isA ? xp : xm);
  const double2 bo0 = cmul(k0, y0), bo1 = cmul(k1, y1), bo2 = cmul(k2, y2);
  const double k2s = kap * kap;
  double2 q;
  q.x = diag * xs.x - ta.x - tb.x + k2s * (s0.x + s1.x + s2.x + s3.x + s4.x + s5.x) - kap * (bo0.x + bo1.x + bo2.x);
  q.y = diag * xs.y - ta.y - tb.y + k2s * (s0.y + s1.y + s2.y + s3.y + s4.y + s5.y) - kap * (bo0.y + bo1.y + bo2.y);
  return q;
}

// out = [b -] (M M^dagger + mu2) in, FP64; |out|^2 into red[red_off], and |b|^2 into red[0]
// with BB.  One pass of the 12-point form.
template <int SPT, bool BB>
__global__ __launch_bounds__(kBlock) void k_normal_slot(const SysDesc* __restrict__ sys, LaunchList L, int s_in,
                                                        int s_b, int s_out, int mode, int red_off, Publish pub) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  (void)sc;
  const Vec<double2> in(d->vec[s_in]);
  const Vec<double2> bv(d->vec[s_b]), out(d->vec[s_out]);
  const PhasePhi<double> ph = phase_of<double>(d);
  const double mu2 = d->mu2;
  auto ld = [=](int k) { return in[k]; };
  double acc = 0.0, bb = 0.0;
#pragma unroll 2
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n >= t_hi) break;
    double2 q = normal12(g, ph, n, mu2, ld);
    const double2 b = bv[n];
    q.x = b.x - q.x;
    q.y = b.y - q.y;
    if (BB) bb += norm2<double>(b);
    out.set(n, q);
    acc += norm2<double>(q);
  }
  double val = block_sum(acc);
  if (BB) {
    const double tb = block_sum(bb);
    if (threadIdx.x == 1) val = tb;
  }
  close_tile<BB ? 2 : 1>(
      L, kk, d, tile, val, BB ? 2 : 1, [=](int q) { return q == 0 ? red_off : 0; },
      [&](Scal* s, int q, double rr, double b2) {
        if (q == 0 && mode == RED_CG_SETUP) cg_setup(s, rr, L.pa[kk] * (BB ? b2 : 1.0) + L.pr[kk] * rr, L.pi[kk]);
      },
      pub);
}

// x = 0, r = b; |b|^2, made NaN where the phase of phi is not finite (so that a non-finite
// phi or b shows in the first reduction the host reads).
template <int SPT>
__global__ __launch_bounds__(kBlock) void k_cg_init_zero(const SysDesc* __restrict__ sys, LaunchList L, int mode,
                                                         Publish pub) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  (void)sc;
  const Vec<double2> b(d->vec[S_B]), x(d->vec[S_X]), r(d->vec[S_R]), ph(d->ph64);
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n < t_hi) {
      const double2 v = b[n];
      const double2 e = ph[n];
      r.set(n, v);
      x.set(n, cz<double2>());
      acc += norm2<double>(v);
      if (!isfinite(e.x) || !isfinite(e.y)) acc = __builtin_nan("");
    }
  }
  const double tot = block_sum(acc);
  close_tile<1>(
      L, kk, d, tile, tot, 1, [](int) { return 0; },
      [&](Scal* s, int, double rr, double) {
        if (mode == RED_CG_SETUP) cg_setup(s, rr, L.pa[kk] + L.pr[kk] * rr, L.pi[kk]);
      },
      pub);
}

// First half of an Arnoldi step: w = A z_j (FP64, the 12-point form) and <v_i, w> = sum
// conj(v_i) w for i <= j, each thread's w fresh in its caches when the basis passes by.  FROM_W: a step
// without an inner solve, where z_j = c64(w_old / |w_old|) is evaluated at the twelve neighbours
// too, so that neither v_j nor z_j has to be there before the launch; w_old and w are in
// different slots.  Each wave sums its two values per i by data-parallel primitives; the
// waves meet once at the end.  With k_cgs this is a step without an inner solve in two
// launches, 21.3 us of kernels for three 24x24x64 systems where seven launches (scaling,
// operator, products, their sum, subtraction, its sum, publication) took 32.
template <int SPT, bool FROM_W>
__global__ __launch_bounds__(kBlock) void k_arnoldi_dots(const SysDesc* __restrict__ sys, LaunchList L, int j) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  const int s_w = L.it[kk];
  const Vec<double2> w(d->vec[s_w]), old(d->vec[S_R + S_U - s_w]), vj(d->vec[S_V0 + j]);
  const Vec<float2> z(d->vec[S_Z0 + j]);
  const PhasePhi<double> ph = phase_of<double>(d);
  const double mu2 = d->mu2, scale = !FROM_W || j == 0 ? L.pa[kk] : 1.0 / sqrt(fmax(sc->red[2 * j], 0.0));
  auto scaled = [=](int k) {
    double2 a = old[k];
    a.x *= scale;
    a.y *= scale;
    return a;
  };
  auto single = [](double2 a) {
    float2 f;
    f.x = (float)a.x;
    f.y = (float)a.y;
    return f;
  };
  auto ld = [=](int k) { return to_c128(FROM_W ? single(scaled(k)) : z[k]); };
#pragma unroll 2
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n >= t_hi) break;
    w.set(n, normal12(g, ph, n, mu2, ld));
    if (FROM_W) {
      const double2 own = scaled(n);
      vj.set(n, own);
      z.set(n, single(own));
    }
  }
  // each thread reads back its own sites only: no barrier
  double2 wv[SPT];
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    wv[m] = cz<double2>();
    if (n < t_hi) wv[m] = w[n];
  }
  __shared__ double sums[kBlock / 64][kMaxRed];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll 2
  for (int q = 0; q <= j; ++q) {
    const Vec<double2> v(d->vec[S_V0 + q]);
    double ar = 0.0, ai = 0.0;
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      const int n = base + m * kBlock;
      if (n < t_hi) {
        const double2 vv = v[n];
        ar += vv.x * wv[m].x + vv.y * wv[m].y;
        ai += vv.x * wv[m].y - vv.y * wv[m].x;
      }
    }
    ar = dpp_wave(ar);
    ai = dpp_wave(ai);
    if (lane == 63) {
      sums[wave][2 * q] = ar;
      sums[wave][2 * q + 1] = ai;
    }
  }
  __syncthreads();
  const int nv = 2 * (j + 1);
  double val = 0.0;
  if ((int)threadIdx.x < nv)
    val = (sums[0][threadIdx.x] + sums[1][threadIdx.x]) + (sums[2][threadIdx.x] + sums[3][threadIdx.x]);
  const Publish none;
  auto off = [](int q) { return q; };
  auto done = [](Scal*, int, double, double) {};
  if (nv <= 8)
    close_tile<8>(L, kk, d, tile, val, nv, off, done, none);
  else if (nv <= 32)
    close_tile<32>(L, kk, d, tile, val, nv, off, done, none);
  else
    close_tile<64>(L, kk, d, tile, val, nv, off, done, none);
}

// w -= sum_i h_i v_i, i <= j, h_i = red[2i] + i red[2i+1]; |w|^2 into red[2j+2].
template <int SPT>
__global__ __launch_bounds__(kBlock) void k_cgs(const SysDesc* __restrict__ sys, LaunchList L, int j, Publish pub) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  const Vec<double2> w(d->vec[L.it[kk]]);
  double2 wv[SPT];
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    wv[m] = cz<double2>();
    if (n < t_hi) wv[m] = w[n];
  }
#pragma unroll 2
  for (int q = 0; q <= j; ++q) {
    const double hr = sc->red[2 * q], hi = sc->red[2 * q + 1];
    const Vec<double2> v(d->vec[S_V0 + q]);
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      const int n = base + m * kBlock;
      if (n < t_hi) {
        const double2 vv = v[n];
        wv[m].x -= hr * vv.x - hi * vv.y;
        wv[m].y -= hr * vv.y + hi * vv.x;
      }
    }
  }
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n < t_hi) {
      w.set(n, wv[m]);
      acc += norm2<double>(wv[m]);
    }
  }
  const double tot = block_sum(acc);
  close_tile<1>(
      L, kk, d, tile, tot, 1, [=](int) { return 2 * (j + 1); }, [](Scal*, int, double, double) {}, pub);
}

// v = pa*src (FP64, stored to s_v if s_v >= 0) and the single-precision CG's start on it:
// r32 = c64(v), z = 0 (the slot pj), |r32|^2 (FP32 sums within a tile).
template <int SPT>
__global__ __launch_bounds__(kBlock) void k_prep_inner(const SysDesc* __restrict__ sys, LaunchList L, int s_v) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  (void)sc;
  const double scale = L.pa[kk];
  const bool store_v = s_v >= 0;
  const Vec<double2> src(d->vec[L.it[kk]]), v(store_v ? d->vec[s_v] : nullptr);
  const Vec<float2> z(d->vec[L.pj[kk]]), r32(d->vec[S_R32]);
  float acc = 0.0f;
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n < t_hi) {
      double2 a = src[n];
      a.x *= scale;
      a.y *= scale;
      if (store_v) v.set(n, a);
      float2 a32;
      a32.x = (float)a.x;
      a32.y = (float)a.y;
      r32.set(n, a32);
      z.set(n, cz<float2>());
      acc += norm2<float>(a32);
    }
  }
  const double tot = (double)block_sum(acc);
  const Publish none;
  close_tile<1>(
      L, kk, d, tile, tot, 1, [](int) { return 0; },
      [&](Scal* s, int, double rr, double) { cg_setup(s, rr, L.pr[kk] * rr, L.pi[kk]); }, none);
}

__global__ __launch_bounds__(kBlock) void k_publish(Publish pub) { publish(pub); }

// x = (set ? 0 : x) + sum_{i < cnt} y_i z_i, y from ys (row of the system's slot), z_i the
// C64 slot S_Z0 + i.
template <int SPT>
__global__ __launch_bounds__(kBlock) void k_xupdate(const SysDesc* __restrict__ sys, LaunchList L,
                                                    const double* __restrict__ ys, int cnt, int set) {
  constexpr int TILE = kBlock * SPT;
  HUB_PROLOGUE_T(TILE)
  (void)sc;
  const double* __restrict__ yrow = ys + (size_t)L.sys[kk] * kYStride;
  const Vec<double2> x(d->vec[S_X]);
  double2 xv[SPT];
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    xv[m] = cz<double2>();
    if (n < t_hi && !set) xv[m] = x[n];
  }
  for (int q = 0; q < cnt; ++q) {
    const double yr = yrow[2 * q], yi = yrow[2 * q + 1];
    const Vec<float2> z(d->vec[S_Z0 + q]);
#pragma unroll
    for (int m = 0; m < SPT; ++m) {
      const int n = base + m * kBlock;
      if (n < t_hi) {
        const float2 zf = z[n];
        const double zr = zf.x, zi = zf.y;
        xv[m].x += yr * zr - yi * zi;
        xv[m].y += yr * zi + yi * zr;
      }
    }
  }
#pragma unroll
  for (int m = 0; m < SPT; ++m) {
    const int n = base + m * kBlock;
    if (n < t_hi) x.set(n, xv[m]);
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------
static inline int tiles_of(int n) { return (n + kTile - 1) / kTile; }

template <bool NT>
static void apply_nt(const Geom& g, const double* phi, const double2* x, double2* y, int batch, bool dag,
                     hipStream_t st) {
  const int nt = (g.n + kPubTile - 1) / kPubTile;
  const int per = pub_group(nt, batch);
  const dim3 grid(nt * ((batch + per - 1) / per)), block(kBlock);
  if (per == 1) {
    if (dag)
      hipLaunchKernelGGL((k_apply<true, NT>), grid, block, 0, st, g, phi, x, y, nt);
    else
      hipLaunchKernelGGL((k_apply<false, NT>), grid, block, 0, st, g, phi, x, y, nt);
  } else {
    if (dag)
      hipLaunchKernelGGL((k_apply_grp<true, NT>), grid, block, 0, st, g, phi, x, y, nt, per, batch);
    else
      hipLaunchKernelGGL((k_apply_grp<false, NT>), grid, block, 0, st, g, phi, x, y, nt, per, batch);
  }
}

hipError_t launch_apply(const Geom& g, const double* phi, const double2* x, double2* y, int batch, bool dag,
                        hipStream_t st, bool to_caller) {
  if (to_caller)
    apply_nt<true>(g, phi, x, y, batch, dag, st);
  else
    apply_nt<false>(g, phi, x, y, batch, dag, st);
  return hipGetLastError();
}


hipError_t launch_force(const Geom& g, const double* phi, const double2* eta, const double2* xi, double scale,
                        int accumulate, double* out, int batch, hipStream_t st) {
  const int nt = tiles_of(g.n);
  // 2048-site tiles: a quarter of the public kernels' workgroups per vector
  const int per = pub_group(4 * nt, batch);
  const dim3 grid(nt * ((batch + per - 1) / per)), block(kBlock);
  if (per == 1)
    hipLaunchKernelGGL(k_force, grid, block, 0, st, g, phi, eta, xi, scale, accumulate, out, nt);
  else
    hipLaunchKernelGGL(k_force_grp, grid, block, 0, st, g, phi, eta, xi, scale, accumulate, out, nt, per,
                       batch);
  return hipGetLastError();
}

hipError_t launch_apply_jobs(const Geom& g, const ApplyJobs& J, int njob, bool dag, hipStream_t st) {
  if (njob < 1 || njob > kMaxSys) return hipErrorInvalidValue;
  const int nt = (g.n + kPubTile - 1) / kPubTile;
  if (dag)
    hipLaunchKernelGGL(k_apply_jobs<true>, dim3(nt * njob), dim3(kBlock), 0, st, g, J, nt);
  else
    hipLaunchKernelGGL(k_apply_jobs<false>, dim3(nt * njob), dim3(kBlock), 0, st, g, J, nt);
  return hipGetLastError();
}

hipError_t launch_terms(const Geom& g, const TermJobs& J, int nchain, bool force, double* part, double* result,
                        hipStream_t st) {
  if (nchain < 1 || J.nterm < 1 || J.nterm > kMaxTerms || nchain * J.nterm > kMaxSys) return hipErrorInvalidValue;
  const int nt = (g.n + kBlock - 1) / kBlock;
  if (force)
    hipLaunchKernelGGL(k_terms<true>, dim3(nt * nchain), dim3(kBlock), 0, st, g, J, nt, part, result);
  else
    hipLaunchKernelGGL(k_terms<false>, dim3(nt * nchain), dim3(kBlock), 0, st, g, J, nt, part, result);
  if (nt > 1)
    hipLaunchKernelGGL(k_dot_finish, dim3(nchain * J.nterm), dim3(kBlock), 0, st, part, nt, result);
  return hipGetLastError();
}

hipError_t launch_phase_jobs(const PhaseJobs& J, int njob, int n, hipStream_t st) {
  if (njob < 1 || njob > kMaxSys) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_phase_jobs, dim3((n + kBlock - 1) / kBlock, njob), dim3(kBlock), 0, st, J, n);
  return hipGetLastError();
}

hipError_t launch_force_sum(const Geom& g, const double* phi, const double2* eta, const double2* xi,
                            const double* scale_host, int accumulate, double* out, int batch, hipStream_t st) {
  if (batch < 1 || batch > kMaxSys) return hipErrorInvalidValue;
  Mu2Arr sc;
  for (int b = 0; b < kMaxSys; ++b) sc.v[b] = b < batch ? scale_host[b] : 0.0;
  hipLaunchKernelGGL(k_force_sum, dim3(tiles_of(g.n)), dim3(kBlock), 0, st, g, phi, eta, xi, sc, accumulate, out,
                     batch);
  return hipGetLastError();
}

hipError_t launch_stream_bytes(const double* phi, const double2* x, double2* y, int n, int mode, hipStream_t st) {
  const dim3 grid((n + kPubTile - 1) / kPubTile), block(kBlock);
  if (mode == 0)
    hipLaunchKernelGGL((k_stream_bytes<false, true>), grid, block, 0, st, phi, x, y, n);
  else if (mode == 1)
    hipLaunchKernelGGL((k_stream_bytes<true, false>), grid, block, 0, st, phi, x, y, n);
  else
    hipLaunchKernelGGL((k_stream_bytes<false, false>), grid, block, 0, st, phi, x, y, n);
  return hipGetLastError();
}

hipError_t launch_dot_re(const Geom& g, const double2* a, const double2* b, int batch, double* part,
                         double* result, hipStream_t st) {
  const int nt = tiles_of(g.n);
  hipLaunchKernelGGL(k_dot_re, dim3(nt * batch), dim3(kBlock), 0, st, g, a, b, nt, part);
  hipLaunchKernelGGL(k_dot_finish, dim3(batch), dim3(kBlock), 0, st, part, nt, result);
  return hipGetLastError();
}

hipError_t launch_md_drift(double* phi, const double* pi, double eps, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_md_drift, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, phi, pi, eps, n);
  return hipGetLastError();
}

hipError_t launch_md_kick(double* pi, const double* phi, const double* G, double cg, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_md_kick, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, pi, phi, G, cg, n);
  return hipGetLastError();
}

hipError_t launch_ms_start(const MsDesc* d, int ntiles, hipStream_t st) {
  hipLaunchKernelGGL(k_ms_start, dim3(ntiles), dim3(kBlock), 0, st, d);
  hipLaunchKernelGGL(k_ms_setup, dim3(1), dim3(kBlock), 0, st, d);
  return hipGetLastError();
}

hipError_t launch_ms_iter(const MsDesc* d, int ntiles, int it, hipStream_t st) {
  hipLaunchKernelGGL(k_ms1, dim3(ntiles), dim3(kBlock), 0, st, d, it);
  hipLaunchKernelGGL(k_ms2, dim3(ntiles), dim3(kBlock), 0, st, d, it);
  return hipGetLastError();
}

// One pass pays for the phases' kernel where the batch is large: from a million sites of all
// vectors on, from half as many with six vectors or more (microseconds of the kernels in two
// passes and in one, buffers resident; rotated: one pass gains more).  Below: 30x30x128, three
// vectors 13.8, 16.9; 90x60x40, two 16.1, 18.0; 24x24x64, five 9.9, 10.2; 102x102x64, one 25.6,
// 31.2.  Above: 30x30x128, five 21.7, 19.3, eight 28.5, 23.4; 64x64x64, two 19.8, 18.8;
// 24x24x64, eight 12.7, 11.9; 102x102x64, two 38.6, 35.8.  Both give the same bits.
static bool normal_one_pass(int n, int batch) {
  return batch > 1 && (long)n * batch >= (batch < 6 ? 1L << 20 : 1L << 19);
}

size_t normal_scratch(const Geom& g, int batch, bool least) {
  return (size_t)g.n * 16 * (least || normal_one_pass(g.n, batch) ? 1 : batch);
}

hipError_t launch_normal(const Geom& g, const double* phi, double2* ws, size_t ws_bytes, const double mu2_host[kMaxSys],
                         const double2* x, double2* y, int batch, hipStream_t st) {
  Mu2Arr m;
  for (int b = 0; b < kMaxSys; ++b) m.v[b] = b < batch ? mu2_host[b] : 0.0;
  if (normal_one_pass(g.n, batch) || ws_bytes < (size_t)g.n * 16 * batch) {
    const int nt = (g.n + kBlock - 1) / kBlock;
    // groups of even size: seven vectors and one in two groups took as long as two of seven
    // (30x30x128, eight vectors 34.7 us, 23.4 with four and four)
    int per = pub_group(nt, batch);
    const int groups = (batch + per - 1) / per;
    per = (batch + groups - 1) / groups;
    hipLaunchKernelGGL(k_phase_pub, dim3(nt), dim3(kBlock), 0, st, phi, ws, g.n);
    hipLaunchKernelGGL(k_normal_pub, dim3(nt * ((batch + per - 1) / per)), dim3(kBlock), 0, st, g, ws, m, x, y, nt, per,
                       batch);
    return hipGetLastError();
  }
  const hipError_t e = launch_apply(g, phi, x, ws, batch, true, st);
  if (e != hipSuccess) return e;
  const int nt = (g.n + kPubTile - 1) / kPubTile;
  hipLaunchKernelGGL(k_normal2_pub, dim3(nt * batch), dim3(kBlock), 0, st, g, phi, m, ws, x, y, nt);
  return hipGetLastError();
}

hipError_t launch_phase(const double* phi, double2* p64, float* p32, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_phase, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, phi, p64, p32, n);
  return hipGetLastError();
}

template <int N>
static CgList<N> cg_list(const LaunchList& L) {
  CgList<N> c;
  std::memset(&c, 0, sizeof(c));
  c.scal = L.scal;
  c.nsys = L.nsys;
  c.total_tiles = L.total_tiles;
  for (int k = 0; k <= N; ++k) c.tile_begin[k] = k <= L.nsys ? L.tile_begin[k] : L.total_tiles;
  for (int k = 0; k < L.nsys; ++k) {
    c.sys[k] = L.sys[k];
    c.pi[k] = L.pi[k];
    c.it[k] = L.it[k];
  }
  return c;
}

// One CG stage (1 or 2) over the list; with events, the launch records its own start and end.
template <typename R, int SPT, typename LL>
static void cg_stage(const SysDesc* sys, const LL& c, int stage, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(c.total_tiles), block(kBlock);
  const bool single = sizeof(R) == 4;
  const int sR = single ? (int)S_R32 : (int)S_R, sP = single ? (int)S_P32 : (int)S_P0,
            sU = single ? (int)S_U32 : (int)S_U;
  auto kern = stage == 1 ? k_cg1<R, LL, SPT> : k_cg2<R, LL, SPT>;
  if (e0)
    hipExtLaunchKernelGGL(kern, grid, block, 0, st, e0, e1, 0, sys, c, sR, sP, sU);
  else
    hipLaunchKernelGGL(kern, grid, block, 0, st, sys, c, sR, sP, sU);
}

template <typename R, int SPT>
static void cg_stage_list(const SysDesc* sys, const LaunchList& L, int stage, hipStream_t st, hipEvent_t e0,
                          hipEvent_t e1) {
  if (L.nsys <= kSmallCg)
    cg_stage<R, SPT>(sys, cg_list<kSmallCg>(L), stage, st, e0, e1);
  else
    cg_stage<R, SPT>(sys, cg_list<kMaxSys>(L), stage, st, e0, e1);
}

template <typename R>
static void cg_stage_any(const SysDesc* sys, const LaunchList& L, int spt, int stage, hipStream_t st,
                         hipEvent_t e0, hipEvent_t e1) {
  if (spt == kSmallSpt)
    cg_stage_list<R, kSmallSpt>(sys, L, stage, st, e0, e1);
  else
    cg_stage_list<R, kSitesPerThread>(sys, L, stage, st, e0, e1);
}

static bool spt_ok(const LaunchList& L) { return L.spt == kSmallSpt || L.spt == kSitesPerThread; }

hipError_t launch_cg_iter(const SysDesc* sys, const LaunchList& L, bool single, hipStream_t st) {
  if (!spt_ok(L)) return hipErrorInvalidValue;
  for (int stage = 1; stage <= 2; ++stage) {
    if (single)
      cg_stage_any<float>(sys, L, L.spt, stage, st, nullptr, nullptr);
    else
      cg_stage_any<double>(sys, L, L.spt, stage, st, nullptr, nullptr);
  }
  return hipGetLastError();
}

hipError_t launch_cg_stage(const SysDesc* sys, const LaunchList& L, bool single, int stage, hipStream_t st,
                           hipEvent_t e0, hipEvent_t e1) {
  if (!spt_ok(L)) return hipErrorInvalidValue;
  if (single)
    cg_stage_any<float>(sys, L, L.spt, stage, st, e0, e1);
  else
    cg_stage_any<double>(sys, L, L.spt, stage, st, e0, e1);
  return hipGetLastError();
}


hipError_t launch_publish(const Publish& pub, hipStream_t st) {
  if (pub.cnt < 1 || pub.cnt > kMaxSys || !pub.d || !pub.h || !pub.flag) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(kBlock), 0, st, pub);
  return hipGetLastError();
}

// Launch KERNEL<..., SPT> for the tile class of L.
#define HUB_BY_CLASS(KERNEL, GRID, ...)                                                       \
  do {                                                                                       \
    if (L.spt == kSmallSpt)                                                                  \
      hipLaunchKernelGGL(KERNEL<kSmallSpt>, GRID, dim3(kBlock), 0, st, __VA_ARGS__);          \
    else                                                                                     \
      hipLaunchKernelGGL(KERNEL<kSitesPerThread>, GRID, dim3(kBlock), 0, st, __VA_ARGS__);    \
  } while (0)

hipError_t launch_normal_slot(const SysDesc* sys, const LaunchList& L, int s_in, int s_b, int s_out, RedMode mode,
                              int red_off, bool with_bb, const Publish& pub, hipStream_t st) {
  if (!spt_ok(L) || red_off < (with_bb ? 1 : 0) || red_off >= kMaxRed) return hipErrorInvalidValue;
  const dim3 grid(L.total_tiles), block(kBlock);
  const bool small = L.spt == kSmallSpt;
  auto kern = with_bb ? (small ? k_normal_slot<kSmallSpt, true> : k_normal_slot<kSitesPerThread, true>)
                      : (small ? k_normal_slot<kSmallSpt, false> : k_normal_slot<kSitesPerThread, false>);
  hipLaunchKernelGGL(kern, grid, block, 0, st, sys, L, s_in, s_b, s_out, (int)mode, red_off, pub);
  return hipGetLastError();
}

hipError_t launch_cg_init_zero(const SysDesc* sys, const LaunchList& L, RedMode mode, const Publish& pub,
                               hipStream_t st) {
  if (!spt_ok(L)) return hipErrorInvalidValue;
  HUB_BY_CLASS(k_cg_init_zero, dim3(L.total_tiles), sys, L, (int)mode, pub);
  return hipGetLastError();
}

hipError_t launch_arnoldi_dots(const SysDesc* sys, const LaunchList& L, int j, bool from_w, hipStream_t st) {
  if (!spt_ok(L) || j < 0 || j >= kMaxRestart) return hipErrorInvalidValue;
  for (int k = 0; k < L.nsys; ++k)
    if (L.it[k] != S_R && L.it[k] != S_U) return hipErrorInvalidValue;
  const bool small = L.spt == kSmallSpt;
  auto kern = from_w ? (small ? k_arnoldi_dots<kSmallSpt, true> : k_arnoldi_dots<kSitesPerThread, true>)
                     : (small ? k_arnoldi_dots<kSmallSpt, false> : k_arnoldi_dots<kSitesPerThread, false>);
  hipLaunchKernelGGL(kern, dim3(L.total_tiles), dim3(kBlock), 0, st, sys, L, j);
  return hipGetLastError();
}

hipError_t launch_cgs(const SysDesc* sys, const LaunchList& L, int j, const Publish& pub, hipStream_t st) {
  if (!spt_ok(L) || j < 0 || j >= kMaxRestart) return hipErrorInvalidValue;
  HUB_BY_CLASS(k_cgs, dim3(L.total_tiles), sys, L, j, pub);
  return hipGetLastError();
}

hipError_t launch_prep_inner(const SysDesc* sys, const LaunchList& L, int s_v, hipStream_t st) {
  if (!spt_ok(L)) return hipErrorInvalidValue;
  HUB_BY_CLASS(k_prep_inner, dim3(L.total_tiles), sys, L, s_v);
  return hipGetLastError();
}

hipError_t launch_xupdate(const SysDesc* sys, const LaunchList& L, const double* ys, int cnt, bool set,
                          hipStream_t st) {
  if (!spt_ok(L)) return hipErrorInvalidValue;
  HUB_BY_CLASS(k_xupdate, dim3(L.total_tiles), sys, L, ys, cnt, set ? 1 : 0);
  return hipGetLastError();
}

}  // namespace hub
