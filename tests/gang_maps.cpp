// Host check of the gang CG's maps (hub_gang.h): every workgroup of a cut is walked as the
// kernel walks it, on a table of its own, and w = M M^dagger r is compared with the plain
// stencil on the whole lattice.  Exit 0: every entry read was written, every element
// received was sent, and the values agree.
#define __host__
#define __device__
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "hub_gang.h"

using namespace hub;
using cd = std::complex<double>;

static unsigned long long seed = 1;
static double rnd() {
  seed = seed * 6364136223846793005ull + 1442695040888963407ull;
  return (double)(seed >> 11) / 9007199254740992.0 - 0.5;
}

struct Lat {
  int L1, L2, Nt;
  double kappa = 0.3, ms = 0.07;
  int at(int t, int s, int i, int j) const {
    t = (t + Nt) % Nt, i = (i + L1) % L1, j = (j + L2) % L2;
    return ((t * 2 + s) * L1 + i) * L2 + j;
  }
  int n() const { return 2 * L1 * L2 * Nt; }
};
static cd link(const Lat& l, const std::vector<double>& phi, int t, int s, int i, int j) {
  t = (t + l.Nt) % l.Nt;
  const double f = phi[l.at(t, s, i, j)], sg = (s == 0 ? t == 0 : t == l.Nt - 1) ? -1.0 : 1.0;
  return sg * (std::polar(1.0, s ? -f : f) - l.ms);
}
static std::vector<cd> apply(const Lat& l, const std::vector<double>& phi, const std::vector<cd>& x, bool dag) {
  std::vector<cd> y(l.n());
  for (int t = 0; t < l.Nt; ++t)
    for (int s = 0; s < 2; ++s)
      for (int i = 0; i < l.L1; ++i)
        for (int j = 0; j < l.L2; ++j) {
          const int d = s ? 1 : -1;
          const cd b = x[l.at(t, 1 - s, i, j)] + x[l.at(t, 1 - s, i + d, j)] + x[l.at(t, 1 - s, i, j + d)];
          const int dt = (s == 0) == dag ? 1 : -1;
          const cd c = dag ? std::conj(link(l, phi, t + dt, s, i, j)) : link(l, phi, t, s, i, j);
          y[l.at(t, s, i, j)] = (s ? 1.0 : -1.0) * (x[l.at(t, s, i, j)] - c * x[l.at(t + dt, s, i, j)]) - l.kappa * b;
        }
  return y;
}

static int fail(const char* what, const Lat& l, int gt, int gi, int gj) {
  std::printf("%s: %dx%dx%d cut %dx%dx%d\n", what, l.L1, l.L2, l.Nt, gt, gi, gj);
  return 1;
}

// A table whose entries know whether they were written in this phase.
struct Table {
  std::vector<cd> v;
  std::vector<char> ok;
  bool bad = false;
  explicit Table(int n) : v(n), ok(n, 0) {}
  void set(int k, cd x) {
    if (k < 0 || k >= (int)v.size()) {
      bad = true;
      return;
    }
    v[k] = x, ok[k] = 1;
  }
  cd get(int k) {
    if (k < 0 || k >= (int)v.size() || !ok[k]) {
      bad = true;
      return 0;
    }
    return v[k];
  }
};

static int check(const Lat& l, int gt, int gi, int gj) {
  const int G = gt * gi * gj;
  std::vector<double> phi(l.n());
  std::vector<cd> r(l.n());
  for (auto& p : phi) p = 4 * rnd();
  for (auto& z : r) z = cd(rnd(), rnd());
  const std::vector<cd> want = apply(l, phi, apply(l, phi, r, true), false);
  const GangBlock big = gang_largest(l.L1, l.L2, l.Nt, gt, gi, gj);
  const int nslot = gang_slots(big);
  std::vector<cd> exch((size_t)G * nslot);
  std::vector<char> sent((size_t)G * nslot, 0);
  std::vector<int> owners(l.n(), 0);
  for (int wg = 0; wg < G; ++wg) {
    const GangBlock B = gang_block(l.L1, l.L2, l.Nt, gt, gi, gj, wg);
    if (B.half > big.half || gang_halos(B) > gang_halos(big) || gang_extras(B) > gang_extras(big) ||
        gang_entries(B) > gang_entries(big))
      return fail("a block beyond the largest", l, gt, gi, gj);
    for (int s = 0; s < 2; ++s)
      for (int k = 0; k < B.half; ++k) {
        const GangSite c = gang_site(B, k);
        const int n = l.at(B.t0 + c.t, s, B.i0 + c.i, B.j0 + c.j);
        owners[n]++;
        auto send = [&](int place) {
          exch[(size_t)wg * nslot + place] = r[n];
          sent[(size_t)wg * nslot + place] = 1;
        };
        if (gang_slots(B) > nslot) return fail("more elements than slots", l, gt, gi, gj);
        if (gang_sent(B, c)) send(s * B.half + k);
        if (gt > 1 && c.t == 0) send(gang_plane(B, 0, s, gang_div(k, B.rT)));
        if (gt > 1 && c.t == B.T - 1) send(gang_plane(B, 1, s, gang_div(k, B.rT)));
      }
  }
  for (int o : owners)
    if (o != 1) return fail("a site without one owner", l, gt, gi, gj);
  double worst = 0.0;
  for (int wg = 0; wg < G; ++wg) {
    const GangBlock B = gang_block(l.L1, l.L2, l.Nt, gt, gi, gj, wg);
    Table F(gang_entries(B)), E(gang_entries(B));
    for (int q = 0; q < B.ea * B.eb; ++q)
      for (int s = 0; s < 2; ++s)
        for (int te = 0; te < B.TS; ++te)
          E.set((q * 2 + s) * B.TS + te, link(l, phi, B.t0 + te - 1, s, B.i0 + q / B.eb - B.oi, B.j0 + q % B.eb - B.oj));
    auto put = [&](Table& t, int e, int te, cd v) {
      t.set(e, v);
      if (B.gt == 1 && te == 1) t.set(e + B.T, v);
      if (B.gt == 1 && te == B.T) t.set(e - B.T, v);
    };
    for (int s = 0; s < 2; ++s)
      for (int k = 0; k < B.half; ++k) {
        const GangSite c = gang_site(B, k);
        put(F, gang_entry(B, c.i, c.j, s, c.t + 1), c.t + 1, r[l.at(B.t0 + c.t, s, B.i0 + c.i, B.j0 + c.j)]);
      }
    for (int e = 0; e < gang_halos(B); ++e) {
      const GangHalo h = gang_halo(B, e);
      int src, k;
      gang_source(B, h, src, k);
      if (src < 0 || src >= G || k < 0 || k >= nslot || !sent[(size_t)src * nslot + k])
        return fail("an element nobody sends", l, gt, gi, gj);
      put(F, gang_entry(B, h.i, h.j, h.s, h.te), h.te, exch[(size_t)src * nslot + k]);
    }
    // the kernel's two passes; v stands for -u on A and u on B
    auto pass = [&](Table& f, int s, int i, int j, int te, bool first) {
      const int a0 = gang_entry(B, i, j, s, te), dh = s ? -B.TS : B.TS;
      int h1, h2;
      gang_bonds(B, i, j, s, te, h1, h2);
      const int dt = ((s == 0) == first) ? 1 : -1;
      const cd c = first ? std::conj(E.get(a0 + dt)) : E.get(a0);
      const double ks = (s ? -l.kappa : l.kappa) * (first ? 1.0 : -1.0);
      return f.get(a0) - c * f.get(a0 + dt) + ks * (f.get(a0 + dh) + f.get(h1) + f.get(h2));
    };
    Table V(gang_entries(B));
    for (int s = 0; s < 2; ++s) {
      for (int k = 0; k < B.half; ++k) {
        const GangSite c = gang_site(B, k);
        put(V, gang_entry(B, c.i, c.j, s, c.t + 1), c.t + 1, pass(F, s, c.i, c.j, c.t + 1, true));
      }
      for (int e = 0; e < gang_extras(B); ++e) {
        int i, j, te;
        gang_extra(B, s, e, i, j, te);
        // with time uncut an extra column is only read at its own slices
        V.set(gang_entry(B, i, j, s, te), pass(F, s, i, j, te, true));
      }
    }
    for (int s = 0; s < 2; ++s)
      for (int k = 0; k < B.half; ++k) {
        const GangSite c = gang_site(B, k);
        const cd w = pass(V, s, c.i, c.j, c.t + 1, false);
        worst = std::max(worst, std::abs(w - want[l.at(B.t0 + c.t, s, B.i0 + c.i, B.j0 + c.j)]));
      }
    if (F.bad || E.bad || V.bad) return fail("an entry read before it was written", l, gt, gi, gj);
  }
  if (!(worst < 1e-13)) {
    std::printf("worst %g ", worst);
    return fail("values", l, gt, gi, gj);
  }
  return 0;
}

template <typename R>
static int chosen(const Lat& l, bool show) {
  const GangCut c = gang_cut<R>(l.L1, l.L2, l.Nt);
  if (c.g == 0) {
    if (show) std::printf("%s %dx%dx%d: none\n", sizeof(R) == 4 ? "f32" : "f64", l.L1, l.L2, l.Nt);
    return 0;
  }
  const GangBlock B = gang_largest(l.L1, l.L2, l.Nt, c.gt, c.gi, c.gj);
  if (c.g != c.gt * c.gi * c.gj || c.g > kGangMaxWgs || gang_class<R>(B) != c.cls || c.nslot != gang_slots(B))
    return fail("the chosen cut", l, c.gt, c.gi, c.gj);
  if (show)
    std::printf("%s %dx%dx%d: %dx%dx%d = %d, class %d half %d halos %d extras %d table %d cost %.2f\n", sizeof(R) == 4 ? "f32" : "f64",
                l.L1, l.L2, l.Nt, c.gt, c.gi, c.gj, c.g, c.cls, B.half, gang_halos(B), gang_extras(B),
                gang_table(B), gang_cost<R>(B, c.cls, c.g));
  return l.n() <= 40000 ? check(l, c.gt, c.gi, c.gj) : 0;
}

int main(int argc, char** argv) {
  const bool show = argc > 1;
  int bad = 0;
  // explicit cuts: uncut, each direction alone, all together; degenerate and uneven extents
  const int lats[][3] = {{1, 1, 1}, {1, 1, 2}, {2, 1, 8}, {1, 3, 2}, {2, 2, 4}, {3, 3, 8}, {5, 7, 6}, {6, 4, 9}, {4, 9, 16}};
  for (auto& x : lats) {
    Lat l{x[0], x[1], x[2]};
    for (int gt = 1; gt <= 4 && gt <= l.Nt; ++gt)
      for (int gi = 1; gi <= 4 && gi <= l.L1; ++gi)
        for (int gj = 1; gj <= 4 && gj <= l.L2; ++gj) bad += check(l, gt, gi, gj);
  }
  // the cut that the rule picks, over the range of lattices
  const int some[][3] = {{2, 1, 64}, {4, 3, 27}, {6, 6, 16}, {6, 6, 64}, {9, 9, 40}, {12, 12, 32}, {11, 11, 42}, {12, 12, 64},
                         {13, 22, 18}, {25, 23, 30}, {24, 24, 32}, {24, 24, 64}, {33, 17, 6}, {48, 48, 16}, {40, 32, 46},
                         {48, 48, 64}, {39, 74, 20}, {102, 102, 16}, {102, 102, 64}, {102, 51, 64}, {1, 1, 3}, {90, 90, 64},
                         {120, 120, 64}, {1, 1, 20000}, {1000, 1, 4}};
  for (auto& x : some) {
    Lat l{x[0], x[1], x[2]};
    bad += chosen<float>(l, show) + chosen<double>(l, show);
  }
  if (bad) std::printf("%d wrong\n", bad);
  return bad ? 1 : 0;
}
