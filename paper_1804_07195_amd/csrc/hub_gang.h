// Geometry of the gang CG: how a lattice is cut over the workgroups that iterate on it
// together, and where every site of a workgroup's block and of its halo lives.  Shared by
// the kernel (hub_gang.hip), the engine that picks the cut, and the host check of the maps.
#pragma once

#include <cstddef>
#include <cstdint>

namespace hub {

constexpr int kGangThreads = 512;              // threads per workgroup: half per sublattice
constexpr int kGangHalf = kGangThreads / 2;
constexpr int kGangMaxWgs = 256;               // workgroups of one launch: one per CU
// LDS of a workgroup: the reductions, the field table, and the table of links a fixed
// distance behind it, so that one address reaches both (the immediate offset of an LDS
// access is 16 bits).
constexpr int kGangHead = 256;
constexpr int kGangLinks = 65280;
constexpr int kGangLdsBytes = kGangHead + 2 * kGangLinks;
constexpr int kGangRecWords = 4;               // 8-byte words of a reduction record
constexpr int kGangCopies = 8;                 // of every record: workgroup k polls copy k mod 8
constexpr int kGangCtlWords = 32;              // 8-byte control words in front of the records

// Classes of the kernel: sites (M), halo elements (H) and extra sites (X) per thread.  The
// kernel's loops over a thread's sites are unrolled (the vectors are in registers), so a
// small block runs a body of its own size: skipping the sites of a larger body costs a
// branch each, three times an iteration of a 6x6x16 system.
struct GangClass {
  int M, H, X;
};
template <typename R> struct GangTab;
template <> struct GangTab<float> {
  static constexpr int n = 7;
  static constexpr GangClass c[n] = {{1, 2, 1}, {2, 3, 1}, {3, 3, 1}, {4, 4, 2}, {6, 5, 2}, {8, 6, 3}, {11, 6, 3}};
};
template <> struct GangTab<double> {
  static constexpr int n = 4;
  static constexpr GangClass c[n] = {{1, 2, 1}, {2, 3, 1}, {3, 4, 2}, {4, 4, 2}};
};

// The cut: gt x gi x gj blocks along t, i and j (g = 0: the system is not iterated by a gang).
struct GangCut {
  int gt, gi, gj, g;
  int nslot;  // exchange elements of the largest block
  int cls;    // class of the largest block
};

// Block k of `parts` along an extent: [start, start + len).
__host__ __device__ inline int gang_start(int extent, int parts, int k) {
  return (int)((long long)k * extent / parts);
}
// The block that holds coordinate x.
__host__ __device__ inline int gang_owner(int extent, int parts, int x) {
  return (int)(((long long)(x + 1) * parts - 1) / extent);
}

// One workgroup's block and its extended block: the cells and slices of the block plus one
// layer in every cut direction.  In an uncut spatial direction the block spans the lattice
// and neighbours wrap inside it; time always has a slot in front and behind (filled from
// the block itself when time is uncut).
struct GangBlock {
  int L1, L2, Nt;
  int gt, gi, gj;
  int t0, T, i0, a, j0, b;
  int oi, oj;  // 1 in a cut direction
  int ea, eb;  // extended cells along i and j
  int TS;      // slots per column of the extended block: T + 2
  int half;    // sites per sublattice: a b T
  float rT, ra, rb, rea, reb;  // reciprocals for gang_div
};

// n / d for 0 <= n < 10^6 from the reciprocal r of d: (n + 1/2) r lies at least 1/(2 d) from
// an integer and carries an error below 3e-7 n / d.
__host__ __device__ inline int gang_div(int n, float r) { return (int)(((float)n + 0.5f) * r); }

__host__ __device__ inline GangBlock gang_block(int L1, int L2, int Nt, int gt, int gi, int gj, int wg) {
  GangBlock B;
  B.L1 = L1, B.L2 = L2, B.Nt = Nt, B.gt = gt, B.gi = gi, B.gj = gj;
  // slices fastest: the largest faces of a block lie towards its neighbours in time, and
  // consecutive workgroups are placed on the same XCD
  const int bt = wg % gt, q = wg / gt, bj = q % gj, bi = q / gj;
  B.t0 = gang_start(Nt, gt, bt), B.T = gang_start(Nt, gt, bt + 1) - B.t0;
  B.i0 = gang_start(L1, gi, bi), B.a = gang_start(L1, gi, bi + 1) - B.i0;
  B.j0 = gang_start(L2, gj, bj), B.b = gang_start(L2, gj, bj + 1) - B.j0;
  B.oi = gi > 1, B.oj = gj > 1;
  B.ea = B.a + 2 * B.oi, B.eb = B.b + 2 * B.oj;
  B.TS = B.T + 2;
  B.half = B.a * B.b * B.T;
  B.rT = 1.0f / (float)B.T, B.ra = 1.0f / (float)B.a, B.rb = 1.0f / (float)B.b, B.rea = 1.0f / (float)B.ea, B.reb = 1.0f / (float)B.eb;
  return B;
}

__host__ __device__ inline int gang_wrap(int x, int n) { return x < 0 ? x + n : (x >= n ? x - n : x); }

// Table entry of cell (i, j) of the extended block (i in [-oi, a + oi), j likewise; a
// coordinate outside an uncut direction wraps), sublattice s, slot te (slice t0 + te - 1).
__host__ __device__ inline int gang_entry(const GangBlock& B, int i, int j, int s, int te) {
  const int ci = B.oi ? i + 1 : gang_wrap(i, B.a), cj = B.oj ? j + 1 : gang_wrap(j, B.b);
  return ((ci * B.eb + cj) * 2 + s) * B.TS + te;
}
__host__ __device__ inline int gang_entries(const GangBlock& B) { return B.ea * B.eb * 2 * B.TS; }

// Own site k < half of one sublattice: slices fastest, then j, then i.
struct GangSite {
  int i, j, t;
};
__host__ __device__ inline GangSite gang_site(const GangBlock& B, int k) {
  GangSite c;
  const int cell = gang_div(k, B.rT);
  c.t = k - cell * B.T;
  c.i = gang_div(cell, B.rb);
  c.j = cell - c.i * B.b;
  return c;
}

// Site q of the block in the order of memory: j fastest, then i, the sublattice, the slice.
struct GangPlace {
  int i, j, s, t;
};
__host__ __device__ inline GangPlace gang_place(const GangBlock& B, int q) {
  GangPlace c;
  const int q1 = gang_div(q, B.rb), q2 = gang_div(q1, B.ra);
  c.j = q - q1 * B.b;
  c.i = q1 - q2 * B.a;
  c.s = q2 & 1;
  c.t = q2 >> 1;
  return c;
}

// What a workgroup sends.  Sites of cells on a face of a cut spatial direction go to their
// place among the block's sites (A sites first, then B sites; a cell's slices adjacent).
// With time cut the first and the last slice go to planes behind them as well, cells
// adjacent: read from their columns, every element of a plane would cost a memory line.
__host__ __device__ inline bool gang_sent(const GangBlock& B, GangSite c) {
  return (B.oi && (c.i == 0 || c.i == B.a - 1)) || (B.oj && (c.j == 0 || c.j == B.b - 1));
}
__host__ __device__ inline int gang_plane(const GangBlock& B, int last, int s, int cell) {
  return 2 * B.half + (2 * last + s) * B.a * B.b + cell;
}
__host__ __device__ inline int gang_slots(const GangBlock& B) { return 2 * B.half + (B.gt > 1 ? 4 * B.a * B.b : 0); }

// The two bonds of a site beside the one inside its cell: A(i, j) has B(i - 1, j) and
// B(i, j - 1), B(i, j) has A(i + 1, j) and A(i, j + 1).  Entries of both at slot te.
__host__ __device__ inline void gang_bonds(const GangBlock& B, int i, int j, int s, int te, int& h1, int& h2) {
  const int d = s ? 1 : -1;
  h1 = gang_entry(B, i + d, j, 1 - s, te);
  h2 = gang_entry(B, i, j + d, 1 - s, te);
}

// Cells of the ring around the block that the 12-point footprint touches: all but the two
// corners (-1, -1) and (a, b).
__host__ __device__ inline int gang_ring(const GangBlock& B) {
  return B.oi * 2 * (B.b + B.oj) + B.oj * 2 * B.a;
}
__host__ __device__ inline void gang_ring_cell(const GangBlock& B, int q, int& i, int& j) {
  const int row = B.b + B.oj;
  if (B.oi && q < row) {
    i = -1, j = q;  // to the corner (-1, b)
  } else if (B.oi && q < 2 * row) {
    i = B.a, j = q - row - B.oj;  // from the corner (a, -1)
  } else {
    q -= B.oi * 2 * row;
    i = q >> 1, j = (q & 1) ? B.b : -1;
  }
}

// Halo element e of this workgroup: an entry of the extended block filled from another
// workgroup.  First the ring at the block's own slices (slices fastest), then, with time
// cut, the slots in front and behind of the ring and of the block itself.
struct GangHalo {
  int i, j, s, te;
};
__host__ __device__ inline int gang_halos(const GangBlock& B) {
  const int ring = gang_ring(B);
  return ring * 2 * B.T + (B.gt > 1 ? (ring + B.a * B.b) * 4 : 0);
}
__host__ __device__ inline GangHalo gang_halo(const GangBlock& B, int e) {
  GangHalo h;
  const int ring = gang_ring(B);
  if (e < ring * 2 * B.T) {
    const int q = e / (2 * B.T), r = e - q * 2 * B.T;
    gang_ring_cell(B, q, h.i, h.j);
    h.s = r / B.T;
    h.te = r - h.s * B.T + 1;
  } else {
    e -= ring * 2 * B.T;
    const int q = e >> 2;
    if (q < ring) {
      gang_ring_cell(B, q, h.i, h.j);
    } else {
      h.i = (q - ring) / B.b, h.j = (q - ring) - h.i * B.b;
    }
    h.s = (e >> 1) & 1;
    h.te = (e & 1) ? B.T + 1 : 0;
  }
  return h;
}
// Where a halo element comes from: the owning workgroup and the element's place there.
__host__ __device__ inline void gang_source(const GangBlock& B, GangHalo h, int& wg, int& k) {
  const int gi_ = gang_wrap(B.i0 + h.i, B.L1), gj_ = gang_wrap(B.j0 + h.j, B.L2),
            gt_ = gang_wrap(B.t0 + h.te - 1, B.Nt);
  const int bt = gang_owner(B.Nt, B.gt, gt_), bi = gang_owner(B.L1, B.gi, gi_), bj = gang_owner(B.L2, B.gj, gj_);
  wg = (bi * B.gj + bj) * B.gt + bt;
  GangBlock O = B;
  const int t0 = gang_start(B.Nt, B.gt, bt), i0 = gang_start(B.L1, B.gi, bi), j0 = gang_start(B.L2, B.gj, bj);
  O.T = gang_start(B.Nt, B.gt, bt + 1) - t0;
  O.a = gang_start(B.L1, B.gi, bi + 1) - i0;
  O.b = gang_start(B.L2, B.gj, bj + 1) - j0;
  O.half = O.a * O.b * O.T;
  const int cell = (gi_ - i0) * O.b + (gj_ - j0);
  if (h.te >= 1 && h.te <= B.T)
    k = h.s * O.half + cell * O.T + (gt_ - t0);
  else
    k = gang_plane(O, h.te == 0, h.s, cell);
}

// Extra sites of sublattice s at which u = M^dagger r is computed here although another
// workgroup owns them: B at (-1, j) and (i, -1) and A at (a, j) and (i, b) (the bonds of
// the block's own rows), and with time cut A one slice in front and B one behind.
__host__ __device__ inline int gang_extras(const GangBlock& B) {
  return (B.oi * B.b + B.oj * B.a) * B.T + (B.gt > 1 ? B.a * B.b : 0);
}
__host__ __device__ inline void gang_extra(const GangBlock& B, int s, int e, int& i, int& j, int& te) {
  const int ni = B.oi * B.b * B.T, nj = B.oj * B.a * B.T;
  if (e < ni) {
    i = s ? -1 : B.a, j = e / B.T, te = e - j * B.T + 1;
  } else if (e < ni + nj) {
    e -= ni;
    i = e / B.T, j = s ? -1 : B.b, te = e - i * B.T + 1;
  } else {
    e -= ni + nj;
    i = e / B.b, j = e - i * B.b, te = s ? B.T + 1 : 0;
  }
}

// The largest block of a cut (every count above grows with each extent).
inline GangBlock gang_largest(int L1, int L2, int Nt, int gt, int gi, int gj) {
  GangBlock B = gang_block(L1, L2, Nt, gt, gi, gj, 0);
  B.T = (Nt + gt - 1) / gt, B.a = (L1 + gi - 1) / gi, B.b = (L2 + gj - 1) / gj;
  B.ea = B.a + 2 * B.oi, B.eb = B.b + 2 * B.oj, B.TS = B.T + 2, B.half = B.a * B.b * B.T;
  return B;
}

// Entries of a table: the extended block, and a column and a half of zeros around an entry
// that stands for sites a thread does not have (every neighbour it reads is zero too).
__host__ __device__ inline int gang_zero(const GangBlock& B) { return gang_entries(B) + B.TS; }
__host__ __device__ inline int gang_table(const GangBlock& B) { return gang_entries(B) + 2 * B.TS + 1; }
// A system of one workgroup in which two field tables fit in front of the links (its body is
// one of the first three classes): the second lies kGangSecond bytes behind the first.
constexpr int kGangSecond = kGangLinks / 2;
template <typename R>
__host__ __device__ inline bool gang_solo(const GangCut& c, int L1, int L2, int Nt) {
  const size_t entries = (size_t)L1 * L2 * 2 * (Nt + 2) + 2 * (Nt + 2) + 1;
  return c.g == 1 && c.cls <= 2 && entries * 2 * sizeof(R) <= (size_t)kGangSecond;
}
// The first class that holds a block, or -1.
template <typename R>
inline int gang_class(const GangBlock& B) {
  if ((size_t)gang_table(B) * 2 * sizeof(R) > (size_t)kGangLinks) return -1;
  for (int k = 0; k < GangTab<R>::n; ++k) {
    const GangClass c = GangTab<R>::c[k];
    if (B.half <= c.M * kGangHalf && gang_halos(B) <= c.H * kGangThreads && gang_extras(B) <= c.X * kGangHalf)
      return k;
  }
  return -1;
}

// Words of a system's exchange memory: control words, two parities of reduction records (copies),
// two parities of sites; and of the state its workgroups keep between launches (r, p, s, z
// in the order of their registers).
template <typename R>
__host__ __device__ inline size_t gang_exch_words(int g, int nslot) {
  return (size_t)kGangCtlWords + 2 * (size_t)g * kGangCopies * kGangRecWords + 2 * (size_t)g * nslot * (sizeof(R) / 2);
}

template <typename R>
__host__ __device__ inline size_t gang_state_words(int g, int cls) {
  return 4 * (size_t)g * GangTab<R>::c[cls].M * kGangThreads * (sizeof(R) / 4);
}

// Time of one CG iteration of a cut in microseconds, fitted to measurements (complex64 /
// complex128; one workgroup 0.95 to 1.3 with one site per thread, 1.5 / 2.2 at 6x6x16;
// 12x12x32 3.25 / 4.7 with 8 workgroups and 2.95 / 3.6 with 16; 24x24x64 3.5 / 5.0 with 64;
// 48x48x64 4.8 with 128, 4.2 / 6.2 with 256; 102x102x64 8.9 with 256, when it was fitted): the
// arithmetic of the largest block, and with more than one workgroup a reduction and an
// exchange of faces.
template <typename R>
inline double gang_cost(const GangBlock& B, int cls, int g) {
  constexpr bool single = sizeof(R) == 4;
  const int M = GangTab<R>::c[cls].M;
  if (g == 1 && cls <= 2) return single ? 0.68 + 0.27 * M : 0.7 + 0.48 * M;
  if (g == 1) return 0.9 + (single ? (M > 6 ? 0.4 : 0.32) : 0.55) * M;
  double l = 0.0;
  for (int k = 2; k <= g; k *= 2) l += 1.0;
  if (single) return 1.75 + 0.14 * l + 0.42 * (M - 1) + (M > 6 ? 0.25 * (M - 6) : 0.0) + 0.3e-3 * gang_halos(B);
  return 2.1 + 0.17 * l + 0.6 * (M - 1) + (M > 3 ? 0.6 : 0.0) + 0.5e-3 * gang_halos(B);
}

// The cut of a lattice; g = 0: none fits.  It depends on the lattice alone, so that a
// system's results do not depend on what it shares a launch with: the shortest iteration
// among the cuts whose workgroups times their time, per site, stay below what a launch full
// of such systems may take: the tiled iteration at a full device (88 and 184 bytes per site
// at 5 TB/s over 256 CUs), less a fifth.  Up to 10,200 complex64 sites a smaller bound keeps
// gangs of four, of which 64, the largest batch, are one launch: 9x6x58 takes 3.68 us an
// iteration alone, 0.245 per system for 16 and 0.065 for 64 with it, and 2.50, 0.172 and 0.088
// with eight workgroups, as the larger bound has it (9x9x40: 3.47, 0.232, 0.062; 2.62, 0.180,
// 0.092).
template <typename R>
inline GangCut gang_cut(int L1, int L2, int Nt) {
  const double n = 2.0 * L1 * L2 * Nt;
  const double room = n * (sizeof(R) == 8 ? 7.5e-3 : n > 10200 ? 3.6e-3 : 3.1e-3);
  GangCut best{0, 0, 0, 0, 0, 0};
  double cost = 0.0;
  for (int gt = 1; gt <= 16 && gt <= Nt; gt *= 2)
    for (int gi = 1; gi <= 16 && gi <= L1; ++gi)
      for (int gj = 1; gj <= 16 && gj <= L2; ++gj) {
        const int g = gt * gi * gj;
        if (g > kGangMaxWgs) break;
        const GangBlock B = gang_largest(L1, L2, Nt, gt, gi, gj);
        const int cls = gang_class<R>(B);
        if (cls < 0) continue;
        // a fifth more where the gangs of a full launch leave CUs over (sixteen systems of
        // 18 workgroups take two launches, of 16 workgroups one: FP64 12x23x15 alone 3.70 us
        // with it and 3.20 without, sixteen 0.303 and 0.469 each); a cut beyond its room counts
        // by how far it is beyond
        const double t = gang_cost<R>(B, cls, g) * (kGangMaxWgs % g == 0 ? 1.0 : 1.2);
        const double c = g == 1 || t * g <= room ? t : 1000.0 * t * g;
        if (best.g == 0 || c < cost) {
          best = GangCut{gt, gi, gj, g, gang_slots(B), cls};
          cost = c;
        }
      }
  return best;
}

}  // namespace hub
