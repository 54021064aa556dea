// The gang CG (gfx950): conjugate gradients on (M M^dagger + mu^2) z = r whose whole state
// stays on the chip.  A system is cut into blocks (hub_gang.h), one workgroup each; every
// workgroup keeps r, p, s = A p and z of its block in registers and the one vector its
// stencil reads at neighbouring sites in LDS, and a launch runs a whole block of
// iterations.
//
// What bounds it: the tiled iteration (k_cg1, k_cg2) moves every vector through the caches
// twice and ends in two kernel boundaries, each of which empties and refills the device;
// here the vectors do not move, and an iteration costs the arithmetic of the largest block
// plus two exchanges between workgroups.  Those exchanges carry the faces of the blocks
// and one reduction record per workgroup, as words of 32 data bits and a 32-bit tag that
// one 8-byte store makes visible at once: the receiver polls the words themselves, so no
// fence, no cache write-back and no separate flag stands in an exchange.
//
// The recurrence has one reduction per iteration (Chronopoulos and Gear's form of CG): with
// u = M^dagger r,  gamma = |r|^2,  delta = <r, A r> = |u|^2 + mu^2 gamma,  w = M u + mu^2 r,
//   beta = gamma / gamma_prev,  alpha = gamma / (delta - beta gamma / alpha_prev),
//   p = r + beta p,  s = w + beta s,  z += alpha p,  r -= alpha s.
// gamma and delta are known after the first half of the operator, so the reduction travels
// while the second half is computed and its faces are sent; the receivers keep r and s of
// their halo, so what they wait for is the faces of w, which travel with the reduction.
//
// Microseconds per iteration, before (tiled, or one workgroup per small complex64 system) and
// here: 12x12x32 7.1 complex64, 13.6 FP64 (16 systems) -> 2.9 and 3.6 for one, 3.1 and 4.75
// for the sixteen; 24x24x64 complex64 11 -> 3.35; 48x48x64 13 and 15 -> 4.0 and 6.4; 102x102x64
// complex64 26 -> 8.5.  By its counters the waves wait for 45% (102x102x64) to 66% (sixteen
// systems in FP64) of the time, for the words of other workgroups and at four barriers, and
// the vector ALU issues in 50% to 23% of its cycles.
//
// A gang needs all its workgroups on the device at once.  They meet at the start of a
// launch before they change anything; a gang that does not fit beside others is refused
// there and launched again, a meeting that does not happen in time (other work holds the
// CUs) is called off by one atomic decision.  Should that go on, the host carries on with
// k_gang_step: the same iteration cut into launches where the workgroups would wait for each
// other, so that none of them has to be there with another one.  It gives the same bits.
// Every wait after a meeting is bounded too.
#include <hip/hip_ext.h>

#include <type_traits>

#include "hub_device.h"
#include "hub_gang.h"

namespace hub {
namespace {

typedef unsigned long long u64;

constexpr int kGangWaves = kGangThreads / 64;
enum GangPart : int { kGangShare, kGangSums, kGangUpdate };  // of an iteration in k_gang_step
constexpr long long kGangMeetTicks = 200 * 1000;  // 2 ms of the 100 MHz wall clock
constexpr int kGangSpins = 1 << 20;               // polls of one wait (seconds)

// Exchange memory is read and written at the scope of the device (sc1, as the compiler's
// own agent-scope atomics: coherent between the XCDs' L2s), 16 bytes at a time: two tagged
// words, each whole by itself.
typedef unsigned gang_q __attribute__((ext_vector_type(4)));
constexpr int kGangAux = 16;  // sc1
struct Mem {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Mem(void* p, size_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000)) {}
  __device__ __forceinline__ gang_q load(unsigned off, unsigned base) const {
    asm volatile("" ::: "memory");  // a poll reads memory every time
    return __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)base, kGangAux);
  }
  __device__ __forceinline__ void store(unsigned off, unsigned base, gang_q v) const {
    // The base goes into the vector offset: behind a 16-byte store with its base in a scalar
    // register the compiler rewrites the data registers at once (it leaves the wait states
    // of a store without one), and words changed on their way out.
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)(off + base), 0, kGangAux);
    asm volatile("" ::: "memory");
  }
};

// State memory: complex values by byte offset (a 64-bit address per value would take the
// registers that it relieves).
typedef unsigned gang_d __attribute__((ext_vector_type(2)));
struct State {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ State(void* p, size_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000)) {}
  __device__ __forceinline__ void get(unsigned off, float2& v) const {
    const gang_d q = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    v.x = __uint_as_float(q.x);
    v.y = __uint_as_float(q.y);
  }
  __device__ __forceinline__ void get(unsigned off, double2& v) const {
    const gang_q q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    v.x = __longlong_as_double((long long)((u64)q.y << 32 | q.x));
    v.y = __longlong_as_double((long long)((u64)q.w << 32 | q.z));
  }
  __device__ __forceinline__ void set(unsigned off, float2 v) const {
    const gang_d q = {__float_as_uint(v.x), __float_as_uint(v.y)};
    __builtin_amdgcn_raw_buffer_store_b64(q, r, (int)off, 0, 0);
  }
  __device__ __forceinline__ void set(unsigned off, double2 v) const {
    const u64 x = (u64)__double_as_longlong(v.x), y = (u64)__double_as_longlong(v.y);
    const gang_q q = {(unsigned)x, (unsigned)(x >> 32), (unsigned)y, (unsigned)(y >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)off, 0, 0);
  }
};

// A complex value as words of 32 data bits and a tag: 2 for complex64, 4 for complex128.
template <typename C> struct Tagged;
template <> struct Tagged<float2> {
  static constexpr int BYTES = 16;
  gang_q q;
  __device__ __forceinline__ void load(const Mem& m, unsigned off, unsigned base) { q = m.load(off, base); }
  __device__ __forceinline__ bool has(unsigned tag) const { return q.y == tag && q.w == tag; }
  __device__ __forceinline__ float2 value() const {
    float2 v;
    v.x = __uint_as_float(q.x);
    v.y = __uint_as_float(q.z);
    return v;
  }
  static __device__ __forceinline__ void store(const Mem& m, unsigned off, unsigned base, float2 v, unsigned tag) {
    gang_q q = {__float_as_uint(v.x), tag, __float_as_uint(v.y), tag};
    m.store(off, base, q);
  }
};
template <> struct Tagged<double2> {
  static constexpr int BYTES = 32;
  gang_q a, b;
  __device__ __forceinline__ void load(const Mem& m, unsigned off, unsigned base) {
    a = m.load(off, base);
    b = m.load(off + 16, base);
  }
  __device__ __forceinline__ bool has(unsigned tag) const {
    return a.y == tag && a.w == tag && b.y == tag && b.w == tag;
  }
  __device__ __forceinline__ double2 value() const {
    double2 v;
    v.x = __longlong_as_double((long long)((u64)a.z << 32 | a.x));
    v.y = __longlong_as_double((long long)((u64)b.z << 32 | b.x));
    return v;
  }
  static __device__ __forceinline__ void store(const Mem& m, unsigned off, unsigned base, double2 v, unsigned tag) {
    const u64 x = (u64)__double_as_longlong(v.x), y = (u64)__double_as_longlong(v.y);
    gang_q a = {(unsigned)x, tag, (unsigned)(x >> 32), tag}, b = {(unsigned)y, tag, (unsigned)(y >> 32), tag};
    m.store(off, base, a);
    m.store(off + 16, base, b);
  }
};

// Workgroups of the gangs of this process that are on the device or on their way to it.  A
// gang that would not fit beside the others is refused before it holds CUs that they wait
// for, so that two streams cannot each hold half of what both need.
__device__ unsigned g_gang_wgs;

typedef HUB_GAS unsigned gang_word;
__device__ __forceinline__ unsigned word_load(const gang_word* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool word_swap(gang_word* p, unsigned& cur, unsigned v) {
  return __hip_atomic_compare_exchange_strong(p, &cur, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gang_release(int g) {
  __hip_atomic_fetch_sub((gang_word*)&g_gang_wgs, (unsigned)g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The workgroups of a system meet.  Control words: [0] arrivals over all launches; [16] the
// decision on launch seq, 2 seq + 1 to go and 2 seq to leave; [32] seq once the gang has
// its place among g_gang_wgs (given back by whoever takes the word back to 0); [48] seq if it
// was refused one.  The first to arrive asks for the place, the last decides to go, and
// anybody who has waited too long decides to leave.
__device__ int gang_meet(unsigned* ctl, int g, unsigned seq, unsigned arrived, int deny) {
  gang_word *dec = (gang_word*)(ctl + 16), *place = (gang_word*)(ctl + 32), *refused = (gang_word*)(ctl + 48);
  auto decide = [&](unsigned what) {
    unsigned cur = word_load(dec);
    while (cur < 2 * seq) {
      if (word_swap(dec, cur, what)) return true;
    }
    return false;
  };
  auto give_back = [&] {
    unsigned cur = seq;
    if (word_swap(place, cur, 0)) gang_release(g);
  };
  const long long t0 = wall_clock64();
  if (arrived == (seq - 1) * (unsigned)g + 1) {
    gang_word* all = (gang_word*)&g_gang_wgs;
    unsigned cur = word_load(all);
    bool room;
    do room = !deny && cur + (unsigned)g <= kGangMaxWgs;
    while (room && !word_swap(all, cur, cur + (unsigned)g));
    if (room) {
      unsigned old = word_load(place);
      while (!word_swap(place, old, seq)) {
      }
      if (word_load(dec) == 2 * seq) give_back();
    } else {
      __hip_atomic_store(refused, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_s_waitcnt(0);
      (void)decide(2 * seq);
    }
  }
  for (;;) {
    const unsigned v = word_load(dec);
    if (v >= 2 * seq) return (v & 1) ? 0 : word_load(refused) == seq ? 3 : 1;
    if (arrived == seq * (unsigned)g && word_load(place) == seq) (void)decide(2 * seq + 1);
    if (wall_clock64() - t0 > kGangMeetTicks && decide(2 * seq)) give_back();
    __builtin_amdgcn_s_sleep(2);
  }
}

// The temporal link of a site: s (e^{i phi} - m) on A, s (e^{-i phi} - m) on B, s = -1 on
// the hop across the antiperiodic boundary.
__device__ __forceinline__ float2 gang_link(const SysDesc* d, float, int n, bool isB, bool wrap) {
  float c, s;
  cis32(Real<float>(d->ph32)[n], c, s);
  const float sg = wrap ? -1.0f : 1.0f;
  float2 e;
  e.x = sg * (c - (float)d->g.ms);
  e.y = isB ? -sg * s : sg * s;
  return e;
}
__device__ __forceinline__ double2 gang_link(const SysDesc* d, double, int n, bool isB, bool wrap) {
  const double2 cs = Vec<double2>(d->ph64)[n];
  const double sg = wrap ? -1.0 : 1.0;
  double2 e;
  e.x = sg * (cs.x - d->g.ms);
  e.y = isB ? -sg * cs.y : sg * cs.y;
  return e;
}

// The sites [0, half) of one sublattice by chunks: chunk c covers the sites c .. c + CH - 1 of
// every thread.  Within a chunk nothing branches (a site that a thread does not have is the
// zero entry), so the loads of several sites are in flight together.
template <int M, int CH, typename F>
__device__ __forceinline__ void gang_chunks(int half, F f) {
#pragma unroll
  for (int c = 0; c < M; c += CH)
    if (c == 0 || half > c * kGangHalf) {
#pragma unroll
      for (int m = c; m < c + CH; ++m)
        if (m < M) f(m);
    }
}

__device__ __forceinline__ double from_lane(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
  return __longlong_as_double((long long)((u64)hi << 32 | lo));
}

// SOLO: a system of one workgroup whose two field tables fit: nothing is exchanged, and r and
// M^dagger r do not share a place, so that an iteration has two barriers instead of four and
// no wave waits for another one's sum (2x1x64 FP64 1.37 -> 0.99 us, 6x6x16 1.75 -> 1.48 us;
// bound by the latency of the two barriers, the LDS and the scalars' divisions).  With more
// workgroups a second table is slower: a record is then stored behind the faces.
// STEP: one part of one iteration (K is a GangPart), everything that another workgroup has to
// have done in an earlier launch: r's faces sent; then u and this workgroup's record; then,
// from the records, the rest of the iteration and the faces of the new r.  The state passes
// through memory, and r of the halo is received anew where the whole loop carries it along
// with its owner's arithmetic: the operations on every value are the same ones.
template <typename R, int CLS, bool SOLO, bool STEP>
__device__ __forceinline__ void gang_run(const SysDesc* __restrict__ d, Scal* sc, const int wg, const int zslot,
                                         const unsigned tag0, const unsigned seq, const unsigned arrived, const int deny,
                                         const int K, char* const lds) {
  using C = typename V2<R>::T;
  using TW = Tagged<C>;
  constexpr int M = GangTab<R>::c[CLS].M, H = GangTab<R>::c[CLS].H, X = GangTab<R>::c[CLS].X;
  constexpr bool single = sizeof(R) == 4;
  constexpr int CH = !single && M > 3 ? 2 : M > 6 ? 4 : M % 3 == 0 ? 3 : M;
  // The largest bodies have no registers left for the solution: it stays in the state
  // memory (the XCD's L2) and is read ahead of its update while the records travel.
  constexpr bool ZMEM = CLS == GangTab<R>::n - 1;
  // Two bonds of a site share a register where a register per bond would not fit.
  constexpr bool PACK = single ? M > 8 : M > 3;
  // The small bodies have registers for every address (12x12x32: an iteration takes 7% longer
  // when they work them out anew); the others do not (FP64 at 48x48x64: 30% longer with them).
  constexpr bool KEEP = M <= (single ? 3 : 2);
  constexpr int sR = single ? (int)S_R32 : (int)S_R;
  double2* const red = reinterpret_cast<double2*>(lds);        // (gamma, |u|^2) of each wave
  double2* const red2 = red + kGangWaves;                      // of each wave's share of the records
  int* const flag = reinterpret_cast<int*>(red2 + kGangMaxWgs / 64);
  int &sh_off = flag[0], &sh_bad = flag[1];
  static_assert((kGangWaves + kGangMaxWgs / 64) * 16 + 8 <= kGangHead, "head of the LDS");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = SOLO ? 1 : d->gang.g, nslot = SOLO ? 0 : d->gang.nslot;
  if (tid == 0) sh_bad = 0;
  const GangBlock B = gang_block(d->g.L1, d->g.L2, d->g.Nt, d->gang.gt, d->gang.gi, d->gang.gj, wg);
  // a part reads the count that no workgroup of its launch writes
  const int it0 = !STEP || K == kGangShare ? sc->git : K == kGangSums ? sc->sit : sc->git - 1;
  C* const F = reinterpret_cast<C*>(lds + kGangHead);               // the field: r, then M^dagger r in its place
  C* const E = reinterpret_cast<C*>(lds + kGangHead + kGangLinks);  // the temporal links
  const Mem mem(d->gang_mem, g > 1 ? gang_exch_words<R>(g, nslot) * 8 : 0);
  const unsigned rec_base = kGangCtlWords * 8, rec_copy = (unsigned)g * (kGangRecWords * 8),
                 rec_half = kGangCopies * rec_copy;
  const unsigned ex_base = rec_base + 2 * rec_half, ex_half = (unsigned)g * nslot * TW::BYTES;

  // This thread's sites: k = k0 + m kGangHalf of sublattice sub (the same in a whole wave).
  // Places in the tables are kept as byte offsets.  Each list is worked out by a rolled loop into LDS and read
  // back by the thread that wrote it: unrolled into registers, the index arithmetic of all
  // sites would be a hundred kilobytes of code.
  const int sub = __builtin_amdgcn_readfirstlane(tid / kGangHalf);
  const int k0 = tid & (kGangHalf - 1);
  constexpr int SZ = (int)sizeof(C);
  const int dh = (sub ? -B.TS : B.TS) * SZ;  // to the bond inside the cell
  const int wrap = B.T * SZ;                 // from a slice to its copy past the end
  auto place = [](int entry) { return kGangHead + entry * SZ; };
  const int zero = place(gang_zero(B));
  int4* const list = reinterpret_cast<int4*>(F);
  int a0[M], h1[M], h2[M];  // packed: both bonds in h1, in units of 8 bytes
  unsigned ends = 0, sent = 0;  // ends: bit m: the first slice, bit M + m: the last
#pragma unroll 1
  for (int k = k0; k < B.half; k += kGangHalf) {
    const GangSite c = gang_site(B, k);
    int4 v;
    v.x = place(gang_entry(B, c.i, c.j, sub, c.t + 1));
    gang_bonds(B, c.i, c.j, sub, c.t + 1, v.y, v.z);
    v.y = place(v.y);
    v.z = place(v.z);
    v.w = (gang_sent(B, c) ? 1 : 0) | (c.t == 0 ? 2 : 0) | (c.t == B.T - 1 ? 4 : 0);
    list[sub * B.half + k] = v;
  }
#pragma unroll
  for (int m = 0; m < M; ++m) {
    a0[m] = h1[m] = h2[m] = zero;
    if (k0 + m * kGangHalf < B.half) {
      const int4 v = list[sub * B.half + k0 + m * kGangHalf];
      a0[m] = v.x;
      h1[m] = v.y;
      h2[m] = v.z;
      sent |= (unsigned)(v.w & 1) << m;
      ends |= (unsigned)(v.w >> 1 & 1) << m | (unsigned)(v.w >> 2 & 1) << (M + m);
    }
    if (PACK) h1[m] = h1[m] >> 3 | h2[m] >> 3 << 16;
  }
  __syncthreads();
  // Halo elements this thread receives: byte offset at the sender; place here and, in the
  // upper bits, which copies it has.
  unsigned hsrc[H], hdst[H];
  unsigned hvalid = 0;
  constexpr unsigned kPlace = (1u << 18) - 1;
  static_assert(kGangLdsBytes <= (1 << 18), "a place fits");
  const int nh = g > 1 ? gang_halos(B) : 0;
#pragma unroll 1
  for (int e = tid; e < nh; e += kGangThreads) {
    const GangHalo el = gang_halo(B, e);
    int src, k;
    gang_source(B, el, src, k);
    int2 v;
    v.x = (int)(((unsigned)src * nslot + k) * TW::BYTES);
    v.y = place(gang_entry(B, el.i, el.j, el.s, el.te)) | (B.gt == 1 && el.te == 1 ? 1 << 18 : 0) |
          (B.gt == 1 && el.te == B.T ? 1 << 19 : 0);
    reinterpret_cast<int2*>(F)[e] = v;
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int e = tid + h * kGangThreads;
    hsrc[h] = hdst[h] = 0;
    if (e < nh) {
      const int2 v = reinterpret_cast<const int2*>(F)[e];
      hsrc[h] = (unsigned)v.x;
      hdst[h] = (unsigned)v.y;
      hvalid |= 1u << h;
    }
  }
  __syncthreads();
  // Extra sites it computes.
  int xa[X], x1[X], x2[X];
  const int nx = g > 1 ? gang_extras(B) : 0;
#pragma unroll 1
  for (int e = k0; e < nx; e += kGangHalf) {
    int i, j, te;
    gang_extra(B, sub, e, i, j, te);
    int4 v;
    v.x = place(gang_entry(B, i, j, sub, te));
    gang_bonds(B, i, j, sub, te, v.y, v.z);
    v.y = place(v.y);
    v.z = place(v.z);
    v.w = 0;
    list[sub * nx + e] = v;
  }
#pragma unroll
  for (int x = 0; x < X; ++x) {
    xa[x] = x1[x] = x2[x] = zero;
    if (k0 + x * kGangHalf < nx) {
      const int4 v = list[sub * nx + k0 + x * kGangHalf];
      xa[x] = v.x;
      x1[x] = v.y;
      x2[x] = v.z;
    }
    if (PACK) x1[x] = x1[x] >> 3 | x2[x] >> 3 << 16;
  }
  __syncthreads();
  auto at = [&](int off) -> C& { return *reinterpret_cast<C*>(lds + off); };
  auto link = [&](int off) -> C& { return *reinterpret_cast<C*>(lds + off + kGangLinks); };

  // links of the extended block (j fastest: consecutive lanes read consecutive sites)
#pragma unroll 4
  for (int q = tid; q < gang_entries(B); q += kGangThreads) {
    const int q1 = gang_div(q, B.reb), cj = q - q1 * B.eb, q2 = gang_div(q1, B.rea), ci = q1 - q2 * B.ea, s = q2 & 1,
              te = q2 >> 1;
    const int gt = gang_wrap(B.t0 + te - 1, B.Nt), gi = gang_wrap(B.i0 + ci - B.oi, B.L1),
              gj = gang_wrap(B.j0 + cj - B.oj, B.L2);
    const int n = ((gt * 2 + s) * B.L1 + gi) * B.L2 + gj;
    E[((ci * B.eb + cj) * 2 + s) * B.TS + te] = gang_link(d, R(0), n, s != 0, s ? gt == B.Nt - 1 : gt == 0);
  }
  for (int q = gang_entries(B) + tid; q < gang_table(B); q += kGangThreads) E[q] = F[q] = cz<C>();

  // Vectors between registers and the state memory (each thread its own places), and
  // between registers and their slots through the field table (j fastest in memory).
  const State state(d->gang_state, gang_state_words<R>(g, CLS) * 8);
  const unsigned svec = (unsigned)(g * M * kGangThreads) * SZ, sown = (unsigned)(wg * M * kGangThreads + tid) * SZ;
  auto load = [&](C* v, int which, int o) {
#pragma unroll
    for (int m = 0; m < M; ++m) state.get(which * svec + sown + (unsigned)o + m * kGangThreads * SZ, v[m]);
  };
  auto save = [&](const C* v, int which) {
#pragma unroll
    for (int m = 0; m < M; ++m) state.set(which * svec + sown + m * kGangThreads * SZ, v[m]);
  };
  auto take = [&](C* v, const void* src) {
    const Vec<C> from(src);
#pragma unroll 4
    for (int q = tid; q < 2 * B.half; q += kGangThreads) {
      const GangPlace c = gang_place(B, q);
      F[gang_entry(B, c.i, c.j, c.s, c.t + 1)] = from[(((B.t0 + c.t) * 2 + c.s) * B.L1 + B.i0 + c.i) * B.L2 + B.j0 + c.j];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = at(a0[m]);
    __syncthreads();
  };
  auto give = [&](const C* v, void* dst) {
    gang_chunks<M, CH>(B.half, [&](int m) { at(a0[m]) = v[m]; });
    __syncthreads();
    const Vec<C> to(dst);
#pragma unroll 4
    for (int q = tid; q < 2 * B.half; q += kGangThreads) {
      const GangPlace c = gang_place(B, q);
      to.set((((B.t0 + c.t) * 2 + c.s) * B.L1 + B.i0 + c.i) * B.L2 + B.j0 + c.j, F[gang_entry(B, c.i, c.j, c.s, c.t + 1)]);
    }
    __syncthreads();
  };
  C r[M], p[M], s[M], z[M];
  if (it0 > 0) {
    load(r, 0, 0);
    load(p, 1, 0);
    load(s, 2, 0);
    if (!ZMEM) load(z, 3, 0);
    __syncthreads();
  } else {
    take(r, d->vec[sR]);
    if (!single) take(z, d->vec[zslot]);  // the inner solve starts from zero
#pragma unroll
    for (int m = 0; m < M; ++m) {
      p[m] = s[m] = cz<C>();
      if (single) z[m] = cz<C>();
    }
    if (ZMEM) save(z, 3);
  }
  double gamma_prev = it0 > 0 ? sc->rrv[(it0 - 1) & 1] : 1.0;
  double alpha_prev = it0 > 0 ? sc->alpha[(it0 - 1) & 1] : 1.0;
  const double mu2 = d->mu2, stop2 = sc->stop2;
  const int maxit = sc->maxit;
  const R rmu2 = (R)mu2;
  const R ks = sub ? -(R)d->g.kappa : (R)d->g.kappa;
  const int dt1 = sub ? -SZ : SZ;  // M^dagger reads t + 1 on A, t - 1 on B; M the other way
  if (SOLO)
    for (int q = gang_entries(B) + tid; q < gang_table(B); q += kGangThreads) F[kGangSecond / SZ + q] = cz<C>();
  if (!STEP && g > 1) {
    if (tid == 0) sh_off = gang_meet((unsigned*)d->gang_mem, g, seq, arrived, deny);
    __syncthreads();
    if (sh_off) {
      if (wg == 0 && tid == 0) sc->gang = sh_off;
      return;
    }
  }

  // Own faces out; a halo element in.
  const unsigned mine = ((unsigned)wg * nslot + sub * B.half + k0) * TW::BYTES;
  const unsigned plane = ((unsigned)wg * nslot + gang_plane(B, 0, sub, 0)) * TW::BYTES;
  auto publish = [&](const C* v, unsigned tag, int o) {
    const unsigned ex = ex_base + (tag & 1) * ex_half, se = sent + (unsigned)o, en = ends + (unsigned)o;
    auto column = [&](int m) {
      if (se >> m & 1) TW::store(mem, mine + (unsigned)((M > 6 ? o : 0) + m * kGangHalf * TW::BYTES), ex, v[m], tag);
    };
    auto planes = [&](int m) {
      const unsigned first = en >> m & 1, last = en >> (M + m) & 1;
      if (first | last) {
        const unsigned cell = plane + (unsigned)(gang_div(k0 + o + m * kGangHalf, B.rT) * TW::BYTES);
        const unsigned up = (unsigned)(2 * B.a * B.b * TW::BYTES);
        if (first) TW::store(mem, cell, ex, v[m], tag);
        if (last) TW::store(mem, cell + up, ex, v[m], tag);
      }
    };
    if (M > 6) {  // one pass over the sites: two keep more in registers
      gang_chunks<M, CH>(B.half, [&](int m) {
        column(m);
        if (B.gt > 1) planes(m);
      });
    } else {
      if (B.oi || B.oj) gang_chunks<M, CH>(B.half, column);
      if (B.gt > 1 && en != 0) gang_chunks<M, CH>(B.half, planes);
    }
  };
  auto receive = [&](unsigned tag, auto use) {
    const unsigned ex = ex_base + (tag & 1) * ex_half;
    unsigned pend = hvalid;
    int spin = 0;
    while (pend) {
      TW w[H];
#pragma unroll
      for (int h = 0; h < H; ++h)
        if (pend >> h & 1) w[h].load(mem, hsrc[h], ex);
#pragma unroll
      for (int h = 0; h < H; ++h)
        if ((pend >> h & 1) && w[h].has(tag)) {
          use(h, w[h].value());
          pend &= ~(1u << h);
        }
      if (pend && ++spin > kGangSpins) {
        sh_bad = 1;
        break;
      }
    }
  };
  // Lanes below kGangCopies of a wave store the copies of this workgroup's record.  By
  // itself a reduction through one copy that all poll takes 0.3 us (16 workgroups) to 0.65 us
  // (256) longer; in the iteration it is what 256 workgroups wait for (48x48x64: 4.35 us with
  // one copy, 4.15 us with eight), fewer of them wait for the faces.
  auto post = [&](double a, double b, unsigned tag) {
    if (lane < kGangCopies)
      Tagged<double2>::store(mem, (unsigned)lane * rec_copy + (unsigned)wg * (kGangRecWords * 8),
                             rec_base + (tag & 1) * rec_half, double2{a, b}, tag);
  };
  // The records of all workgroups, 64 to a wave, in a fixed order, into red2.
  const int nw = g > 1 ? (g + 63) / 64 : 1;
  auto collect = [&](unsigned tag) {
    const unsigned rec = rec_base + (tag & 1) * rec_half + (unsigned)(wg % kGangCopies) * rec_copy;
    const int c = wave * 64 + lane;
    double2 q = cz<double2>();
    if (c < g) {
      Tagged<double2> w;
      int spin = 0;
      for (;;) {
        w.load(mem, (unsigned)c * (kGangRecWords * 8), rec);
        if (w.has(tag)) break;
        if (++spin > kGangSpins) {
          sh_bad = 1;
          break;
        }
      }
      q = w.value();
    }
    q.x = dpp_wave(q.x);
    q.y = dpp_wave(q.y);
    if (lane == 63) red2[wave] = q;
  };
  // o is zero in these (see the iteration loop)
  auto put = [&](unsigned dst, C v, int o) {
    dst += (unsigned)o;
    const int a = (int)(dst & kPlace);
    at(a) = v;
    if (B.gt == 1) {
      if (dst >> 18 & 1) at(a + wrap) = v;
      if (dst >> 19 & 1) at(a - wrap) = v;
    }
  };
  auto put_own = [&](const C* v, int o, int behind = 0) {
    gang_chunks<M, CH>(B.half, [&](int m) { at(a0[m] + behind) = v[m]; });
    if (SOLO || B.gt == 1) {
      const unsigned en = ends + (unsigned)o;
      const int up = o + wrap + behind, down = o - wrap + behind;
      gang_chunks<M, CH>(B.half, [&](int m) {
        if (en >> m & 1) at(a0[m] + up) = v[m];
        if (en >> (M + m) & 1) at(a0[m] + down) = v[m];
      });
    }
  };
  // Half an operator application at one site: own - e x(t + dt) + k sum of bonds, with e
  // conjugated for M^dagger (eg = -1).
  auto half_op = [&](C e, auto adj, C xt, C x0, C y1, C y2, R k, C own) {
    constexpr bool ADJ = decltype(adj)::value;
    C v;
    v.x = fma(k, x0.x + y1.x + y2.x, fma(ADJ ? -e.y : e.y, xt.y, fma(-e.x, xt.x, own.x)));
    v.y = fma(k, x0.y + y1.y + y2.y, fma(ADJ ? e.y : -e.y, xt.x, fma(-e.x, xt.y, own.y)));
    return v;
  };
  // The two outer bonds of a site (o is zero, see the iteration loop).
  auto low = [&](int b1) -> C { return at(b1 << 3 & 0x7fff8); };
  auto high = [&](int b1) -> C { return at((int)((unsigned)b1 >> 13 & 0x7fff8)); };
  static_assert(!(SOLO && (PACK || ZMEM)), "small bodies");
  auto bond1 = [&](int b1, int o, int behind = 0) -> C { return PACK ? low(b1 + o) : at(b1 + behind); };
  auto bond2 = [&](int b1, int b2, int o, int behind = 0) -> C { return PACK ? high(b1 + o) : at(b2 + behind); };

  // The parts of an iteration.  A zero in every offset, which the compiler cannot see through:
  // it would work out the address of every neighbour of every site once for all iterations
  // (or, with one zero for all passes, once for both passes) and run out of registers.
  auto unseen = [] {
    int o = 0;
    if (!KEEP) asm volatile("" : "+v"(o));
    return o;
  };
  // v = M^dagger r (times -1 on A) here and at the extra sites; gamma, |u|^2 of each wave
  auto first_half = [&](C* v, C* xv) {
    const int o = unseen(), o_h = o + dh, o_t = o + dt1;
    R acc_g = 0, acc_u = 0;
    gang_chunks<M, CH>(B.half, [&](int m) {
      v[m] = half_op(link(a0[m] + o_t), std::true_type{}, at(a0[m] + o_t), at(a0[m] + o_h), bond1(h1[m], o),
                     bond2(h1[m], h2[m], o), ks, r[m]);
      acc_g = fma(r[m].x, r[m].x, fma(r[m].y, r[m].y, acc_g));
      acc_u = fma(v[m].x, v[m].x, fma(v[m].y, v[m].y, acc_u));
    });
    gang_chunks<X, X>(nx, [&](int x) {
      xv[x] = half_op(link(xa[x] + o_t), std::true_type{}, at(xa[x] + o_t), at(xa[x] + o_h), bond1(x1[x], o),
                      bond2(x1[x], x2[x], o), ks, at(xa[x]));
    });
    acc_g = dpp_wave(acc_g);
    acc_u = dpp_wave(acc_u);
    if (lane == 63) red[wave] = double2{(double)acc_g, (double)acc_u};
    __syncthreads();
    return o;
  };
  // the sums of the waves: this workgroup's record
  auto record = [&](unsigned tag) {
    if (wave == 0) {
      const double2 q = lane < kGangWaves ? red[lane] : cz<double2>();
      const double sg = dpp_row(q.x), su = dpp_row(q.y);
      if (g > 1)
        post(from_lane(sg, 15), from_lane(su, 15), tag);
      else if (lane == 15)
        red2[0] = double2{sg, su};
    }
  };
  // w = M u + mu^2 r, in v
  auto second_half = [&](C* v, C* xv, int o) {
    put_own(v, o);
    if (g > 1) gang_chunks<X, X>(nx, [&](int x) { at(xa[x]) = xv[x]; });
    __syncthreads();
    o = unseen();
    const int o_h = o + dh, o_t = o - dt1;
    gang_chunks<M, CH>(B.half, [&](int m) {
      v[m] = half_op(link(a0[m]), std::false_type{}, at(a0[m] + o_t), at(a0[m] + o_h), bond1(h1[m], o),
                     bond2(h1[m], h2[m], o), -ks, v[m]);
      v[m].x = fma(rmu2, r[m].x, v[m].x);
      v[m].y = fma(rmu2, r[m].y, v[m].y);
    });
    return o;
  };
  // gamma and |u|^2 from the waves' shares of the records
  auto totals = [&](double& gamma, double& uu) {
    gamma = red2[0].x;
    uu = red2[0].y;
    for (int k = 1; k < nw; ++k) {
      gamma += red2[k].x;
      uu += red2[k].y;
    }
  };
  auto step_of = [&](int it, double gamma, double uu, double& beta, double& alpha) {
    beta = it == 0 ? 0.0 : gamma / gamma_prev;
    alpha = gamma / (fma(mu2, gamma, uu) - (it == 0 ? 0.0 : beta * gamma / alpha_prev));
  };
  auto advance = [&](const C* v, R rb, R ra) {
    const int o = unseen();
    gang_chunks<M, CH>(B.half, [&](int m) {
      s[m].x = fma(rb, s[m].x, v[m].x);
      s[m].y = fma(rb, s[m].y, v[m].y);
      p[m].x = fma(rb, p[m].x, r[m].x);
      p[m].y = fma(rb, p[m].y, r[m].y);
      r[m].x = fma(-ra, s[m].x, r[m].x);
      r[m].y = fma(-ra, s[m].y, r[m].y);
      z[m].x = fma(ra, p[m].x, z[m].x);
      z[m].y = fma(ra, p[m].y, z[m].y);
      if (ZMEM) state.set(3 * svec + sown + (unsigned)o + m * kGangThreads * SZ, z[m]);
    });
    return o;
  };

  if constexpr (STEP) {
    const bool mark = wg == 0 && tid == 0;
    auto lost = [&] {
      if (sh_bad && tid == 0) {
        sc->gang = 2;
        store_active(sc, 0);
      }
      return sh_bad != 0;
    };
    put_own(r, 0);
    if (K == kGangShare) {
      publish(r, tag0 + 1, 0);
      if (mark) {
        sc->sit = it0;
        sc->gang = 4;
      }
      return;
    }
    receive(tag0 + 1, [&](int h, C v) { put(hdst[h], v, 0); });
    __syncthreads();
    if (lost()) return;
    C v[M], xv[X];
    int o = first_half(v, xv);
    if (K == kGangSums) {
      record(tag0 + 1);
      if (mark) sc->git = it0 + 1;  // the rest of the iteration follows
      return;
    }
    o = second_half(v, xv, o);
    if (ZMEM) load(z, 3, o);
    if (wave < nw) collect(tag0 + 1);
    __syncthreads();
    if (lost()) return;
    double gamma, uu, beta, alpha;
    totals(gamma, uu);
    if (it0 > 0 && (!(gamma > stop2) || it0 >= maxit)) {
      __syncthreads();
      give(z, d->vec[zslot]);
      if (mark) {
        sc->rrv[it0 & 1] = gamma;
        sc->iters = it0;
        store_active(sc, 2);  // the next launch makes it 0: others of this one have yet to read it
      }
      return;
    }
    step_of(it0, gamma, uu, beta, alpha);
    o = advance(v, (R)beta, (R)alpha);
    save(r, 0);
    save(p, 1);
    save(s, 2);
    if (!ZMEM) save(z, 3);
    publish(r, tag0 + 2, o);
    if (mark) {
      sc->rrv[it0 & 1] = gamma;
      sc->alpha[it0 & 1] = alpha;
      sc->sit = it0 + 1;
    }
    return;
  }

  // r and s of the halo: sent once per launch, then carried along with the owner's own
  // arithmetic, so that the faces of w can travel while the reduction does.
  C rh[H], sh[H];
#pragma unroll
  for (int h = 0; h < H; ++h) rh[h] = sh[h] = cz<C>();
  put_own(r, 0);
  if (g > 1) {
    publish(r, tag0 + 1, 0);
    if (it0 > 0) publish(s, tag0 + 2, 0);
    receive(tag0 + 1, [&](int h, C v) {
      rh[h] = v;
      put(hdst[h], v, 0);
    });
    if (it0 > 0) receive(tag0 + 2, [&](int h, C v) { sh[h] = v; });
    // nobody writes over these faces before all have read them
    __syncthreads();
    if (wave == 0) post(0.0, 0.0, tag0 + 2);
    if (wave < nw) collect(tag0 + 2);
  }
  __syncthreads();
  int it = it0;
  bool stopped = false;
  double gamma = 0.0;
  if constexpr (SOLO) {
    // waves without a site only take part in the barriers and the stopping test
    const bool any = __builtin_amdgcn_readfirstlane(k0) < B.half;
    constexpr int D = kGangSecond;
#pragma unroll 1
    for (int step = 0; step < K; ++step, ++it) {
      C v[M];
      R acc_g = 0, acc_u = 0;
      if (any) {
        gang_chunks<M, CH>(B.half, [&](int m) {
          v[m] = half_op(link(a0[m] + dt1), std::true_type{}, at(a0[m] + dt1), at(a0[m] + dh), bond1(h1[m], 0),
                         bond2(h1[m], h2[m], 0), ks, r[m]);
          acc_g = fma(r[m].x, r[m].x, fma(r[m].y, r[m].y, acc_g));
          acc_u = fma(v[m].x, v[m].x, fma(v[m].y, v[m].y, acc_u));
        });
        put_own(v, 0, D);
        acc_g = dpp_wave(acc_g);
        acc_u = dpp_wave(acc_u);
      }
      if (lane == 63) red[wave] = double2{(double)acc_g, (double)acc_u};
      __syncthreads();
      // every wave sums the waves' shares, in one order
      double2 q[kGangWaves];
#pragma unroll
      for (int k = 0; k < kGangWaves; ++k) q[k] = red[k];
#pragma unroll
      for (int n = kGangWaves / 2; n > 0; n /= 2)
#pragma unroll
        for (int k = 0; k < n; ++k) q[k].x += q[k + n].x, q[k].y += q[k + n].y;
      gamma = q[0].x;
      if (it > 0 && (!(gamma > stop2) || it >= maxit)) {
        stopped = true;
        break;
      }
      double beta, alpha;
      step_of(it, gamma, q[0].y, beta, alpha);
      const R rb = (R)beta, ra = (R)alpha;
      if (any) {
        gang_chunks<M, CH>(B.half, [&](int m) {
          C w = half_op(link(a0[m]), std::false_type{}, at(a0[m] + D - dt1), at(a0[m] + D + dh), bond1(h1[m], 0, D),
                        bond2(h1[m], h2[m], 0, D), -ks, v[m]);
          w.x = fma(rmu2, r[m].x, w.x);
          w.y = fma(rmu2, r[m].y, w.y);
          s[m].x = fma(rb, s[m].x, w.x);
          s[m].y = fma(rb, s[m].y, w.y);
          p[m].x = fma(rb, p[m].x, r[m].x);
          p[m].y = fma(rb, p[m].y, r[m].y);
          r[m].x = fma(-ra, s[m].x, r[m].x);
          r[m].y = fma(-ra, s[m].y, r[m].y);
          z[m].x = fma(ra, p[m].x, z[m].x);
          z[m].y = fma(ra, p[m].y, z[m].y);
        });
        put_own(r, 0);
      }
      __syncthreads();
      gamma_prev = gamma;
      alpha_prev = alpha;
    }
  }
#pragma unroll 1
  for (int step = 0; !SOLO && step < K; ++step, ++it) {
    const unsigned tag = tag0 + (unsigned)step + 3;
    C v[M], xv[X];
    int o = first_half(v, xv);
    record(tag);
    // w; its faces out
    o = second_half(v, xv, o);
    if (g > 1) publish(v, tag, o);
    if (ZMEM) load(z, 3, o);
    if (g > 1 && wave < nw) collect(tag);
    __syncthreads();
    if (sh_bad) {
      if (wg == 0 && tid == 0) {
        sc->gang = 2;
        store_active(sc, 0);
        gang_release(g);
      }
      return;
    }
    // totals and step_of, written out: called here, they make the bodies of three sites 1%
    // slower (24x24x64 complex64 3.34 and 3.38 us)
    gamma = red2[0].x;
    double uu = red2[0].y;
    for (int k = 1; k < nw; ++k) {
      gamma += red2[k].x;
      uu += red2[k].y;
    }
    // the stopping test of iteration it (at it = 0 the CG setup decided)
    if (it > 0 && (!(gamma > stop2) || it >= maxit)) {
      stopped = true;
      break;
    }
    const double beta = it == 0 ? 0.0 : gamma / gamma_prev;
    const double alpha = gamma / (fma(mu2, gamma, uu) - (it == 0 ? 0.0 : beta * gamma / alpha_prev));
    const R rb = (R)beta, ra = (R)alpha;
    o = advance(v, rb, ra);
    put_own(r, o);
    if (g > 1)
      receive(tag, [&](int h, C w) {
        sh[h].x = fma(rb, sh[h].x, w.x);
        sh[h].y = fma(rb, sh[h].y, w.y);
        rh[h].x = fma(-ra, sh[h].x, rh[h].x);
        rh[h].y = fma(-ra, sh[h].y, rh[h].y);
        put(hdst[h], rh[h], o);
      });
    __syncthreads();
    gamma_prev = gamma;
    alpha_prev = alpha;
  }
  // a system that stopped leaves its solution, any other its state
  if (stopped) {
    __syncthreads();
    give(z, d->vec[zslot]);
  } else {
    save(r, 0);
    save(p, 1);
    save(s, 2);
    if (!ZMEM) save(z, 3);
  }
  if (wg == 0 && tid == 0) {
    if (!stopped) {
      sc->rrv[(it - 1) & 1] = gamma_prev;
      sc->alpha[(it - 1) & 1] = alpha_prev;
    } else {
      sc->rrv[it & 1] = gamma;
      sc->iters = it;
      store_active(sc, 0);
    }
    sc->git = it;
    sc->gang = 0;
    if (g > 1) gang_release(g);
  }
}

// The body of the system's class.
template <typename R, bool STEP>
__device__ __forceinline__ void gang_bodies(const SysDesc* __restrict__ d, Scal* sc, int wg, int zslot, unsigned tag,
                                            unsigned seq, unsigned arrived, int deny, int K, char* lds) {
  static_assert(GangTab<float>::n == 7 && GangTab<double>::n == 4, "the cases below");
  constexpr int last = GangTab<R>::n - 1;
  switch (d->gang.cls) {
    case 0: return gang_run<R, 0, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    case 1: return gang_run<R, 1, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    case 2: return gang_run<R, 2, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    case 3: return gang_run<R, 3, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    case 4: return gang_run<R, last < 4 ? last : 4, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    case 5: return gang_run<R, last < 5 ? last : 5, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
    default: return gang_run<R, last, false, STEP>(d, sc, wg, zslot, tag, seq, arrived, deny, K, lds);
  }
}

template <typename R>
__global__ __launch_bounds__(kGangThreads) void k_gang(const SysDesc* __restrict__ sys, GangList L, int K) {
  extern __shared__ __attribute__((aligned(16))) char gang_mem_lds[];
  const int kk = L.list[blockIdx.x], wg = L.wg[blockIdx.x];
  if (kk == kGangNone) return;
  const SysDesc* __restrict__ d = sys + L.sys[kk];
  Scal* sc = L.scal + L.sys[kk];
  // every workgroup of a launch counts among the arrivals, also of a system that has stopped
  unsigned arrived = 0;
  if (d->gang.g > 1 && threadIdx.x == 0)
    arrived = __hip_atomic_fetch_add((HUB_GAS unsigned*)d->gang_mem, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
  if (load_active(sc) != 1) return;
  const int zslot = L.pi[kk];
  const unsigned tag = L.tag[kk], seq = L.seq[kk];
  if (gang_solo<R>(d->gang, d->g.L1, d->g.L2, d->g.Nt)) {
    switch (d->gang.cls) {
      case 0: return gang_run<R, 0, true, false>(d, sc, wg, zslot, tag, seq, arrived, 0, K, gang_mem_lds);
      case 1: return gang_run<R, 1, true, false>(d, sc, wg, zslot, tag, seq, arrived, 0, K, gang_mem_lds);
      default: return gang_run<R, 2, true, false>(d, sc, wg, zslot, tag, seq, arrived, 0, K, gang_mem_lds);
    }
  }
  gang_bodies<R, false>(d, sc, wg, zslot, tag, seq, arrived, L.deny, K, gang_mem_lds);
}

// One part of an iteration of every system of L (all of several workgroups).  Bound by its
// set-up, the lists and links that k_gang works out once for its hundreds of iterations: 13 us
// a launch in FP64 and 17 in complex64 over lattices from 12x12x32 to 102x77x64, some 30 us an
// iteration (k_gang 3 to 9, the tiled kernels 26 at 102x102x64).  It runs where k_gang cannot.
template <typename R>
__global__ __launch_bounds__(kGangThreads) void k_gang_step(const SysDesc* __restrict__ sys, GangList L, int part) {
  extern __shared__ __attribute__((aligned(16))) char gang_mem_lds[];
  const int kk = L.list[blockIdx.x], wg = L.wg[blockIdx.x];
  if (kk == kGangNone) return;
  const SysDesc* __restrict__ d = sys + L.sys[kk];
  Scal* sc = L.scal + L.sys[kk];
  // read once for the whole workgroup: others of the launch may write it
  int* const active = reinterpret_cast<int*>(gang_mem_lds);
  if (threadIdx.x == 0) *active = load_active(sc);
  __syncthreads();
  const int a = *active;
  __syncthreads();
  if (part == kGangUpdate ? a == 0 : a != 1) {
    if (a == 2 && wg == 0 && threadIdx.x == 0) store_active(sc, 0);
    return;
  }
  gang_bodies<R, true>(d, sc, wg, L.pi[kk], L.tag[kk], 0, 0, 0, part, gang_mem_lds);
}

__global__ __launch_bounds__(kBlock) void k_gang_clear(u64* p, size_t n) {
  for (size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x; k < n; k += (size_t)gridDim.x * kBlock) p[k] = 0;
}

}  // namespace

template <typename R>
static hipError_t gang_launch(const SysDesc* sys, const GangList& L, int K, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(L.nblock), block(kGangThreads);
  // the tables exceed the default limit of dynamic LDS
  const hipError_t e = hipFuncSetAttribute((const void*)k_gang<R>, hipFuncAttributeMaxDynamicSharedMemorySize, kGangLdsBytes);
  if (e != hipSuccess) return e;
  if (e0)
    hipExtLaunchKernelGGL(k_gang<R>, grid, block, kGangLdsBytes, st, e0, e1, 0, sys, L, K);
  else
    hipLaunchKernelGGL(k_gang<R>, grid, block, kGangLdsBytes, st, sys, L, K);
  return hipGetLastError();
}

hipError_t launch_gang(const SysDesc* sys, const GangList& L, int K, bool single, hipStream_t st, hipEvent_t e0,
                       hipEvent_t e1) {
  if (L.nsys < 1 || L.nsys > kMaxSys || K < 1 || L.nblock < 1 || L.nblock > kGangMaxWgs)
    return hipErrorInvalidValue;
  return single ? gang_launch<float>(sys, L, K, st, e0, e1) : gang_launch<double>(sys, L, K, st, e0, e1);
}

template <typename R>
static hipError_t gang_steps(const SysDesc* sys, GangList L, int K, hipStream_t st) {
  const dim3 grid(L.nblock), block(kGangThreads);
  const hipError_t e =
      hipFuncSetAttribute((const void*)k_gang_step<R>, hipFuncAttributeMaxDynamicSharedMemorySize, kGangLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_gang_step<R>, grid, block, kGangLdsBytes, st, sys, L, (int)kGangShare);
  for (int k = 0; k < K; ++k) {
    hipLaunchKernelGGL(k_gang_step<R>, grid, block, kGangLdsBytes, st, sys, L, (int)kGangSums);
    hipLaunchKernelGGL(k_gang_step<R>, grid, block, kGangLdsBytes, st, sys, L, (int)kGangUpdate);
    for (int q = 0; q < L.nsys; ++q) ++L.tag[q];
  }
  // also ends a system that the last update has stopped
  hipLaunchKernelGGL(k_gang_step<R>, grid, block, kGangLdsBytes, st, sys, L, (int)kGangShare);
  return hipGetLastError();
}

hipError_t launch_gang_steps(const SysDesc* sys, const GangList& L, int K, bool single, hipStream_t st) {
  if (L.nsys < 1 || L.nsys > kMaxSys || K < 1 || L.nblock < 1 || L.nblock > kGangMaxWgs) return hipErrorInvalidValue;
  return single ? gang_steps<float>(sys, L, K, st) : gang_steps<double>(sys, L, K, st);
}

hipError_t launch_gang_clear(unsigned long long* mem, size_t words, hipStream_t st) {
  const size_t blocks = (words + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(k_gang_clear, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(kBlock), 0, st, mem, words);
  return hipGetLastError();
}

}  // namespace hub
