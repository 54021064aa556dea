// Host check of the solver engine (csrc/hub_engine.hip) and the C ABI's drivers
// (csrc/hub_api.hip) against a device that is played by this file: every launch takes effect at once, with numbers that lead the engine where the
// scenario wants it.  Usage: engine_host <scenario>; exit 0: the engine did as it should.
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "hub_engine.h"

using namespace hub;

// ---- the device ---------------------------------------------------------------------
namespace {
struct Device {
  bool lose_flag = false;  // the sequence number of an Arnoldi step's publication does not arrive
  double resid2 = 9e-20;   // |b - A x|^2 that the next true residuals show (|b| = 1)
  int cgs = 0;             // second halves of Arnoldi steps so far
  int steps = 0;           // blocks of a system in steps
  bool fail = false;       // launches of gangs fail
  int cus = 256, masked = 256;  // of the device, of the stream
  size_t freed = 0;        // hipFree calls
  std::function<void(const SysDesc*, const GangList&, int, bool)> gang;
  std::function<void(const SysDesc&, Scal&)> tiled;  // a block of one system
} dev;

void publish(const Publish& pub, bool lose = false) {
  if (!pub.flag) return;
  std::memcpy((void*)pub.h, (const void*)pub.d, sizeof(Scal) * pub.cnt);
  if (!lose) *pub.flag = pub.seq;
}
void start(Scal& sc, int maxit) {
  sc.active = 1;
  sc.iters = sc.git = sc.gang = 0;
  sc.maxit = maxit;
}
void stop(Scal& sc) {
  sc.active = 0;
  sc.iters = 10;
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { return std::free(p), ++dev.freed, hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { return *f = *t = (size_t)8 << 30, hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = (void*)s, hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "an error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)std::malloc(1), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void*)s), hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = dev.cus, hipSuccess; }
hipError_t hipExtStreamGetCUMask(hipStream_t, uint32_t n, uint32_t* mask) {
  for (uint32_t k = 0; k < n; ++k) mask[k] = 0;
  for (int k = 0; k < dev.masked; ++k) mask[k / 32] |= 1u << k % 32;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)std::malloc(1), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void*)e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0.0f, hipSuccess; }
}

namespace hub {
hipError_t launch_apply(const Geom&, const double*, const double2*, double2*, int, bool, hipStream_t, bool) { return hipSuccess; }
hipError_t launch_force(const Geom&, const double*, const double2*, const double2*, double, int, double*, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_dot_re(const Geom&, const double2*, const double2*, int, double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_phase(const double*, double2*, float*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_phase_jobs(const PhaseJobs&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_normal(const Geom&, const double*, double2*, size_t, const double*, const double2*, double2*, int,
                         hipStream_t) {
  return hipSuccess;
}
size_t normal_scratch(const Geom& g, int batch, bool least) { return (size_t)g.n * 16 * (least ? 1 : batch); }
hipError_t launch_force_sum(const Geom&, const double*, const double2*, const double2*, const double*, int, double*, int,
                            hipStream_t) {
  return hipSuccess;
}
hipError_t launch_stream_bytes(const double*, const double2*, double2*, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_publish(const Publish& pub, hipStream_t) { return publish(pub), hipSuccess; }
hipError_t launch_xupdate(const SysDesc*, const LaunchList&, const double*, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_gang_clear(unsigned long long*, size_t, hipStream_t) { return hipSuccess; }
hipError_t launch_gang_steps(const SysDesc*, const GangList& L, int K, bool, hipStream_t) {
  for (int k = 0; k < L.nsys; ++k) {
    Scal& sc = L.scal[L.sys[k]];
    if (sc.active != 1) continue;
    sc.git += K;
    sc.gang = 4;
    ++dev.steps;
    if (sc.git >= 100) stop(sc);
  }
  return hipSuccess;
}
hipError_t launch_cg_init_zero(const SysDesc*, const LaunchList& L, RedMode mode, const Publish& pub, hipStream_t) {
  for (int k = 0; k < L.nsys; ++k) {
    L.scal[L.sys[k]].red[0] = 1.0;
    if (mode == RED_CG_SETUP) start(L.scal[L.sys[k]], L.pi[k]);
  }
  return publish(pub), hipSuccess;
}
hipError_t launch_normal_slot(const SysDesc*, const LaunchList& L, int, int, int, RedMode mode, int off, bool, const Publish& pub,
                              hipStream_t) {
  for (int k = 0; k < L.nsys; ++k) {
    L.scal[L.sys[k]].red[off] = dev.resid2;
    if (mode == RED_CG_SETUP) start(L.scal[L.sys[k]], L.pi[k]);
  }
  return publish(pub), hipSuccess;
}
hipError_t launch_prep_inner(const SysDesc*, const LaunchList& L, int, hipStream_t) {
  for (int k = 0; k < L.nsys; ++k) start(L.scal[L.sys[k]], L.pi[k]);
  return hipSuccess;
}
hipError_t launch_arnoldi_dots(const SysDesc*, const LaunchList& L, int j, bool, hipStream_t) {
  for (int k = 0; k < L.nsys; ++k)
    for (int i = 0; i <= 2 * j + 1; ++i) L.scal[L.sys[k]].red[i] = i == 2 * j ? 1.0 : 0.0;
  return hipSuccess;
}
hipError_t launch_cgs(const SysDesc*, const LaunchList& L, int j, const Publish& pub, hipStream_t) {
  ++dev.cgs;
  for (int k = 0; k < L.nsys; ++k) L.scal[L.sys[k]].red[2 * j + 2] = 0.9;
  return publish(pub, dev.lose_flag), hipSuccess;
}
hipError_t launch_gang(const SysDesc* sys, const GangList& L, int K, bool single, hipStream_t, hipEvent_t, hipEvent_t) {
  if (dev.fail) return hipErrorLaunchFailure;
  if (dev.gang) return dev.gang(sys, L, K, single), hipSuccess;
  for (int k = 0; k < L.nsys; ++k) stop(L.scal[L.sys[k]]);
  return hipSuccess;
}
hipError_t launch_cg_iter(const SysDesc* sys, const LaunchList& L, bool, hipStream_t) {
  for (int k = 0; k < L.nsys; ++k) {
    if (dev.tiled) dev.tiled(sys[L.sys[k]], L.scal[L.sys[k]]);
    stop(L.scal[L.sys[k]]);
  }
  return hipSuccess;
}
hipError_t launch_cg_stage(const SysDesc* sys, const LaunchList& L, bool single, int, hipStream_t st, hipEvent_t, hipEvent_t) {
  return launch_cg_iter(sys, L, single, st);
}
}  // namespace hub

// ---- scenarios ----------------------------------------------------------------------
namespace {
#define CHECK(c)                                                    \
  do {                                                              \
    if (!(c)) {                                                     \
      std::printf("line %d: %s does not hold\n", __LINE__, #c);     \
      std::exit(1);                                                 \
    }                                                               \
  } while (0)

hub_solve_opts options(hub_solver solver) {
  hub_solve_opts o{};
  o.solver = solver;
  o.max_iter = solver == HUB_CG_FP64 ? 20000 : 3;
  o.restart_m = 10;
  o.inner_max_iter = 4000;
  o.tol = 1e-10;
  o.inner_a = 5.0;
  o.inner_floor = 1e-5;
  o.check_every = 8;
  return o;
}
System system_of(int L1, int L2, int Nt, hub_solver solver) {
  static double field;
  hub_lattice lat{};
  lat.L1 = L1, lat.L2 = L2, lat.Nt = Nt, lat.kappa_t = 0.2;
  System s;
  s.g = make_geom(lat);
  s.phi = &field;
  s.opts = options(solver);
  return s;
}
constexpr size_t kPlenty = (size_t)8 << 30;

// A publication whose number does not arrive while the next Arnoldi step is on the device
// already: the records there are the next step's, and must not pass for the ones waited for.
// Where nothing came after it, they are the right ones.
void lost_publication() {
  for (bool next_on_the_way : {true, false}) {
    dev = Device{};
    Pool pool(0, kPlenty);
    Engine eng(&pool, nullptr);
    System s = system_of(6, 6, 8, HUB_FGMRES_MIXED);
    if (!next_on_the_way) s.opts.restart_m = 1;
    CHECK(eng.add(&s) == Engine::ADD_OK);
    dev.lose_flag = true;
    bool failed = false;
    for (int k = 0; k < 50 && !s.done && !failed; ++k) failed = eng.step() != hipSuccess;
    CHECK(dev.cgs > 0);
    CHECK(failed == next_on_the_way);
    CHECK(failed || s.done);
    eng.remove(&s);
  }
}

// A block that does not fit beside those in use is refused with the cached blocks kept: none
// of them would make room for it.
void refusal_keeps_cache() {
  constexpr size_t MB = (size_t)1 << 20;
  Pool pool(0, 10 * MB);
  void *held = pool.alloc(4 * MB, nullptr), *cached = pool.alloc(4 * MB, nullptr);
  CHECK(held && cached);
  pool.release(cached, nullptr);
  CHECK(!pool.alloc(8 * MB, nullptr));
  CHECK(dev.freed == 0 && pool.reserved() == 8 * MB);
  void* fits = pool.alloc(6 * MB, nullptr);  // in the place of the cached one
  CHECK(fits && dev.freed == 1 && pool.reserved() == 10 * MB);
  pool.release(held, nullptr);
  pool.release(fits, nullptr);
}

// What the tables of several fields may take: a workspace of one block each for the tables and
// the vectors of every system is enough, also where blocks of a power of two would not be.
void tables_of_fields() {
  for (hub_solver solver : {HUB_CG_FP64, HUB_FGMRES_MIXED})
    for (int fields : {1, 3, 5, 33, 64})
      for (int Nt : {3, 16, 64, 100}) {
        dev = Device{};
        dev.resid2 = 0.0;
        const System s = system_of(4, 2, Nt, solver);
        const size_t n = s.g.n;
        hub_ctx* ctx = nullptr;
        CHECK(hub_create(&ctx, 0, fields * Engine::workspace_bytes(s.g, s.opts)) == HUB_OK);
        std::vector<double> phi(fields * n), mu2(fields);
        std::vector<hub_c128> b(fields * n), x(fields * n);
        std::vector<hub_solve_info> info(fields);
        hub_lattice lat{};
        lat.L1 = 4, lat.L2 = 2, lat.Nt = Nt, lat.kappa_t = 0.2;
        const hub_status st = hub_solve_fields(ctx, &lat, phi.data(), 1, mu2.data(), fields, b.data(), x.data(), &s.opts,
                                               info.data(), nullptr);
        if (st != HUB_OK) std::printf("solver %d, %d fields, Nt %d: %s\n", solver, fields, Nt, hub_last_error());
        CHECK(st == HUB_OK);
        CHECK(hub_destroy(ctx) == HUB_OK);
      }
}

// One request on buffers of its own.
struct Request {
  hub_request r{};
  std::vector<double> phi;
  std::vector<hub_c128> chi, x;
  uint64_t ticket = 0;
  Request(int L1, int L2, int Nt, double mu2, hub_solver solver) {
    r.lat.L1 = L1, r.lat.L2 = L2, r.lat.Nt = Nt, r.lat.kappa_t = 0.2;
    r.mu2 = mu2;
    const size_t n = 2 * (size_t)L1 * L2 * Nt;
    phi.resize(n), chi.resize(n), x.resize(n);
    r.phi = phi.data(), r.chi = chi.data(), r.x_out = x.data();
    r.opts = options(solver);
  }
  void submit(hub_ctx* ctx) { CHECK(hub_submit(ctx, &r, &ticket) == HUB_OK); }
  hub_status wait(hub_ctx* ctx) {
    int32_t done = 0;
    hub_status st = HUB_OK;
    while (!done) st = hub_poll(ctx, ticket, &done, nullptr);
    return st;
  }
};

// A gang whose wait runs out ends its own system; the others, of the same call or of other
// requests, are solved.
void gang_without_an_answer() {
  for (hub_solver solver : {HUB_CG_FP64, HUB_FGMRES_MIXED}) {
    dev = Device{};
    dev.resid2 = 0.0;
    dev.gang = [](const SysDesc* sys, const GangList& L, int, bool) {
      for (int k = 0; k < L.nsys; ++k) {
        Scal& sc = L.scal[L.sys[k]];
        if (sc.active == 1 && sys[L.sys[k]].mu2 == 0.5) sc.gang = 2;
        stop(sc);
      }
    };
    Pool pool(0, kPlenty);
    {
      Engine eng(&pool, nullptr);
      std::vector<System> s{system_of(6, 6, 8, solver), system_of(6, 6, 8, solver)};
      std::vector<void*> owned;
      s[0].mu2 = 0.5;
      for (System& q : s) CHECK(eng.add(&q) == Engine::ADD_OK);
      bool room = false;
      CHECK(eng.join_gangs({&s[0], &s[1]}, owned, room) == hipSuccess && room);
      int ended = 0;
      for (System& q : s) q.on_done = [&](System*) { ++ended; };
      for (int k = 0; k < 50 && !(s[0].done && s[1].done); ++k) CHECK(eng.step() == hipSuccess);
      CHECK(s[0].status == HUB_ERR_HIP && s[1].status == HUB_OK && ended == 2);
      for (System& q : s) eng.remove(&q, &owned);
      pool.release_all(owned, nullptr);
    }
    // requests, of other lattices too
    hub_ctx* ctx = nullptr;
    CHECK(hub_create(&ctx, 0, 0) == HUB_OK);
    std::vector<Request> rs;
    for (int k = 0; k < 6; ++k) rs.emplace_back(4 + k, 5, 8, k == 2 ? 0.5 : 0.1, solver);
    for (Request& r : rs) r.submit(ctx);
    for (int k = 0; k < 6; ++k) CHECK(rs[k].wait(ctx) == (k == 2 ? HUB_ERR_HIP : HUB_OK));
    CHECK(hub_destroy(ctx) == HUB_OK);
  }
}

// A gang that is never met, or always refused, goes on in steps after a bounded number of
// attempts, tries again ever more rarely, and its place in the next solve begins there.
void gangs_that_never_meet() {
  for (int outcome : {1, 3}) {
    dev = Device{};
    dev.resid2 = 0.0;
    int tries = 0;
    dev.gang = [&](const SysDesc*, const GangList& L, int, bool) {
      for (int k = 0; k < L.nsys; ++k)
        if (L.scal[L.sys[k]].active == 1) L.scal[L.sys[k]].gang = outcome, ++tries;
    };
    Pool pool(0, kPlenty);
    Engine eng(&pool, nullptr);
    for (int solve = 0; solve < 2; ++solve) {
      System s = system_of(12, 12, 32, HUB_CG_FP64);
      std::vector<void*> owned;
      tries = dev.steps = 0;
      CHECK(eng.add(&s) == Engine::ADD_OK);
      bool room = false;
      CHECK(eng.join_gangs({&s}, owned, room) == hipSuccess && room);
      CHECK(s.desc.gang.g > 1);
      for (int k = 0; k < 100 && !s.done; ++k) CHECK(eng.step() == hipSuccess);
      CHECK(s.done && s.status == HUB_OK);
      CHECK(dev.steps == 7);  // 16 iterations each
      // three and one on its way, then two after 1, 2 and 4 blocks; later fewer
      CHECK(solve == 0 ? tries > kGangMisses && tries <= 10 : tries <= 4);
      eng.remove(&s, &owned);
      pool.release_all(owned, nullptr);
    }
  }
}

// Which kernels iterate on a request depends on the request and the budget, not on what else
// is in flight: it is the same alone and in company, for budgets from one workspace to plenty.
void kernels_by_request() {
  std::mutex mu;
  std::map<double, std::string> path;  // of the request with that shift
  std::map<double, int> launches;
  auto note = [&](double mu2, const char* what) {
    std::lock_guard<std::mutex> lk(mu);
    if (path[mu2].find(what) == std::string::npos) path[mu2] += what;
  };
  for (hub_solver solver : {HUB_CG_FP64, HUB_FGMRES_MIXED}) {
    const System s = system_of(12, 12, 32, solver);
    const size_t ws = Engine::workspace_bytes(s.g, s.opts);
    Pool pool(0, kPlenty);
    System like = s;
    const size_t gang = Engine(&pool, nullptr).gang_bytes({&like});
    bool seen[2] = {false, false};
    for (double part : {1.0, 1.2, 1.5, 2.0, 2.5, 3.0, 3.7, 4.0, 5.0, 100.0}) {
      dev = Device{};
      dev.resid2 = 0.0;
      dev.tiled = [&](const SysDesc& d, Scal& sc) {
        if (sc.active) note(d.mu2, "tiled ");
      };
      dev.gang = [&](const SysDesc* sys, const GangList& L, int, bool) {
        for (int k = 0; k < L.nsys; ++k) {
          const double m = sys[L.sys[k]].mu2;
          if (L.scal[L.sys[k]].active) note(m, "gang ");
          if (++launches[m] % 20 == 0) stop(L.scal[L.sys[k]]);  // in flight for some while
        }
      };
      std::string alone;
      for (int company : {1, 4}) {
        path.clear();
        hub_ctx* ctx = nullptr;
        CHECK(hub_create(&ctx, 0, (size_t)(part * (double)ws)) == HUB_OK);
        std::vector<Request> rs;
        for (int k = 0; k < company; ++k) rs.emplace_back(12, 12, 32, 0.1 + k, solver);
        for (Request& r : rs) r.submit(ctx);
        for (Request& r : rs) CHECK(r.wait(ctx) == HUB_OK);
        CHECK(hub_destroy(ctx) == HUB_OK);
        if (company == 1) alone = path[0.1];
        CHECK(alone == "gang " || alone == "tiled ");
        for (const Request& r : rs) CHECK(path[r.r.mu2] == alone);
      }
      seen[alone == "gang "] = true;
    }
    CHECK(seen[0] && seen[1]);
    // a call beside a served request that holds most of the budget
    dev = Device{};
    dev.resid2 = 0.0;
    path.clear();
    std::atomic<int> served{0};
    dev.tiled = [&](const SysDesc& d, Scal& sc) {
      if (sc.active) note(d.mu2, "tiled ");
    };
    dev.gang = [&](const SysDesc* sys, const GangList& L, int, bool) {
      for (int k = 0; k < L.nsys; ++k) {
        const double m = sys[L.sys[k]].mu2;
        note(m, "gang ");
        if (m == 0.7 || ++served > 2000) stop(L.scal[L.sys[k]]);
      }
    };
    hub_ctx* ctx = nullptr;
    CHECK(hub_create(&ctx, 0, 2 * ws + gang) == HUB_OK);
    Request r(12, 12, 32, 0.1, solver);
    r.submit(ctx);
    while (served == 0) std::this_thread::yield();
    Request c(12, 12, 32, 0.7, solver);
    hub_solve_info info;
    CHECK(hub_solve(ctx, &c.r.lat, c.r.phi, &c.r.mu2, 1, c.r.chi, c.r.x_out, &c.r.opts, &info, nullptr) == HUB_OK);
    CHECK(path[0.7] == "gang ");
    CHECK(r.wait(ctx) == HUB_OK);
    CHECK(hub_destroy(ctx) == HUB_OK);
    // one that would not fit without it either does not wait: the request ends after the call
    path.clear();
    served = 0;
    std::atomic<bool> returned{false};
    dev.gang = [&](const SysDesc* sys, const GangList& L, int, bool) {
      for (int k = 0; k < L.nsys; ++k) {
        ++served;
        note(sys[L.sys[k]].mu2, "gang ");
        if (returned) stop(L.scal[L.sys[k]]);
      }
    };
    const int many = 8;
    System small = system_of(6, 6, 64, solver);
    const size_t others = Engine::workspace_bytes(small.g, small.opts) + Engine(&pool, nullptr).gang_bytes({&small});
    CHECK(hub_create(&ctx, 0, many * ws + others) == HUB_OK);
    Request r2(6, 6, 64, 0.1, solver);
    r2.submit(ctx);
    while (served == 0) std::this_thread::yield();
    std::vector<hub_c128> b(many * c.x.size()), x(many * c.x.size());
    std::vector<hub_solve_info> infos(many);
    const std::vector<double> mu2(many, 0.7);
    CHECK(hub_solve(ctx, &c.r.lat, c.r.phi, mu2.data(), many, b.data(), x.data(), &c.r.opts, infos.data(), nullptr) == HUB_OK);
    CHECK(path[0.7] == "tiled ");
    returned = true;
    CHECK(r2.wait(ctx) == HUB_OK && path[0.1] == "gang ");
    CHECK(hub_destroy(ctx) == HUB_OK);
  }
}

// Turns are taken in the order of asking, as many at once as fit; an engine at work gives its
// own up when another one waits, after a block or two, and when a step fails.
void turns() {
  GangTurns& t = GangTurns::of(7);
  CHECK(t.take(100) && t.take(100) && !t.wanted());
  std::mutex mu;
  std::string order;
  std::vector<std::thread> ts;
  auto ask = [&](char name, int wgs) {
    const bool before = t.wanted();
    ts.emplace_back([&, name, wgs] {
      CHECK(t.take(wgs));
      std::lock_guard<std::mutex> lk(mu);
      order += name;
    });
    while (!before && !t.wanted()) std::this_thread::yield();
    std::this_thread::sleep_for(std::chrono::milliseconds(20));
  };
  ask('a', 256);
  ask('b', 10);  // would fit, but came later
  CHECK(order.empty());
  t.give(100);
  t.give(100);
  while (order.size() < 1) std::this_thread::yield();
  CHECK(order == "a");
  t.give(256);
  for (std::thread& x : ts) x.join();
  CHECK(order == "ab" && !t.wanted());
  CHECK(!t.take(250));  // a second later: without
  CHECK(t.take(246) && !t.wanted());
  t.give(246);
  t.give(10);

  Pool pool(0, kPlenty);
  for (bool fails : {false, true}) {
    dev = Device{};
    dev.resid2 = 0.0;
    std::atomic<int> launches{0};
    dev.gang = [&](const SysDesc*, const GangList&, int, bool) { ++launches; };  // never stops
    Engine eng(&pool, nullptr);
    System s = system_of(48, 48, 64, HUB_CG_FP64);
    std::vector<void*> owned;
    bool room = false;
    CHECK(eng.add(&s) == Engine::ADD_OK);
    CHECK(eng.join_gangs({&s}, owned, room) == hipSuccess && room && s.desc.gang.g == kGangMaxWgs);
    for (int k = 0; k < 10; ++k) CHECK(eng.step() == hipSuccess);
    GangTurns& u = GangTurns::of(0);
    CHECK(!u.wanted());
    std::atomic<bool> got{false};
    std::thread other([&] {
      CHECK(u.take(1));
      got = true;
      u.give(1);
    });
    while (!u.wanted() && !got) std::this_thread::yield();
    const int before = launches;
    if (fails) {
      dev.fail = true;
      CHECK(eng.step() != hipSuccess);
    } else {
      CHECK(eng.step() == hipSuccess);
      CHECK(eng.step() == hipSuccess);
    }
    other.join();
    CHECK(got && launches <= before + 2);
    dev.fail = false;
    eng.remove(&s, &owned);
    pool.release_all(owned, nullptr);
    CHECK(u.take(kGangMaxWgs));  // nothing is left behind
    u.give(kGangMaxWgs);
  }
}

// Without the CUs for a full launch a system of several workgroups has no gang; one engine
// sees its stream change (the handle may be another stream's by the next call).
void cus_of_the_stream() {
  Pool pool(0, kPlenty);
  dev = Device{};
  Engine eng(&pool, nullptr);
  for (auto c : {std::pair<int, int>{256, 256}, {256, 255}, {32, 32}, {256, 256}, {304, 304}}) {
    dev.cus = c.first, dev.masked = c.second;
    for (int L : {6, 12}) {
      System s = system_of(L, L, L == 6 ? 16 : 32, HUB_FGMRES_MIXED);
      std::vector<void*> owned;
      bool room = false;
      const bool want = L == 6 || c.second >= 256;
      CHECK((eng.gang_bytes({&s}) > 0) == want);
      CHECK(eng.add(&s) == Engine::ADD_OK);
      CHECK(eng.join_gangs({&s}, owned, room) == hipSuccess && room);
      CHECK(s.gang == want && (s.desc.gang.g == 1) == (L == 6));
      eng.remove(&s, &owned);
      pool.release_all(owned, nullptr);
    }
  }
}

// Systems that stop at about the same time share a launch, in whatever order they are given:
// a launch holds its CUs until its last system is through.
void like_with_like() {
  dev = Device{};
  dev.resid2 = 0.0;
  int launches = 0, distinct = 0;  // shifts of a launch, over all launches
  dev.gang = [&](const SysDesc* sys, const GangList& L, int, bool) {
    ++launches;
    std::set<double> seen;
    for (int k = 0; k < L.nsys; ++k) {
      const SysDesc& d = sys[L.sys[k]];
      seen.insert(d.mu2);
      CHECK(L.pi[k] == S_X && L.tag[k] == 0 && L.seq[k] == 1);
      stop(L.scal[L.sys[k]]);
    }
    distinct += (int)seen.size();
  };
  Pool pool(0, (size_t)64 << 30);
  Engine eng(&pool, nullptr);
  std::vector<System> s;
  const double shifts[4] = {0.1, 0.0, 1.0, 0.01};
  for (int k = 0; k < 40; ++k) {
    s.push_back(system_of(12, 12, 32, HUB_CG_FP64));
    s.back().mu2 = shifts[(k * k + k / 3) % 4];
  }
  std::vector<System*> all;
  std::vector<void*> owned;
  bool room = false;
  for (System& q : s) {
    CHECK(eng.add(&q) == Engine::ADD_OK);
    all.push_back(&q);
  }
  CHECK(eng.join_gangs(all, owned, room) == hipSuccess && room);
  for (int k = 0; k < 3 && launches == 0; ++k) CHECK(eng.step() == hipSuccess);
  CHECK(launches == (40 * s[0].desc.gang.g + 255) / 256 && distinct <= 4 + launches - 1);
  for (System& q : s) eng.remove(&q, &owned);
  pool.release_all(owned, nullptr);
}

const std::map<std::string, void (*)()> scenarios = {
    {"like_with_like", like_with_like},
    {"cus_of_the_stream", cus_of_the_stream},
    {"turns", turns},
    {"kernels_by_request", kernels_by_request},
    {"gangs_that_never_meet", gangs_that_never_meet},
    {"gang_without_an_answer", gang_without_an_answer},
    {"tables_of_fields", tables_of_fields},
    {"refusal_keeps_cache", refusal_keeps_cache},
    {"lost_publication", lost_publication},
};
}  // namespace

int main(int argc, char** argv) {
  const auto it = argc > 1 ? scenarios.find(argv[1]) : scenarios.end();
  if (it == scenarios.end()) return std::printf("no such scenario\n"), 2;
  it->second();
  return 0;
}
