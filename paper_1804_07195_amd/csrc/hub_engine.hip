// Host orchestration of the solves: workspace pool, the batched engine that runs
// FP64 CG (Sec. 3) and the flexible GMRES with single-precision CG preconditioning
// of Appendix A (Algorithm A.1) for many systems at once, and the small Hessenberg
// least-squares problem of the FGMRES update.
#include <algorithm>
#include <chrono>
#include <map>
#include <cmath>
#include <cstring>

#include "hub_engine.h"

namespace hub {

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string t_err;
void set_error(const std::string& msg) { t_err = msg; }
const char* get_error() { return t_err.c_str(); }

// ---------------------------------------------------------------------------
// geometry
// ---------------------------------------------------------------------------
Geom make_geom(const hub_lattice& lat) {
  Geom g{};
  g.L1 = lat.L1;
  g.L2 = lat.L2;
  g.Nt = lat.Nt;
  g.P = lat.L1 * lat.L2;
  g.n = 2 * g.P * lat.Nt;
  g.dL2 = make_fastdiv((uint32_t)lat.L2);
  g.dL1 = make_fastdiv((uint32_t)lat.L1);
  g.kappa = lat.kappa_t;
  g.ms = lat.ms_t;
  return g;
}

int ntiles_of(int n) { return (n + kTile - 1) / kTile; }

// ---------------------------------------------------------------------------
// Pool
// ---------------------------------------------------------------------------
static constexpr size_t kGran = size_t(2) << 20;

size_t Pool::rounded(size_t bytes) {
  if (bytes >= kGran) return (bytes + kGran - 1) / kGran * kGran;
  size_t r = 4096;
  while (r < bytes) r <<= 1;
  return r;
}

Pool::Pool(int device, size_t budget) : device_(device), budget_(budget) {}

Pool::~Pool() {
  (void)hipSetDevice(device_);
  for (auto& f : free_)
    for (auto& b : f.second) {
      drop_event(b.ev, true);
      (void)hipFree(b.p);
    }
  for (auto& l : live_) (void)hipFree(l.first);
}

void Pool::drop_event(SharedEvent* e, bool wait) {
  if (!e) return;
  if (wait && e->ev) (void)hipEventSynchronize(e->ev);
  if (--e->refs == 0) {
    if (e->ev) (void)hipEventDestroy(e->ev);
    delete e;
  }
}

size_t Pool::in_use() const {
  std::lock_guard<std::mutex> lk(mu_);
  return used_;
}

bool Pool::fits(size_t bytes) const {
  std::lock_guard<std::mutex> lk(mu_);
  return used_ + rounded(bytes) <= budget_;
}

size_t Pool::reserved() const {
  std::lock_guard<std::mutex> lk(mu_);
  return reserved_;
}

void* Pool::alloc(size_t bytes, hipStream_t st) {
  const size_t sz = rounded(bytes == 0 ? 1 : bytes);
  std::lock_guard<std::mutex> lk(mu_);
  // reuse a cached block of the same size: at once on the stream that released it,
  // on another stream once the work before the release has finished
  auto same = free_.find(sz);
  if (same != free_.end()) {
    auto& f = same->second;
    for (size_t k = 0; k < f.size(); ++k) {
      Block& b = f[k];
      if (b.st != st && b.ev && b.ev->ev && hipEventQuery(b.ev->ev) != hipSuccess) continue;
      void* p = b.p;
      drop_event(b.ev, false);
      f.erase(f.begin() + (long)k);
      if (f.empty()) free_.erase(same);
      live_.emplace(p, sz);
      used_ += sz;
      return p;
    }
  }
  // release cached blocks, the largest first, until the new one fits; none where even all
  // of them would not make room
  if (used_ + sz > budget_) {
    set_error("workspace of " + std::to_string(sz) + " bytes exceeds the HBM budget (" +
              std::to_string(used_) + " of " + std::to_string(budget_) + " bytes in use)");
    return nullptr;
  }
  while (reserved_ + sz > budget_ && !free_.empty()) {
    auto last = std::prev(free_.end());
    Block b = last->second.back();
    last->second.pop_back();
    if (last->second.empty()) free_.erase(last);
    drop_event(b.ev, true);
    (void)hipFree(b.p);
    reserved_ -= b.bytes;
  }
  void* p = nullptr;
  if (hipMalloc(&p, sz) != hipSuccess) {
    (void)hipGetLastError();
    set_error("hipMalloc of " + std::to_string(sz) + " bytes failed");
    return nullptr;
  }
  reserved_ += sz;
  used_ += sz;
  live_.emplace(p, sz);
  return p;
}

void Pool::release(void* p, hipStream_t st) {
  if (p) release_all(std::vector<void*>{p}, st);
}

void Pool::release_all(const std::vector<void*>& ps, hipStream_t st) {
  std::lock_guard<std::mutex> lk(mu_);
  SharedEvent* e = nullptr;
  for (void* p : ps) {
    if (!p) continue;
    const auto l = live_.find(p);
    if (l == live_.end()) continue;
    if (!e) {
      e = new SharedEvent;
      if (hipEventCreateWithFlags(&e->ev, hipEventDisableTiming) != hipSuccess ||
          hipEventRecord(e->ev, st) != hipSuccess) {
        // no event to order later users after the stream's work: wait for it here
        if (e->ev) (void)hipEventDestroy(e->ev);
        e->ev = nullptr;
        (void)hipStreamSynchronize(st);
      }
    }
    e->refs++;
    free_[l->second].push_back(Block{p, l->second, st, e});
    used_ -= l->second;
    live_.erase(l);
  }
}

// ---------------------------------------------------------------------------
// least squares  min | beta e_1 - H y |  for a (k+1) x k upper Hessenberg H
// (Algorithm A.1 solves the normal equations by Cholesky; Givens rotations give
// the same minimiser with better conditioning).
// ---------------------------------------------------------------------------
std::vector<std::complex<double>> hessenberg_lsq(const std::vector<std::complex<double>>& Hin, int ldh, int k,
                                                 double beta, double* resid) {
  using cd = std::complex<double>;
  std::vector<cd> H(Hin);
  std::vector<cd> gvec(k + 1, cd(0.0));
  gvec[0] = beta;
  auto at = [&](int i, int j) -> cd& { return H[(size_t)j * ldh + i]; };
  for (int i = 0; i < k; ++i) {
    const cd a = at(i, i), b = at(i + 1, i);
    const double r = std::sqrt(std::norm(a) + std::norm(b));
    if (r == 0.0) continue;
    double c;
    cd s;
    if (std::abs(a) == 0.0) {
      c = 0.0;
      s = 1.0;
    } else {
      c = std::abs(a) / r;
      s = (a / std::abs(a)) * std::conj(b) / r;
    }
    for (int j = i; j < k; ++j) {
      const cd u = at(i, j), v = at(i + 1, j);
      at(i, j) = c * u + s * v;
      at(i + 1, j) = -std::conj(s) * u + c * v;
    }
    const cd u = gvec[i], v = gvec[i + 1];
    gvec[i] = c * u + s * v;
    gvec[i + 1] = -std::conj(s) * u + c * v;
  }
  // the rotated right-hand side's last entry is the minimal residual
  if (resid) *resid = std::abs(gvec[k]);
  std::vector<cd> y(k, cd(0.0));
  for (int i = k - 1; i >= 0; --i) {
    cd acc = gvec[i];
    for (int j = i + 1; j < k; ++j) acc -= at(i, j) * y[j];
    y[i] = at(i, i) == cd(0.0) ? cd(0.0) : acc / at(i, i);
  }
  return y;
}

// ---------------------------------------------------------------------------
// Engine
// ---------------------------------------------------------------------------
enum Phase : int {
  PH_NEW = 0,
  PH_CG_ITER,
  PH_CG_CONFIRM,
  PH_F_INNER,
  PH_F_POST_INIT,
  PH_F_ARNOLDI,
  PH_F_POST_ARNOLDI,
  PH_F_LSQ,
  PH_LOST,  // a workgroup of the system's gang did not answer
  PH_DONE
};

#define HUB_TRY(expr)                        \
  do {                                       \
    hipError_t e_ = (expr);                  \
    if (e_ != hipSuccess) return e_;         \
  } while (0)

constexpr size_t kScalBytes = sizeof(Scal) * kMaxSys + sizeof(unsigned) * kScalCounters;

GangTurns& GangTurns::of(int device) {
  static std::mutex& mu = *new std::mutex;  // never destroyed: engines may outlive statics
  static auto& all = *new std::map<int, GangTurns>;
  std::lock_guard<std::mutex> lk(mu);
  return all[device];
}

bool GangTurns::take(int wgs) {
  std::unique_lock<std::mutex> lk(mu_);
  const unsigned my = asked_++;
  auto mine = [&] {
    while (left_.erase(served_)) ++served_;
    return served_ == my && held_ + wgs <= kGangMaxWgs;
  };
  const bool got = cv_.wait_for(lk, std::chrono::seconds(1), mine);
  if (got) {
    held_ += wgs;
    ++served_;
  } else {
    left_.insert(my);
    while (left_.erase(served_)) ++served_;
  }
  cv_.notify_all();
  return got;
}

bool GangTurns::add(int wgs) {
  std::lock_guard<std::mutex> lk(mu_);
  if (wanted() || held_ + wgs > kGangMaxWgs) return false;
  held_ += wgs;
  return true;
}

void GangTurns::give(int wgs) {
  std::lock_guard<std::mutex> lk(mu_);
  held_ -= wgs;
  cv_.notify_all();
}

Engine::Engine(Pool* pool, hipStream_t st)
    : pool_(pool), st_(st), slots_(kMaxSys, nullptr), turns_(GangTurns::of(pool->device())) {
  ok_ = hipMalloc(&d_desc_, sizeof(SysDesc) * kMaxSys) == hipSuccess &&
        hipHostMalloc(&h_desc_, sizeof(SysDesc) * kMaxSys, hipHostMallocDefault) == hipSuccess &&
        hipMalloc(&d_y_, sizeof(double) * kYStride * kMaxSys) == hipSuccess &&
        hipHostMalloc(&h_y_, sizeof(double) * kYStride * kMaxSys, hipHostMallocDefault) == hipSuccess &&
        hipMalloc(&d_scal_, kScalBytes) == hipSuccess &&
        hipHostMalloc(&h_scal_, sizeof(Scal) * kMaxSys, hipHostMallocDefault) == hipSuccess &&
        hipHostMalloc(&h_flags_, sizeof(Scal) * kMaxSys * 4 + 256, hipHostMallocCoherent) == hipSuccess &&
        hipHostMalloc(&h_pub_, sizeof(Scal) * kMaxSys * 2 + 256, hipHostMallocCoherent) == hipSuccess &&
        hipMemsetAsync(d_scal_, 0, kScalBytes, st_) == hipSuccess;
  if (ok_) {
    std::memset(h_scal_, 0, sizeof(Scal) * kMaxSys);
    std::memset(h_pub_, 0, sizeof(Scal) * kMaxSys * 2 + 256);
    h_pub_flag_ = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(h_pub_) + sizeof(Scal) * kMaxSys * 2);
    std::memset(h_flags_, 0, sizeof(Scal) * kMaxSys * 4 + 256);
    h_blk_flag_ = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(h_flags_) + sizeof(Scal) * kMaxSys * 4);
  }
}

void Engine::set_profiling(bool on) {
  profiling_ = on;
  for (auto& a : stat)
    for (auto& b : a) b = KernelStat{};
}

Engine::~Engine() {
  (void)hipStreamSynchronize(st_);
  for (hipEvent_t e : events_) (void)hipEventDestroy(e);
  for (System* s : slots_)
    if (s) remove(s);
  end_turn();
  if (d_desc_) (void)hipFree(d_desc_);
  if (h_desc_) (void)hipHostFree(h_desc_);
  if (d_y_) (void)hipFree(d_y_);
  if (h_y_) (void)hipHostFree(h_y_);
  if (d_scal_) (void)hipFree(d_scal_);
  if (h_scal_) (void)hipHostFree(h_scal_);
  if (h_flags_) (void)hipHostFree(h_flags_);
  if (h_pub_) (void)hipHostFree(h_pub_);
}

bool Engine::idle() const {
  for (System* s : slots_)
    if (s && !s->done) return false;
  return true;
}

int Engine::count() const {
  int c = 0;
  for (System* s : slots_) c += s != nullptr;
  return c;
}

static bool is_fgmres(const hub_solve_opts& o) { return o.solver == HUB_FGMRES_MIXED; }

size_t Engine::workspace_bytes(const Geom& g, const hub_solve_opts& o) {
  const size_t n = (size_t)g.n;
  const size_t part = Pool::rounded((size_t)tile_geo(g, spt_of(g.n)).ntiles * (kMaxRed + 2) * sizeof(double));
  // vectors + the phase tables that `add` computes when the caller brings none
  // (FP64 phase n * 16; the mixed solver's float angle n * 4)
  if (!is_fgmres(o)) return 5 * Pool::rounded(n * 16) + part;
  const int m = o.restart_m;
  return (size_t)(m + 4) * Pool::rounded(n * 16) + (size_t)(m + 4) * Pool::rounded(n * 8) +
         Pool::rounded(n * 4) + part;
}

Engine::AddResult Engine::add(System* s) {
  int slot = -1;
  for (int k = 0; k < kMaxSys; ++k)
    if (!slots_[k]) {
      slot = k;
      break;
    }
  if (slot < 0) {
    set_error("engine full");
    return ADD_NO_ROOM;
  }
  const size_t n = (size_t)s->g.n;
  SysDesc& d = s->desc;
  std::memset(&d, 0, sizeof(d));
  d.g = s->g;
  d.mu2 = s->mu2;
  d.phi = s->phi;
  d.spt = spt_of(s->g.n);
  const TileGeo tg = tile_geo(s->g, d.spt);
  d.tnb = tg.nb;
  d.tbsz = tg.bsz;
  d.tseg = tg.seg;
  d.ntiles = tg.ntiles;
  d.sc = d_scal_ + slot;
  s->bytes = 0;
  auto get = [&](size_t bytes) -> void* {
    void* p = pool_->alloc(bytes, st_);
    if (p) s->owned.push_back(p);
    if (p) s->bytes += Pool::rounded(bytes);
    return p;
  };
  bool ok = true, hip_ok = true;
  d.part = (double*)get((size_t)d.ntiles * (kMaxRed + 2) * sizeof(double));
  ok = ok && d.part;
  if (ok) {
    d.part1 = d.part + (size_t)d.ntiles * kMaxRed;
    d.part2 = d.part1 + d.ntiles;
  }
  d.vec[S_B] = (void*)s->b;
  d.vec[S_X] = (void*)s->x;
  if (!is_fgmres(s->opts)) {
    for (int k : {(int)S_R, (int)S_P0, (int)S_P0 + 1, (int)S_U}) {
      d.vec[k] = get(n * 16);
      ok = ok && d.vec[k];
    }
  } else {
    const int m = s->opts.restart_m;
    for (int k : {(int)S_R, (int)S_U}) {
      d.vec[k] = get(n * 16);
      ok = ok && d.vec[k];
    }
    for (int k = 0; k <= m && ok; ++k) {
      d.vec[S_V0 + k] = get(n * 16);
      ok = ok && d.vec[S_V0 + k];
    }
    for (int k : {(int)S_R32, (int)S_P32, (int)S_P32 + 1, (int)S_U32}) {
      if (!ok) break;
      d.vec[k] = get(n * 8);
      ok = ok && d.vec[k];
    }
    for (int k = 0; k < m && ok; ++k) {
      d.vec[S_Z0 + k] = get(n * 8);
      ok = ok && d.vec[S_Z0 + k];
    }
  }
  // the phase e^{i phi} of the solver kernels (shared with other systems when the
  // caller precomputed it)
  const bool want32 = is_fgmres(s->opts);
  if (ok && (!s->ph64 || (want32 && !s->ph32))) {
    double2* p64 = (double2*)get(n * 16);
    float* p32 = want32 ? (float*)get(n * 4) : nullptr;
    ok = ok && p64 && (!want32 || p32);
    if (ok && launch_phase(s->phi, p64, p32, (int)n, st_) != hipSuccess) ok = hip_ok = false;
    if (ok) {
      s->ph64 = p64;
      s->ph32 = p32;
    }
  }
  d.ph64 = s->ph64;
  d.ph32 = s->ph32;
  if (!ok) {
    pool_->release_all(s->owned, st_);
    s->owned.clear();
    if (!hip_ok) set_error("phase launch failed");
    return hip_ok ? ADD_NO_ROOM : ADD_HIP;
  }
  s->slot = slot;
  s->phase = PH_NEW;
  s->done = s->gang = false;
  s->info = hub_solve_info{};
  slots_[slot] = s;
  upload_desc(s);
  return ADD_OK;
}

// A stream with fewer CUs than a gang launch may have workgroups (a mask, a partition of the
// device) would miss its meetings: there, only systems of one workgroup have a gang.
void Engine::look_at_device() {
  constexpr int kWords = 32;
  uint32_t mask[kWords] = {0};
  int cus = 0, masked = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, pool_->device()) != hipSuccess) cus = 0;
  if (hipExtStreamGetCUMask(st_, kWords, mask) == hipSuccess) {
    for (uint32_t m : mask) masked += __builtin_popcount(m);
    cus = std::min(cus, masked);
  } else {
    (void)hipGetLastError();
  }
  all_cus_ = cus >= kGangMaxWgs;
}

GangCut Engine::cut_of(const Geom& g, bool single) {
  const int k = single ? 1 : 0;
  int* e = cut_ext_[k];
  if (e[0] != g.L1 || e[1] != g.L2 || e[2] != g.Nt) {
    cut_[k] = single ? gang_cut<float>(g.L1, g.L2, g.Nt) : gang_cut<double>(g.L1, g.L2, g.Nt);
    e[0] = g.L1, e[1] = g.L2, e[2] = g.Nt;
  }
  return all_cus_ || cut_[k].g == 1 ? cut_[k] : GangCut{};
}

// 8-byte words of a gang's exchange memory and of its state.
static size_t exch(const GangCut& c, bool single) {
  return single ? gang_exch_words<float>(c.g, c.nslot) : gang_exch_words<double>(c.g, c.nslot);
}
static size_t state(const GangCut& c, bool single) {
  return single ? gang_state_words<float>(c.g, c.cls) : gang_state_words<double>(c.g, c.cls);
}

size_t Engine::gang_bytes(const std::vector<System*>& v) {
  look_at_device();
  size_t words = 0;
  for (System* s : v) {
    const bool single = is_fgmres(s->opts);
    const GangCut c = cut_of(s->g, single);
    if (c.g > 0) words += state(c, single) + (c.g > 1 ? exch(c, single) : 0);
  }
  return words > 0 ? Pool::rounded(words * 8) : 0;
}

hipError_t Engine::join_gangs(const std::vector<System*>& v, std::vector<void*>& owned, bool& room) {
  room = true;
  look_at_device();
  size_t words = 0, clear = 0;
  for (System* s : v) {
    const bool single = is_fgmres(s->opts);
    const GangCut c = cut_of(s->g, single);
    if (c.g > 1) clear += exch(c, single);
    if (c.g > 0) words += state(c, single);
  }
  unsigned long long* mem = nullptr;
  if (words > 0) {
    mem = (unsigned long long*)pool_->alloc((clear + words) * 8, st_);
    if (mem) {
      owned.push_back(mem);
      if (clear > 0) HUB_TRY(launch_gang_clear(mem, clear, st_));
    } else {
      set_error("");
      room = pool_->fits((clear + words) * 8);
      if (!room) return hipSuccess;
    }
  }
  unsigned long long* st = mem + clear;
  for (System* s : v) {
    const bool single = is_fgmres(s->opts);
    const GangCut c = cut_of(s->g, single);
    s->desc.gang = c;
    s->desc.gang_mem = s->desc.gang_state = nullptr;
    s->gang = c.g > 0 && mem;
    s->gang_tag = s->gang_seq = s->gang_decided = 0;
    s->gang_missed = s->gang_steps = s->gang_backoff = 0;
    if (c.g > 1 && c.g >= tight_g_) {
      s->gang_missed = kGangMisses - 1;  // one more and it is back there
      s->gang_steps = s->gang_backoff = tight_backoff_;
    }
    if (s->gang) {
      if (c.g > 1) {
        s->desc.gang_mem = mem;
        mem += exch(c, single);
      }
      s->desc.gang_state = st;
      st += state(c, single);
    }
    upload_desc(s);
  }
  return hipSuccess;
}

void Engine::remove(System* s, std::vector<void*>* owned) {
  // drain blocks that still reference the system
  for (auto& q : inflight_) {
    bool refs = false;
    for (auto& b : q)
      for (System* x : b.v) refs = refs || x == s;
    if (!refs) continue;
    // an error here surfaces again at the next synchronising call of the stream
    for (auto& b : q) (void)finish_block(b);
    q.clear();
  }
  if (inflight_[0].empty() && inflight_[1].empty()) end_turn();
  if (s->slot >= 0 && slots_[s->slot] == s) slots_[s->slot] = nullptr;
  if (owned)
    owned->insert(owned->end(), s->owned.begin(), s->owned.end());
  else
    pool_->release_all(s->owned, st_);
  s->owned.clear();
  s->slot = -1;
}

void Engine::upload_desc(System* s) {
  h_desc_[s->slot] = s->desc;
  desc_lo_ = std::min(desc_lo_, s->slot);
  desc_hi_ = std::max(desc_hi_, s->slot);
}

void Engine::upload_y(System* s, const std::vector<std::complex<double>>& y) {
  static_assert(sizeof(std::complex<double>) == 2 * sizeof(double), "complex layout");
  double* row = h_y_ + (size_t)s->slot * kYStride;
  for (size_t i = 0; i < y.size() && (int)i < kMaxRestart; ++i) {
    row[2 * i] = y[i].real();
    row[2 * i + 1] = y[i].imag();
  }
  y_lo_ = std::min(y_lo_, s->slot);
  y_hi_ = std::max(y_hi_, s->slot);
}

hipError_t Engine::flush_desc() {
  if (desc_hi_ < desc_lo_) return hipSuccess;
  const hipError_t e = hipMemcpyAsync(d_desc_ + desc_lo_, h_desc_ + desc_lo_, sizeof(SysDesc) * (desc_hi_ - desc_lo_ + 1),
                                      hipMemcpyHostToDevice, st_);
  desc_lo_ = kMaxSys;
  desc_hi_ = -1;
  return e;
}

hipError_t Engine::flush_y() {
  if (y_hi_ < y_lo_) return hipSuccess;
  const hipError_t e = hipMemcpyAsync(d_y_ + (size_t)y_lo_ * kYStride, h_y_ + (size_t)y_lo_ * kYStride,
                                      sizeof(double) * kYStride * (y_hi_ - y_lo_ + 1), hipMemcpyHostToDevice, st_);
  y_lo_ = kMaxSys;
  y_hi_ = -1;
  return e;
}

LaunchList Engine::list(const std::vector<System*>& v) const {
  LaunchList L;
  std::memset(&L, 0, sizeof(L));
  L.scal = d_scal_;
  L.nsys = (int)v.size();
  // every system of a list has the same tile class (callers group them)
  L.spt = v.empty() ? kSitesPerThread : v.front()->desc.spt;
  int acc = 0;
  for (int k = 0; k < L.nsys; ++k) {
    L.tile_begin[k] = acc;
    L.sys[k] = v[k]->slot;
    acc += v[k]->desc.ntiles;
  }
  L.tile_begin[L.nsys] = acc;
  for (int k = L.nsys + 1; k <= kMaxSys; ++k) L.tile_begin[k] = acc;
  L.total_tiles = acc;
  return L;
}

Publish Engine::publication(const std::vector<System*>& v) {
  int lo = kMaxSys, hi = -1;
  for (System* s : v) {
    lo = std::min(lo, s->slot);
    hi = std::max(hi, s->slot);
  }
  Publish pub;
  pub.d = d_scal_ + lo;
  pub.seq = ++pub_seq_;
  pub.h = h_pub_ + (size_t)(pub.seq & 1) * kMaxSys + lo;
  pub.cnt = hi - lo + 1;
  pub.flag = h_pub_flag_;
  return pub;
}

// A kernel writes the records and then a sequence number to host-coherent memory and
// the host polls the number: about half the latency of a copy plus a stream
// synchronisation.  Two publications may be under way, into buffers of their own.
// hipStreamQuery bounds the wait.  Should the stream drain without the number showing, the
// records are read through a copy where nothing was published after them; where something
// was, the device holds the later records, and that is an error.
hipError_t Engine::wait_publication(const Publish& pub) {
  const size_t lo = pub.d - d_scal_;
  for (unsigned spin = 1;; ++spin) {
    if ((int)(__atomic_load_n(h_pub_flag_, __ATOMIC_ACQUIRE) - pub.seq) >= 0) break;
    if ((spin & 255) == 0) {
      const hipError_t q = hipStreamQuery(st_);
      if (q == hipErrorNotReady) continue;
      if (q != hipSuccess) return q;
      if ((int)(__atomic_load_n(h_pub_flag_, __ATOMIC_ACQUIRE) - pub.seq) >= 0) break;
      if (pub.seq != pub_seq_) {
        set_error("results of a solver step not published");
        return hipErrorUnknown;
      }
      HUB_TRY(hipMemcpyAsync(h_scal_ + lo, pub.d, sizeof(Scal) * pub.cnt, hipMemcpyDeviceToHost, st_));
      return hipStreamSynchronize(st_);
    }
  }
  std::memcpy(h_scal_ + lo, pub.h, sizeof(Scal) * pub.cnt);
  return hipSuccess;
}

hipError_t Engine::read_scal(const std::vector<System*>& v) {
  if (v.empty()) return hipSuccess;
  const Publish pub = publication(v);
  HUB_TRY(launch_publish(pub, st_));
  return wait_publication(pub);
}

void Engine::finish(System* s, hub_status st) {
  s->status = st;
  s->phase = PH_DONE;
  s->done = true;
  s->info.converged = st == HUB_OK ? 1 : 0;
}

// No further Arnoldi step of this cycle.
static bool cycle_ends(const System* s) {
  return s->err < s->opts.tol * s->bnorm || s->wnorm == 0.0 || !std::isfinite(s->wnorm);
}

// Arnoldi step j of the systems v; `pub` is published at its end.  w stays in its slot after
// an inner solve (v_j holds the old one) and changes slots in a step that reads the old w at
// the neighbours.
hipError_t Engine::launch_arnoldi(const std::vector<System*>& v, int j, Publish& pub) {
  for (bool plain : {false, true}) {
    std::vector<System*> u;
    for (System* s : v)
      if (s->plain == plain) u.push_back(s);
    if (u.empty()) continue;
    LaunchList L = list(u);
    for (size_t q = 0; q < u.size(); ++q) {
      if (plain) u[q]->wslot = S_R + S_U - u[q]->wslot;
      L.it[q] = u[q]->wslot;
      L.pa[q] = 1.0 / u[q]->wnorm;
    }
    HUB_TRY(launch_arnoldi_dots(d_desc_, L, j, plain, st_));
  }
  LaunchList L = list(v);
  for (size_t q = 0; q < v.size(); ++q) L.it[q] = v[q]->wslot;
  pub = publication(v);
  return launch_cgs(d_desc_, L, j, pub, st_);
}

// One host-side transition for a group of systems at the same phase (and, in
// FGMRES, the same Arnoldi step): one launch per kernel over the group's systems and
// one read-back for all of them (the per-system arithmetic is that of a system alone).
hipError_t Engine::group_phase(int phase, const std::vector<System*>& g) {
  const int j = g.front()->j;
  switch (phase) {
    case PH_NEW: {
      // the group shares the solver and whether x0 is used
      const hub_solve_opts& og = g.front()->opts;
      LaunchList L = list(g);
      if (!is_fgmres(og)) {
        // FP64 CG: r = b - A x (x = 0 or x0) and the CG start
        if (!og.use_x0) {
          for (size_t q = 0; q < g.size(); ++q) {
            L.pa[q] = 0.0;
            L.pr[q] = g[q]->opts.tol * g[q]->opts.tol;
            L.pi[q] = g[q]->opts.max_iter;
          }
          HUB_TRY(launch_cg_init_zero(d_desc_, L, RED_CG_SETUP, Publish{}, st_));
        } else {
          for (size_t q = 0; q < g.size(); ++q) {
            L.pa[q] = g[q]->opts.tol * g[q]->opts.tol;
            L.pr[q] = 0.0;
            L.pi[q] = g[q]->opts.max_iter;
            g[q]->info.applies++;
          }
          HUB_TRY(launch_normal_slot(d_desc_, L, S_X, S_B, S_R, RED_CG_SETUP, 1, true, Publish{}, st_));
        }
        for (System* s : g) {
          s->enq = 0;
          s->gen++;
          s->phase = PH_CG_ITER;
        }
        return hipSuccess;
      }
      // FGMRES: r = b (or b - A x0), |b|
      const Publish pub = publication(g);
      if (!og.use_x0)
        HUB_TRY(launch_cg_init_zero(d_desc_, L, RED_STORE, pub, st_));
      else
        HUB_TRY(launch_normal_slot(d_desc_, L, S_X, S_B, S_R, RED_STORE, 1, true, pub, st_));
      HUB_TRY(wait_publication(pub));
      std::vector<System*> run, zero;
      for (System* s : g) {
        const Scal& sc = h_scal_[s->slot];
        s->bb = sc.red[0];
        s->err = og.use_x0 ? std::sqrt(sc.red[1]) : std::sqrt(s->bb);
        if (og.use_x0) s->info.applies++;
        s->bnorm = std::sqrt(s->bb);
        if (!std::isfinite(s->bb) || !std::isfinite(s->err)) {
          // phi, b or the initial guess holds a non-finite value
          finish(s, HUB_ERR_ARG);
        } else if (s->bnorm == 0.0) {
          zero.push_back(s);
        } else if (s->err <= s->opts.tol * s->bnorm) {
          s->info.true_rel_resid = s->err / s->bnorm;
          finish(s, HUB_OK);
        } else {
          run.push_back(s);
        }
      }
      if (!zero.empty()) {
        // b = 0: x = 0 exactly
        HUB_TRY(launch_cg_init_zero(d_desc_, list(zero), RED_STORE, Publish{}, st_));
        for (System* s : zero) {
          s->info.true_rel_resid = 0.0;
          finish(s, HUB_OK);
        }
      }
      if (run.empty()) return hipSuccess;
      // initial single-precision solve on r (Algorithm A.1, first line)
      LaunchList R = list(run);
      for (size_t q = 0; q < run.size(); ++q) {
        const System* s = run[q];
        const hub_solve_opts& o = s->opts;
        const double tau = std::max(std::min(o.tol * o.inner_a * s->bnorm / s->err, 1.0), o.inner_floor);
        R.pa[q] = 1.0;
        R.pr[q] = tau * tau;
        R.pi[q] = o.inner_max_iter;
        R.pj[q] = S_Z0;
        R.it[q] = S_R;
      }
      HUB_TRY(launch_prep_inner(d_desc_, R, -1, st_));
      for (System* s : run) {
        s->enq = 0;
        s->gen++;
        s->phase = PH_F_INNER;
        s->post = PH_F_POST_INIT;
      }
      return hipSuccess;
    }
    case PH_CG_CONFIRM: {
      // FP64 true residual of the CG iterate; restart the CG from x if it misses tol.
      // |b|^2 comes from the CG start, whose reduction is NaN when phi or b holds a
      // non-finite value: such systems stop here.
      std::vector<System*> ok;
      for (System* s : g) {
        if (!std::isfinite(s->bb))
          finish(s, HUB_ERR_ARG);
        else
          ok.push_back(s);
      }
      if (ok.empty()) return hipSuccess;
      return confirm(ok);
    }
    case PH_LOST: {
      for (System* s : g) finish(s, HUB_ERR_HIP);
      return hipSuccess;
    }
    case PH_F_POST_INIT: {
      // x = z_0 (or x0 + z_0), r = b - A x, ERR = |r|
      for (System* s : g) upload_y(s, {std::complex<double>(1.0, 0.0)});
      HUB_TRY(flush_y());
      const LaunchList L = list(g);
      HUB_TRY(launch_xupdate(d_desc_, L, d_y_, 1, !g.front()->opts.use_x0, st_));
      const Publish pub = publication(g);
      HUB_TRY(launch_normal_slot(d_desc_, L, S_X, S_B, S_R, RED_STORE, 0, false, pub, st_));
      HUB_TRY(wait_publication(pub));
      for (System* s : g) {
        const hub_solve_opts& o = s->opts;
        s->info.applies++;
        s->err = std::sqrt(h_scal_[s->slot].red[0]);
        s->info.true_rel_resid = s->err / s->bnorm;
        if (s->err <= o.tol * s->bnorm) {
          finish(s, HUB_OK);
          continue;
        }
        s->j = 0;
        s->wslot = S_R;
        s->rate = 1.0;
        s->wnorm = s->err;
        s->rnorm_cycle = s->err;
        s->H.assign((size_t)(o.restart_m + 1) * o.restart_m, std::complex<double>(0.0));
        s->phase = PH_F_ARNOLDI;
      }
      return hipSuccess;
    }
    case PH_F_ARNOLDI: {
      // v_j = w / |w|; z_j from the single-precision CG when TOL a |b| / ERR < 1, else z_j = v_j
      std::vector<System*> act;
      for (System* s : g) {
        if (cycle_ends(s))
          s->phase = PH_F_LSQ;
        else
          act.push_back(s);
      }
      if (act.empty()) return hipSuccess;
      // without an inner solve the step itself makes v_j and z_j (k_arnoldi_dots)
      std::vector<System*> inner;
      std::vector<double> tau;
      for (System* s : act) {
        const hub_solve_opts& o = s->opts;
        const double ratio = o.tol * o.inner_a * s->bnorm / s->err;
        s->plain = !(ratio < 1.0) || o.inner_max_iter < 1;
        if (s->plain) {
          s->phase = PH_F_POST_ARNOLDI;
          continue;
        }
        inner.push_back(s);
        tau.push_back(std::max(ratio, o.inner_floor));
      }
      if (inner.empty()) return hipSuccess;
      LaunchList L = list(inner);
      for (size_t q = 0; q < inner.size(); ++q) {
        System* s = inner[q];
        L.pa[q] = 1.0 / s->wnorm;
        L.pj[q] = S_Z0 + j;
        L.it[q] = s->wslot;
        L.pr[q] = tau[q] * tau[q];
        L.pi[q] = s->opts.inner_max_iter;
        s->enq = 0;
        s->gen++;
        s->phase = PH_F_INNER;
        s->post = PH_F_POST_ARNOLDI;
      }
      return launch_prep_inner(d_desc_, L, S_V0 + j, st_);
    }
    case PH_F_POST_ARNOLDI: {
      // w = A z_j, classical Gram-Schmidt against v_0 .. v_j, h_{j+1,j} = |w|, ERR *= |w|.
      // Steps without an inner solve follow each other on the device: the next one is
      // enqueued before the host has this one's result.  It is in vain when this one
      // converges (its vectors lie past those that the update reads), so it is not enqueued
      // where the last reduction of ERR suggests that.  (25x23x30 1356 -> 1301 us, a
      // Hasenbusch force at 24x24x64 7.08 -> 6.84 ms.)
      std::vector<System*> v = g;
      Publish pub, next;
      HUB_TRY(launch_arnoldi(v, j, pub));
      for (int i = j;; ++i) {
        bool ahead = i + 1 < v.front()->opts.restart_m;
        for (System* s : v)
          ahead = ahead && s->plain && i + 1 < s->opts.restart_m && s->err * s->rate >= s->opts.tol * s->bnorm;
        if (ahead) HUB_TRY(launch_arnoldi(v, i + 1, next));
        HUB_TRY(wait_publication(pub));
        std::vector<System*> on;
        for (System* s : v) {
          const int m = s->opts.restart_m;
          s->info.applies++;
          const Scal& sc = h_scal_[s->slot];
          for (int k = 0; k <= i; ++k) s->H[(size_t)i * (m + 1) + k] = {sc.red[2 * k], sc.red[2 * k + 1]};
          const double hn = std::sqrt(std::max(sc.red[2 * (i + 1)], 0.0));
          s->H[(size_t)i * (m + 1) + i + 1] = hn;
          s->wnorm = hn;
          // ERR: the residual of the best iterate of the cycle so far, the least-squares
          // residual of the Arnoldi relation (Algorithm A.1's ERR * |w| is this quantity
          // while every step's inner solve meets its tolerance, and not after an
          // unpreconditioned step, where it ends cycles that have not converged)
          double res = s->err;
          (void)hessenberg_lsq(s->H, m + 1, i + 1, s->rnorm_cycle, &res);
          s->rate = s->plain && s->err > 0.0 ? res / s->err : 1.0;
          s->err = res;
          s->j = i + 1;
          s->phase = (s->j == m) ? PH_F_LSQ : PH_F_ARNOLDI;
          if (ahead && !cycle_ends(s)) on.push_back(s);
        }
        if (on.empty()) return hipSuccess;
        v = on;
        pub = next;
      }
    }
    case PH_F_LSQ: {
      // y = argmin |(|r|, 0, ..) - H y|, x += sum y_i z_i, true residual, restart or stop
      const int k = j;
      const LaunchList L = list(g);
      if (k > 0) {
        for (System* s : g) upload_y(s, hessenberg_lsq(s->H, s->opts.restart_m + 1, k, s->rnorm_cycle));
        HUB_TRY(flush_y());
        HUB_TRY(launch_xupdate(d_desc_, L, d_y_, k, false, st_));
      }
      const Publish pub = publication(g);
      HUB_TRY(launch_normal_slot(d_desc_, L, S_X, S_B, S_R, RED_STORE, 0, false, pub, st_));
      HUB_TRY(wait_publication(pub));
      for (System* s : g) {
        const hub_solve_opts& o = s->opts;
        s->info.applies++;
        s->cycles++;
        s->info.outer_iters = s->cycles;
        s->err = std::sqrt(h_scal_[s->slot].red[0]);
        s->info.true_rel_resid = s->err / s->bnorm;
        if (s->err <= o.tol * s->bnorm) {
          finish(s, HUB_OK);
        } else if (s->cycles >= o.max_iter || !std::isfinite(s->err) || k == 0) {
          finish(s, HUB_ERR_NOCONV);
        } else {
          s->j = 0;
          s->wslot = S_R;
          s->rate = 1.0;
          s->wnorm = s->err;
          s->rnorm_cycle = s->err;
          std::fill(s->H.begin(), s->H.end(), std::complex<double>(0.0));
          s->phase = PH_F_ARNOLDI;
        }
      }
      return hipSuccess;
    }
    default:
      return hipSuccess;
  }
}

// FP64 true residual of the CG iterates of g (finite |b|^2); restart a CG from x where it
// misses tol, or stop the system.
hipError_t Engine::confirm(const std::vector<System*>& g) {
  LaunchList L = list(g);
  for (size_t q = 0; q < g.size(); ++q) {
    const System* s = g[q];
    L.pa[q] = s->opts.tol * s->opts.tol * s->bb;
    L.pr[q] = 0.0;
    L.pi[q] = std::max(1, s->opts.max_iter - s->cg_total);
  }
  const Publish pub = publication(g);
  HUB_TRY(launch_normal_slot(d_desc_, L, S_X, S_B, S_R, RED_CG_SETUP, 1, false, pub, st_));
  HUB_TRY(wait_publication(pub));
  for (System* s : g) {
    const hub_solve_opts& o = s->opts;
    s->info.applies++;
    const double rr = h_scal_[s->slot].red[1];
    s->info.true_rel_resid = s->bb > 0 ? std::sqrt(rr / s->bb) : 0.0;
    if (s->info.true_rel_resid <= o.tol) {
      finish(s, HUB_OK);
    } else if (!std::isfinite(rr) && s->cg_total == 0) {
      // r = b - A x0 is not finite before any iteration: phi or x0 is not finite
      finish(s, HUB_ERR_ARG);
    } else if (s->cg_total >= o.max_iter || !std::isfinite(rr)) {
      finish(s, HUB_ERR_NOCONV);
    } else {
      s->info.outer_iters++;
      s->enq = 0;
      s->gen++;
      s->phase = PH_CG_ITER;
    }
  }
  return hipSuccess;
}

hipError_t Engine::take_event(std::vector<hipEvent_t>& dst) {
  if (events_.empty()) {
    hipEvent_t ev;
    HUB_TRY(hipEventCreate(&ev));
    events_.push_back(ev);
  }
  dst.push_back(events_.back());
  events_.pop_back();
  return hipSuccess;
}

// System s joins the launch G, of whose blocks `taken` are given away per XCD; false: no room.
// Blocks go to the XCDs in turn (block b to XCD b mod 8), so a gang takes its blocks with a
// stride, consecutive workgroups on one XCD: a reduction among 16 workgroups by itself takes
// 2.0 us on one XCD and 2.45 us over all.  More than about a dozen of one gang on an XCD get
// into each other's way (the FP64 iteration of a 48x48x64 system cut in some 140 blocks 8.1 us
// with 28 on each of five XCDs, 7.0 us with 18 on each of eight).
bool Engine::gang_entry(GangList& G, int (&taken)[kNumXcd], System* s, bool single) const {
  constexpr int kPer = kGangMaxWgs / kNumXcd;  // blocks per XCD
  constexpr int kSpread = 12;                  // workgroups of a gang per XCD, while others are free
  if (G.nsys == 0) std::memset(G.list, kGangNone, sizeof(G.list));
  int room[kNumXcd], total = 0;
  for (int x = 0; x < kNumXcd; ++x) total += room[x] = kPer - taken[x];
  const int g = s->desc.gang.g;
  if (g > total || G.nsys == kMaxSys) return false;
  // the XCDs with the most room, an even share on each
  int order[kNumXcd];
  for (int x = 0; x < kNumXcd; ++x) order[x] = x;
  std::stable_sort(order, order + kNumXcd, [&](int a, int b) { return room[a] > room[b]; });
  int nx = 0, sum = 0;
  while (nx < kNumXcd && (sum < g || nx * kSpread < g)) sum += room[order[nx++]];
  int left = g, wg = 0;
  for (int k = 0; k < nx; ++k) {
    const int x = order[k];
    int later = 0;
    for (int q = k + 1; q < nx; ++q) later += room[order[q]];
    int n = std::max(std::min((left + nx - k - 1) / (nx - k), room[x]), left - later);
    left -= n;
    for (; n > 0; --n) {
      const int b = x + kNumXcd * taken[x]++;
      G.list[b] = (unsigned char)G.nsys;
      G.wg[b] = (unsigned char)wg++;
      G.nblock = std::max(G.nblock, b + 1);
    }
  }
  static_assert(kPer * kNumXcd == kGangMaxWgs && kGangMaxWgs <= 256 && kMaxSys < kGangNone, "block table");
  G.scal = d_scal_;
  G.sys[G.nsys] = s->slot;
  G.pi[G.nsys] = single ? S_Z0 + s->j : S_X;
  G.tag[G.nsys] = s->gang_tag;
  G.seq[G.nsys] = s->gang_seq + 1;
  ++G.nsys;
  return true;
}

// Gang launches over the systems of v, as many systems to a launch as the device has CUs
// for: every workgroup of a launch has to be on the device for its gang to meet.  Systems
// whose gang keeps missing its meetings come first, in steps, which need no meeting.  The
// others go by their shift, so that those of a launch stop at about the same time: its CUs
// are taken until the last one does.  (64 systems of 11x88x22 with four shifts in any order,
// FP64: 28.8 ms as they come, 20.2 ms by shift, 24.7 ms with the tiled kernels.)
hipError_t Engine::launch_gangs(const std::vector<System*>& v, bool single, Block& b) {
  std::vector<System*> meet, step;
  for (System* s : v) (s->gang_steps > 0 ? step : meet).push_back(s);
  std::stable_sort(meet.begin(), meet.end(), [](const System* a, const System* b) { return a->mu2 < b->mu2; });
  for (int steps = 1; steps >= 0; --steps) {
    const std::vector<System*>& w = steps ? step : meet;
    for (size_t q = 0; q < w.size();) {
      GangList G;
      std::memset(&G, 0, sizeof(G));
      int taken[kNumXcd] = {0};
      for (; q < w.size(); ++q)
        if (!gang_entry(G, taken, w[q], single)) break;
      const int iters = steps ? kGangSteps : G.nsys == 1 ? kGangItersAlone : kGangIters;
      for (size_t k = q - G.nsys; k < q; ++k) {
        w[k]->gang_tag += iters + 2;  // a launch uses two tags before its iterations'
        w[k]->enq += iters;
        if (steps)
          --w[k]->gang_steps;
        else
          ++w[k]->gang_seq;
      }
      if (steps) {
        HUB_TRY(launch_gang_steps(d_desc_, G, iters, single, st_));
        continue;
      }
      G.deny = (int)(deny_ >> (gang_launches_++ & 31) & 1);
      hipEvent_t e0 = nullptr, e1 = nullptr;
      if (profiling_) {
        HUB_TRY(take_event(b.gev));
        HUB_TRY(take_event(b.gev));
        e0 = b.gev[b.gev.size() - 2];
        e1 = b.gev.back();
      }
      HUB_TRY(launch_gang(d_desc_, G, iters, single, st_, e0, e1));
    }
  }
  return hipSuccess;
}

void Engine::end_turn() {
  if (turn_ > 0) turns_.give(turn_);
  turn_ = 0;
}

// Before gangs are launched in the given precision: the turn for them.  One that is held goes
// on, unless it is too small now or another engine waits; then what is in flight is read back
// first.
hipError_t Engine::begin_turn(bool single) {
  auto need = [&] {
    int wgs = 0;
    for (System* s : slots_)
      if (s && !s->done && s->gang && s->gang_steps == 0 && s->phase == (single ? (int)PH_F_INNER : (int)PH_CG_ITER))
        wgs += s->desc.gang.g > 1 ? s->desc.gang.g : 0;
    return std::min(wgs, kGangMaxWgs);
  };
  int wgs = need();
  if (wgs == 0) return hipSuccess;
  if (turn_ > 0 && turn_ < wgs && turns_.add(wgs - turn_)) turn_ = wgs;
  if (turn_ > 0 && (turn_ < wgs || turns_.wanted())) {
    for (auto& q : inflight_) {
      for (auto& b : q) HUB_TRY(finish_block(b));
      q.clear();
    }
    end_turn();
    wgs = need();
  }
  if (turn_ == 0 && wgs > 0 && turns_.take(wgs)) turn_ = wgs;
  return hipSuccess;
}

// Enqueue one block of CG iterations over every system that is iterating in the
// given precision, followed by an asynchronous read-back of their flags.
hipError_t Engine::launch_block(bool single, bool& launched) {
  launched = false;
  HUB_TRY(begin_turn(single));
  std::vector<System*> v, gangs;
  int k = 1 << 30;
  for (System* s : slots_) {
    if (!s || s->done) continue;
    if ((single && s->phase == PH_F_INNER) || (!single && s->phase == PH_CG_ITER)) {
      if (s->gang) {
        gangs.push_back(s);
        continue;
      }
      v.push_back(s);
      int ks = std::max(1, s->opts.check_every);
      // near the iteration count of the system's previous CG run, enqueue short
      // blocks: launches after convergence return at once but still cost a launch
      if (s->pred > 0 && s->enq + ks > s->pred - kTailBlock) ks = std::min(ks, kTailBlock);
      k = std::min(k, ks);
    }
  }
  if (v.empty() && gangs.empty()) return hipSuccess;
  if (v.empty()) k = 0;
  // tiled systems by the tile size of their CG stages: one launch per size class
  std::vector<System*> ordered;
  std::vector<int> cls_spt, cls_end;
  for (int spt : {(int)kSitesPerThread, (int)kSmallSpt}) {
    for (System* s : v)
      if (s->desc.spt == spt) ordered.push_back(s);
    if (!ordered.empty() && (cls_end.empty() || (int)ordered.size() > cls_end.back())) {
      cls_spt.push_back(spt);
      cls_end.push_back((int)ordered.size());
    }
    if (kSmallSpt == kSitesPerThread) break;
  }
  const int ntile = (int)ordered.size();
  v = ordered;
  const int ncls = (int)cls_spt.size();
  Block b;
  b.single = single;
  b.k = k;
  b.v = v;
  b.v.insert(b.v.end(), gangs.begin(), gangs.end());
  b.cls_end = cls_end;
  for (System* s : b.v) b.gen.push_back(s->gen);
  b.buf = next_buf_[single ? 1 : 0];
  next_buf_[single ? 1 : 0] ^= 1;
  std::vector<LaunchList> Ls;
  for (int c = 0; c < ncls; ++c) {
    const int q0 = c == 0 ? 0 : cls_end[c - 1];
    std::vector<System*> vc(v.begin() + q0, v.begin() + cls_end[c]);
    LaunchList L = list(vc);
    // The solution slot of the initial single-precision solve is S_Z0 (j = 0 then).
    for (size_t q = 0; q < vc.size(); ++q) L.pi[q] = single ? S_Z0 + vc[q]->j : S_X;
    Ls.push_back(L);
  }
  if (profiling_)
    for (int e = 0; e < 4 * k * ncls; ++e) HUB_TRY(take_event(b.kev));
  HUB_TRY(launch_gangs(gangs, single, b));
  for (System* s : b.v) b.gang_seq.push_back(s->gang_seq);
  for (int it = 0; it < k && ntile > 0; ++it) {
    std::vector<int> its(ntile);
    for (int q = 0; q < ntile; ++q) its[q] = v[q]->enq++;
    for (int c = 0; c < ncls; ++c) {
      const int q0 = c == 0 ? 0 : cls_end[c - 1];
      for (int q = q0; q < cls_end[c]; ++q) Ls[c].it[q - q0] = its[q];
    }
    if (!profiling_) {
      for (int c = 0; c < ncls; ++c) HUB_TRY(launch_cg_iter(d_desc_, Ls[c], single, st_));
      continue;
    }
    b.its.push_back(its);
    for (int stage = 1; stage <= 2; ++stage)
      for (int c = 0; c < ncls; ++c) {
        const int e = 4 * (it * ncls + c) + 2 * (stage - 1);
        HUB_TRY(launch_cg_stage(d_desc_, Ls[c], single, stage, st_, b.kev[e], b.kev[e + 1]));
      }
  }
  int lo = kMaxSys, hi = -1;
  for (System* s : b.v) {
    lo = std::min(lo, s->slot);
    hi = std::max(hi, s->slot);
  }
  // The block's flags go to host-coherent memory through a kernel that then writes the
  // block's sequence number (k_publish): unlike a device-to-host copy followed by an
  // event, it adds no barrier packet, so the next block's kernels follow at once.
  Scal* dst = h_flags_ + (size_t)((single ? 2 : 0) + b.buf) * kMaxSys;
  b.seq = ++blk_seq_;
  Publish pub;
  pub.d = d_scal_ + lo;
  pub.h = dst + lo;
  pub.cnt = hi - lo + 1;
  pub.seq = b.seq;
  pub.flag = h_blk_flag_;
  HUB_TRY(launch_publish(pub, st_));
  inflight_[single ? 1 : 0].push_back(std::move(b));
  launched = true;
  return hipSuccess;
}

// Wait until the flags of the block with sequence number seq are in host memory.  Blocks
// publish in stream order, so a later number showing implies this block's records.  The
// spin checks the stream every so often: an error ends it, and a drained stream without
// the number (which a completed publish kernel rules out) is reported as an error.
hipError_t Engine::wait_block(unsigned seq) {
  for (unsigned spin = 1;; ++spin) {
    if ((int)(__atomic_load_n(h_blk_flag_, __ATOMIC_ACQUIRE) - seq) >= 0) return hipSuccess;
    if ((spin & 255) == 0) {
      const hipError_t q = hipStreamQuery(st_);
      if (q == hipErrorNotReady) continue;
      if (q != hipSuccess) return q;
      if ((int)(__atomic_load_n(h_blk_flag_, __ATOMIC_ACQUIRE) - seq) >= 0) return hipSuccess;
      set_error("CG block flags not published");
      return hipErrorUnknown;
    }
  }
}

// Wait for a block's flags and move the systems that stopped iterating on.
hipError_t Engine::finish_block(Block& b) {
  HUB_TRY(wait_block(b.seq));
  const bool single = b.single;
  const Scal* flags = h_flags_ + (size_t)((single ? 2 : 0) + b.buf) * kMaxSys;
  if (profiling_ && !b.kev.empty()) {
    // A system did work in the launch of iteration `it` iff it < its final count
    // (or it is still iterating).
    const int ncls = (int)b.cls_end.size();
    for (int it = 0; it < b.k; ++it) {
      for (int c = 0; c < ncls; ++c) {
        const int q0 = c == 0 ? 0 : b.cls_end[c - 1];
        for (int stage = 0; stage < 2; ++stage) {
          double bytes = 0.0;
          for (int q = q0; q < b.cls_end[c]; ++q) {
            const Scal& sc = flags[b.v[q]->slot];
            const int its = b.its[it][q];
            if (sc.active || its < sc.iters) bytes += (double)b.v[q]->g.n * cg_bytes(single, stage + 1, its);
          }
          const int e = 4 * (it * ncls + c) + 2 * stage;
          float ms = 0.0f;
          HUB_TRY(hipEventElapsedTime(&ms, b.kev[e], b.kev[e + 1]));
          KernelStat& ks = stat[single ? 1 : 0][stage];
          ks.launches++;
          ks.ms += ms;
          ks.bytes += bytes;
        }
      }
    }
  }
  for (size_t e = 0; e + 1 < b.gev.size(); e += 2) {
    float ms = 0.0f;
    HUB_TRY(hipEventSynchronize(b.gev[e + 1]));
    HUB_TRY(hipEventElapsedTime(&ms, b.gev[e], b.gev[e + 1]));
    KernelStat& ks = stat[single ? 1 : 0][2];
    ks.launches++;
    ks.ms += ms;
  }
  for (hipEvent_t e : b.kev) events_.push_back(e);
  for (hipEvent_t e : b.gev) events_.push_back(e);
  b.kev.clear();
  b.gev.clear();
  for (size_t q = 0; q < b.v.size(); ++q) {
    System* s = b.v[q];
    const bool want = single ? (s->phase == PH_F_INNER) : (s->phase == PH_CG_ITER);
    // skip a system that an earlier block already moved on (its flags here
    // belong to a finished CG run)
    if (s->done || !want || s->gen != b.gen[q]) continue;
    const Scal& sc = flags[s->slot];
    if (s->gang) {
      if (sc.gang == 2) {
        // its iterate is not whole; the systems beside it have exchanged nothing with it
        s->phase = PH_LOST;
        continue;
      }
      const int g = s->desc.gang.g;
      if (sc.gang == 1 || sc.gang == 3) {
        // (a launch that was on its way when steps were decided on counts for nothing)
        if (b.gang_seq[q] > s->gang_decided && ++s->gang_missed >= kGangMisses) {
          s->gang_decided = s->gang_seq;
          s->gang_steps = s->gang_backoff = std::min(std::max(1, 2 * s->gang_backoff), kGangStepBlocks);
          tight_g_ = std::min(tight_g_, g);
          tight_backoff_ = s->gang_backoff;
        }
      } else if (sc.gang == 0 && g > 1) {
        s->gang_missed = s->gang_backoff = 0;
        if (g >= tight_g_) tight_g_ = kGangMaxWgs + 1;
      }
    }
    if (sc.active) continue;
    s->pred = sc.iters;
    if (single) {
      s->info.inner_iters += sc.iters;
      s->phase = s->post;
    } else {
      s->cg_total += sc.iters;
      s->info.inner_iters = s->cg_total;
      if (s->bb < 0) s->bb = sc.red[0];
      s->phase = PH_CG_CONFIRM;
    }
  }
  return hipSuccess;
}

hipError_t Engine::advance() {
  // 0. descriptors of systems added since the last step
  HUB_TRY(flush_desc());
  // 1. keep the GPU busy: enqueue the next block for every system still iterating
  //    (speculatively: a system that converged in the block still in flight runs
  //    empty launches, which return at once)
  bool launched[2] = {false, false};
  HUB_TRY(launch_block(false, launched[0]));
  HUB_TRY(launch_block(true, launched[1]));
  // 2. read back older blocks: keep one in flight while that precision iterates
  for (int k = 0; k < 2; ++k) {
    auto& q = inflight_[k];
    const size_t keep = launched[k] ? 1 : 0;
    while (q.size() > keep) {
      HUB_TRY(finish_block(q.front()));
      q.erase(q.begin());
    }
  }
  // 3. host-side phases of the systems that are not iterating, in groups of systems
  //    at the same phase (and Arnoldi step)
  bool progressed = true;
  while (progressed) {
    progressed = false;
    for (int ph : {(int)PH_LOST, (int)PH_NEW, (int)PH_CG_CONFIRM, (int)PH_F_POST_INIT, (int)PH_F_LSQ, (int)PH_F_POST_ARNOLDI,
                   (int)PH_F_ARNOLDI}) {
      // key: Arnoldi step, solver, whether x0 is used (the start's and the first
      // update's kernels depend on them) and tile class (one per launch)
      std::map<int, std::vector<System*>> groups;
      for (System* s : slots_)
        if (s && !s->done && s->phase == ph)
          groups[8 * s->j + (s->desc.spt == kSmallSpt ? 4 : 0) + (is_fgmres(s->opts) ? 2 : 0) +
                 (s->opts.use_x0 ? 1 : 0)]
              .push_back(s);
      for (auto& kv : groups) {
        HUB_TRY(group_phase(ph, kv.second));
        progressed = true;
        for (System* s : kv.second)
          if (s->done && s->on_done) s->on_done(s);
      }
    }
    bool all_wait = true;
    for (System* s : slots_)
      if (s && !s->done && s->phase != PH_F_INNER && s->phase != PH_CG_ITER) all_wait = false;
    if (all_wait) break;
  }
  return hipSuccess;
}

}  // namespace hub

namespace hub {

hipError_t Engine::finalize(System* s, const double2* chi, double* dSdphi, double* S) {
  const Geom& g = s->g;
  double2* xi = (double2*)s->desc.vec[S_U];
  HUB_TRY(launch_dot_re(g, chi, s->x, 1, s->desc.part, &d_scal_[s->slot].red[kMaxRed - 1], st_));
  if (dSdphi) {
    HUB_TRY(launch_apply(g, s->phi, s->x, xi, 1, true, st_));
    HUB_TRY(launch_force(g, s->phi, s->x, xi, 1.0, 0, dSdphi, 1, st_));
  }
  HUB_TRY(read_scal({s}));
  *S = h_scal_[s->slot].red[kMaxRed - 1];
  return hipSuccess;
}

}  // namespace hub
