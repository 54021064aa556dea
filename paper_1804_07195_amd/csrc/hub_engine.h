// Host side of libhub: workspace pool and the batched solver engine.
#pragma once

#include <atomic>
#include <complex>
#include <condition_variable>
#include <cstdint>
#include <deque>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <unordered_map>
#include <vector>

#include "hub.h"
#include "hub_internal.h"

namespace hub {

// Thread-local error message behind hub_last_error().
void set_error(const std::string& msg);
const char* get_error();

// Stream-ordered caching allocator of device memory, bounded by a byte budget.
// A freed block is reused by the same stream at once and by other streams once
// the work enqueued before its release has finished.
class Pool {
 public:
  Pool(int device, size_t budget);
  ~Pool();
  // Returns nullptr (and sets the error) when the budget would be exceeded.
  void* alloc(size_t bytes, hipStream_t st);
  void release(void* p, hipStream_t st);
  // Release several blocks after the same stream work: one event orders all of them.
  void release_all(const std::vector<void*>& ps, hipStream_t st);
  size_t budget() const { return budget_; }
  int device() const { return device_; }
  size_t in_use() const;
  bool fits(size_t bytes) const;  // within the budget, now
  // Served requests that hold workspace or are about to, and synchronous calls that wait for
  // them to give it back; no request is admitted while one waits.
  std::atomic<int> requests{0}, waiting{0};
  size_t reserved() const;
  // Bytes a request of this size takes from the budget (granularity rounding).
  static size_t rounded(size_t bytes);

 private:
  // An event recorded after the work that used a group of released blocks, destroyed
  // when the last block of the group is handed out again or freed.
  struct SharedEvent {
    hipEvent_t ev = nullptr;
    int refs = 0;
  };
  struct Block {
    void* p;
    size_t bytes;
    hipStream_t st;
    SharedEvent* ev;
  };
  void drop_event(SharedEvent* e, bool wait);
  int device_;
  size_t budget_;
  size_t reserved_ = 0;  // bytes obtained from hipMalloc
  size_t used_ = 0;      // bytes handed out
  // by size and by address: a solve of 64 systems takes and gives back some 350 blocks.
  // Searching lists, one event per system and counting the free blocks of a gang launch
  // anew for each system took 0.3 ms of such a solve (32 chains of 2x1x64 through a
  // trajectory of 18 solves: 14.4 -> 8.9 ms).
  std::map<size_t, std::deque<Block>> free_;
  std::unordered_map<void*, size_t> live_;
  mutable std::mutex mu_;
};

// The workgroups of gangs that the engines of this process may have on one device at a time,
// handed out in the order of asking.  An engine holds its share from before a block of gang
// launches to the last of them that was read back; while another one waits it launches none
// ahead and asks anew for each block.  (Left to the refusals on the device, a gang of all
// CUs gets in only where a launch of another context happens not to follow the last one.)
class GangTurns {
 public:
  static GangTurns& of(int device);
  // False after a second: whoever holds the others has other troubles, the device decides.
  bool take(int wgs);
  void give(int wgs);
  // So many beside those held, if nobody waits and they are free.
  bool add(int wgs);
  bool wanted() const { return asked_.load() != served_.load(); }

 private:
  std::mutex mu_;
  std::condition_variable cv_;
  int held_ = 0;
  std::atomic<unsigned> asked_{0}, served_{0};
  std::set<unsigned> left_;  // askers that gave up before their turn
};

// Block length (CG iterations between flag reads) near a system's expected end.
constexpr int kTailBlock = 4;
// Iterations of a gang launch (a gang leaves its launch at convergence), and of one that holds
// a single system.  The launches of a stream follow one another, so a system that has stopped
// waits for the rest of its launch and for the other launches of the engine, two blocks of
// them where one is ahead; a launch costs 12 us (6x6x16) to 32 us (102x102x64) before its
// first iteration.  With 128 for every launch of the server, a request of 6x6x16 that comes
// while another one runs took 3.54 ms instead of 3.77 beside 24x24x64 (mixed; FP64 3.32 and
// 4.01), 12.6 instead of 12.3 beside three of 48x48x64 and 9.5 in both beside 102x102x64,
// and the requests together 2 to 3% longer.
constexpr int kGangIters = 128, kGangItersAlone = 512;
// Meetings in a row that a gang may miss (or be refused) before it goes on in steps; and how:
// blocks of so many iterations (half a millisecond; an attempt takes 2 ms to fail), one of
// them before the next attempt to meet, twice as many after each attempt that fails, up to
// kGangStepBlocks.
constexpr int kGangMisses = 3, kGangSteps = 16, kGangStepBlocks = 64;

// Host-side state of one linear system (M M^dagger + mu2) x = b.
struct System {
  // inputs
  Geom g;
  double mu2 = 0.0;
  const double* phi = nullptr;
  const double2* ph64 = nullptr;  // (cos phi, sin phi); computed on add if NULL
  const float* ph32 = nullptr;    // reduced float phi (mixed solver); computed on add if NULL
  const double2* b = nullptr;
  double2* x = nullptr;
  hub_solve_opts opts{};
  // outputs
  hub_solve_info info{};
  hub_status status = HUB_OK;
  bool done = false;
  // engine bookkeeping
  int slot = -1;
  int phase = 0;
  int post = 0;         // what follows the running single-precision CG
  int j = 0;            // Arnoldi step
  int wslot = 0;        // the slot of S_R, S_U that holds the residual or the Arnoldi vector w
  bool plain = false;   // the Arnoldi step runs without an inner solve
  double rate = 1.0;    // what the last such step left of ERR
  int cycles = 0;
  int cg_total = 0;     // FP64 CG iterations over all restarts
  int enq = 0;          // CG iterations enqueued since the last CG setup
  int gen = 0;          // number of CG setups so far (tags in-flight blocks)
  int pred = 0;         // iterations of the system's previous CG run (0: none yet)
  bool gang = false;    // CG iterations by a gang of workgroups (desc.gang, desc.gang_mem)
  unsigned gang_tag = 0, gang_seq = 0;  // exchange tags handed out, launches so far
  int gang_missed = 0;  // meetings missed in a row
  int gang_steps = 0;   // blocks in steps before the gang tries to meet again
  int gang_backoff = 0; // of them after the last attempts failed
  unsigned gang_decided = 0;  // launches made when that was decided
  double bnorm = 0.0, err = 0.0, wnorm = 0.0, rnorm_cycle = 0.0, bb = -1.0;
  std::vector<std::complex<double>> H;  // (m+1) x m, column-major
  std::vector<void*> owned;             // workspace blocks of this system
  size_t bytes = 0;                     // what they take of the budget
  SysDesc desc{};
  std::function<void(System*)> on_done; // serving: S, force and completion
  void* user = nullptr;
};

// Drives any number (<= kMaxSys) of systems of any lattice sizes to convergence on
// one stream.  Systems iterate together, whatever their phase or shape: by gangs, as many of
// them to a launch as the device has CUs for, or by the tiled kernels, one pair of launches
// per iteration over all systems that use them.
class Engine {
 public:
  Engine(Pool* pool, hipStream_t st);
  ~Engine();
  // False if the engine's own device or pinned buffers could not be allocated.
  bool ok() const { return ok_; }
  // Allocate workspace and join.  ADD_NO_ROOM (with the error set): no free slot or
  // the workspace is over budget; ADD_HIP: a HIP call failed while joining.
  enum AddResult { ADD_OK = 0, ADD_NO_ROOM = 1, ADD_HIP = 2 };
  AddResult add(System* s);
  // Bytes of the budget that systems like these take for their gangs, in one block (0: no
  // lattice of theirs has a cut).
  size_t gang_bytes(const std::vector<System*>& v);
  // Let the systems of v that have just been added iterate by gangs, where their lattice has a
  // cut; their memory is one block, appended to `owned`.  room = false: the budget has none
  // just now, nothing was done and the systems keep the tiled kernels.  They also do should
  // the device be out of memory within the budget.  The kernels that iterate on a system, and
  // with them its bits, must not depend on what else is in flight: the callers wait for room
  // that others hold, and settle for the tiled kernels only where the system or the call does
  // not fit by itself.
  hipError_t join_gangs(const std::vector<System*>& v, std::vector<void*>& owned, bool& room);
  // Remove a finished system and return its workspace to the pool.
  // Takes s out; its workspace blocks go to `owned` if given (the caller releases them,
  // those of all its systems after one event), else back to the pool.
  void remove(System* s, std::vector<void*>* owned = nullptr);
  // Advance every system: host-side phases, then one block of CG iterations.
  // Returns the HIP error if any.
  hipError_t step() {
    const hipError_t e = advance();
    if (e != hipSuccess || (inflight_[0].empty() && inflight_[1].empty())) end_turn();
    return e;
  }
  bool idle() const;
  int count() const;
  hipStream_t stream() const { return st_; }
  // Workspace bytes a system of this shape and solver needs.
  static size_t workspace_bytes(const Geom& g, const hub_solve_opts& o);
  // Kernel timing of the CG stages (HIP events around every launch).
  struct KernelStat {
    int64_t launches = 0;
    double ms = 0.0;
    double bytes = 0.0;
  };
  void set_profiling(bool on);
  // For tests: launch n of a gang of several workgroups, counted on the engine, is refused as
  // by a full device where bit n mod 32 of the mask is set.
  void deny_meetings(unsigned mask) { deny_ = mask; gang_launches_ = 0; }
  // [single][kernel]: stage 1, stage 2 of the tiled CG; the gang launches
  KernelStat stat[2][3];
  // Serving epilogue of a converged system: S = Re chi^dagger x (host), and
  // dS/dphi into dSdphi (device, may be null).  Synchronises the stream.
  hipError_t finalize(System* s, const double2* chi, double* dSdphi, double* S);

 private:
  // One host-side transition of a group of systems at the same phase.
  hipError_t group_phase(int phase, const std::vector<System*>& g);
  // FP64 CG: the true residual of the iterates of g; restart or stop each system.
  hipError_t confirm(const std::vector<System*>& g);
  // A block of CG iterations enqueued for the systems of one precision, whose
  // convergence flags are read back asynchronously.
  struct Block {
    bool single = false;
    int k = 0;
    int buf = 0;
    std::vector<System*> v;             // grouped by tile class, then the gangs' systems
    std::vector<int> cls_end;           // end of each tile class in v
    std::vector<hipEvent_t> gev;        // start/stop of the gang launches (profiling)
    std::vector<int> gen;               // System::gen of each system at enqueue
    std::vector<unsigned> gang_seq;     // its gang launches so far
    std::vector<std::vector<int>> its;  // iteration index per launch and system (profiling)
    std::vector<hipEvent_t> kev;        // kernel start/stop events (profiling)
    unsigned seq = 0;                   // the block's flags are home once *h_blk_flag_ reaches seq
  };
  hipError_t launch_block(bool single, bool& launched);
  hipError_t finish_block(Block& b);
  hipError_t wait_block(unsigned seq);
  hipError_t launch_gangs(const std::vector<System*>& v, bool single, Block& b);
  bool gang_entry(GangList& G, int (&taken)[kNumXcd], System* s, bool single) const;
  hipError_t advance();
  hipError_t begin_turn(bool single);
  void end_turn();
  hipError_t take_event(std::vector<hipEvent_t>& dst);
  GangCut cut_of(const Geom& g, bool single);
  void look_at_device();
  hipError_t read_scal(const std::vector<System*>& v);
  // The publication of the Scal records of v at the end of a following launch, and the wait
  // for it (h_scal_ holds the records then).
  hipError_t launch_arnoldi(const std::vector<System*>& v, int j, Publish& pub);
  Publish publication(const std::vector<System*>& v);
  hipError_t wait_publication(const Publish& pub);
  // Descriptors and FGMRES update coefficients go to pinned staging rows (slot-indexed)
  // and reach the device in one copy per kind: flush_desc at the start of every step,
  // flush_y before the update kernel.  A row is rewritten only after the kernels that
  // read its last copy have been waited for.
  void upload_desc(System* s);
  void upload_y(System* s, const std::vector<std::complex<double>>& y);
  hipError_t flush_desc();
  hipError_t flush_y();
  // Launch list over v (systems of one tile class).
  LaunchList list(const std::vector<System*>& v) const;
  void finish(System* s, hub_status st);

  Pool* pool_;
  hipStream_t st_;
  bool ok_ = false;
  SysDesc* d_desc_ = nullptr;
  SysDesc* h_desc_ = nullptr;   // pinned staging of d_desc_
  double* d_y_ = nullptr;       // update coefficients, kYStride doubles per slot
  double* h_y_ = nullptr;       // pinned staging of d_y_
  int desc_lo_ = kMaxSys, desc_hi_ = -1, y_lo_ = kMaxSys, y_hi_ = -1;  // rows to copy
  Scal* d_scal_ = nullptr;      // kMaxSys records, then kScalCounters counters
  Scal* h_scal_ = nullptr;      // pinned mirror
  Scal* h_pub_ = nullptr;       // host-coherent, two buffers of published records, then their flag
  unsigned* h_pub_flag_ = nullptr;
  unsigned pub_seq_ = 0;
  std::vector<System*> slots_;
  bool profiling_ = false;
  std::vector<hipEvent_t> events_;      // pool for kernel timing
  std::vector<Block> inflight_[2];      // per precision, oldest first
  Scal* h_flags_ = nullptr;             // host-coherent, 4 buffers x kMaxSys, then h_blk_flag_
  unsigned* h_blk_flag_ = nullptr;      // sequence number of the last block whose flags were written
  unsigned blk_seq_ = 0;
  GangCut cut_[2] = {};                 // the last cut computed per precision, of extents cut_ext_
  int cut_ext_[2][3] = {};
  bool all_cus_ = true;  // the stream has the CUs that gangs of several workgroups count on
  // The smallest gang that went on in steps lately, and for how many blocks: where the CUs are
  // taken for long, the systems of the next solve begin with that.
  int tight_g_ = kGangMaxWgs + 1, tight_backoff_ = 0;
  GangTurns& turns_;
  int turn_ = 0;  // workgroups it holds there
  unsigned gang_launches_ = 0;
  unsigned deny_ = 0;
  int next_buf_[2] = {0, 0};
};

// y = argmin |beta e_1 - H y| for the (k+1) x k upper Hessenberg H (column-major, leading
// dimension ldh), by Givens rotations; *resid (if not NULL) receives the minimal residual.
std::vector<std::complex<double>> hessenberg_lsq(const std::vector<std::complex<double>>& H, int ldh, int k,
                                                 double beta, double* resid = nullptr);

Geom make_geom(const hub_lattice& lat);
int ntiles_of(int n);

}  // namespace hub
