// cg_runtime.h - host runtime types of the stencil CG library.
#pragma once
#include <hip/hip_runtime.h>

#include <condition_variable>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/cg.h"
#include "cg_arena.h"
#include "cg_internal.h"

namespace cgr {

struct Plan {
  int variant = 0;
  bool refined = false;
  int fp32g = 0;     // geometry of the FP32 lanes (4 columns per lane)
  bool wg = false;   // whole solve inside one work-group
  bool rr = false;   // ... with the vectors on chip (register-resident solver)
  int rr_threads = 0;  // ... its threads, and rows of a thread
  int rr_rows = 0;
  bool fixed = false;  // fixed-point solve, one work-group (cg_fixed.hip)
  int precond = 0;     // Chebyshev preconditioner steps (classic FP64, tile passes)
  int cheb_rows = 0;   // ... rows of a Chebyshev item / partial tile
  int cheb_tiles = 0;  // ... partials of the Chebyshev pass
  int cheb_grid = 8;   // ... work-groups of the Chebyshev pass
  int fx_threads = 0;
  bool vc = false;     // variable-coefficient operator (four coefficient arrays)
  int width = 0;       // padded row length of one vector, in elements
  int il = 1;          // FP64 vectors with interleaved rows (g.pitch = il * width)
  int rr_period = 0;   // pipelined: residual replacement every rr_period iterations
  bool on_side() const { return rr || fixed; }  // batch: whole solve beside the steps
  cgk::Geo g{};
  int grid = 8;      // work-groups per pass
  size_t v64 = 0, v32 = 0, part = 0, footprint = 0;
};

struct Pin {
  int rows = 0;
  int grid = 0;
  int cpl = 0;  // columns per lane; 0 = default (2 for FP64, 4 for refined)
};

// A captured chunk of iterations holds every pass argument, so its key names
// everything that shapes them: the workspace, the geometry and operator, the
// iteration and the buffer parities.
struct GraphKey {
  const void* mem;
  int v[16];  // nx, ny, rows, grid, variant, refined, iters, mpar, ipar, precond,
              // fp32g, plane, vc, cheb_rows, rr_period, iteration within the period
  bool operator<(const GraphKey& o) const {
    if (mem != o.mem) return mem < o.mem;
    for (int i = 0; i < 16; ++i)
      if (v[i] != o.v[i]) return v[i] < o.v[i];
    return false;
  }
};

struct KStat {
  int64_t launches = 0;
  double seconds = 0.0, bytes = 0.0;
};

struct PendingEv {
  hipEvent_t a, b;
  const char* name;
  double bytes;
};

// Workspace of one resident solve, carved from the arena.
struct Work {
  Plan pl;
  char* mem = nullptr;
  size_t extra = 0;          // bytes past the footprint: the resident loop's exchange area
  uint64_t* sync = nullptr;  // ... or null, where the arena had no room for it
  uint32_t seq = 1;          // ... the number of its next meeting
  double *b = nullptr, *x = nullptr, *r = nullptr, *w[2] = {}, *z = nullptr, *q = nullptr,
         *p = nullptr, *pc[2] = {};
  float *rf = nullptr, *df = nullptr, *pf[2] = {};
  float* zf = nullptr;  // refinement, preconditioned: z = M^-1 r_in
  double* cheb = nullptr;  // preconditioner coefficients (c0, c1[s-1], c2[s-1])
  double *u = nullptr, *sv = nullptr, *mv = nullptr;  // preconditioned pipelined
  double* kc = nullptr;  // variable coefficients: west, south, east, north arrays
  double* part[2] = {};
  cgk::State* S[2] = {};
  int m = 0;  // passes issued (state/partial parity)
  int i = 0;  // iterations issued (vector ping-pong parity)
  int maxit = 0;
  bool check = false;  // the passes being issued only classify the final state
};

// The resident loop (cg_resident.hip) of a solve: its kind, strips per
// wavefront and work-groups; wgs == 0: the solve runs by passes.
struct Resident {
  int kind = 0, strips = 0, wgs = 0;
  bool near = false;  // all work-groups on one XCD
};

// The stream of a device's latest resident launch, unless that is known to have
// ended (a context clears what names its streams before it destroys them).
struct ResidentTurn {
  std::mutex m;
  hipStream_t last = nullptr;
  uint64_t number = 0;  // of the launch
  hipEvent_t ended = nullptr;
};
ResidentTurn& resident_turn_of(int device);

struct Ctx;
double now_s();
Resident resident_of(const Ctx& c, const Plan& pl);
// The solve as it stands, for a launch of `budget` iterations; numbers its meetings.
cgk::ResSolve resident_solve(Work& w, const cgk::State* st, const double* part, int budget,
                             int spin);
// After a launch: counts its abandoned solves, and pauses the loop if there are any.
void resident_outcome(Ctx& c, int abandoned);
// Counts a launch of the loop in the context's statistics; an abandoned solve
// is counted under kResidentAbandoned.
void count_resident(Ctx& c, int kind, int rows, int strips, bool near);
constexpr const char* kResidentAbandoned = "resident_abandoned";
// Issues a resident launch (`launch`, on `st`) in its turn on the device: the
// work-groups of a launch wait for each other, so two that both fit alone must
// not share it.  The device itself waits for a launch of another stream that may
// be in flight, and no lock is held meanwhile: launches of all contexts follow
// each other in the order they were issued, each of a bounded number of
// iterations.
template <class F>
hipError_t resident_turn(int device, hipStream_t st, uint64_t& number, F launch) {
  ResidentTurn& t = resident_turn_of(device);
  std::lock_guard<std::mutex> lk(t.m);
  hipError_t e = hipSuccess;
  if (t.last && t.last != st) {
    if (!t.ended) e = hipEventCreateWithFlags(&t.ended, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(t.ended, t.last);
    if (e == hipSuccess) e = hipStreamWaitEvent(st, t.ended, 0);
  }
  if (e == hipSuccess) e = launch();
  if (e == hipSuccess) {
    t.last = st;
    number = ++t.number;
  }
  return e;
}
// The host has waited for the launch of this number; for all of a stream's.
void resident_ended(int device, uint64_t number);
void resident_ended(int device, hipStream_t st);
bool carve(Ctx& c, Work& w);
int stage_in(Ctx& c, Work& w, const cg_problem* p);
cgk::State initial_state(const cg_problem* p);
// c0, c1[s-1], c2[s-1] of the Chebyshev preconditioner with s steps
void cheb_coeffs(int nx, int ny, int s, double* out);
// stage_in without waiting: the initial state is copied from `pinned` (host
// memory the caller keeps unchanged until the stream has passed the copy).
int stage_in_async(Ctx& c, Work& w, const cg_problem* p, const cgk::State* pinned);
int stage_out(Ctx& c, Work& w, const cg_problem* p, const cgk::State& s);
void fill_result(const cgk::State& s, cg_result* res, double secs, bool refined);

int validate(const cg_problem* p);
// CG_PREC_AUTO's choice: FP64 below kAutoRefineDof unknowns, FP32-refined from
// there; any other precision unchanged.  The line was drawn where both ran by
// steps (refinement 0.81x FP64's solves/s at 128^2, 1.17x at 181^2); in batches of
// the resident loop refinement measures 0.71x at 128^2, 0.96x at 181^2, 1.14x at
// 256^2 and 1.75x at 1024^2.  It stays: the choice decides a request's bits.
constexpr int64_t kAutoRefineDof = 20480;
cg_problem resolve_precision(const cg_problem& p);
size_t footprint_of(const cg_problem* p);
cgk::Geo make_geo(int nx, int ny, int fp32g, int rows);
cgk::Geo make_geo3(int nx, int plane, int nz, int zc);
int default_rows(int nx, int ny, int fp32g);

class Server;  // serving scheduler (cg_serve.cpp)

// The lock of a context: recursive, and handed over in order of arrival.  The
// server's thread takes its context again right after each of its turns; an
// ordinary mutex would let it do so before a waiting caller wakes up.
class ContextLock {
 public:
  void lock() {
    std::unique_lock<std::mutex> lk(m_);
    if (depth_ && owner_ == std::this_thread::get_id()) {
      ++depth_;
      return;
    }
    const uint64_t turn = next_++;
    cv_.wait(lk, [&] { return !depth_ && turn == now_; });
    owner_ = std::this_thread::get_id();
    depth_ = 1;
  }
  void unlock() {
    {
      std::lock_guard<std::mutex> lk(m_);
      if (--depth_) return;
      ++now_;
    }
    cv_.notify_all();
  }
  // Whether another thread waits for the holder, who asks.
  bool wanted() {
    std::lock_guard<std::mutex> lk(m_);
    return next_ > now_ + 1;
  }

 private:
  std::mutex m_;
  std::condition_variable cv_;
  std::thread::id owner_;
  int depth_ = 0;
  uint64_t next_ = 0, now_ = 0;
};

struct Ctx {
  int device = 0;
  int num_cu = 256;
  hipStream_t st = nullptr;
  hipStream_t side = nullptr;  // register-resident solves of a batch, beside the steps
  hipStream_t loop = nullptr;  // resident iteration loops of a batch, beside the steps
  hipStream_t user_stream = nullptr;
  hipEvent_t user_ev = nullptr;
  void* own_arena = nullptr;
  Arena arena;
  int max_slots = 256;
  std::string tune_path;
  ContextLock mu;
  char* host_state = nullptr;  // pinned staging for state words
  int graph_chunk = 32;        // iterations per captured chunk; 0 = plain launches
  int wg_max_dof = 16384;      // whole-solve-in-one-work-group threshold (FP64)
  bool rr_enabled = true;      // register-resident solver for grids that fit it
  int step_chunk = 32;         // batch: steps between harvests
  int serve_chunk = 8;         // serving: steps between admissions
  bool resident_on = true;     // iteration loops of mid-size solves in one launch
  int resident_budget = 1024;  // ... iterations of one launch
  int resident_spin = 1 << 16; // ... polls before a wait is given up (some tens of ms)
  double resident_after = 0.0; // ... not before this time: a solve was abandoned
  double resident_pause = 0.0; // ... and the pause that followed (0: none, or a launch
                               // has gone through since)
  int resident_strips = 0;     // ... strips per wavefront (0: by the grid)
  bool resident_near = true;   // ... on one XCD where it fits
  int cheb_item_div = 1;       // Chebyshev items per pass: resident work-groups / this
  int step_chunk_for(bool serving) const { return serving ? serve_chunk : step_chunk; }
  size_t engine_bytes() const {  // control block of the multi-solve engine
    return (size_t)max_slots * (sizeof(cgk::Slot) + 2 * 256 * sizeof(cgk::Item) +
                                2 * sizeof(int) + sizeof(cgk::State)) + 8192;
  }
  bool capturing = false;
  bool prof = false;
  std::string last_error;
  std::map<uint64_t, Pin> pins;  // tile shape pinned per grid shape
  std::map<GraphKey, hipGraphExec_t> graphs;
  std::map<std::string, KStat> stats;
  std::vector<PendingEv> pending;
  std::vector<hipEvent_t> ev_free;
  Server* server = nullptr;
  std::mutex server_mu;  // guards `server` only (submit/poll never wait for an epoch)

  // pins are kept per grid shape, precision and variant (the refined inner
  // solve is classic whatever the variant, so refined pins use variant 0)
  static uint64_t key(int nx, int ny, int fp32g, int variant) {
    const uint64_t v = fp32g ? 0 : (uint64_t)(variant & 1);
    return ((uint64_t)(uint32_t)nx << 34) | ((uint64_t)(uint32_t)ny << 2) | (v << 1) |
           (uint64_t)(fp32g & 1);
  }
  std::string arch;      // gcnArchName of the device (tune cache key)
  int hip_version = 0;   // hipRuntimeGetVersion (tune cache key)
  int init(const cg_config* cfg);
  ~Ctx();
  bool use_wg(const cg_problem* p) const;
  bool use_rr(const cg_problem* p) const;
  // allow_rr = false: the tile geometry even where the register-resident
  // solver would run the problem (building blocks use tiles)
  // interleave: lay the FP64 vectors of a tile-pass solve out with their rows
  // interleaved (off for the building blocks' scratch vectors)
  Plan plan(const cg_problem* p, bool allow_rr = true, bool interleave = true);
  // strip height of a tile-pass solve when no tile shape is pinned
  int unpinned_rows(const cg_problem* p, int fp32g) const;
  int solve(const cg_problem* p, cg_result* res);
  int solve_batch(const cg_problem* p, int n, cg_result* res);
  int apply_or_dot(int kind, int nx, int ny, cg_memspace mem, const double* u, const double* y_in,
                   double* y_out, double* dot_out);
  int tune(int nx, int ny, int variant, int precision);
  void load_tune_cache();
  void save_tune_cache();
  int order_after_user();
  hipError_t pass(int kind, int fp32g, const cgk::PassArgs& a, int grid, bool check = false);
  int stream_probe(int pattern, size_t elems, int reps, double* seconds, double* bytes);
  int mul_probe(int rounds, int reps, double* seconds, double* ops);
  hipEvent_t event();
  void prof_add(const char* name, double seconds, double bytes, int64_t launches);
  void prof_collect();
  void forget_graphs(const void* mem);
};

}  // namespace cgr

// Serving front end (cg_serve.cpp).
int cgr_server_submit(cgr::Ctx* c, const cg_problem* p, uint64_t* ticket);
int cgr_server_poll(cgr::Ctx* c, uint64_t ticket, cg_result* res);
void cgr_server_stop(cgr::Ctx* c);
