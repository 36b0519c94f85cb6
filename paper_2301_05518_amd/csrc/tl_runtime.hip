// Host runtime behind the C ABI of twolink.h: contexts, argument validation,
// resident plans (packing, work lists, tuning, HIP graph capture), reductions.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <list>
#include <map>
#include <mutex>
#include <new>
#include <optional>
#include <sstream>
#include <string>
#include <utility>
#include <vector>

#include <unistd.h>

#include "tl_internal.h"
#include "twolink.h"

using tl::StepConfig;
using tl::StepGroup;

static_assert(TL_F64 == tl::F64 && TL_F32 == tl::F32 && TL_F16S == tl::F16S && TL_BF16 == tl::BF16,
              "precision codes");
static_assert((TL_W12 & 3) == 0 && (TL_ONELINK & 3) == 0 && TL_W12 != TL_ONELINK,
              "TL_W12 and TL_ONELINK are bits above the precision codes");

// A tuned step tiling: cfg, and when cfg runs several steps per launch the one-step tiling
// `single` that an odd step count ends with (variant 8) or that runs of fewer than kRunMinSteps
// steps use (variant 9); single.variant < 0: none.
struct Tuned {
  StepConfig cfg{0, 256, 4, 0, 0, 0, 0};
  StepConfig single{-1, 0, 0, 0, 0, 0, 0};
};

// What whole-run launches of one plan share: control block and exchange scratch.  Their tags only
// grow, so a pair is never cleared again, and never separated.
struct RunMem {
  tl::RunCtl* ctl = nullptr;
  char* scratch = nullptr;
  size_t bytes = 0;   // of scratch
};

// The contexts on one device, for the order of their whole-run launches (see RunTurn).
struct RunLane {
  std::mutex m;
  std::vector<tl_ctx*> ctxs;
  uint64_t seq = 0;   // launches recorded
};

struct tl_ctx {
  int device = -1;
  hipStream_t stream = nullptr;
  std::string err;
  int n_cu = 0;
  std::string arch;
  bool log = false;
  bool fault_alloc = false;   // TL_FAULT=alloc: internal allocations report failure
  bool fault_launch = false;  // TL_FAULT=launch: launches report failure without running
  bool fault_exchange = false;  // TL_FAULT=exchange: memory of whole-run launches cannot be cleared
  bool fault_team = false;      // TL_FAULT=team: whole-run launches run with the teams that are there at once
  bool fault_wait = false;    // TL_FAULT=wait: whole-run launches give up a halo word that is not there at once
  bool big_lds = false;       // dynamic-LDS limit raised for the LDS-staged step kernels
  void* scratch = nullptr;
  size_t scratch_bytes = 0;
  // device memory of plans that are gone, kept for the next ones (see mem_get)
  struct MemBlock {
    void* p;
    size_t bytes;
  };
  std::vector<MemBlock> pool;
  size_t pool_bytes = 0;
  std::vector<RunMem> run_pool;
  // pinned host words, one per plan with whole-run launches: set by the kernel when a wait between
  // workgroups ran out (kFailWords; plans beyond that share the last one)
  uint32_t* run_fail = nullptr;
  std::vector<char> fail_used;
  // whole-run launches among several contexts (see RunTurn; guarded by the lane's mutex)
  RunLane* lane = nullptr;
  hipEvent_t run_event = nullptr;   // recorded after the latest one
  uint64_t run_seq = 0;             // its number on the device, 0: none
  uint64_t run_waited = 0;          // numbers up to this one that the context's stream waits for
  double run_load = 0.0;            // share of the chip those that may still run take
  double* noalloc = nullptr;  // this device's fixed partial-sum area of tl_reduce_noalloc
  std::string noalloc_err;    // why it is missing (lookup failed at tl_create)
  std::map<std::string, Tuned> tune;       // tuned step tilings by workload key
  std::string tune_file;                   // TL_TUNE_CACHE: tuning results persisted across processes
  std::list<std::pair<std::string, tl_plan*>> smear_plans;   // tl_smear(TL_GRAPH) plans, most recent first
  tl_ctx_stats stats{};
};

namespace {

thread_local std::string g_create_err;

int vfail(tl_ctx* c, int code, const char* fmt, va_list ap) {
  char buf[1024];
  vsnprintf(buf, sizeof buf, fmt, ap);
  if (c) c->err = buf; else g_create_err = buf;
  return code;
}

int fail(tl_ctx* c, int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vfail(c, code, fmt, ap);
  va_end(ap);
  return code;
}

// No C++ exception may cross the C interface: an entry point whose host-side bookkeeping
// throws (in practice a failed host allocation) reports TL_ERR_NOMEM instead.
int host_failure(tl_ctx* c) noexcept {
  try {
    if (c) c->err = "host allocation failed"; else g_create_err = "host allocation failed";
  } catch (...) {
  }
  return TL_ERR_NOMEM;
}

#define HIP_TRY(ctx, expr)                                                                     \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess) return fail((ctx), TL_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

#define TL_TRY(expr)            \
  do {                          \
    int rc_ = (expr);           \
    if (rc_ != TL_OK) return rc_; \
  } while (0)

// Makes the context's device current for the duration of a call.
struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

// Makes the context's device current for the rest of the enclosing entry point, or fails
// the call (nothing queued) when the runtime refuses to switch to it.
#define TL_ON_DEVICE(c)                                                                  \
  DeviceGuard dg_((c)->device);                                                          \
  if (!dg_.ok) return fail((c), TL_ERR_DEVICE, "hipSetDevice(%d) failed", (c)->device)

// Internal format code of a public precision argument (precision, optionally | TL_W12 and
// | TL_ONELINK), -1 if invalid.
int fmt_code(int p) {
  const int base = p & ~(TL_W12 | TL_ONELINK);
  if (base < TL_F64 || base > TL_BF16) return -1;
  return base | ((p & TL_W12) ? tl::W12 : 0) | ((p & TL_ONELINK) ? tl::ONE : 0);
}

bool valid_prec(int p) { return fmt_code(p) >= 0; }

int check_geom(tl_ctx* c, const tl_geom* g) {
  if (!g) return fail(c, TL_ERR_ARG, "geometry is NULL");
  for (int d = 0; d < 4; d++)
    if (g->L[d] < 1 || g->L[d] > 4096)
      return fail(c, TL_ERR_SHAPE, "extent L[%d] = %d outside [1, 4096]", d, g->L[d]);
  const int64_t v3 = (int64_t)g->L[0] * g->L[1] * g->L[2];
  if (v3 > (int64_t(1) << 27)) return fail(c, TL_ERR_SHAPE, "slice volume %lld exceeds 2^27 sites", (long long)v3);
  return TL_OK;
}

int64_t vol3(const tl_geom& g) { return (int64_t)g.L[0] * g.L[1] * g.L[2]; }

int need_device(tl_ctx* c) {
  if (c->device < 0) return fail(c, TL_ERR_DEVICE, "host-only context (created with device -1) cannot run device work");
  return TL_OK;
}

void run_free(RunMem& m) {
  if (m.ctl) (void)hipFree(m.ctl);
  if (m.scratch) (void)hipFree(m.scratch);
  m = RunMem{};
}

// Frees everything the context keeps of plans that are gone.
void mem_drain(tl_ctx* c) {
  (void)hipStreamSynchronize(c->stream);
  for (auto& b : c->pool) (void)hipFree(b.p);
  for (auto& m : c->run_pool) run_free(m);
  c->pool.clear();
  c->run_pool.clear();
  c->pool_bytes = 0;
}

int dev_alloc(tl_ctx* c, void** p, size_t bytes) {
  *p = nullptr;
  if (bytes == 0) bytes = 256;
  if (c->fault_alloc) return fail(c, TL_ERR_NOMEM, "device allocation of %zu bytes failed (TL_FAULT=alloc)", bytes);
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess && (!c->pool.empty() || !c->run_pool.empty())) {   // what the context keeps goes first
    (void)hipGetLastError();
    mem_drain(c);
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
    return fail(c, TL_ERR_NOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
  }
  return TL_OK;
}

// Plan memory: a block given back after its last work has finished (see plan_free) serves a later
// plan of the same context, which saves the allocator's round trips.  At most kPoolBlocks blocks and
// kPoolBytes in all are kept (the newest), none over twice the size asked for is handed out, and
// tl_destroy frees them.
constexpr size_t kPoolBlocks = 12, kPoolBytes = size_t(256) << 20;

int mem_get(tl_ctx* c, void** p, size_t* bytes) {
  *bytes = std::max<size_t>((*bytes + 4095) / 4096 * 4096, 4096);
  size_t best = c->pool.size();
  if (!c->fault_alloc)
    for (size_t i = 0; i < c->pool.size(); i++)
      if (c->pool[i].bytes >= *bytes && c->pool[i].bytes <= 2 * *bytes &&
          (best == c->pool.size() || c->pool[i].bytes < c->pool[best].bytes))
        best = i;
  if (best < c->pool.size()) {
    *p = c->pool[best].p;
    *bytes = c->pool[best].bytes;
    c->pool_bytes -= *bytes;
    c->pool.erase(c->pool.begin() + (std::ptrdiff_t)best);
    return TL_OK;
  }
  return dev_alloc(c, p, *bytes);
}

void mem_put(tl_ctx* c, bool keep, void* p, size_t bytes) {
  if (!p) return;
  if (keep && bytes <= kPoolBytes) {
    // the blocks kept longest make room: a pool full of sizes that no plan asks for any more would
    // send every later call to the allocator (16^3 FP32, 20 steps: 83 instead of 61 us)
    while (!c->pool.empty() && (c->pool.size() >= kPoolBlocks || c->pool_bytes + bytes > kPoolBytes)) {
      (void)hipFree(c->pool.front().p);
      c->pool_bytes -= c->pool.front().bytes;
      c->pool.erase(c->pool.begin());
    }
    try {
      c->pool.push_back({p, bytes});
      c->pool_bytes += bytes;
      return;
    } catch (...) {   // no host memory for the list: free the block
    }
  }
  (void)hipFree(p);
}

// Whole-run launches of several contexts take turns.  A team needs all its workgroups on the chip
// at once, and launches that are dispatched together get a part of it each: every team then waits,
// and runs incomplete (four contexts with 48^3 FP32 plans of 40 steps: 1550 us for a run each, 1460 with
// step launches, 560 in turn; 48^3 BF16 12 RHS 4200, 3010, 1920).  So a context's stream waits for other contexts' launches, the
// oldest first, until what may run beside its own fits (four 16^3 plans do).  Work of one context
// is in order anyway, so a context that is alone on its device does nothing here; launches in a
// graph the caller captured are not ordered.  Waits go to launches queued earlier only.
RunLane& run_lane(int device) {
  static std::mutex m;
  static auto* lanes = new std::map<int, RunLane>();   // as long as the process: contexts may outlive static objects
  std::lock_guard<std::mutex> lock(m);
  return (*lanes)[device];
}

// Takes the turn of a launch that needs `load` of the chip, until it goes out of scope; the launch is
// queued in between.
class RunTurn {
 public:
  RunTurn(tl_ctx* c, double load) : c_(c), lane_(*c->lane), lock_(lane_.m), load_(load) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (lane_.ctxs.size() < 2 || !c->run_event ||
        (c->stream && (hipStreamIsCapturing(c->stream, &st) != hipSuccess || st != hipStreamCaptureStatusNone))) {
      lock_.unlock();
      return;
    }
    std::vector<tl_ctx*> others;
    for (tl_ctx* o : lane_.ctxs)
      if (o != c && o->run_seq > c->run_waited && o->run_load > 0.0) {
        others.push_back(o);
        load += o->run_load;
      }
    std::sort(others.begin(), others.end(), [](const tl_ctx* a, const tl_ctx* b) { return a->run_seq < b->run_seq; });
    for (tl_ctx* o : others) {
      if (load <= 1.0) break;
      if (hipStreamWaitEvent(c->stream, o->run_event, 0) != hipSuccess) (void)hipGetLastError();
      c->run_waited = o->run_seq;
      load -= o->run_load;
    }
  }
  ~RunTurn() {
    if (!lock_.owns_lock()) return;
    if (hipEventRecord(c_->run_event, c_->stream) != hipSuccess) {
      (void)hipGetLastError();
      return;
    }
    c_->run_seq = ++lane_.seq;
    c_->run_load = std::max(c_->run_load, load_);
  }
  // The context's stream is idle.
  static void idle(tl_ctx* c) {
    if (!c->run_event) return;
    std::lock_guard<std::mutex> lock(c->lane->m);
    c->run_load = 0.0;
  }

 private:
  tl_ctx* c_;
  RunLane& lane_;
  std::unique_lock<std::mutex> lock_;
  double load_;
};

// Queue one library launch; TL_FAULT=launch makes it fail before anything is queued.
template <class F>
int launch(tl_ctx* c, const char* what, F&& f) {
  if (c->fault_launch) return fail(c, TL_ERR_HIP, "%s launch failed (TL_FAULT=launch)", what);
  const hipError_t e = f();
  if (e != hipSuccess) return fail(c, TL_ERR_HIP, "%s launch: %s", what, hipGetErrorString(e));
  return TL_OK;
}

// Context scratch: grows on demand; stream-ordered reuse is safe because every
// user queues on the context stream and waits before overwriting host tables.
int ctx_scratch(tl_ctx* c, size_t bytes, char** out) {
  if (bytes > c->scratch_bytes) {
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    if (c->scratch) HIP_TRY(c, hipFree(c->scratch));
    c->scratch = nullptr;
    c->scratch_bytes = 0;
    void* p = nullptr;
    TL_TRY(dev_alloc(c, &p, bytes));
    c->scratch = p;
    c->scratch_bytes = bytes;
  }
  *out = static_cast<char*>(c->scratch);
  return TL_OK;
}

// A whole-run launch whose wait between workgroups ran out ends, with NaNs spreading from where it
// gave up.  That is reported once, by the next call that looks: calls on that plan, or tl_sync.
constexpr size_t kFailWords = 1024;

bool fail_taken(uint32_t* word) {
  if (!word || *static_cast<volatile uint32_t*>(word) == 0) return false;
  *static_cast<volatile uint32_t*>(word) = 0;
  return true;
}

int run_failure(tl_ctx* c) {
  return fail(c, TL_ERR_HIP, "a whole-run smearing launch gave up waiting for another workgroup; its fields are not valid");
}

// Plans are made ready (tables, memory, tuning) outside a caller's stream capture: under it the
// uploads would only be recorded, and whatever runs before the graph is replayed would read tables
// that were never written.
int need_eager(tl_ctx* c, const char* what) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (!c->stream) return TL_OK;   // the null stream is never captured
  HIP_TRY(c, hipStreamIsCapturing(c->stream, &st));
  if (st != hipStreamCaptureStatusNone) return fail(c, TL_ERR_HIP, "%s while the context's stream is being captured", what);
  return TL_OK;
}

// Upload of a host table onto the context stream (never under capture, see need_eager).  A small
// one travels in a kernel's arguments, which are copied when the launch is queued, so nothing has
// to wait for it.
int upload(tl_ctx* c, void* dst, const void* src, size_t bytes) {
  if (bytes == 0) return TL_OK;
  if (bytes <= tl::kUploadArgs && bytes % 4 == 0 && !c->fault_launch) {
    HIP_TRY(c, tl::launch_upload(dst, src, bytes, c->stream));
    return TL_OK;
  }
  HIP_TRY(c, hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return TL_OK;
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// Slot of slice t in a two-link field built for w_slices (NULL = all slices).
int slot_of(const tl_geom& g, const int32_t* w_slices, int n_w, int t) {
  if (t < 0 || t >= g.L[3]) return -1;
  if (!w_slices) return t;
  for (int j = 0; j < n_w; j++)
    if (w_slices[j] == t) return j;
  return -1;
}

int check_wslices(tl_ctx* c, const tl_geom& g, const int32_t* w_slices, int n_w) {
  if (!w_slices) return TL_OK;
  if (n_w < 1 || n_w > g.L[3]) return fail(c, TL_ERR_ARG, "n_w_slices = %d outside [1, Lt=%d]", n_w, g.L[3]);
  for (int j = 0; j < n_w; j++)
    if (w_slices[j] < 0 || w_slices[j] >= g.L[3])
      return fail(c, TL_ERR_SHAPE, "w_slices[%d] = %d outside [0, %d)", j, w_slices[j], g.L[3]);
  return TL_OK;
}

// Coefficients of one smearing step, out = alpha in + beta sum_hops:
//   two-link (eq. tlSmear with eq. tlLapl1): in + (s/4)(sum_hops - 6 in), s = sigma/n
//   one-link (Sec. 2, nabla^2 = H - 6):      in + s (sum_hops - 6 in)
void step_coeffs(bool one, int n_steps, double sigma, double* alpha, double* beta) {
  const double s = sigma / (double)n_steps;
  const double q = one ? s : 0.25 * s;
  *alpha = 1.0 - 6.0 * q;
  *beta = q;
}

// Largest sigma/n for which every step factor lies in [-1, 1] (a contraction for unitary links).
double max_step(bool one) { return one ? 1.0 / 6.0 : 2.0 / 3.0; }

// A step configuration a cache entry or TL_TILE may name.
bool valid_cfg(const StepConfig& g) {
  return g.variant >= 0 && g.variant <= 9 && g.block >= 64 && g.block <= (g.variant >= 5 ? 512 : 256) &&
         g.block % 64 == 0 && g.tz >= 1 && (g.nt == 0 || g.nt == 1) && (g.flip == 0 || g.flip == 1) &&
         g.width >= 0 && g.width <= 4;
}

// Up to 7 comma-separated integers "variant,block,tz,grid,nt,flip,width" at v into c (missing
// ones 0); returns how many were read and sets *end past them.
int parse_cfg(const char* v, StepConfig* c, const char** end) {
  int* f[7] = {&c->variant, &c->block, &c->tz, &c->grid, &c->nt, &c->flip, &c->width};
  *c = StepConfig{};
  int n = 0;
  const char* q = v;
  while (n < 7) {
    char* e = nullptr;
    const long x = strtol(q, &e, 10);
    if (e == q || x < -(1L << 30) || x > (1L << 30)) break;
    *f[n++] = (int)x;
    q = e;
    if (*q != ',') break;
    q++;
  }
  *end = q;
  return n;
}

// "variant,block,tz,grid[,nt[,flip[,width]]]" with an optional ";..." naming the one-step tiling
// of a two-step one (six or seven fields); n_min: fields the first part needs.
bool parse_tuned(const char* v, int n_min, Tuned* out) {
  Tuned t;
  const char* end = nullptr;
  const int n = parse_cfg(v, &t.cfg, &end);
  if (n < n_min || !valid_cfg(t.cfg)) return false;
  if (*end == ';') {
    if (n < 6 || parse_cfg(end + 1, &t.single, &end) < 6 || *end != '\0' || !valid_cfg(t.single) ||
        t.single.variant >= 8)
      return false;
  } else if (*end != '\0') {
    return false;
  }
  if (t.cfg.variant < 8) t.single = StepConfig{-1, 0, 0, 0, 0, 0, 0};
  else if (t.single.variant < 0) t.single = StepConfig{0, 256, 4, 0, 0, 0, 0};
  *out = t;
  return true;
}

std::string cfg_text(const StepConfig& g) {
  return std::to_string(g.variant) + "," + std::to_string(g.block) + "," + std::to_string(g.tz) + "," +
         std::to_string(g.grid) + "," + std::to_string(g.nt) + "," + std::to_string(g.flip) +
         (g.width > 0 ? "," + std::to_string(g.width) : std::string());
}

// Tuning cache file (TL_TUNE_CACHE): a JSON object {"<workload key>": "variant,block,tz,grid,nt,flip[,width]",
// ...} (a two-step tiling followed by ";" and its one-step companion).  The keys (architecture,
// precision code, group width, launch mode, each group's dims and RHS) hold no quote or
// backslash, so the file is read and written with plain string handling; a missing,
// unreadable or malformed file is an empty cache.
void tune_file_load(tl_ctx* c) {
  std::ifstream in(c->tune_file);
  if (!in) return;
  std::stringstream ss;
  ss << in.rdbuf();
  const std::string t = ss.str();
  size_t pos = 0;
  while (true) {
    const size_t k0 = t.find('"', pos);
    if (k0 == std::string::npos) break;
    const size_t k1 = t.find('"', k0 + 1);
    const size_t v0 = k1 == std::string::npos ? k1 : t.find('"', k1 + 1);
    const size_t v1 = v0 == std::string::npos ? v0 : t.find('"', v0 + 1);
    if (v1 == std::string::npos) break;
    Tuned tu;
    const std::string val = t.substr(v0 + 1, v1 - v0 - 1);
    if (parse_tuned(val.c_str(), 6, &tu)) c->tune[t.substr(k0 + 1, k1 - k0 - 1)] = tu;
    pos = v1 + 1;
  }
}

// Rewrite the whole file (a temporary then a rename, so a reader never sees half a file).
void tune_file_save(const tl_ctx* c) {
  const std::string tmp = c->tune_file + ".tmp" + std::to_string((long)getpid());
  {
    std::ofstream out(tmp);
    if (!out) return;
    out << "{\n";
    size_t k = 0;
    for (const auto& kv : c->tune) {
      const Tuned& g = kv.second;
      out << "  \"" << kv.first << "\": \"" << cfg_text(g.cfg)
          << (g.cfg.variant >= 8 ? ";" + cfg_text(g.single) : std::string()) << "\""
          << (++k < c->tune.size() ? ",\n" : "\n");
    }
    out << "}\n";
    if (!out) return;
  }
  (void)std::rename(tmp.c_str(), c->tune_file.c_str());
}

}  // namespace

// ====================================================================== plans

// A whole-run launch (variant 9): its units and everything the launch needs but the pointers.
struct RunShape {
  tl::RunConfig cfg{};
  std::vector<tl::RunUnit> units;
  int np = 0, subs = 1, halo = 0, team_size = 1, n_teams = 0, n_tiles = 0;
  int n_shares = 1, steps = 1;   // shares the teams take the units in; steps per launch at most
  size_t scratch = 0;
};

struct tl_plan {
  tl_ctx* ctx = nullptr;
  int prec = 0, n_steps = 0;     // prec: internal format code (tl::vprec(prec) for the vectors)
  double sigma = 0.0, alpha = 1.0, beta = 0.0;
  unsigned flags = 0;

  struct JobCopy {
    tl_job job;
    std::vector<int32_t> t_of_rhs, w_slices;
    int64_t V3 = 0, Vp = 0;
    std::vector<int> res_index;   // job RHS r -> resident RHS index
  };
  std::vector<JobCopy> jobs;

  struct Res {
    int job, r, slot;
    int64_t off;                  // byte offset in each resident buffer
  };
  std::vector<Res> res;           // resident order: grouped by (job, slot)

  struct Group {
    int job, slot, first, nr;     // resident RHS [first, first + nr)
  };
  std::vector<Group> groups;
  int width = 1;

  size_t buf_bytes = 0;
  size_t buf_cap[2] = {0, 0}, tables_cap = 0;   // bytes of the blocks behind buf and tables
  char* buf[2] = {nullptr, nullptr};
  int cur = 0;
  bool of_call = false;                         // of a tl_smear call: no caller can have captured it

  // device tables: the step groups of both tilings (group_cap entries each), whole-run units,
  // per-job pack offsets, reduction fields, partials
  char* tables = nullptr;
  size_t group_cap = 0;
  int64_t* packoff_dev = nullptr;
  std::vector<int64_t> packoff_first;   // index of job j's first entry in packoff_dev
  tl::RedField* red_dev = nullptr;
  double* partials = nullptr;
  int64_t max_v3 = 0;

  // A step tiling and its work list (device table dev, host copy host).
  struct Tiling {
    StepConfig cfg{0, 256, 4, 0, 0, 0, 0};
    StepGroup* dev = nullptr;
    std::vector<StepGroup> host;
    int n_tiles = 0;
    int64_t lds = 0;                    // dynamic LDS bytes of its launches (variants 5-8)
    RunShape run;                       // variant 9: its units and launch (host, n_tiles unused but for info)
  };
  Tiling tile;                          // the step tiling
  Tiling single;                        // when tile runs two steps per launch: the one-step
                                        // tiling of the last step of an odd count
  tl::RunUnit* run_units = nullptr;     // whole-run launches: units table (in tables)
  RunMem run;                           // and their shared memory (taken when first used)
  uint32_t* fail = nullptr;             // their failure word
  bool ready = false;                   // tuning done (or not requested) and tables uploaded

  hipGraphExec_t graph[2] = {nullptr, nullptr};

  tl_plan_info info{};
};

namespace {

// RHS per step group of a configuration: the plan's groups, or narrower ones (cfg.width).
int eff_width(const tl_plan* p, const StepConfig& cfg) {
  return cfg.width > 0 ? std::min(cfg.width, p->width) : p->width;
}

// Work list of a plan for one step configuration.
int make_groups(const tl_plan* p, const StepConfig& cfg, std::vector<StepGroup>* out) {
  out->clear();
  int tiles = 0;
  const int ew = eff_width(p, cfg);
  for (const auto& gr0 : p->groups) {
    for (int first = gr0.first; first < gr0.first + gr0.nr; first += ew) {   // the plan's group, or its parts
      const auto& jc = p->jobs[gr0.job];
      const tl_geom& g = jc.job.g;
      const int nr = std::min(ew, gr0.first + gr0.nr - first);
      StepGroup s{};
      const int64_t wslot = (int64_t)gr0.slot * 3 * jc.Vp * tl::kWBytes[p->prec];
      s.W = static_cast<const char*>(jc.job.W) + wslot;
      s.w_mu_stride = jc.Vp * tl::kWBytes[p->prec];
      s.psi_off = p->res[first].off;
      s.rhs_stride = nr > 1 ? p->res[first + 1].off - p->res[first].off : 0;
      s.Lx = g.L[0];
      s.Ly = g.L[1];
      s.Lz = g.L[2];
      s.Vp = (int32_t)jc.Vp;
      s.nr = nr;
      if (cfg.variant == 8) {   // two steps per launch: blocks of k rows of one y chain
        const int D = tl::hop_of(p->prec);
        const int R = (tl::vprec(p->prec) == tl::F64) ? 1 : ew;
        s.rows = tl::fuse_rows(p->prec, R, g.L[0], g.L[1], cfg.block, 160 * 1024);
        if (s.rows == 0) return TL_ERR_UNSUPPORTED;
        const int ychains = (D == 2 && !(g.L[1] & 1)) ? 2 : 1;
        s.n_xy_tiles = ychains * (g.L[1] / ychains / s.rows);
      } else if (cfg.variant >= 5) {   // full-row tiles
        s.rows = tl::lds_rows(g.L[0], g.L[1], cfg.block);
        if (s.rows == 0) return TL_ERR_UNSUPPORTED;
        s.n_xy_tiles = g.L[1] / s.rows;
      } else {
        s.rows = 0;
        s.n_xy_tiles = (int32_t)(((int64_t)g.L[0] * g.L[1] + cfg.block - 1) / cfg.block);
      }
      if (cfg.variant >= 6) {   // chains of planes z, z+2, ...: two for even Lz, one for odd (and for
        const int chains = (tl::is_one(p->prec) || (g.L[2] & 1)) ? 1 : 2;   // one-links: consecutive planes)
        const int clen = g.L[2] / chains;
        s.n_z_tiles = chains * ((clen + cfg.tz - 1) / cfg.tz);
      } else {
        s.n_z_tiles = (g.L[2] + cfg.tz - 1) / cfg.tz;
      }
      s.tile_begin = tiles;
      const int64_t nt = (int64_t)s.n_xy_tiles * s.n_z_tiles;
      if (tiles + nt > (int64_t)1 << 30) return TL_ERR_UNSUPPORTED;
      tiles += (int)nt;
      out->push_back(s);
    }
  }
  return TL_OK;
}

// Dynamic LDS bytes of a configuration (variants 5-8), -1 if it does not fit.
int64_t plan_lds(const tl_plan* p, const StepConfig& cfg, const std::vector<StepGroup>& gs) {
  if (cfg.variant < 5) return 0;
  int64_t mx = 0;
  const int R = (tl::vprec(p->prec) == tl::F64) ? 1 : eff_width(p, cfg);
  for (const auto& g : gs)
    mx = std::max(mx, cfg.variant == 8 ? tl::lds_bytes_fuse2(p->prec, R, g.Lx, g.rows)
                                       : tl::lds_bytes(p->prec, R, g.Lx, g.rows));
  return mx <= 160 * 1024 ? mx : -1;
}

// Runs of fewer steps use one launch per step: a whole-run launch reads every two-link twice
// (once as the forward and once as the backward one of a site) before its first step.
constexpr int kRunMinSteps = 4;
// Steps the autotuner times of a whole run at most: what a run costs once is a few steps' time, and
// 200 launches of all steps of a long run would take minutes.
constexpr int kTuneSteps = 60;

// Unit-steps of a whole-run launch per team at most; longer runs take several launches.  A member
// without a tile waits for the others at the end of a team's share, and every wait of the kernel
// is given up after kSpinLimit polls (several seconds): at 2 to 10 us per unit-step a share takes
// 0.1 to 0.3 s, so no run is long enough to run into that, and other streams get their turn.
constexpr int kRunMaxUnitSteps = 32768;

// Cut a cell of extents c into at most `team` tiles of at most `sites` sites that a workgroup of
// `subs` thread sets can hold.  First the fewest waves per SIMD (a phase's arithmetic time), then
// the cheapest exchange: sites read from other tiles, and eight times the 128-byte lines they lie
// in (across x every site has its own: 64^3 FP32 24 RHS takes 52 us per step in tiles of 32x4x4
// and 62 in 8x8x8, which read fewer sites).  Returns the tile count, 0 if none fits.
int cut_cell(const int32_t c[3], int prec, int width, int subs, int sites, int team, int32_t b[3], int32_t t[3],
             int* halo) {
  int best = 0;
  int64_t best_cost = 0;
  for (int tx = 1; tx <= c[0] && tx <= team; tx++) {
    const int bx = (c[0] + tx - 1) / tx;
    if ((c[0] + bx - 1) / bx != tx) continue;
    for (int ty = 1; ty <= c[1] && tx * ty <= team; ty++) {
      const int by = (c[1] + ty - 1) / ty;
      if ((c[1] + by - 1) / by != ty) continue;
      for (int tz = 1; tz <= c[2] && tx * ty * tz <= team; tz++) {
        const int bz = (c[2] + tz - 1) / tz;
        if ((c[2] + bz - 1) / bz != tz || (int64_t)bx * by * bz > sites) continue;
        const int np = (bx * by * bz + 63) / 64 * 64;
        const int fx = tx > 1 ? by * bz : 0, fy = ty > 1 ? bx * bz : 0, fz = tz > 1 ? bx * by : 0;
        const int h = 2 * (fx + fy + fz);
        const int lines = 2 * (fx + (fy ? bz * ((bx + 7) / 8) : 0) + (fz + 7) / 8);
        if (subs * h > 64 * tl::kFetch * ((tl::run_max_threads(prec) - np * subs) / 64) ||
            tl::run_lds(prec, width, subs, np, h) > 160 * 1024)
          continue;
        const int64_t cost = ((int64_t)((np / 64 * subs + 3) / 4) << 32) + h + 8 * lines;
        if (best && cost >= best_cost) continue;
        best = tx * ty * tz;
        best_cost = cost;
        *halo = h;
        b[0] = bx; b[1] = by; b[2] = bz;
        t[0] = tx; t[1] = ty; t[2] = tz;
      }
    }
  }
  return best;
}

// Places a whole run's units (sorted, teams known) in their teams.  A team is as large as the
// largest cells need, and a step costs about as much on few sites per SIMD as on many (BF16, 3
// RHS: 2.1 us at one wave of sites per SIMD, 2.5 at two), so the units of a smaller lattice run
// several at once, each on a part of the team, where a team has several of them: the number that
// makes rounds * (4 + waves per SIMD) least.  Plans of one lattice size have the team size
// itself for that.  Two slices of 32^3 beside four of 48^3: 4.2 -> 2.2 us per step.
void place_units(int prec, int sites, RunShape* r, int* halo) {
  const int n_units = (int)r->units.size(), shares = std::min(n_units, r->n_teams);
  for (int i = 0, j; i < n_units; i = j) {
    tl::RunUnit cut = r->units[i];
    for (j = i; j < n_units && r->units[j].shape == cut.shape; j++) {}
    auto waves = [&](int np) { return (np / 64 * r->subs + 3) / 4; };
    auto padded = [](const int32_t b[3]) { return (b[0] * b[1] * b[2] + 63) / 64 * 64; };
    const int each = (j - i + shares - 1) / shares;   // units of this size per share
    int at_once = 1;
    int64_t best = (int64_t)each * (4 + waves(padded(cut.b)));
    for (int m = 2; j - i < n_units && m <= std::min(each, r->team_size); m++) {
      int32_t b[3], t[3];
      int h = 0;
      if (!cut_cell(cut.c, prec, r->cfg.width, r->subs, sites, r->team_size / m, b, t, &h)) break;
      const int np = std::max(r->np, padded(b)), hm = std::max(*halo, h);
      const int64_t cost = (int64_t)((each + m - 1) / m) * (4 + waves(padded(b)));
      if (cost >= best || r->subs * hm > 64 * tl::kFetch * ((tl::run_max_threads(prec) - np * r->subs) / 64) ||
          tl::run_lds(prec, r->cfg.width, r->subs, np, hm) > 160 * 1024)
        continue;
      best = cost;
      at_once = m;
      std::copy(b, b + 3, cut.b);
      std::copy(t, t + 3, cut.t);
      r->np = np;
      *halo = hm;
    }
    const int n = cut.t[0] * cut.t[1] * cut.t[2];
    for (int u = i; u < j; u++) {
      tl::RunUnit& g = r->units[u];
      std::copy(cut.b, cut.b + 3, g.b);
      std::copy(cut.t, cut.t + 3, g.t);
      g.first = (u - i) / shares % at_once * n;   // a share takes every shares-th unit
      g.span = at_once * n;
      r->n_tiles += n;
    }
  }
}

// The whole-run launch of a plan for configuration cfg (block: threads per workgroup at most, tz:
// workgroups per team at most, grid: workgroups, flip: 1 every RHS of a group gets threads of its
// own, else nt: 1 two sets of threads share a group's RHS, 0 one thread takes them in turn).  Returns the reason it does not apply, or NULL.
const char* make_run(const tl_plan* p, const StepConfig& cfg, RunShape* out) {
  const int prec = tl::vprec(p->prec), hop = tl::hop_of(p->prec);
  RunShape r;
  if (p->flags & TL_PLAIN) return "TL_PLAIN runs one step per launch";
  r.subs = cfg.flip ? p->width : cfg.nt ? std::min(2, p->width) : 1;
  r.cfg.width = (p->width + r.subs - 1) / r.subs;
  const int sites = cfg.block / r.subs / 64 * 64;
  if (sites < 64) return "too few threads per RHS";
  int halo = 0;
  for (const auto& gr : p->groups) {
    const auto& jc = p->jobs[gr.job];
    const tl_geom& g = jc.job.g;
    tl::RunUnit u{};
    u.W = static_cast<const char*>(jc.job.W) + (int64_t)gr.slot * 3 * jc.Vp * tl::kWBytes[p->prec];
    u.w_mu_stride = jc.Vp * tl::kWBytes[p->prec];
    u.psi_off = p->res[gr.first].off;
    u.rhs_stride = gr.nr > 1 ? p->res[gr.first + 1].off - p->res[gr.first].off : 0;
    u.Lx = g.L[0];
    u.Ly = g.L[1];
    u.Lz = g.L[2];
    u.Vp = (int32_t)jc.Vp;
    u.nr = gr.nr;
    int chains[3];
    for (int d = 0; d < 3; d++) {
      chains[d] = (hop == 2 && !(g.L[d] & 1)) ? 2 : 1;
      u.c[d] = g.L[d] / chains[d];
    }
    int h = 0;
    int n = 0;
    // groups of one lattice are neighbours in the list: reuse the cut
    if (!r.units.empty() && r.units.back().Lx == u.Lx && r.units.back().Ly == u.Ly && r.units.back().Lz == u.Lz) {
      std::copy(r.units.back().b, r.units.back().b + 3, u.b);
      std::copy(r.units.back().t, r.units.back().t + 3, u.t);
      u.shape = r.units.back().shape;
      n = u.t[0] * u.t[1] * u.t[2];
    } else {
      n = cut_cell(u.c, prec, r.cfg.width, r.subs, sites, std::min(cfg.tz, tl::kRunMaxTeam), u.b, u.t, &h);
      u.shape = (int32_t)r.units.size();
      if (n == 0) return "a cell does not fit a team of workgroups";
      r.np = std::max(r.np, (u.b[0] * u.b[1] * u.b[2] + 63) / 64 * 64);
      halo = std::max(halo, h);
      r.team_size = std::max(r.team_size, n);
    }
    for (int z = 0; z < chains[2]; z++)
      for (int y = 0; y < chains[1]; y++)
        for (int x = 0; x < chains[0]; x++) {
          u.p[0] = x;
          u.p[1] = y;
          u.p[2] = z;
          r.units.push_back(u);
        }
  }
  // the largest cells first: teams take units in this order
  std::stable_sort(r.units.begin(), r.units.end(), [](const tl::RunUnit& a, const tl::RunUnit& b) {
    return (int64_t)a.c[0] * a.c[1] * a.c[2] > (int64_t)b.c[0] * b.c[1] * b.c[2];
  });
  r.cfg.grid = std::max(8, (cfg.grid > 0 ? cfg.grid : std::max(p->ctx->n_cu, 1)) / 8 * 8);
  const int per = r.cfg.grid / 8;
  if (per >= r.team_size) {
    r.n_teams = 8 * (per / r.team_size);
  } else {
    int xpt = 2;
    while (xpt < 8 && xpt * per < r.team_size) xpt *= 2;
    r.n_teams = 8 / xpt;
  }
  place_units(prec, sites, &r, &halo);
  // fetch waves: one halo entry per thread as far as the workgroup has room
  const int room = (tl::run_max_threads(prec) - r.np * r.subs) / 64, entries = r.subs * halo;
  r.cfg.fetch = std::min(room, (entries + 63) / 64);
  if (64 * tl::kFetch * r.cfg.fetch < entries) return "too many threads per workgroup";
  r.halo = halo;
  r.cfg.lds = tl::run_lds(prec, r.cfg.width, r.subs, r.np, halo);
  if (r.cfg.lds > 160 * 1024) return "tiling needs more LDS than this device allows";
  const int64_t plane = (int64_t)r.subs * r.cfg.width * tl::kRunWords[prec] * r.team_size * r.np * 16;
  if (r.n_teams > tl::kMaxRunTeams || r.cfg.grid > tl::kMaxRunGrid || plane > INT32_MAX || r.units.size() > p->res.size() * 8)
    return "work list too long for the whole-run kernel";
  r.n_shares = std::min((int)r.units.size(), r.n_teams);
  r.steps = std::max(1, kRunMaxUnitSteps / (((int)r.units.size() + r.n_shares - 1) / r.n_shares));
  r.scratch = r.cfg.fetch ? (size_t)(r.n_teams * 2 * plane) : 0;
  *out = std::move(r);
  return nullptr;
}

// Whether cfg applies to this plan (its work list exists and fits in LDS); reason on failure.
bool tiling_applies(const tl_plan* p, const StepConfig& cfg, const char** reason) {
  if (cfg.variant == 9) {
    RunShape r;
    *reason = make_run(p, cfg, &r);
    if (!*reason && !p->ctx->big_lds) *reason = "tiling needs more LDS than this device allows";
    return !*reason;
  }
  if (tl::is_one(p->prec) && cfg.variant != 0 && cfg.variant != 4 && cfg.variant != 7 && cfg.variant != 8) {
    *reason = "one-link smearing runs the step variants 0, 4, 7 and 8 only";
    return false;
  }
  if (cfg.variant >= 5 && tl::vprec(p->prec) == tl::F64 && eff_width(p, cfg) > 1) {
    *reason = "the LDS-staged step kernels take FP64 groups of one RHS only";
    return false;
  }
  if (cfg.variant == 8 && (p->flags & TL_PLAIN)) {
    *reason = "TL_PLAIN runs one step per launch";
    return false;
  }
  std::vector<StepGroup> gs;
  if (make_groups(p, cfg, &gs) != TL_OK) {
    *reason = "work list too long, or tiling not applicable to these lattices";
    return false;
  }
  const int64_t lds = plan_lds(p, cfg, gs);
  if (lds < 0 || (lds > 0 && !p->ctx->big_lds)) {
    *reason = "tiling needs more LDS than this device allows";
    return false;
  }
  return true;
}

// Device memory that starts as zeros (queued on the context's stream).
int dev_zeroed(tl_ctx* c, void** m, size_t bytes) {
  TL_TRY(dev_alloc(c, m, bytes));
  const hipError_t e = c->fault_exchange ? hipErrorOutOfMemory : hipMemsetAsync(*m, 0, bytes, c->stream);
  if (e == hipSuccess) return TL_OK;
  (void)hipGetLastError();
  (void)hipFree(*m);
  *m = nullptr;
  return fail(c, e == hipErrorOutOfMemory ? TL_ERR_NOMEM : TL_ERR_HIP, "clearing %zu bytes: %s", bytes, hipGetErrorString(e));
}

// Build a whole-run tiling: units table, control block and exchange scratch.  The control block
// and new scratch start as zeros; afterwards tags only grow, so scratch is never cleared again.
int upload_run(tl_plan* p, const StepConfig& cfg, tl_plan::Tiling* t) {
  tl_ctx* c = p->ctx;
  RunShape r;
  const char* why = make_run(p, cfg, &r);
  if (!why && !c->big_lds) why = "tiling needs more LDS than this device allows";
  if (why) return fail(c, TL_ERR_UNSUPPORTED, "%s", why);
  if (!c->run_fail) {
    if (c->fault_alloc) return fail(c, TL_ERR_NOMEM, "host allocation failed (TL_FAULT=alloc)");
    c->fail_used.resize(kFailWords, 0);
    void* h = nullptr;
    if (hipHostMalloc(&h, kFailWords * sizeof(uint32_t), hipHostMallocMapped) != hipSuccess) {
      (void)hipGetLastError();
      return fail(c, TL_ERR_NOMEM, "hipHostMalloc failed");
    }
    std::memset(h, 0, kFailWords * sizeof(uint32_t));
    c->run_fail = static_cast<uint32_t*>(h);
  }
  if (!c->run_event && hipEventCreateWithFlags(&c->run_event, hipEventDisableTiming) != hipSuccess) {
    (void)hipGetLastError();
    c->run_event = nullptr;   // without it the context's launches are not ordered
  }
  if (!p->fail) {
    const size_t k = std::find(c->fail_used.begin(), c->fail_used.end() - 1, 0) - c->fail_used.begin();
    c->fail_used[k] = 1;
    p->fail = c->run_fail + k;
  }
  if (!p->run.ctl) {
    // a pair whose scratch is large enough, else any (its scratch is replaced below)
    auto it = c->run_pool.end();
    for (auto k = c->run_pool.begin(); k != c->run_pool.end(); ++k)
      if (it == c->run_pool.end() || (it->bytes < r.scratch && k->bytes > it->bytes) ||
          (k->bytes >= r.scratch && k->bytes < it->bytes))
        it = k;
    if (it != c->run_pool.end() && !c->fault_alloc) {
      p->run = *it;
      c->run_pool.erase(it);
    } else {
      void* m = nullptr;
      TL_TRY(dev_zeroed(c, &m, sizeof(tl::RunCtl)));
      p->run.ctl = static_cast<tl::RunCtl*>(m);
    }
  }
  if (r.scratch > p->run.bytes) {
    if (p->run.scratch) {
      HIP_TRY(c, hipStreamSynchronize(c->stream));
      (void)hipFree(p->run.scratch);
    }
    p->run.scratch = nullptr;
    p->run.bytes = 0;
    void* m = nullptr;
    TL_TRY(dev_zeroed(c, &m, r.scratch));
    p->run.scratch = static_cast<char*>(m);
    p->run.bytes = r.scratch;
  }
  TL_TRY(upload(c, p->run_units, r.units.data(), r.units.size() * sizeof(tl::RunUnit)));
  t->cfg = cfg;
  t->cfg.width = 1;   // every RHS is advanced by itself
  t->lds = r.cfg.lds;
  t->n_tiles = r.n_tiles;
  t->host.clear();
  t->run = std::move(r);
  return TL_OK;
}

// Tiling t's host side for a step configuration: its work list and launch numbers.
int describe_tiling(tl_plan* p, const StepConfig& cfg, tl_plan::Tiling* t) {
  const char* why = nullptr;
  if (!tiling_applies(p, cfg, &why)) return fail(p->ctx, TL_ERR_UNSUPPORTED, "%s", why);
  std::vector<StepGroup> gs;
  (void)make_groups(p, cfg, &gs);
  if (gs.size() > p->group_cap)   // the device table holds one entry per RHS at most
    return fail(p->ctx, TL_ERR_UNSUPPORTED, "work list of %zu groups exceeds the table (%zu)", gs.size(), p->group_cap);
  t->cfg = cfg;
  t->cfg.rows64 = std::all_of(gs.begin(), gs.end(), [](const StepGroup& g) { return g.Lx == 64; }) ? 1 : 0;
  t->lds = plan_lds(p, cfg, gs);
  t->n_tiles = gs.empty() ? 0 : gs.back().tile_begin + gs.back().n_xy_tiles * gs.back().n_z_tiles;
  t->host = std::move(gs);
  return TL_OK;
}

// Build cfg's work list and upload it into tiling t's device table.
int upload_tiling(tl_plan* p, const StepConfig& cfg, tl_plan::Tiling* t) {
  if (cfg.variant == 9) return upload_run(p, cfg, t);
  TL_TRY(describe_tiling(p, cfg, t));
  return upload(p->ctx, t->dev, t->host.data(), t->host.size() * sizeof(StepGroup));
}

// The plan's tilings from a tuned pair.
int upload_tuned(tl_plan* p, const Tuned& tu) {
  if (tu.cfg.variant == 9 && p->n_steps < kRunMinSteps) return upload_tiling(p, tu.single, &p->tile);
  TL_TRY(upload_tiling(p, tu.cfg, &p->tile));
  if (tu.cfg.variant == 8) TL_TRY(upload_tiling(p, tu.single, &p->single));
  return TL_OK;
}

// One launch of tiling t over every group (batched) or over one group (plain mode, g >= 0),
// from buffer `in` to buffer `out`: one step, two for variant 8, `steps` for variant 9 (in launches
// of at most run.steps steps, the later ones in place, see plan_flips).  k: index of the launch
// in its sequence (odd launches run reversed when the tiling flips).
int plan_launch(tl_plan* p, const tl_plan::Tiling& t, hipStream_t s, const char* in, char* out, int g, int k, int steps) {
  tl_ctx* c = p->ctx;
  if (t.cfg.variant == 9) {
    tl::RunArgs a{};
    a.units = p->run_units;
    a.ctl = p->run.ctl;
    a.scratch = p->run.scratch;
    a.fail = p->fail;
    a.spins = c->fault_wait ? 0 : tl::kSpinLimit;
    a.in = in;
    a.out = out;
    a.n_units = (int32_t)t.run.units.size();
    a.n_shares = t.run.n_shares;
    a.n_teams = t.run.n_teams;
    a.team_size = t.run.team_size;
    a.np = t.run.np;
    a.subs = t.run.subs;
    a.halo = t.run.halo;
    a.hop = tl::hop_of(p->prec);
    a.w12 = tl::is_w12(p->prec);
    for (int done = 0; done < steps; done += a.n_steps, a.in = out) {
      a.n_steps = std::min(t.run.steps, steps - done);
      // the launch's time at 3 us per unit-step and share, between 100 us and 2 ms
      a.patience = c->fault_team ? 0 : (int)std::clamp<int64_t>(6 * (int64_t)a.n_steps * ((a.n_units + a.n_shares - 1) / a.n_shares), 200, 4000);
      TL_TRY(launch(c, "smearing run", [&] { return tl::launch_run(tl::vprec(p->prec), t.run.cfg, a, p->alpha, p->beta, s); }));
    }
    return TL_OK;
  }
  int base = 0, n = t.n_tiles;
  if (g >= 0) {
    base = t.host[g].tile_begin;
    n = t.host[g].n_xy_tiles * t.host[g].n_z_tiles;
  }
  StepConfig cfg = t.cfg;
  cfg.rev = (cfg.flip && (k & 1)) ? 1 : 0;
  return launch(c, "smearing step", [&] {
    return tl::launch_step(p->prec, eff_width(p, cfg), cfg, t.dev, (int)t.host.size(), base, n, in, out, p->alpha, p->beta,
                           t.lds, s);
  });
}

int plan_step(tl_plan* p, hipStream_t s, int parity, int g, int k, int steps = 1) {
  return plan_launch(p, p->tile, s, p->buf[parity], p->buf[parity ^ 1], g, k, steps);
}

// Whether a run of the n steps ends in the other resident buffer: every step or two-step launch
// goes from one to the other.  A whole run ends where n one-step launches would, so that a
// captured run of an even number of steps advances the field with every replay.  It may write the
// buffer it reads, because a site is read and written by the one thread that holds it (its
// neighbours get it through the exchange words), and read before anything is written.
bool plan_flips(const tl_plan* p) {
  return (p->tile.cfg.variant == 8 ? p->n_steps / 2 + (p->n_steps & 1) : p->n_steps) & 1;
}

// The share of every CU that a whole-run launch takes (registers by its waves, LDS).
double run_load(const RunShape& r, int prec) {
  const double waves = (double)(r.np * r.subs + 64 * r.cfg.fetch) / tl::run_max_threads(tl::vprec(prec));
  return std::max(waves, (double)r.cfg.lds / (160 * 1024));
}

// Queue the n steps starting from buffer `parity` on stream s.
int plan_enqueue(tl_plan* p, hipStream_t s, int parity) {
  if (p->flags & TL_PLAIN) {
    for (int g = 0; g < (int)p->tile.host.size(); g++) {
      int q = parity;
      for (int k = 0; k < p->n_steps; k++) {
        TL_TRY(plan_step(p, s, q, g, k));
        q ^= 1;
      }
    }
  } else if (p->tile.cfg.variant == 9) {
    TL_TRY(plan_launch(p, p->tile, s, p->buf[parity], p->buf[plan_flips(p) ? parity ^ 1 : parity], -1, 0, p->n_steps));
  } else if (p->tile.cfg.variant == 8) {
    int q = parity;
    for (int k = 0; k < p->n_steps / 2; k++) {
      TL_TRY(plan_step(p, s, q, -1, k));
      q ^= 1;
    }
    if (p->n_steps & 1) TL_TRY(plan_launch(p, p->single, s, p->buf[q], p->buf[q ^ 1], -1, 0, 1));
  } else {
    int q = parity;
    for (int k = 0; k < p->n_steps; k++) {
      TL_TRY(plan_step(p, s, q, -1, k));
      q ^= 1;
    }
  }
  return TL_OK;
}

// What a plan's tuned tiling depends on.  "c2" is the set of candidates: entries of a cache file
// from before whole-run launches do not name it and are tuned again.  Batched plans name the power
// of two below n (32 at most; 2 also for 3 steps): fewer than two steps have no two-step and fewer
// than four no whole-run candidates, and those spread what a run costs once (about 10 us) over n.
std::string tune_key(const tl_plan* p) {
  std::string k = p->ctx->arch + "|c2|p" + std::to_string(p->prec) + "|w" + std::to_string(p->width) +
                  ((p->flags & TL_PLAIN) ? "|plain" : "|batch") + ((p->flags & TL_ONE_STEP) ? "|one" : "");
  if (!(p->flags & (TL_PLAIN | TL_ONE_STEP))) {
    int n = 1;
    while (n < 32 && 2 * n <= p->n_steps) n *= 2;
    k += "|n" + std::to_string(n);
  }
  for (const auto& g : p->groups) {
    const tl_geom& ge = p->jobs[g.job].job.g;
    k += "|" + std::to_string(ge.L[0]) + "x" + std::to_string(ge.L[1]) + "x" + std::to_string(ge.L[2]) + ":" +
         std::to_string(g.nr);
  }
  return k;
}

// Captures what enqueue(stream) queues in a graph.
template <class F>
int capture_graph(tl_ctx* c, hipGraphExec_t* exec, F&& enqueue) {
  hipStream_t cs = nullptr;
  HIP_TRY(c, hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
  hipGraph_t graph = nullptr;
  int rc = TL_OK;
  if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    rc = fail(c, TL_ERR_HIP, "hipStreamBeginCapture failed");
  } else {
    rc = enqueue(cs);
    hipError_t e = hipStreamEndCapture(cs, &graph);
    if (rc == TL_OK && e != hipSuccess) rc = fail(c, TL_ERR_HIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
  }
  if (rc == TL_OK) {
    hipError_t e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    if (e != hipSuccess) rc = fail(c, TL_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
  }
  if (graph) (void)hipGraphDestroy(graph);
  (void)hipStreamDestroy(cs);
  return rc;
}

int plan_capture(tl_plan* p, int parity) {
  if (p->graph[parity]) return TL_OK;
  TL_TRY(capture_graph(p->ctx, &p->graph[parity], [&](hipStream_t cs) { return plan_enqueue(p, cs, parity); }));
  p->ctx->stats.graphs_captured++;
  return TL_OK;
}

// Time every candidate tiling on the plan's own data (buffer cur -> cur^1,
// which leaves the input untouched), require each candidate's output to be
// bit-identical to the first candidate's, keep the fastest.  Then, for batched
// plans of two or more steps, time the two-step tilings against two launches
// of that winner (output bit-identical to them, time per step compared).
int plan_autotune(tl_plan* p) {
  tl_ctx* c = p->ctx;
  const std::string key = tune_key(p);
  auto hit = c->tune.find(key);
  if (hit != c->tune.end()) {
    // a cached tiling that does not apply to this plan (a cache file written by another
    // version of the library, or edited) is dropped and the plan tuned again
    const char* why = nullptr;
    const Tuned& tu = hit->second;
    if (tiling_applies(p, tu.cfg, &why) && (tu.cfg.variant < 8 || tiling_applies(p, tu.single, &why))) {
      c->stats.tune_hits++;
      const int rc = upload_tuned(p, tu);
      return rc == TL_ERR_NOMEM && tu.cfg.variant == 9 ? upload_tiling(p, tu.single, &p->tile) : rc;
    }
    if (c->log) fprintf(stderr, "[twolink] tune %s: cached tiling %s does not apply (%s), tuning again\n", key.c_str(),
                        cfg_text(tu.cfg).c_str(), why);
    c->tune.erase(hit);
  }
  c->stats.tune_sweeps++;
  std::vector<StepConfig> cands, cands2;
  const int cu = std::max(c->n_cu, 1);
  // the plan's RHS groups, and (batched plans with wider groups) every RHS on its own tiles:
  // more parallel work for small lattices at the price of loading each two-link once per RHS
  std::vector<int> widths{0};
  if (!(p->flags & TL_PLAIN) && p->width > 1) widths.push_back(1);
  for (int wd : widths)
    for (int variant : {0, 2, 3, 4, 5, 6, 7}) {
      const bool lds_variant = variant >= 5;
      const int ew = wd > 0 ? wd : p->width;
      if (tl::is_one(p->prec) && variant != 0 && variant != 4 && variant != 7) continue;   // one-link: hops of one site
      if ((variant == 2 || variant == 3 || lds_variant) && tl::vprec(p->prec) == tl::F64 && ew > 1) continue;   // would run variant 0
      if (lds_variant && !c->big_lds) continue;
      const std::vector<int> tzs = (variant == 0 || variant == 4) ? std::vector<int>{1, 2, 4}
                                   : (variant >= 6 ? std::vector<int>{4, 8, 16} : std::vector<int>{8, 16, 32});
      const std::vector<int> blocks = lds_variant ? std::vector<int>{512, 256} : std::vector<int>{256, 128, 64};
      for (int block : blocks)
        for (int tz : tzs)
          for (int grid : {0, cu, 8 * cu})   // one workgroup per tile, or persistent: 1 or 8 per CU
            for (int nt : {0, 1})
              for (int flip : {0, 1}) {
                StepConfig g{variant, block, tz, grid, nt, flip, 0};
                g.width = wd;
                cands.push_back(g);
              }
    }
  if (!(p->flags & (TL_PLAIN | TL_ONE_STEP)) && p->n_steps >= 2 && c->big_lds &&
      !(tl::vprec(p->prec) == tl::F64 && p->width > 1))
    for (int block : {512, 448, 384, 320, 256})
      for (int tz : {4, 8, 16, 32})
        for (int grid : {0, cu})
          for (int nt : {0, 1})
            for (int flip : {0, 1}) cands2.push_back({8, block, tz, grid, nt, flip, 0});
  // whole-run launches: every team size that changes the cut, RHS of a group sharing threads or not
  std::vector<StepConfig> cands9;
  if (!(p->flags & (TL_PLAIN | TL_ONE_STEP)) && p->n_steps >= kRunMinSteps && c->big_lds)
    for (int subs = 1; subs <= 3; subs++)   // one set of threads per group, two, one per RHS
      for (int block : {512, 256})
        for (int team : {1, 2, 4, 8, 16, 32, 64, 128, 256})
          if (subs == 1 || (subs == 2 ? p->width > 2 : p->width > 1))
            cands9.push_back({9, block, team, 0, subs == 2, subs == 3, 0});
  void* ref = nullptr;
  void* flag_mem = nullptr;
  TL_TRY(dev_alloc(c, &ref, p->buf_bytes));
  int rc = dev_alloc(c, &flag_mem, 256);
  if (rc != TL_OK) {
    (void)hipFree(ref);
    return rc;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
    rc = fail(c, TL_ERR_HIP, "hipEventCreate failed");
  // Batched plans time their one launch per step.  Plain plans (one launch per group) time one
  // group of each distinct lattice shape and weigh it by the number of groups of that shape,
  // so that the tiling suits every shape of the batch, not only the first.
  std::vector<std::pair<int, int>> timed{{-1, 1}};   // (group, weight); -1: every group at once
  if (p->flags & TL_PLAIN) {
    timed.clear();
    for (int g = 0; g < (int)p->groups.size(); g++) {
      const tl_geom& ge = p->jobs[p->groups[g].job].job.g;
      bool seen = false;
      for (auto& tw : timed) {
        const tl_geom& gt = p->jobs[p->groups[tw.first].job].job.g;
        if (gt.L[0] == ge.L[0] && gt.L[1] == ge.L[1] && gt.L[2] == ge.L[2] && p->groups[tw.first].nr == p->groups[g].nr) {
          tw.second++;
          seen = true;
          break;
        }
      }
      if (!seen) timed.push_back({g, 1});
    }
  }
  // time reps launches of p->tile (after two untimed) for each timed group, then compare the
  // output with ref (have_ref false: keep it as ref instead); ms: per launch
  const int whole = std::min(p->n_steps, kTuneSteps);
  auto trial = [&](bool have_ref, float* ms, bool* same, int warm = 2, int reps = 10) -> int {
    *ms = 0.0f;
    for (const auto& tw : timed) {
      for (int w = 0; w < warm; w++) TL_TRY(plan_step(p, c->stream, p->cur, tw.first, w, whole));
      (void)hipEventRecord(e0, c->stream);
      for (int k = 0; k < reps; k++) TL_TRY(plan_step(p, c->stream, p->cur, tw.first, k, whole));
      (void)hipEventRecord(e1, c->stream);
      if (hipEventSynchronize(e1) != hipSuccess) return fail(c, TL_ERR_HIP, "autotune timing failed");
      float t = 0.0f;
      (void)hipEventElapsedTime(&t, e0, e1);
      *ms += t / reps * tw.second;
    }
    *same = true;
    if (!have_ref) {
      if (hipMemcpyAsync(ref, p->buf[p->cur ^ 1], p->buf_bytes, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
        return fail(c, TL_ERR_HIP, "autotune reference copy failed");
    } else {
      int one = 0;
      (void)hipMemsetAsync(flag_mem, 0, sizeof(int), c->stream);
      (void)tl::launch_compare(static_cast<const char*>(ref), p->buf[p->cur ^ 1], (int64_t)p->buf_bytes,
                               static_cast<int*>(flag_mem), c->stream);
      (void)hipMemcpyAsync(&one, flag_mem, sizeof(int), hipMemcpyDeviceToHost, c->stream);
      (void)hipStreamSynchronize(c->stream);
      *same = one == 0;
    }
    return TL_OK;
  };
  auto log = [&](const StepConfig& g, float ms_step, bool same) {
    if (c->log)
      fprintf(stderr, "[twolink] tune %s variant=%d block=%d tz=%d grid=%d nt=%d flip=%d width=%d: %.4f ms/step%s\n",
              key.c_str(), g.variant, g.block, g.tz, g.grid, g.nt, g.flip, eff_width(p, g), ms_step,
              same ? "" : "  OUTPUT DIFFERS - rejected");
  };
  float best = 1e30f;
  StepConfig best_cfg = cands[0];
  bool have_ref = false;
  for (size_t ci = 0; ci < cands.size() && rc == TL_OK; ci++) {
    const char* why = nullptr;
    if (!tiling_applies(p, cands[ci], &why)) continue;
    rc = upload_tiling(p, cands[ci], &p->tile);
    if (rc != TL_OK) break;
    float ms = 0.0f;
    bool same = true;
    rc = trial(have_ref, &ms, &same);
    if (rc != TL_OK) break;
    have_ref = true;
    log(p->tile.cfg, ms, same);
    if (same && ms < best) {
      best = ms;
      best_cfg = p->tile.cfg;
    }
  }
  Tuned tu;
  tu.cfg = best_cfg;
  if (rc == TL_OK && !cands2.empty()) {
    // reference: two launches of the one-step winner, buffer cur -> cur^1 -> ref
    rc = upload_tiling(p, best_cfg, &p->single);
    if (rc == TL_OK) rc = plan_launch(p, p->single, c->stream, p->buf[p->cur], p->buf[p->cur ^ 1], -1, 0, 1);
    if (rc == TL_OK) rc = plan_launch(p, p->single, c->stream, p->buf[p->cur ^ 1], static_cast<char*>(ref), -1, 1, 1);
    float best2 = 1e30f;
    StepConfig best2_cfg{};
    for (size_t ci = 0; ci < cands2.size() && rc == TL_OK; ci++) {
      const char* why = nullptr;
      if (!tiling_applies(p, cands2[ci], &why)) continue;
      rc = upload_tiling(p, cands2[ci], &p->tile);
      if (rc != TL_OK) break;
      float ms = 0.0f;
      bool same = true;
      rc = trial(true, &ms, &same);
      if (rc != TL_OK) break;
      log(p->tile.cfg, ms / 2, same);
      if (same && ms / 2 < best2) {
        best2 = ms / 2;
        best2_cfg = p->tile.cfg;
      }
    }
    if (rc == TL_OK && best2 < best) {
      tu.cfg = best2_cfg;
      tu.single = best_cfg;
      best = best2;
    }
  }
  if (rc == TL_OK && !cands9.empty()) {
    // whole-run launches (all n steps each, up to kTuneSteps), against as many launches of the
    // one-step winner from buffer to buffer.  The winner so far is timed over such a run too (launches
    // that all read one buffer find their input in the caches, those of a run do not), replayed from
    // a graph if the plan's runs are.
    rc = upload_tiling(p, best_cfg, &p->single);
    if (rc == TL_OK && tu.cfg.variant == 8) rc = upload_tiling(p, tu.cfg, &p->tile);
    char* pair[2] = {p->buf[p->cur ^ 1], static_cast<char*>(ref)};
    auto sequence = [&](const tl_plan::Tiling& t, int launches, hipStream_t s) -> int {
      for (int k = 0; k < launches; k++)
        TL_TRY(plan_launch(p, t, s, k ? pair[(k - 1) & 1] : p->buf[p->cur], pair[k & 1], -1, k, 1));
      return TL_OK;
    };
    const tl_plan::Tiling& winner = tu.cfg.variant == 8 ? p->tile : p->single;
    const int launches = tu.cfg.variant == 8 ? whole / 2 : whole;
    hipGraphExec_t replay = nullptr;
    if (rc == TL_OK && (p->flags & TL_GRAPH))
      rc = capture_graph(c, &replay, [&](hipStream_t s) { return sequence(winner, launches, s); });
    for (int rep = 0; rep < 2 && rc == TL_OK; rep++) {   // one untimed
      const int runs = replay ? 1 + 2 * rep : 1;
      (void)hipEventRecord(e0, c->stream);
      for (int k = 0; k < runs && rc == TL_OK; k++) {
        if (!replay) rc = sequence(winner, launches, c->stream);
        else if (hipGraphLaunch(replay, c->stream) != hipSuccess) rc = fail(c, TL_ERR_HIP, "autotune graph launch failed");
      }
      (void)hipEventRecord(e1, c->stream);
      float ms = 0.0f;
      if (rc == TL_OK && (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        rc = fail(c, TL_ERR_HIP, "autotune timing failed");
      best = ms / (runs * (tu.cfg.variant == 8 ? whole / 2 * 2 : whole));
    }
    if (replay) (void)hipGraphExecDestroy(replay);
    if (rc == TL_OK) rc = sequence(p->single, whole, c->stream);
    if (rc == TL_OK && (whole & 1) &&
        hipMemcpyAsync(ref, pair[0], p->buf_bytes, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
      rc = fail(c, TL_ERR_HIP, "autotune reference copy failed");
    float best9 = 1e30f;
    StepConfig best9_cfg{};
    for (size_t ci = 0; ci < cands9.size() && rc == TL_OK; ci++) {
      const char* why = nullptr;
      if (!tiling_applies(p, cands9[ci], &why)) continue;
      rc = upload_tiling(p, cands9[ci], &p->tile);
      if (rc == TL_ERR_NOMEM) {   // no exchange memory: not a candidate
        rc = TL_OK;
        continue;
      }
      if (rc != TL_OK) break;
      float ms = 0.0f;
      bool same = true;
      rc = trial(true, &ms, &same, 1, 3);
      if (rc != TL_OK) break;
      if (fail_taken(p->fail)) same = false;   // it gave up waiting: not a candidate
      log(p->tile.cfg, ms / whole, same);
      if (same && ms / whole < best9) {
        best9 = ms / whole;
        best9_cfg = p->tile.cfg;
      }
    }
    if (rc == TL_OK && best9 < best) {
      tu.cfg = best9_cfg;
      tu.single = best_cfg;
    }
  }
  (void)hipStreamSynchronize(c->stream);
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(ref);
  (void)hipFree(flag_mem);
  if (rc != TL_OK) return rc;
  c->tune[key] = tu;
  if (!c->tune_file.empty()) tune_file_save(c);
  return upload_tuned(p, tu);
}

// TL_TILE="variant,block,tz,grid[,nt[,flip]]" fixes the step tiling of every plan (no tuning):
// used to profile or sweep one tiling at a time.  A two-step tiling (variant 8) may name its
// one-step companion after a ";" (default: variant 0, 256 threads, tz 4).
bool tile_override(Tuned* tu) {
  const char* e = getenv("TL_TILE");
  return e && parse_tuned(e, 4, tu);
}

// Microseconds of a plan's run in one launch, and in n launches of the direct kernel: estimates for
// default_run, fitted to 4500 measured points (4^3 to 96^3, odd extents, 1 to 96 slices of 1 to 4
// RHS, every format, 4 to 32 steps).  A whole-run launch costs a few us, each round of units its
// link loads and then a step for every step: both grow with the waves per SIMD and the RHS per
// thread, and for teams over several XCDs.  A direct launch costs what its bytes or its arithmetic
// take, and never less than the chain of a tile's loads and products.
double run_estimate(const tl_plan* p, const RunShape& r, bool* one_round) {
  const bool f64 = tl::vprec(p->prec) == tl::F64;
  const double w = r.cfg.width;
  double longest = 0.0;
  *one_round = true;
  for (int share = 0; share < r.n_shares; share++) {   // a team takes every n_shares-th unit
    double us = 6.0;
    int rounds = 0, shape = -1;
    for (size_t u = share; u < r.units.size(); u += r.n_shares) {
      const tl::RunUnit& g = r.units[u];
      if (g.first != 0) continue;   // runs beside the one before
      const int waves = ((g.b[0] * g.b[1] * g.b[2] + 63) / 64 * r.subs + 3) / 4;
      const bool across = g.span > r.cfg.grid / 8;
      double step = f64 ? 0.7 + 1.2 * w + 0.5 * waves + (across ? 1.8 : 0.0) : 0.5 + w * (0.5 + 0.1 * waves) + (across ? 0.5 : 0.0);
      double once = 4.0 + 3.0 * waves + 0.8 * w + (across ? 3.0 : 0.0);
      if (g.t[0] * g.t[1] * g.t[2] == 1) {   // nothing to exchange
        step *= 0.7;
        once = 4.0 * waves;
      }
      if (shape >= 0 && g.shape != shape) once += across ? 8.0 : 3.0;   // a team barrier
      shape = g.shape;
      us += once + p->n_steps * step;
      rounds++;
    }
    longest = std::max(longest, us);
    *one_round = *one_round && rounds == 1;
  }
  return longest;
}
double direct_estimate(const tl_plan* p) {
  const int vp = tl::vprec(p->prec);
  const double w = p->width;
  const double chain = vp == tl::F64 ? 5.0 + 9.0 * w : 4.5 + 2.5 * w;
  const double tbs = vp == tl::F64 ? 4.0 : 4.6;
  const double tflops = vp == tl::F64 ? 5.5 - 0.5 * w : vp == tl::F32 ? 15.0 : vp == tl::F16S ? 19.0 : 28.0;
  const double work = std::max(p->info.bytes_per_step / tbs, p->info.flops_per_step / tflops) * 1e-6;
  return p->n_steps * std::max(chain, 0.5 * chain + work);
}

// The tiling of a plan that is neither tuned nor fixed: all steps in one launch where the cells
// fit teams of one XCD (up to 32 workgroups) or a few, else the direct kernel, one step per
// launch.  Where one round of units does all the work one launch was faster at every point measured
// from four steps on (20 steps of 16^3 FP32 3 RHS: 50 instead of 350 us).  With several rounds of
// few steps the link loads of each round can cost more than they save (4 steps of 96 slices of
// 33x33x17 BF16 1 RHS: 368 instead of 202 us), so there the estimates decide: of the 4500 points
// three then take longer than with the other choice's time, by 17% at most (95, by up to 2.2
// times, with one launch for all), and two of 134 random batches of 1 to 24 lattices, by 33%.  Team size: every unit
// at once if the chip has room, a wave or more of sites per tile; FP64 threads hold one RHS
// where that fits (its registers are full with one).
bool default_run(const tl_plan* p, StepConfig* cfg) {
  if ((p->flags & (TL_PLAIN | TL_ONE_STEP)) || p->n_steps < kRunMinSteps || !p->ctx->big_lds) return false;
  int64_t units = 0, sites = 1;
  for (const auto& gr : p->groups) {
    const tl_geom& g = p->jobs[gr.job].job.g;
    int64_t cell = 1, cells = 1;
    for (int d = 0; d < 3; d++) {
      const int ch = (tl::hop_of(p->prec) == 2 && !(g.L[d] & 1)) ? 2 : 1;
      cells *= ch;
      cell *= g.L[d] / ch;
    }
    units += cells;
    sites = std::max(sites, cell);
  }
  int team = 1;
  while (team < 32 && 2 * team * units <= std::max(p->ctx->n_cu, 8) && sites / (2 * team) >= 64) team *= 2;
  RunShape r;
  for (; team <= 256; team *= 2)
    for (int split : {1, 0})
      if (split == (tl::vprec(p->prec) == tl::F64 && p->width > 1) || (!split && tl::vprec(p->prec) == tl::F64)) {
        *cfg = {9, 512, team, 0, 0, split, 0};
        if (make_run(p, *cfg, &r)) continue;
        bool one_round = false;
        const double us = run_estimate(p, r, &one_round);
        return one_round || us < direct_estimate(p);
      }
  return false;
}

// The tiling of an untuned plan, made ready when the plan is created, so that its first run
// queues launches only and may be captured by the caller.  Step launches need no exchange memory,
// so they serve where there is none.
int prepare_untuned(tl_plan* p) {
  StepConfig run{};
  if (default_run(p, &run)) {
    const int rc = upload_run(p, run, &p->tile);
    if (rc != TL_ERR_NOMEM) return rc;
  }
  return upload_tiling(p, p->tile.cfg, &p->tile);
}

int plan_prepare(tl_plan* p) {
  if (p->ready) return TL_OK;
  Tuned forced;
  if (tile_override(&forced)) {
    TL_TRY(need_eager(p->ctx, "first run of a plan (TL_TILE)"));
    TL_TRY(upload_tuned(p, forced));
  } else if (p->flags & TL_AUTOTUNE) {
    TL_TRY(need_eager(p->ctx, "first run of a plan (TL_AUTOTUNE)"));
    TL_TRY(plan_autotune(p));
  }
  p->ready = true;
  return TL_OK;
}

// The same for a plan's whole-run memory: at most four pairs, 256 MB of scratch in all, are kept.
void run_put(tl_ctx* c, bool keep, RunMem m) {
  size_t held = m.bytes;
  for (const auto& k : c->run_pool) held += k.bytes;
  if (keep && c->run_pool.size() < 4 && held <= kPoolBytes) {
    try {
      c->run_pool.push_back(m);
      return;
    } catch (...) {
    }
  }
  run_free(m);
}

// Waits for the plan's work: afterwards its memory and the jobs' fields may go, on whatever
// stream they are used next.  A caller may have captured a created plan's calls and replay them on
// streams the context does not know, so there the whole device is waited for (which hipFree would
// do as well).  Returns whether a whole-run launch of the plan gave up unreported.
bool plan_free(tl_plan* p) {
  if (!p) return false;
  bool failed = false;
  if (p->ctx && p->ctx->device >= 0) {
    DeviceGuard dg(p->ctx->device);
    tl_ctx* c = p->ctx;
    const bool idle = (p->of_call ? hipStreamSynchronize(c->stream) : hipDeviceSynchronize()) == hipSuccess;
    if (!idle) (void)hipGetLastError();   // the blocks then go back through hipFree
    RunTurn::idle(c);
    failed = fail_taken(p->fail);
    for (auto& g : p->graph)
      if (g) (void)hipGraphExecDestroy(g);
    for (int k = 0; k < 2; k++) mem_put(c, idle, p->buf[k], p->buf_cap[k]);
    mem_put(c, idle, p->tables, p->tables_cap);
    if (p->run.ctl) run_put(c, idle, p->run);
    if (p->fail) {
      const size_t k = p->fail - c->run_fail;
      if (k + 1 < kFailWords) c->fail_used[k] = 0;
    }
  }
  delete p;
  return failed;
}

}  // namespace

// ====================================================================== C ABI

extern "C" {

int tl_version(void) { return 10100; }

int tl_create(tl_ctx** out, int device, void* stream) {
  tl_ctx* c = nullptr;
  try {
    if (!out) return fail(nullptr, TL_ERR_ARG, "out is NULL");
    *out = nullptr;
    c = new (std::nothrow) tl_ctx();
    if (!c) return fail(nullptr, TL_ERR_NOMEM, "host allocation failed");
    const char* lg = getenv("TL_LOG");
    c->log = lg && lg[0] == '1';
    const char* tf = getenv("TL_TUNE_CACHE");
    if (tf && tf[0]) {
      c->tune_file = tf;
      tune_file_load(c);
    }
    const char* fl = getenv("TL_FAULT");
    if (fl) {
      c->fault_alloc = strcmp(fl, "alloc") == 0;
      c->fault_launch = strcmp(fl, "launch") == 0;
      c->fault_exchange = strcmp(fl, "exchange") == 0;
      c->fault_team = strcmp(fl, "team") == 0;
      c->fault_wait = strcmp(fl, "wait") == 0;
    }
    if (device == -1) {
      c->device = -1;
      *out = c;
      return TL_OK;
    }
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || device < 0 || device >= n) {
      delete c;
      c = nullptr;
      return fail(nullptr, TL_ERR_DEVICE, "device %d not available (%d devices%s%s)", device, e == hipSuccess ? n : 0,
                  e == hipSuccess ? "" : ": ", e == hipSuccess ? "" : hipGetErrorString(e));
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
      delete c;
      c = nullptr;
      return fail(nullptr, TL_ERR_DEVICE, "hipGetDeviceProperties(%d) failed", device);
    }
    {
      // the LDS-staged step kernels need more than the default dynamic-LDS limit;
      // without it their tilings are simply not offered
      DeviceGuard dg(device);
      if (!dg.ok) {
        delete c;
        c = nullptr;
        return fail(nullptr, TL_ERR_DEVICE, "hipSetDevice(%d) failed", device);
      }
      c->big_lds = tl::init_kernel_attributes() == hipSuccess;
      (void)hipGetLastError();
      // the fixed device area of tl_reduce_noalloc: its address on this device, looked up
      // once per device; a failure here only disables that entry point
      const hipError_t ne = tl::noalloc_scratch_init(device);
      c->noalloc = tl::noalloc_scratch(device);
      if (ne != hipSuccess || !c->noalloc) {
        c->noalloc = nullptr;
        c->noalloc_err = std::string("hipGetSymbolAddress: ") + hipGetErrorString(ne);
        (void)hipGetLastError();
      }
    }
    c->stream = static_cast<hipStream_t>(stream);
    c->n_cu = prop.multiProcessorCount;
    c->arch = prop.gcnArchName;
    c->lane = &run_lane(device);
    {
      std::lock_guard<std::mutex> lock(c->lane->m);
      c->lane->ctxs.push_back(c);
    }
    c->device = device;
    *out = c;
    return TL_OK;
  } catch (...) {   // a half-built context is released; *out stays NULL
    if (out) *out = nullptr;
    delete c;
    return host_failure(nullptr);
  }
}

int tl_destroy(tl_ctx* c) {
  try {
    if (!c) return TL_ERR_ARG;
    for (auto& sp : c->smear_plans) plan_free(sp.second);
    c->smear_plans.clear();
    if (c->device >= 0) {
      DeviceGuard dg(c->device);   // teardown goes on even if the switch fails
      (void)hipStreamSynchronize(c->stream);
      if (c->scratch) (void)hipFree(c->scratch);
      mem_drain(c);
      if (c->run_fail) (void)hipHostFree(c->run_fail);
      std::lock_guard<std::mutex> lock(c->lane->m);
      auto& all = c->lane->ctxs;
      all.erase(std::remove(all.begin(), all.end(), c), all.end());
      if (c->run_event) (void)hipEventDestroy(c->run_event);
    }
    delete c;
    return TL_OK;
  } catch (...) {
    return host_failure(nullptr);
  }
}

int tl_set_stream(tl_ctx* c, void* stream) {
  try {
    if (!c) return TL_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (c->device >= 0 && s != c->stream) {
      // Context scratch and plan buffers are reused in stream order.  Work already queued on
      // the old stream may still read them, so the new stream waits for it (an event, no host
      // wait) before anything queued through this context runs there.
      TL_ON_DEVICE(c);
      hipEvent_t ev = nullptr;
      HIP_TRY(c, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
      hipError_t e = hipEventRecord(ev, c->stream);
      if (e == hipSuccess) e = hipStreamWaitEvent(s, ev, 0);
      (void)hipEventDestroy(ev);
      if (e != hipSuccess) return fail(c, TL_ERR_HIP, "ordering the new stream after the old: %s", hipGetErrorString(e));
    }
    c->stream = s;
    return TL_OK;
  } catch (...) {
    return host_failure(c);
  }
}

int tl_sync(tl_ctx* c) {
  try {
    if (!c) return TL_ERR_ARG;
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    HIP_TRY(c, hipGetLastError());
    RunTurn::idle(c);
    bool failed = false;
    if (c->run_fail)
      for (size_t k = 0; k < kFailWords; k++) failed = fail_taken(c->run_fail + k) || failed;
    return failed ? run_failure(c) : TL_OK;
  } catch (...) {
    return host_failure(c);
  }
}

const char* tl_last_error(const tl_ctx* c) { return c ? c->err.c_str() : g_create_err.c_str(); }

int tl_check_geom(const tl_geom* g) {
  try {
    tl_ctx tmp;
    return check_geom(&tmp, g);
  } catch (...) {
    return host_failure(nullptr);
  }
}

size_t tl_twolinks_bytes(const tl_geom* g, int prec, int n_slices) {
  if (tl_check_geom(g) != TL_OK || !valid_prec(prec) || n_slices < 0 || n_slices > g->L[3]) return 0;
  return (size_t)n_slices * 3 * (size_t)tl::padded_sites(vol3(*g)) * tl::kWBytes[fmt_code(prec)];
}

namespace {

// Shared by tl_build_twolinks (two-links, no TL_ONELINK bit) and tl_pack_links (one-links,
// TL_ONELINK bit required).
int build_links(tl_ctx* c, const tl_geom* g, const void* U, const int32_t* slices, int n_slices, int prec,
                void* W, bool one) {
  if (!c) return TL_ERR_ARG;
  TL_TRY(check_geom(c, g));
  if (!valid_prec(prec)) return fail(c, TL_ERR_PRECISION, "unknown precision %d", prec);
  if (tl::is_one(fmt_code(prec)) != one)
    return fail(c, TL_ERR_PRECISION, one ? "tl_pack_links needs TL_ONELINK in prec"
                                         : "TL_ONELINK fields are built by tl_pack_links");
  if (!U || !W) return fail(c, TL_ERR_ARG, "U and W must be non-NULL device pointers");
  if (!slices) {
    if (n_slices != 0 && n_slices != g->L[3])
      return fail(c, TL_ERR_ARG, "slices is NULL but n_slices = %d (expected 0 or Lt = %d)", n_slices, g->L[3]);
    n_slices = g->L[3];
  } else {
    if (n_slices < 1 || n_slices > g->L[3])
      return fail(c, TL_ERR_ARG, "n_slices = %d outside [1, Lt=%d]", n_slices, g->L[3]);
    std::vector<char> seen(g->L[3], 0);
    for (int j = 0; j < n_slices; j++) {
      if (slices[j] < 0 || slices[j] >= g->L[3])
        return fail(c, TL_ERR_SHAPE, "slices[%d] = %d outside [0, %d)", j, slices[j], g->L[3]);
      if (seen[slices[j]]++) return fail(c, TL_ERR_ARG, "slice %d listed twice", slices[j]);
    }
  }
  TL_TRY(need_device(c));
  TL_ON_DEVICE(c);
  const int code = fmt_code(prec);
  if (!slices) return launch(c, "two-link build", [&] { return tl::launch_build(code, U, g->L, 0, 0, n_slices, W, c->stream); });
  // runs of consecutive slices share a launch
  int j = 0;
  while (j < n_slices) {
    int k = j + 1;
    while (k < n_slices && slices[k] == slices[k - 1] + 1) k++;
    TL_TRY(launch(c, "two-link build", [&] { return tl::launch_build(code, U, g->L, slices[j], j, k - j, W, c->stream); }));
    j = k;
  }
  return TL_OK;
}

}  // namespace

int tl_build_twolinks(tl_ctx* c, const tl_geom* g, const void* U, const int32_t* slices, int n_slices, int prec,
                      void* W) {
  try {
    return build_links(c, g, U, slices, n_slices, prec, W, false);
  } catch (...) {
    return host_failure(c);
  }
}

int tl_pack_links(tl_ctx* c, const tl_geom* g, const void* U, const int32_t* slices, int n_slices, int prec,
                  void* W) {
  try {
    return build_links(c, g, U, slices, n_slices, prec, W, true);
  } catch (...) {
    return host_failure(c);
  }
}

// Slices up to this many sites take the Laplacian in one launch on the natural fields, which reads
// each neighbour's 48 bytes; a larger one no longer finds most of them in the caches, and a field of
// 16-bit vectors is then packed first.  us, one launch against pack, step and unpack: F16S 104^3
// (1.1 M sites) 83 / 86, 112^3 122 / 94, 192^3 664 / 454; BF16 104^3 63 / 77, 112^3 97 / 86, 192^3
// 536 / 419.  FP32 and FP64 fields stay ahead or level in one launch up to 47 M sites (256^3 1663 / 1651 and
// 2699 / 3446).
constexpr int64_t kLapNaturalSites = 1200000;

int tl_laplacian(tl_ctx* c, const tl_geom* g, const void* W, const int32_t* w_slices, int n_w_slices, int prec,
                 int t, const void* in, void* out) {
  try {
    if (!c) return TL_ERR_ARG;
    TL_TRY(check_geom(c, g));
    if (!valid_prec(prec)) return fail(c, TL_ERR_PRECISION, "unknown precision %d", prec);
    if (!W || !in || !out) return fail(c, TL_ERR_ARG, "W, in and out must be non-NULL device pointers");
    TL_TRY(check_wslices(c, *g, w_slices, n_w_slices));
    const int slot = slot_of(*g, w_slices, n_w_slices, t);
    if (slot < 0) return fail(c, TL_ERR_SHAPE, "slice t = %d is not in the two-link field", t);
    const int64_t V3 = vol3(*g), Vp = tl::padded_sites(V3);
    const size_t nat_bytes = (size_t)V3 * 48;
    const char* a = static_cast<const char*>(in);
    const char* b = static_cast<const char*>(out);
    if (a < b + nat_bytes && b < a + nat_bytes) return fail(c, TL_ERR_ARG, "in and out overlap");
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    const int code = fmt_code(prec);
    const char* slice = static_cast<const char*>(W) + (int64_t)slot * 3 * Vp * tl::kWBytes[code];
    // Lap = alpha in + beta sum_hops: two-link -3/2, 1/4 (eq. tlLapl1); one-link -6, 1 (H - 6)
    const double la = tl::is_one(code) ? -6.0 : -1.5, lb = tl::is_one(code) ? 1.0 : 0.25;
    const int vp = tl::vprec(code);
    if ((vp != tl::F16S && vp != tl::BF16) || V3 <= kLapNaturalSites)
      return launch(c, "laplacian", [&] { return tl::launch_laplacian(code, slice, (int)Vp, g->L, in, out, la, lb, c->stream); });
    // pack, one step, unpack on context scratch (which a captured launch must not hold)
    TL_TRY(need_eager(c, "tl_laplacian of a large slice"));
    const size_t fb = align256((size_t)Vp * tl::kVBytes[vp]);
    char* s = nullptr;
    TL_TRY(ctx_scratch(c, 1024 + 2 * fb, &s));
    const StepConfig cfg{0, 256, 4, 0, 0};
    struct {
      StepGroup g;
      int64_t off0;
    } tab{};
    tab.g.W = slice;
    tab.g.w_mu_stride = Vp * tl::kWBytes[code];
    tab.g.Lx = g->L[0];
    tab.g.Ly = g->L[1];
    tab.g.Lz = g->L[2];
    tab.g.Vp = (int32_t)Vp;
    tab.g.nr = 1;
    tab.g.n_xy_tiles = (int32_t)(((int64_t)g->L[0] * g->L[1] + cfg.block - 1) / cfg.block);
    tab.g.n_z_tiles = (g->L[2] + cfg.tz - 1) / cfg.tz;
    TL_TRY(upload(c, s, &tab, sizeof tab));
    const StepGroup* gdev = reinterpret_cast<const StepGroup*>(s);
    const int64_t* offdev = reinterpret_cast<const int64_t*>(s + offsetof(decltype(tab), off0));
    char *A = s + 1024, *B = A + fb;
    TL_TRY(launch(c, "pack", [&] { return tl::launch_pack(vp, in, A, offdev, 1, V3, Vp, c->stream); }));
    TL_TRY(launch(c, "laplacian", [&] { return tl::launch_step(code, 1, cfg, gdev, 1, 0, tab.g.n_xy_tiles * tab.g.n_z_tiles, A, B, la, lb,
                                        0, c->stream); }));
    return launch(c, "unpack", [&] { return tl::launch_unpack(vp, B, out, offdev, 1, V3, Vp, c->stream); });
  } catch (...) {
    return host_failure(c);
  }
}

}  // extern "C"

namespace {

// tl_plan_create; of_call: a plan of tl_smear, which is loaded before it runs.
int plan_create(tl_ctx* c, const tl_job* jobs, int n_jobs, int n_steps, double sigma, int prec, unsigned flags,
                bool of_call, tl_plan** out) {
  try {
    if (!c) return TL_ERR_ARG;
    if (!out) return fail(c, TL_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (!jobs || n_jobs < 1) return fail(c, TL_ERR_ARG, "need at least one job");
    if (!valid_prec(prec)) return fail(c, TL_ERR_PRECISION, "unknown precision %d", prec);
    if (flags & ~(unsigned)(TL_PLAIN | TL_GRAPH | TL_AUTOTUNE | TL_ONE_STEP))
      return fail(c, TL_ERR_ARG, "unknown flag bits 0x%x", flags);
    if ((flags & TL_PLAIN) && (flags & TL_GRAPH)) return fail(c, TL_ERR_ARG, "TL_PLAIN runs eager launches; it excludes TL_GRAPH");
    if (n_steps < 0) return fail(c, TL_ERR_ARG, "n_steps = %d is negative", n_steps);
    if (!std::isfinite(sigma)) return fail(c, TL_ERR_ARG, "sigma is not finite");
    const bool one = tl::is_one(fmt_code(prec));
    if (n_steps > 0) {
      const double s = sigma / n_steps;
      if (s < 0.0 || s > max_step(one))
        return fail(c, TL_ERR_ARG, "sigma/n = %g outside [0, %s]", s, one ? "1/6" : "2/3");
    }
    for (int j = 0; j < n_jobs; j++) {
      const tl_job& jb = jobs[j];
      TL_TRY(check_geom(c, &jb.g));
      if (!jb.W || !jb.psi) return fail(c, TL_ERR_ARG, "job %d: W and psi must be non-NULL", j);
      if (jb.n_rhs < 1 || !jb.t_of_rhs) return fail(c, TL_ERR_ARG, "job %d: needs n_rhs >= 1 and t_of_rhs", j);
      TL_TRY(check_wslices(c, jb.g, jb.w_slices, jb.n_w_slices));
      for (int r = 0; r < jb.n_rhs; r++)
        if (slot_of(jb.g, jb.w_slices, jb.n_w_slices, jb.t_of_rhs[r]) < 0)
          return fail(c, TL_ERR_SHAPE, "job %d RHS %d: slice %d not in the two-link field", j, r, jb.t_of_rhs[r]);
    }
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    TL_TRY(need_eager(c, "plan created"));
  
    tl_plan* p = new (std::nothrow) tl_plan();
    if (!p) return fail(c, TL_ERR_NOMEM, "host allocation failed");
    struct Release {   // frees the plan on every exit but the successful one
      tl_plan* p;
      ~Release() { plan_free(p); }
    } release{p};
    p->ctx = c;
    p->prec = fmt_code(prec);
    p->n_steps = n_steps;
    p->sigma = sigma;
    p->flags = flags;
    p->of_call = of_call;
    if (n_steps > 0) step_coeffs(one, n_steps, sigma, &p->alpha, &p->beta);
    const int max_width = (flags & TL_PLAIN) ? 1 : 4;
  
    // resident order: per job, per slot (in slice order), RHS in job order;
    // groups of up to max_width RHS, balanced within a slot.
    size_t off = 0;
    for (int j = 0; j < n_jobs; j++) {
      tl_plan::JobCopy jc;
      jc.job = jobs[j];
      jc.t_of_rhs.assign(jobs[j].t_of_rhs, jobs[j].t_of_rhs + jobs[j].n_rhs);
      if (jobs[j].w_slices) jc.w_slices.assign(jobs[j].w_slices, jobs[j].w_slices + jobs[j].n_w_slices);
      jc.job.t_of_rhs = jc.t_of_rhs.data();
      jc.job.w_slices = jobs[j].w_slices ? jc.w_slices.data() : nullptr;
      jc.V3 = vol3(jc.job.g);
      jc.Vp = tl::padded_sites(jc.V3);
      jc.res_index.assign(jc.job.n_rhs, -1);
      p->max_v3 = std::max(p->max_v3, jc.V3);
      std::map<int, std::vector<int>> by_slot;
      for (int r = 0; r < jc.job.n_rhs; r++)
        by_slot[slot_of(jc.job.g, jc.job.w_slices, jc.job.n_w_slices, jc.t_of_rhs[r])].push_back(r);
      const size_t rb = align256((size_t)jc.Vp * tl::kVBytes[p->prec]);
      for (auto& kv : by_slot) {
        const int k = (int)kv.second.size();
        const int ng = (k + max_width - 1) / max_width;
        int done = 0;
        for (int q = 0; q < ng; q++) {
          const int nr = (k - done + (ng - q) - 1) / (ng - q);
          tl_plan::Group gr{j, kv.first, (int)p->res.size(), nr};
          for (int i = 0; i < nr; i++) {
            const int r = kv.second[done + i];
            jc.res_index[r] = (int)p->res.size();
            p->res.push_back({j, r, kv.first, (int64_t)off});
            off += rb;
          }
          done += nr;
          p->width = std::max(p->width, nr);
          p->groups.push_back(gr);
        }
      }
      p->jobs.push_back(std::move(jc));
    }
    p->buf_bytes = std::max<size_t>(off, 256);
  
    // device memory: two resident buffers and the tables
    int rc = TL_OK;
    for (int k = 0; k < 2 && rc == TL_OK; k++) {
      void* b = nullptr;
      size_t bytes = p->buf_bytes;
      rc = mem_get(c, &b, &bytes);
      if (rc == TL_OK) {
        p->buf[k] = static_cast<char*>(b);
        p->buf_cap[k] = bytes;
      }
    }
    const size_t n_res = p->res.size();
    // two tilings' step groups: a tiling may split the plan's groups down to one RHS each
    p->group_cap = n_res;
    const size_t gbytes = 2 * align256(n_res * sizeof(StepGroup));
    const size_t ubytes = align256(n_res * 8 * sizeof(tl::RunUnit));
    const size_t obytes = align256(n_res * sizeof(int64_t));
    const size_t rbytes = align256(n_res * sizeof(tl::RedField));
    const size_t pbytes = align256((size_t)tl::red_partials_doubles((int)n_res, p->max_v3) * sizeof(double));
    if (rc == TL_OK) {
      void* t = nullptr;
      size_t bytes = gbytes + ubytes + obytes + rbytes + pbytes;
      rc = mem_get(c, &t, &bytes);
      if (rc == TL_OK) {
        p->tables = static_cast<char*>(t);
        p->tables_cap = bytes;
      }
    }
    if (rc == TL_OK) {
      p->tile.dev = reinterpret_cast<StepGroup*>(p->tables);
      p->single.dev = reinterpret_cast<StepGroup*>(p->tables + gbytes / 2);
      p->run_units = reinterpret_cast<tl::RunUnit*>(p->tables + gbytes);
      p->packoff_dev = reinterpret_cast<int64_t*>(p->tables + gbytes + ubytes);
      p->red_dev = reinterpret_cast<tl::RedField*>(p->tables + gbytes + ubytes + obytes);
      p->partials = reinterpret_cast<double*>(p->tables + gbytes + ubytes + obytes + rbytes);
      // pack offsets and reduction fields: neighbours in the tables, one upload
      std::vector<char> host(obytes + rbytes, 0);
      int64_t* po = reinterpret_cast<int64_t*>(host.data());
      tl::RedField* rf = reinterpret_cast<tl::RedField*>(host.data() + obytes);
      int64_t k = 0, oo = 0;
      for (auto& jc : p->jobs) {
        p->packoff_first.push_back(k);
        for (int r = 0; r < jc.job.n_rhs; r++, k++) {
          const int64_t o = p->res[jc.res_index[r]].off;
          po[k] = o;
          rf[k] = {o, o, jc.V3, jc.Vp, oo};
          oo += jc.V3;
        }
      }
      rc = upload(c, p->packoff_dev, host.data(), host.size());
    }
    if (rc == TL_OK && (!of_call || (flags & TL_AUTOTUNE))) {
      // zero the resident buffers so tuning runs never see stale bit patterns
      for (int k = 0; k < 2 && rc == TL_OK; k++)
        if (hipMemsetAsync(p->buf[k], 0, p->buf_bytes, c->stream) != hipSuccess)
          rc = fail(c, TL_ERR_HIP, "hipMemsetAsync failed");
    }
    if (rc == TL_OK) rc = describe_tiling(p, p->tile.cfg, &p->tile);
    if (rc != TL_OK) return rc;
    // info
    tl_plan_info& in = p->info;
    in.n_groups = (int32_t)p->groups.size();
    in.group_width = p->width;
    in.launches_per_step = (flags & TL_PLAIN) ? in.n_groups : 1;
    double bytes = 0.0, flops = 0.0;
    int64_t rs = 0;
    for (auto& gr : p->groups) {
      const double v3 = (double)p->jobs[gr.job].V3;
      bytes += v3 * (3.0 * tl::kWBytes[p->prec] + 2.0 * gr.nr * tl::kVBytes[p->prec]);
      flops += v3 * (444.0 * gr.nr + (tl::is_w12(p->prec) ? 3 * 42.0 : 0.0));
      rs += (int64_t)p->jobs[gr.job].V3 * gr.nr;
    }
    in.rhs_sites = rs;
    in.bytes_per_step = bytes;
    in.flops_per_step = flops;
    in.resident_bytes = (int64_t)(p->buf_cap[0] + p->buf_cap[1] + p->tables_cap);
    if (!(flags & TL_AUTOTUNE)) TL_TRY(prepare_untuned(p));   // a tuned one: its first run
    release.p = nullptr;
    *out = p;
    return TL_OK;
  } catch (...) {
    return host_failure(c);
  }
}

}  // namespace

extern "C" {

int tl_plan_create(tl_ctx* c, const tl_job* jobs, int n_jobs, int n_steps, double sigma, int prec, unsigned flags,
                   tl_plan** out) {
  return plan_create(c, jobs, n_jobs, n_steps, sigma, prec, flags, false, out);
}

int tl_plan_load(tl_plan* p) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    TL_ON_DEVICE(c);
    for (size_t j = 0; j < p->jobs.size(); j++) {
      const auto& jc = p->jobs[j];
      TL_TRY(launch(c, "pack", [&] { return tl::launch_pack(tl::vprec(p->prec), jc.job.psi, p->buf[p->cur], p->packoff_dev + p->packoff_first[j],
                                          jc.job.n_rhs, jc.V3, jc.Vp, c->stream); }));
    }
    return TL_OK;
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_plan_run(tl_plan* p) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    if (p->n_steps == 0) return TL_OK;
    TL_ON_DEVICE(c);
    if (fail_taken(p->fail)) return run_failure(c);
    TL_TRY(plan_prepare(p));
    std::optional<RunTurn> turn;
    if (p->tile.cfg.variant == 9) turn.emplace(c, run_load(p->tile.run, p->prec));
    // a tuned run that is one launch needs no graph
    if ((p->flags & TL_GRAPH) && !(p->tile.cfg.variant == 9 && (p->flags & TL_AUTOTUNE))) {
      TL_TRY(plan_capture(p, p->cur));
      if (c->fault_launch) return fail(c, TL_ERR_HIP, "graph launch failed (TL_FAULT=launch)");
      HIP_TRY(c, hipGraphLaunch(p->graph[p->cur], c->stream));
    } else {
      TL_TRY(plan_enqueue(p, c->stream, p->cur));
    }
    if (plan_flips(p)) p->cur ^= 1;
    return TL_OK;
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_plan_store(tl_plan* p) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    TL_ON_DEVICE(c);
    if (fail_taken(p->fail)) return run_failure(c);
    for (size_t j = 0; j < p->jobs.size(); j++) {
      const auto& jc = p->jobs[j];
      TL_TRY(launch(c, "unpack", [&] { return tl::launch_unpack(tl::vprec(p->prec), p->buf[p->cur], jc.job.psi, p->packoff_dev + p->packoff_first[j],
                                            jc.job.n_rhs, jc.V3, jc.Vp, c->stream); }));
    }
    return TL_OK;
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_plan_reduce(tl_plan* p, int kind, const tl_plan* other, double* out) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    if (kind < TL_NORM2 || kind > TL_SITE_NORM) return fail(c, TL_ERR_ARG, "unknown reduction kind %d", kind);
    if (!out) return fail(c, TL_ERR_ARG, "out is NULL");
    const char* b = nullptr;
    if (kind == TL_DOT) {
      if (!other) return fail(c, TL_ERR_ARG, "TL_DOT needs a second plan");
      if (other->ctx != c || tl::vprec(other->prec) != tl::vprec(p->prec) || other->buf_bytes != p->buf_bytes || other->res.size() != p->res.size())
        return fail(c, TL_ERR_ARG, "TL_DOT: plans differ in context, precision or shape");
      for (size_t i = 0; i < p->res.size(); i++)
        if (other->res[i].off != p->res[i].off) return fail(c, TL_ERR_ARG, "TL_DOT: plans differ in layout");
      b = other->buf[other->cur];
    }
    TL_ON_DEVICE(c);
    if (fail_taken(p->fail) || (kind == TL_DOT && fail_taken(other->fail))) return run_failure(c);
    // a (this) is the second argument of <other, this>
    return launch(c, "reduction", [&] { return tl::launch_reduce(kind, tl::vprec(p->prec), p->buf[p->cur], b, p->red_dev, (int)p->res.size(), p->max_v3,
                                          p->partials, out, c->stream); });
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_plan_time(tl_plan* p, int reps, double* ms_per_step) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    if (reps < 1 || !ms_per_step) return fail(c, TL_ERR_ARG, "need reps >= 1 and an output pointer");
    if (p->n_steps == 0) return fail(c, TL_ERR_ARG, "plan has no steps");
    TL_ON_DEVICE(c);
    TL_TRY(tl_plan_run(p));   // tuning and graph capture happen outside the timed region
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = TL_OK;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
      if (e0) (void)hipEventDestroy(e0);
      return fail(c, TL_ERR_HIP, "hipEventCreate failed");
    }
    (void)hipEventRecord(e0, c->stream);
    for (int k = 0; k < reps && rc == TL_OK; k++) rc = tl_plan_run(p);
    (void)hipEventRecord(e1, c->stream);
    float ms = 0.0f;
    if (rc == TL_OK) {
      if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
        rc = fail(c, TL_ERR_HIP, "event timing failed");
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc == TL_OK && fail_taken(p->fail)) rc = run_failure(c);
    if (rc == TL_OK) *ms_per_step = ms / ((double)reps * p->n_steps * p->info.launches_per_step);
    return rc;
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_stream_time(tl_ctx* c, void* buf, int64_t bytes, int n_in, int kinds, int grid, int reps, double* ms) {
  try {
    if (!c) return TL_ERR_ARG;
    if (!buf || !ms || reps < 1) return fail(c, TL_ERR_ARG, "need a buffer, an output pointer and reps >= 1");
    if (n_in < 1 || n_in > 16) return fail(c, TL_ERR_ARG, "n_in = %d outside [1, 16]", n_in);
    if (kinds < 0 || kinds > 3 || grid < 0) return fail(c, TL_ERR_ARG, "bad kinds %d or grid %d", kinds, grid);
    if (reinterpret_cast<uintptr_t>(buf) % 256) return fail(c, TL_ERR_ARG, "buffer not 256-byte aligned");
    const int64_t n_words = bytes / 16 / (n_in + 1);
    if (n_words < 1) return fail(c, TL_ERR_ARG, "buffer of %lld bytes too small", (long long)bytes);
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    const int g = grid > 0 ? grid : 16 * std::max(c->n_cu, 1);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
      if (e0) (void)hipEventDestroy(e0);
      return fail(c, TL_ERR_HIP, "hipEventCreate failed");
    }
    int rc = launch(c, "stream", [&] { return tl::launch_stream(buf, n_words, n_in, kinds, g, c->stream); });
    if (rc == TL_OK) (void)hipEventRecord(e0, c->stream);
    for (int k = 0; k < reps && rc == TL_OK; k++)
      rc = launch(c, "stream", [&] { return tl::launch_stream(buf, n_words, n_in, kinds, g, c->stream); });
    float t = 0.0f;
    if (rc == TL_OK) {
      (void)hipEventRecord(e1, c->stream);
      if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&t, e0, e1) != hipSuccess)
        rc = fail(c, TL_ERR_HIP, "event timing failed");
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc == TL_OK) *ms = t / reps;
    return rc;
  } catch (...) {
    return host_failure(c);
  }
}

int tl_plan_get_info(const tl_plan* p, tl_plan_info* info) {
  try {
    if (!p || !info) return TL_ERR_ARG;
    *info = p->info;
    info->resident_bytes += (int64_t)p->run.bytes + (p->run.ctl ? (int64_t)sizeof(tl::RunCtl) : 0);
    const tl_plan::Tiling& t = p->tile;
    info->n_tiles = t.n_tiles;
    info->variant = t.cfg.variant;
    info->block = t.cfg.block;
    info->tz = t.cfg.tz;
    info->grid = t.cfg.variant == 9 ? t.run.cfg.grid : t.cfg.grid > 0 ? std::min(t.cfg.grid, t.n_tiles) : t.n_tiles;
    info->nt = t.cfg.nt;
    info->flip = t.cfg.flip;
    info->steps_per_launch = t.cfg.variant == 8 ? 2 : 1;
    info->tile_width = eff_width(p, t.cfg);
    return TL_OK;
  } catch (...) {
    return host_failure(p ? p->ctx : nullptr);
  }
}

int tl_plan_destroy(tl_plan* p) {
  try {
    if (!p) return TL_ERR_ARG;
    tl_ctx* c = p->ctx;
    return plan_free(p) ? run_failure(c) : TL_OK;
  } catch (...) {
    return host_failure(nullptr);
  }
}

}  // extern "C"

namespace {

constexpr size_t kSmearPlans = 4;   // tl_smear(TL_GRAPH) plans a context keeps

// Everything a tl_smear plan depends on: the job list (geometries, device pointers, slice lists,
// RHS slices), n, sigma (its bits), the precision code and the flags.
std::string smear_signature(const tl_job* jobs, int n_jobs, int n_steps, double sigma, int prec, unsigned flags) {
  std::string k;
  char buf[128];
  uint64_t sb;
  std::memcpy(&sb, &sigma, sizeof sb);
  snprintf(buf, sizeof buf, "n%d|s%llx|p%d|f%u|j%d", n_steps, (unsigned long long)sb, prec, flags, n_jobs);
  k += buf;
  for (int j = 0; j < n_jobs; j++) {
    const tl_job& b = jobs[j];
    snprintf(buf, sizeof buf, "|%d,%d,%d,%d:%p:%p:%d:", b.g.L[0], b.g.L[1], b.g.L[2], b.g.L[3], b.W, b.psi, b.n_rhs);
    k += buf;
    for (int r = 0; r < b.n_rhs; r++) k += std::to_string(b.t_of_rhs[r]) + ",";
    if (b.w_slices) {
      k += "w";
      for (int i = 0; i < b.n_w_slices; i++) k += std::to_string(b.w_slices[i]) + ",";
    }
  }
  return k;
}

}  // namespace

extern "C" {

int tl_smear(tl_ctx* c, const tl_job* jobs, int n_jobs, int n_steps, double sigma, int prec, unsigned flags) {
  try {
    if (!c) return TL_ERR_ARG;
    // the signature reads the jobs' host arrays: malformed jobs are not kept (tl_plan_create refuses them)
    bool keep = (flags & TL_GRAPH) && jobs && n_jobs >= 1;
    for (int j = 0; keep && j < n_jobs; j++)
      if (jobs[j].n_rhs < 1 || !jobs[j].t_of_rhs || (jobs[j].w_slices && jobs[j].n_w_slices < 1)) keep = false;
    std::string sig;
    if (keep) {
      sig = smear_signature(jobs, n_jobs, n_steps, sigma, prec, flags);
      for (auto it = c->smear_plans.begin(); it != c->smear_plans.end(); ++it) {
        if (it->first != sig) continue;
        c->smear_plans.splice(c->smear_plans.begin(), c->smear_plans, it);   // most recent first
        tl_plan* p = c->smear_plans.front().second;
        TL_ON_DEVICE(c);
        TL_TRY(need_eager(c, "tl_smear"));
        c->stats.smear_plan_hits++;
        p->cur = 0;   // the sources are packed afresh, into the buffer whose graph was captured first
        int rc = tl_plan_load(p);
        if (rc == TL_OK) rc = tl_plan_run(p);
        if (rc == TL_OK) rc = tl_plan_store(p);
        return rc;
      }
    }
    tl_plan* p = nullptr;
    TL_TRY(plan_create(c, jobs, n_jobs, n_steps, sigma, prec, flags, true, &p));
    int rc = tl_plan_load(p);
    if (rc == TL_OK) rc = tl_plan_run(p);
    if (rc == TL_OK) rc = tl_plan_store(p);
    if (!keep || rc != TL_OK) {
      if (plan_free(p) && rc == TL_OK) rc = run_failure(c);   // waits for the queued work
      return rc;
    }
    c->smear_plans.emplace_front(std::move(sig), p);
    if (c->smear_plans.size() > kSmearPlans) {
      plan_free(c->smear_plans.back().second);
      c->smear_plans.pop_back();
    }
    return rc;
  } catch (...) {
    return host_failure(c);
  }
}

int tl_get_stats(const tl_ctx* c, tl_ctx_stats* out) {
  if (!c || !out) return TL_ERR_ARG;
  *out = c->stats;
  return TL_OK;
}

namespace {

int check_reduce_args(tl_ctx* c, int kind, int64_t n_sites, int n_rhs, const void* psi, const void* phi,
                      const double* out) {
  if (kind < TL_NORM2 || kind > TL_SITE_NORM) return fail(c, TL_ERR_ARG, "unknown reduction kind %d", kind);
  if (n_sites < 1 || n_rhs < 1) return fail(c, TL_ERR_ARG, "need n_sites >= 1 and n_rhs >= 1");
  if (!psi || !out || (kind == TL_DOT && !phi)) return fail(c, TL_ERR_ARG, "NULL field or output");
  if (n_sites > (int64_t(1) << 40)) return fail(c, TL_ERR_SHAPE, "n_sites too large");
  return TL_OK;
}

}  // namespace

int tl_reduce_noalloc(tl_ctx* c, int kind, int64_t n_sites, int n_rhs, const void* psi, const void* phi,
                      double* out) {
  try {
    if (!c) return TL_ERR_ARG;
    TL_TRY(check_reduce_args(c, kind, n_sites, n_rhs, psi, phi, out));
    if (kind != TL_SITE_NORM) {
      const int64_t need = tl::red_partials_doubles(n_rhs, n_sites);
      if (need > tl::kNoallocPartials)
        return fail(c, TL_ERR_SHAPE,
                    "tl_reduce_noalloc: %lld partial sums needed, the fixed area holds %lld "
                    "(n_rhs * ceil(n_sites / 4096) must not exceed %lld)",
                    (long long)need, (long long)tl::kNoallocPartials, (long long)(tl::kNoallocPartials / 2));
    }
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    if (!c->noalloc) return fail(c, TL_ERR_HIP, "no fixed reduction area on device %d (%s)", c->device, c->noalloc_err.c_str());
    return launch(c, "reduction", [&] { return tl::launch_reduce_flat(kind, psi, phi, n_sites, n_rhs, c->noalloc, out, c->stream); });
  } catch (...) {
    return host_failure(c);
  }
}

int tl_reduce(tl_ctx* c, int kind, int64_t n_sites, int n_rhs, const void* psi, const void* phi, double* out) {
  try {
    if (!c) return TL_ERR_ARG;
    TL_TRY(check_reduce_args(c, kind, n_sites, n_rhs, psi, phi, out));
    TL_TRY(need_device(c));
    TL_ON_DEVICE(c);
    char* s = nullptr;
    if (kind != TL_SITE_NORM) TL_TRY(ctx_scratch(c, (size_t)tl::red_partials_doubles(n_rhs, n_sites) * sizeof(double), &s));
    // psi, phi: <phi, psi>
    return launch(c, "reduction", [&] { return tl::launch_reduce_flat(kind, psi, phi, n_sites, n_rhs, reinterpret_cast<double*>(s), out, c->stream); });
  } catch (...) {
    return host_failure(c);
  }
}

}  // extern "C"
