// A device for the library's host code on the CPU (tests only). Streams hold
// their work in order; it runs, in the calling thread, whenever the host makes a runtime call and
// nothing stands in its way: the stream is held, waits for an event, or a resident kernel leaves no
// room for the wide workgroups of a bulk solve. Kernels are stand-ins that
// reach the library's result by a plain search: what is tested is the order of
// work, waits, deadlines, memory and routes, not the kernels.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <queue>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "hip/hip_runtime.h"
#include "mlmq_cut.h"
#include "mlmq_internal.h"
#include "mlmq_shape.h"
#include "mlmq_step.h"
#include "mlmq_tile.h"

using namespace mlmq;
using Clock = std::chrono::steady_clock;

struct SimEvent {
  uint64_t recorded = 0, done = 0;
  Clock::time_point at{};
};
struct Op {
  std::function<bool()> run;  // false: not yet
};
struct SimStream {
  std::deque<Op> ops;
  bool held = false, nonblocking = false, running = false;
};
struct SimGraph {
  std::vector<Op> ops;
};

namespace {

std::recursive_mutex g_mu;
SimStream g_null;
std::set<SimStream*> g_streams = {&g_null};
thread_local SimGraph* g_capture = nullptr;
thread_local SimStream* g_capture_stream = nullptr;
thread_local hipError_t g_last = hipSuccess;
std::map<uintptr_t, size_t> g_mem;  // device allocations
std::map<uintptr_t, size_t> g_given;  // memory a test calls device memory
size_t g_used = 0, g_room = ~size_t(0), g_largest = ~size_t(0);
std::map<std::string, uint64_t> g_count;
// How the stand-in kernels behave.
uint32_t g_steps = 6;          // launches after which a bulk solve reports its end
double g_worker_ms = 0, g_worker_more = 0, g_served_ms = 0, g_step_ms = 0;
int g_resident = 0;            // server kernels on the device
std::map<const void*, std::pair<const int32_t*, const uint64_t*>> g_tiled;  // id_of -> rows

hipError_t err(hipError_t e) {
  if (e != hipSuccess && e != hipErrorNotReady) g_last = e;
  return e;
}
SimStream* of(hipStream_t s) {
  if (s && !g_streams.count(s)) {
    fprintf(stderr, "hostsim: unknown stream\n");
    abort();
  }
  return s ? s : &g_null;
}
void note(const char* what) { g_count[what] += 1; }

void pump() {
  for (bool any = true; any;) {
    any = false;
    for (SimStream* s : std::set<SimStream*>(g_streams)) {
      if (s->running || s->held) continue;
      s->running = true;
      while (!s->ops.empty() && !s->held) {
        if (!s->ops.front().run()) break;
        s->ops.pop_front();
        any = true;
      }
      s->running = false;
    }
  }
}
// Work of the null stream and that of blocking streams wait for each other;
// the library makes no blocking streams, so each stream is on its own here.
void enqueue(hipStream_t s, std::function<bool()> f) {
  if (g_capture && g_capture_stream == of(s)) {
    g_capture->ops.push_back({std::move(f)});
    return;
  }
  of(s)->ops.push_back({std::move(f)});
  pump();
}

void search(const int32_t* off, const uint64_t* adj, uint32_t n, uint32_t src, bool unit, uint32_t* out, bool* over) {
  std::vector<uint64_t> d(n, ~0ull);
  typedef std::pair<uint64_t, uint32_t> E;
  std::priority_queue<E, std::vector<E>, std::greater<E>> q;
  d[src] = 0;
  q.push({0, src});
  while (!q.empty()) {
    auto [x, v] = q.top();
    q.pop();
    if (x != d[v]) continue;
    for (int32_t e = off[v]; e < off[v + 1]; ++e) {
      const uint32_t u = (uint32_t)adj[e];
      const uint64_t y = x + (unit ? 1 : adj[e] >> 32);
      if (y >= kInf) {
        if (over) *over = true;
        continue;
      }
      if (y < d[u]) {
        d[u] = y;
        q.push({y, u});
      }
    }
  }
  for (uint32_t v = 0; v < n; ++v) out[v] = d[v] >= kInf ? kInf : (uint32_t)d[v];
}

std::function<bool()> timed(double ms, std::function<void()> f) {
  auto start = std::make_shared<Clock::time_point>();
  return [=]() {
    if (*start == Clock::time_point()) *start = Clock::now();
    if (std::chrono::duration<double, std::milli>(Clock::now() - *start).count() < ms) return false;
    f();
    return true;
  };
}

// A launch of a bulk solve: it begins as soon as it is its turn and there is room.
std::function<bool()> bulk_launch(const char* what, uint32_t i, std::vector<std::function<void(uint32_t)>> rows) {
  auto body = timed(g_step_ms, [=] {
    note(what);
    for (auto& r : rows) r(i);
  });
  return [=]() { return g_resident == 0 && body(); };
}

void step_row(const StepArgs& a, uint32_t i) {
  a.host->begun = i;
  if (i < g_steps || a.host->state) return;
  search(a.off, a.adj, a.n, a.source, a.unit_w, a.lab, nullptr);
  uint32_t mx = 0;
  for (uint32_t v = 0; v < a.n; ++v) {
    const uint32_t d = a.lab[a.ord_of ? a.ord_of[v] : v];
    if (a.ord_of) a.out[v] = d;
    if (d != kInf && d > mx) mx = d;
  }
  a.host->max_label = mx;
  a.host->state = 1;
}
void tile_row(const TileArgs& a, uint32_t i) {
  a.host->begun = i;
  if (i < g_steps || a.host->state) return;
  const auto rows = g_tiled.at(a.g.id_of);
  uint32_t src = 0;
  while (a.g.id_of[src] != a.source) ++src;
  search(rows.first, rows.second, a.g.n, src, a.unit_w, a.out, nullptr);
  uint32_t mx = 0;
  for (uint32_t v = 0; v < a.g.n; ++v)
    if (a.out[v] != kInf && a.out[v] > mx) mx = a.out[v];
  a.host->max_label = mx;
  a.host->state = 1;
}

void solve_query(const QueryDesc& q) {
  bool over = false;
  search(q.off, q.adj, q.n, q.source, q.unit_w, q.dist, &over);
  q.ctrl->error.v = kStOk;
  q.ctrl->overflow.v = over ? 1u : 0u;
  q.ctrl->stats[kCtWaveTicks] = 1000000;  // 10 ms of waves: bulk solves report none
}

}  // namespace

// ------------------------------------------------------------ runtime

hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
  std::memset(p, 0, sizeof(*p));
  p->multiProcessorCount = 256;
  p->sharedMemPerBlock = p->maxSharedMemoryPerMultiProcessor = 160 << 10;
  std::strcpy(p->gcnArchName, "sim");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 100000, hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t sim_malloc(void** p, size_t n) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  note("hipMalloc");
  if (n > g_largest || g_used + n > g_room) {
    *p = nullptr;
    return err(hipErrorOutOfMemory);
  }
  *p = std::malloc(n ? n : 1);
  std::memset(*p, 0xA5, n);
  g_mem[(uintptr_t)*p] = n;
  g_used += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  std::unique_lock<std::recursive_mutex> lk(g_mu);
  note("hipFree");
  // waits for everything on the device
  for (;;) {
    pump();
    bool busy = g_resident > 0;
    for (SimStream* s : g_streams) busy = busy || !s->ops.empty();
    if (!busy) break;
    lk.unlock();
    std::this_thread::sleep_for(std::chrono::microseconds(200));
    lk.lock();
  }
  auto it = g_mem.find((uintptr_t)p);
  if (it == g_mem.end()) {
    fprintf(stderr, "hostsim: hipFree of unknown memory\n");
    abort();
  }
  std::memset(p, 0x5A, it->second);
  g_used -= it->second;
  g_mem.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t sim_host_malloc(void** p, size_t n) { return *p = std::calloc(1, n ? n : 1), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  pump();
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  enqueue(st, [=] { return std::memcpy(d, s, n), true; });
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  enqueue(st, [=] { return std::memset(d, v, n), true; });
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  a->type = hipMemoryTypeHost;
  for (auto* m : {&g_mem, &g_given}) {
    auto it = m->upper_bound((uintptr_t)p);
    if (it != m->begin() && (--it, (uintptr_t)p < it->first + it->second)) a->type = hipMemoryTypeDevice;
  }
  return a->type == hipMemoryTypeDevice ? hipSuccess : err(hipErrorInvalidValue);
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  *s = new SimStream();
  (*s)->nonblocking = f & hipStreamNonBlocking;
  g_streams.insert(*s);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  g_streams.erase(s);
  delete s;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  pump();
  return of(s)->ops.empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  while (hipStreamQuery(s) == hipErrorNotReady) std::this_thread::sleep_for(std::chrono::microseconds(50));
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t ev, unsigned) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  auto left = std::shared_ptr<SimEvent>(ev, [](SimEvent*) {});
  const uint64_t k = ev->recorded;
  enqueue(s, [=] { return left->done >= k; });
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  g_capture = new SimGraph();
  g_capture_stream = of(s);
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = g_capture;
  g_capture = nullptr;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return *e = new SimEvent(), hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }  // waits may still name it
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const uint64_t k = ++e->recorded;
  enqueue(s, [=] {
    e->done = k;
    e->at = Clock::now();
    return true;
  });
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  pump();
  return e->done >= e->recorded ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  while (hipEventQuery(e) == hipErrorNotReady) std::this_thread::sleep_for(std::chrono::microseconds(50));
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = std::chrono::duration<float, std::milli>(b->at - a->at).count();
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, void*, char*, size_t) {
  return *x = new SimGraph(*g), hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete g, hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t g) { return delete g, hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t g, hipStream_t s) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  note("hipGraphLaunch");
  for (Op& o : g->ops) of(s)->ops.push_back(o);
  pump();
  return hipSuccess;
}

// ------------------------------------------------------------ launchers

namespace mlmq {

// A launch reports the last error of its thread, as hipGetLastError() after a
// launch does.
static hipError_t launched(hipStream_t s, std::function<bool()> f) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) enqueue(s, std::move(f));
  return e;
}
template <class F>
static hipError_t launched_now(hipStream_t s, F f) {
  return launched(s, [=] { return f(), true; });
}

size_t worker_lds_bytes(uint32_t, uint32_t l1, bool two, bool stage) {
  return 8ull * (64ull + (uint64_t)l1 * (two ? 2u : 1u) + (stage ? 512ull : 0ull));
}
hipError_t worker_occupancy(uint32_t, size_t, bool, int* k) { return *k = 12, hipSuccess; }
hipError_t server_occupancy(size_t, bool, int* k) { return *k = 12, hipSuccess; }
hipError_t launch_init(const QueryDesc* q, BatchCtrl* b, int nq, uint32_t, hipStream_t s) {
  return launched_now(s, [=] {
    std::memset(static_cast<void*>(b), 0, sizeof(*b));
    for (int i = 0; i < nq; ++i) {
      std::memset(static_cast<void*>(q[i].ctrl), 0, sizeof(QueryCtrl));
      for (uint32_t v = 0; v < q[i].n; ++v) q[i].dist[v] = kInf;
    }
  });
}
hipError_t launch_worker(const LaunchArgs& a, uint32_t, uint32_t, size_t, hipStream_t s) {
  g_worker_ms += g_worker_more;
  return launched(s, timed(g_worker_ms, [=] {
                    note("worker");
                    for (int i = 0; i < a.nq; ++i) {
                      if (a.batch->cancel.v || g_worker_ms * 1e5 > (double)a.timeout_ticks)
                        a.queries[i].ctrl->error.v = kStTimeout;
                      else
                        solve_query(a.queries[i]);
                    }
                  }));
}
hipError_t launch_overflow_check(const QueryDesc* q, uint32_t* flag, hipStream_t s) {
  return launched_now(s, [=] {
    note("overflow check");
    for (uint32_t v = 0; v < q->n; ++v)
      if (q->dist[v] != kInf)
        for (int32_t e = q->off[v]; e < q->off[v + 1]; ++e)
          if (q->dist[(uint32_t)q->adj[e]] == kInf) *flag = 1;
  });
}
hipError_t launch_unorder(const uint32_t* lab, const uint32_t* ord, uint32_t n, uint32_t* out, hipStream_t s) {
  return launched_now(s, [=] {
    for (uint32_t v = 0; v < n; ++v) out[v] = lab[ord[v]];
  });
}
hipError_t launch_gather(const QueryDesc* q, int nq, QueryResult* out, hipStream_t s) {
  return launched_now(s, [=] {
    for (int i = 0; i < nq; ++i) {
      out[i].error = q[i].ctrl->error.v;
      out[i].overflow = q[i].ctrl->overflow.v;
      std::memset(out[i].stats, 0, sizeof(out[i].stats));
    }
  });
}
// The resident kernel stays until it is told to stop and serves the slots that
// are open; while it is there no wide workgroup finds room.
hipError_t launch_server_worker(const ServerArgs& a, uint32_t, size_t, hipStream_t s) {
  auto on = std::make_shared<bool>(false);
  return launched(s, [=] {
    if (!*on) {
      *on = true;
      g_resident += 1;
      note("server kernel");
      g_count["launches before it"] = g_count["step"] + g_count["tile"];
    }
    for (int i = 0; i < a.nslots; ++i) {
      const uint64_t w = a.join[i];
      if (w == 0 || (w >> 63) || !(uint32_t)(w >> 32)) continue;
      static std::map<const void*, Clock::time_point> began;
      auto& t = began[a.join + i];
      if (t == Clock::time_point()) t = Clock::now();
      if (std::chrono::duration<double, std::milli>(Clock::now() - t).count() < g_served_ms) continue;
      t = Clock::time_point();
      solve_query(a.slots[i]);
      a.join[i] = 0;
      __atomic_store_n(&a.done_host[i], (uint64_t)(uint32_t)(w >> 32), __ATOMIC_RELEASE);
    }
    if (!a.ctl->stop.v) return false;
    g_resident -= 1;
    return true;
  });
}
hipError_t launch_server_admit(const QueryDesc& q, QueryDesc* slot, uint64_t* join, uint64_t word, uint32_t,
                               hipStream_t s) {
  return launched_now(s, [=] {
    *slot = q;
    std::memset(static_cast<void*>(q.ctrl), 0, sizeof(QueryCtrl));
    *join = word & ~(1ull << 63);
  });
}
hipError_t launch_server_signal(uint32_t* w, uint32_t v, hipStream_t s) {
  return launched_now(s, [=] { *w = v; });
}
hipError_t launch_check(const int32_t*, const uint64_t*, const uint32_t*, uint32_t, uint32_t, uint32_t, uint8_t*,
                        unsigned long long*, hipEvent_t, hipEvent_t, hipStream_t) {
  return hipErrorUnknown;
}
hipError_t launch_latency_probes(const int32_t*, const uint64_t*, uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t*,
                                 uint32_t, uint64_t, uint64_t*, hipStream_t) {
  return hipErrorUnknown;
}
hipError_t noalloc_scratch(int, void** out) {
  static void* p = nullptr;
  if (!p) p = std::malloc(kNoAllocScratchBytes);
  return *out = p, hipSuccess;
}

hipError_t launch_step_init(const StepArgs& a, uint32_t, hipStream_t s) {
  return launched_now(s, [=] {
    note("step init");
    for (uint32_t v = 0; v < a.n; ++v) a.lab[v] = kInf;
  });
}
hipError_t launch_step(const StepArgs& a, uint32_t i, uint32_t, hipStream_t s) {
  return launched(s, bulk_launch("step", i, {[=](uint32_t k) { step_row(a, k); }}));
}
hipError_t launch_step_many(const StepArgs* d, uint32_t n, uint32_t i, uint32_t, hipStream_t s) {
  std::vector<std::function<void(uint32_t)>> rows;
  for (uint32_t r = 0; r < n; ++r)
    rows.push_back([=](uint32_t k) {
      if (k) return step_row(d[r], k);
      for (uint32_t v = 0; v < d[r].n; ++v) d[r].lab[v] = kInf;
    });
  return launched(s, bulk_launch("step", i, rows));
}
hipError_t launch_sort_rows(const int32_t* off, const uint64_t* in, uint64_t* out, uint32_t n, uint32_t, hipStream_t s) {
  return launched_now(s, [=] { std::memcpy(out, in, 8ull * off[n]); });
}
hipError_t launch_transpose(const int32_t* off, const uint64_t* adj, uint32_t n, uint32_t m, int32_t* ioff,
                            uint64_t* iadj, uint32_t* scratch, hipStream_t s) {
  return launched_now(s, [=] {
    std::memset(scratch, 0, 4ull * (n + 1ull + n / 4096 + 2));
    std::memset(iadj, 0, 8ull * m);
    std::memcpy(ioff, off, 4ull * (n + 1ull));
    (void)adj;
  });
}
size_t tile_lds_bytes(uint32_t sbits, uint32_t xcap, uint32_t threads) {
  return 4ull * (128u + (6ull << sbits) + xcap + ((1u << sbits) + 8u) / 2u + threads / 64u * kTileQueue / 2u);
}
hipError_t tile_set_lds(size_t) { return hipSuccess; }
hipError_t launch_tile_init(const TileArgs&, hipStream_t s) {
  return launched_now(s, [] { note("tile init"); });
}
hipError_t launch_tile_round(const TileArgs& a, uint32_t i, uint32_t, uint32_t, hipStream_t s) {
  return launched(s, bulk_launch("tile", i, {[=](uint32_t k) { tile_row(a, k); }}));
}
hipError_t launch_tile_many(const TileArgs* d, uint32_t n, uint32_t i, uint32_t, uint32_t, size_t, hipStream_t s) {
  std::vector<std::function<void(uint32_t)>> rows;
  for (uint32_t r = 0; r < n; ++r)
    rows.push_back([=](uint32_t k) {
      if (k) tile_row(d[r], k);
    });
  return launched(s, bulk_launch("tile", i, rows));
}
hipError_t launch_tile_ids(const TileBuild&, hipStream_t s) {
  return launched_now(s, [] {});
}
hipError_t launch_tile_count(const TileBuild& b, hipStream_t s) {
  return launched_now(s, [=] { g_tiled[b.id_of] = {b.off, b.adj}; });
}
hipError_t launch_tile_fill(const TileBuild&, hipStream_t s) {
  return launched_now(s, [] {});
}

}  // namespace mlmq

// ------------------------------------------------------------ for the tests

extern "C" {
// Leaves something else than zeros where the next call's locals will be.
__attribute__((noinline)) int sim_dirty_stack() {
  volatile uint64_t words[4096];
  for (auto& w : words) w = 0xA5A5A5A5A5A5A5A5ull;
  return (int)words[17];
}
void* sim_alloc(size_t n) {
  void* p = nullptr;
  return sim_malloc(&p, n) == hipSuccess ? p : nullptr;
}
void* sim_stream() {
  hipStream_t s;
  (void)hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  return s;
}
// A stream held does nothing until it is let go: other work is on it.
void sim_hold(void* s, int held) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  of(static_cast<hipStream_t>(s))->held = held != 0;
  pump();
}
void sim_fill(void* s, uint32_t* p, uint32_t n, uint32_t v) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  enqueue(static_cast<hipStream_t>(s), [=] {
    note("fill");
    for (uint32_t i = 0; i < n; ++i) p[i] = v;
    return true;
  });
}
void sim_wait(void* s, double ms) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  enqueue(static_cast<hipStream_t>(s), timed(ms, [] {}));
}
void sim_set(const char* what, double v) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  const std::string w = what;
  if (w == "steps") g_steps = (uint32_t)v;
  if (w == "worker_ms") g_worker_ms = v;
  if (w == "worker_more") g_worker_more = v;  // each run takes that much longer than the last
  if (w == "served_ms") g_served_ms = v;
  if (w == "step_ms") g_step_ms = v;
  if (w == "room") g_room = v < 0 ? ~size_t(0) : g_used + (size_t)v;
  if (w == "largest") g_largest = v < 0 ? ~size_t(0) : (size_t)v;
  if (w == "reset") g_count.clear();
}
double sim_get(const char* what) {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  if (!std::strcmp(what, "used")) return (double)g_used;
  if (!std::strcmp(what, "resident")) return g_resident;
  return (double)g_count[what];
}
// info: tiles (0: refused), cut edges, extra edges
void sim_cut(int32_t n, const int32_t* off, const int32_t* col, uint32_t sbits, uint32_t xcap, uint32_t most,
             uint32_t threads, uint32_t* id_of, uint32_t* verts, uint64_t* info) {
  TileCut c;
  const bool ok = cut_into_tiles(n, off, col, sbits, xcap, most, threads, &c);
  info[0] = ok ? c.verts.size() : 0;
  info[1] = c.cut;
  info[2] = c.extra;
  if (!ok) return;
  std::memcpy(id_of, c.id_of.data(), 4ull * n);
  std::memcpy(verts, c.verts.data(), 4ull * c.verts.size());
}
uint32_t sim_radius(int32_t n, const int32_t* off, const int32_t* col) { return estimate_radius(n, off, col); }
void sim_pump() {
  std::lock_guard<std::recursive_mutex> lk(g_mu);
  pump();
}
}
