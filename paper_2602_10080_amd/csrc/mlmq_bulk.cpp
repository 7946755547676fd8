// Solves that run as a sequence of launches (stepping and tiled), alone or
// several in the same launches.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/mlmq.h"
#include "mlmq_api_internal.h"
#include "mlmq_drive.h"
#include "mlmq_internal.h"

using namespace mlmq;

namespace mlmq {

namespace {

// Groups of solves in flight at once in a batch: stepping ones, tiled ones and
// tiled ones of graphs that are one tile.
constexpr int kLanes = 3;
// Solves that share their launches, and the memory they may take together.
constexpr size_t kGroup = 32;
constexpr size_t kGroupBytes = 16ull << 30;

// Streams of one batch at a time; a few sets are kept for the next ones.
struct Streams {
  hipStream_t s[kLanes] = {};
};
std::mutex g_streams_mu;
std::vector<Streams*> g_streams;
constexpr size_t kKeptSets = 4;

hipError_t streams_acquire(Streams** out) {
  {
    std::lock_guard<std::mutex> lk(g_streams_mu);
    if (!g_streams.empty()) {
      *out = g_streams.back();
      g_streams.pop_back();
      return hipSuccess;
    }
  }
  Streams* t = new Streams();
  hipError_t e = hipSuccess;
  for (hipStream_t& s : t->s)
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
  if (e != hipSuccess) {
    for (hipStream_t s : t->s)
      if (s) (void)hipStreamDestroy(s);
    delete t;
    return e;
  }
  *out = t;
  return hipSuccess;
}

void streams_release(Streams* t) {
  {
    std::lock_guard<std::mutex> lk(g_streams_mu);
    if (g_streams.size() < kKeptSets) {
      g_streams.push_back(t);
      return;
    }
  }
  for (hipStream_t s : t->s) (void)hipStreamDestroy(s);
  delete t;
}

}  // namespace

static void note_end(const mlmq_graph* g, bool unit_weights, bool done);

hipError_t BulkSolve::launch(uint32_t i) {
  return g_->tiles ? launch_tiles(tile_, i, blocks_, stream_) : launch_step(step_, i, blocks_, stream_);
}

int BulkSolve::prepare(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c,
                       hipStream_t stream, bool unit_weights, bool dev_out, bool timed, Deadline* deadline) {
  *this = BulkSolve();
  g_ = g;
  c_ = c;
  dist_out_ = dist_out;
  stream_ = stream;
  unit_ = unit_weights;
  dev_out_ = dev_out;
  deadline_ = deadline;
  const bool ordered = g->d_ord_of != nullptr;
  const size_t mem = align_up(g->tiles ? tile_memory(g, !dev_out) : step_memory(g, ordered || !dev_out, ordered && !dev_out), 256);
  const size_t words = std::max(sizeof(StepHost), sizeof(TileHost));
  const int rc = slab_acquire(mem + align_up(sizeof(QueryDesc), 256) + 256, words + sizeof(QueryDesc) + 64, &slab_);
  if (rc == MLMQ_ERR_OUT_OF_MEMORY) {
    no_room_ = true;  // the queues may need less
    return MLMQ_OK;
  }
  if (rc) return rc;
  char* const base = static_cast<char*>(slab_->dev);
  desc_ = base + mem;
  std::memset(slab_->host, 0, words);
  if (g->tiles) {
    blocks_ = tile_arguments(g, base, source, dist_out, dev_out, unit_weights, c.stats_out != nullptr, &tile_);
    TileHost* h = tile_.host = static_cast<TileHost*>(slab_->host);
    begun_ = &h->begun;
    state_ = &h->state;
    final_ = tile_.out;
    limit_ = kTileRounds;
  } else {
    blocks_ = step_arguments(g, base, source, dist_out, dev_out, unit_weights, c.stats_out != nullptr, &step_);
    StepHost* h = step_.host = static_cast<StepHost*>(slab_->host);
    begun_ = &h->begun;
    state_ = &h->state;
    final_ = step_.out;
    limit_ = kStepMax;
  }
  if (timed && c.stats_out) {
    e_ = hipEventCreate(&ev0_);
    if (e_ == hipSuccess) e_ = hipEventCreate(&evw_);
    if (e_ == hipSuccess) e_ = hipEventCreate(&ev1_);
    if (e_ == hipSuccess) e_ = hipEventRecord(ev0_, stream);
  }
  return MLMQ_OK;
}

void BulkSolve::begin() {
  if (no_room_) return;
  if (e_ == hipSuccess)
    e_ = g_->tiles ? launch_tile_init(tile_, stream_) : launch_step_init(step_, std::max(64u, blocks_), stream_);
  if (e_ == hipSuccess && evw_) e_ = hipEventRecord(evw_, stream_);
}

bool BulkSolve::advance() {
  if (no_room_) return true;
  while (e_ == hipSuccess && !__atomic_load_n(state_, __ATOMIC_ACQUIRE)) {
    if (issued_ + 1 < limit_ && issued_ < *begun_ + kAhead) {
      e_ = launch(++issued_);
      continue;
    }
    if ((++spins_ & 1023u) == 0) {
      const uint32_t begun = *begun_;
      if (begun) deadline_->begun();
      if (deadline_->over()) {
        late_ = true;
        return true;
      }
      if (issued_ + 1 >= limit_ && begun >= issued_) return true;  // no launch is left
      const hipError_t q = hipStreamQuery(stream_);
      if (q != hipSuccess && q != hipErrorNotReady) e_ = q;
    }
    return e_ != hipSuccess;
  }
  return true;
}

// A wait on the stream itself would also wait for what other threads go on
// putting there; an event of its own costs some 8 us (uniform graph of 150,001
// vertices 360 -> 368). So the stream is looked at while its end may be near: at
// most five launches of 2 us are left.
hipError_t wait_issued(hipStream_t stream, Slab* slab, Deadline::clk::time_point by) {
  const auto soon = Deadline::clk::now() + std::chrono::microseconds(50);
  hipError_t e;
  while ((e = hipStreamQuery(stream)) == hipErrorNotReady && Deadline::clk::now() < soon) __builtin_ia32_pause();
  if (e != hipErrorNotReady) return e;
  e = slab->done ? hipSuccess : hipEventCreateWithFlags(&slab->done, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventRecord(slab->done, stream);
  if (e != hipSuccess) return e;
  for (uint32_t spins = 1; (e = hipEventQuery(slab->done)) == hipErrorNotReady; ++spins) {
    if ((spins & 1023u) == 0 && Deadline::clk::now() > by) break;
    __builtin_ia32_pause();
  }
  return e;
}

int BulkSolve::finish(bool* finished) {
  return finish(finished, no_room_ ? hipSuccess : wait_issued(stream_, slab_, deadline_->drained_by()));
}

int BulkSolve::finish(bool* finished, hipError_t waited) {
  *finished = !no_room_;
  if (no_room_) return MLMQ_OK;
  if (waited == hipErrorNotReady) {
    // launches of this solve are still to come: its memory is never reused
    return set_error(MLMQ_ERR_TIMEOUT, "the stream did not get through the solve within its timeout of %u ms",
                     deadline_->ms());
  }
  if (e_ == hipSuccess) e_ = waited;
  const bool done = e_ == hipSuccess && __atomic_load_n(state_, __ATOMIC_ACQUIRE) == 1;
  int rc = MLMQ_OK;
  if (e_ != hipSuccess)
    rc = hip_fail(e_, "solve");
  else if (done)
    rc = deliver();
  else if (late_)
    rc = set_error(MLMQ_ERR_TIMEOUT, "the solve overran its timeout of %u ms", deadline_->ms());
  else
    *finished = false;  // out of launches, or a list ran over
  if (done || !*finished) note_end(g_, unit_, done);
  for (hipEvent_t ev : {ev0_, evw_, ev1_})
    if (ev) (void)hipEventDestroy(ev);
  slab_release(slab_);
  slab_ = nullptr;
  return rc;
}

// After the last launch: the overflow test, the copy to a host buffer, the counters.
int BulkSolve::deliver() {
  int rc = MLMQ_OK;
  hipError_t e = hipSuccess;
  float ms = 0, wms = 0;
  if (ev1_) {
    e = hipEventRecord(ev1_, stream_);
    if (e == hipSuccess) e = hipEventSynchronize(ev1_);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev0_, ev1_);
    if (e == hipSuccess) e = hipEventElapsedTime(&wms, evw_, ev1_);
    if (e != hipSuccess) return hip_fail(e, "solve");
  }
  const uint32_t max_label = g_->tiles ? tile_.host->max_label : step_.host->max_label;
  if (!g_->overflow_safe && !unit_ && (uint64_t)max_label + g_->max_w >= kInf) {
    // Some candidate may have been too large to store: exact test, an edge
    // from a finite label to an unreachable one.
    QueryDesc* h_desc = reinterpret_cast<QueryDesc*>(static_cast<char*>(slab_->host) +
                                                     std::max(sizeof(StepHost), sizeof(TileHost)));
    uint32_t* h_flag = reinterpret_cast<uint32_t*>(h_desc + 1);
    std::memset(h_desc, 0, sizeof(*h_desc));
    h_desc->off = g_->d_off;
    h_desc->adj = g_->d_adj;
    h_desc->dist = final_;
    h_desc->n = (uint32_t)g_->n;
    QueryDesc* d_desc = reinterpret_cast<QueryDesc*>(desc_);
    uint32_t* d_flag = reinterpret_cast<uint32_t*>(desc_ + align_up(sizeof(QueryDesc), 256));
    *h_flag = 0;
    e = hipMemcpyAsync(d_desc, h_desc, sizeof(QueryDesc), hipMemcpyHostToDevice, stream_);
    if (e == hipSuccess) e = hipMemcpyAsync(d_flag, h_flag, 4, hipMemcpyHostToDevice, stream_);
    if (e == hipSuccess) e = launch_overflow_check(d_desc, d_flag, stream_);
    if (e == hipSuccess) e = hipMemcpyAsync(h_flag, d_flag, 4, hipMemcpyDeviceToHost, stream_);
    if (e == hipSuccess) e = hipStreamSynchronize(stream_);
    if (e != hipSuccess) return hip_fail(e, "overflow check");
    if (*h_flag) rc = set_error(MLMQ_ERR_DISTANCE_OVERFLOW, "a reachable distance does not fit below 2^32-1");
  }
  if (!dev_out_) {
    e = hipMemcpyAsync(dist_out_, final_, 4ull * g_->n, hipMemcpyDeviceToHost, stream_);
    if (e == hipSuccess) e = hipStreamSynchronize(stream_);
    if (e != hipSuccess) return hip_fail(e, "copying distances");
  }
  if (c_.stats_out) {
    QueryCtrl t;
    std::memset(&t, 0, sizeof(t));
    const uint64_t* s = g_->tiles ? tile_.host->stats : step_.host->stats;
    t.stats[kCtExpansions] = s[0];
    t.stats[kCtStale] = g_->tiles ? 0 : s[1];
    t.stats[kCtEdges] = g_->tiles ? s[1] : s[2];
    t.stats[kCtPushes] = g_->tiles ? s[2] : s[3];
    t.stats[kCtAtomics] = g_->tiles ? s[3] : s[4];
    fill_stats(c_.stats_out, t, ms, wms, blocks_, 0);
  }
  return rc;
}

namespace {
std::mutex g_turn_mu;
uint32_t g_resident = 0, g_under_way = 0;
}  // namespace

BulkTurn::BulkTurn() {
  std::lock_guard<std::mutex> lk(g_turn_mu);
  mine_ = g_resident == 0;
  if (mine_) ++g_under_way;
}
BulkTurn::~BulkTurn() {
  if (!mine_) return;
  std::lock_guard<std::mutex> lk(g_turn_mu);
  --g_under_way;
}
void resident_begin() {
  std::lock_guard<std::mutex> lk(g_turn_mu);
  ++g_resident;
}
bool resident_has_room() {
  std::lock_guard<std::mutex> lk(g_turn_mu);
  return g_under_way == 0;
}
bool resident_waits() {
  std::lock_guard<std::mutex> lk(g_turn_mu);
  return g_resident != 0;
}
void resident_end() {
  std::lock_guard<std::mutex> lk(g_turn_mu);
  --g_resident;
}

bool bulk_solves(const mlmq_graph* g, const mlmq_config& c, bool unit_weights) {
  if (!(g->tiles || (g->step_ready && g->step_for[unit_weights])) || !is_default_choice(g, c, unit_weights))
    return false;
  std::atomic<uint32_t>& skip = g->bulk_skip[unit_weights];
  for (uint32_t k = skip.load(); k;)
    if (skip.compare_exchange_weak(k, k - 1)) return false;
  return true;
}

// A solve that did not come to its end cost its launches (2.5 ms) on top of the
// worker's time, and the next one on the graph most likely does as well (a long
// tail on a power-law graph, 2000 vertices on RMAT-18: 7.5 ms by the worker alone, 10.5
// with the attempt): the next 7 calls do without one, 63 after another failure,
// and so on until one succeeds.
static void note_end(const mlmq_graph* g, bool unit_weights, bool done) {
  std::atomic<uint32_t>& failed = g->bulk_failed[unit_weights];
  if (done) {
    if (failed.load()) failed.store(0);
    return;
  }
  g->bulk_skip[unit_weights].store(failed.fetch_add(1) ? 63u : 7u);
}

int run_bulk(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c, bool unit_weights,
             bool dev_out, bool* finished, uint32_t* left_ms) {
  Deadline deadline(c.timeout_ms);
  BulkSolve s;
  const int rc =
      s.prepare(g, source, dist_out, c, reinterpret_cast<hipStream_t>(c.stream), unit_weights, dev_out, true, &deadline);
  *finished = true;
  if (rc) return rc;
  s.begin();
  while (!s.advance()) __builtin_ia32_pause();
  const int end = s.finish(finished);
  *left_ms = deadline.left_ms();
  if (!*finished && !*left_ms) {
    *finished = true;
    return set_error(MLMQ_ERR_TIMEOUT, "the solve overran its timeout of %u ms", deadline.ms());
  }
  return end;
}

namespace {

// Solves of one kind in lockstep: one launch serves all of them, a grid row
// each, until every one has reported its end.
class BulkGroup {
 public:
  // Takes queries from which[*next] on while they are of one kind and fit.
  void begin(const mlmq_graph* const* graphs, const uint32_t* sources, uint32_t* const* dist_outs,
             const mlmq_config* conf, const std::vector<int32_t>& which, size_t* next, hipStream_t stream,
             Deadline* deadline, int32_t* status, std::vector<int32_t>* left);
  bool advance();
  // False: the stream did not get through; it must be left alone.
  bool finish(int32_t* status, std::vector<int32_t>* left);
  bool busy() const { return !solves_.empty(); }

 private:
  std::vector<BulkSolve> solves_;
  std::vector<int32_t> query_;
  Slab* args_ = nullptr;
  hipStream_t stream_ = nullptr;
  bool tiled_ = false, late_ = false;
  uint32_t blocks_ = 0, limit_ = 0, issued_ = 0, spins_ = 0;
  hipError_t e_ = hipSuccess;
  Deadline* deadline_ = nullptr;  // of the whole batch

  hipError_t launch(uint32_t i) {
    const uint32_t n = (uint32_t)solves_.size();
    if (tiled_)
      return launch_tiles_many(static_cast<const TileArgs*>(args_->dev), solves_[0].tile_args().g, n, i, blocks_, stream_);
    return launch_step_many(static_cast<const StepArgs*>(args_->dev), n, i, blocks_, stream_);
  }
};

void BulkGroup::begin(const mlmq_graph* const* graphs, const uint32_t* sources, uint32_t* const* dist_outs,
                      const mlmq_config* conf, const std::vector<int32_t>& which, size_t* next, hipStream_t stream,
                      Deadline* deadline, int32_t* status, std::vector<int32_t>* left) {
  *this = BulkGroup();
  stream_ = stream;
  deadline_ = deadline;
  size_t bytes = 0;
  uint32_t most = 0, tiles = 0;
  while (*next < which.size() && solves_.size() < kGroup) {
    const int32_t i = which[*next];
    const mlmq_graph* g = graphs[i];
    const size_t mem = g->tiles ? tile_memory(g, false) : step_memory(g, g->d_ord_of != nullptr, false);
    if (!solves_.empty() && bytes + mem > kGroupBytes) break;
    BulkSolve s;
    const int rc = s.prepare(g, sources[i], dist_outs[i], conf[i], stream, false, true, false, deadline_);
    if (s.no_room() && !solves_.empty()) break;  // as many as fit now, the others after them
    ++*next;
    if (rc) {
      status[i] = rc;
      continue;
    }
    if (s.no_room()) {
      left->push_back(i);
      continue;
    }
    bytes += mem;
    tiled_ = g->tiles != nullptr;
    most = std::max(most, s.blocks());
    if (tiled_) tiles = std::max(tiles, tile_count(g));
    solves_.push_back(s);
    query_.push_back(i);
  }
  if (solves_.empty()) return;
  // The rows share the device. Stepping solves fill it by themselves in their
  // large steps, and a wave pays for itself in the list counters it reads (16
  // sources on RMAT-20: two / four / eight launches' worth of workgroups 5.9 /
  // 4.6 / 4.3 ms); a tiled round has tiles for one launch's worth (8 sources on
  // a 1024 x 1024 grid: one / two / four 10.4 / 10.2 / 11.5 ms, 32 sources 18.7 /
  // 19.1 / 20.0).
  const uint32_t n = (uint32_t)solves_.size();
  const uint32_t all = (tiled_ ? 1u : 8u) * most;
  blocks_ = std::min(most, std::max((all + n - 1u) / n, most / 16u + 1u));
  if (tiled_) blocks_ = std::max(blocks_, (tiles + kTileVisits - 1u) / kTileVisits);
  limit_ = tiled_ ? kTileRounds : kStepMax;
  const size_t one = tiled_ ? sizeof(TileArgs) : sizeof(StepArgs);
  if (slab_acquire(one * n, one * n, &args_) != MLMQ_OK) {
    e_ = hipErrorOutOfMemory;  // finish() reports it
    return;
  }
  for (uint32_t i = 0; i < n; ++i) {
    char* to = static_cast<char*>(args_->host) + one * i;
    if (tiled_)
      std::memcpy(to, &solves_[i].tile_args(), one);
    else
      std::memcpy(to, &solves_[i].step_args(), one);
  }
  e_ = hipMemcpyAsync(args_->dev, args_->host, one * n, hipMemcpyHostToDevice, stream);
  if (e_ == hipSuccess) e_ = launch(0);
}

bool BulkGroup::advance() {
  for (;;) {
    if (e_ != hipSuccess) return true;
    bool over = true;
    uint32_t begun = 0;  // all rows of a launch begin together
    for (const BulkSolve& s : solves_) {
      over = over && s.over();
      begun = std::max(begun, s.begun());
    }
    if (over) return true;
    if (issued_ + 1 < limit_ && issued_ < begun + kAhead) {
      e_ = launch(++issued_);
      continue;
    }
    if ((++spins_ & 1023u) == 0) {
      if (begun) deadline_->begun();
      if (deadline_->over()) {
        late_ = true;
        return true;
      }
      if (issued_ + 1 >= limit_ && begun >= issued_) return true;
      const hipError_t q = hipStreamQuery(stream_);
      if (q != hipSuccess && q != hipErrorNotReady) e_ = q;
    }
    return e_ != hipSuccess;
  }
}

bool BulkGroup::finish(int32_t* status, std::vector<int32_t>* left) {
  Slab* const any = args_ ? args_ : solves_[0].slab();
  const hipError_t waited = wait_issued(stream_, any, deadline_->drained_by());
  for (size_t i = 0; i < solves_.size(); ++i) {
    if (e_ != hipSuccess) solves_[i].fail(e_);
    if (late_) solves_[i].set_late();
    bool finished = true;
    status[query_[i]] = solves_[i].finish(&finished, waited);
    if (!finished) left->push_back(query_[i]);
  }
  solves_.clear();
  if (waited != hipErrorNotReady) slab_release(args_);
  args_ = nullptr;
  return waited != hipErrorNotReady;
}

}  // namespace

// The library's own streams do not wait for the null stream by themselves:
// what the caller has put on its stream (a fill of an output buffer, say), the
// null stream included, comes before what they are given next.
hipError_t start_after(hipStream_t after, const hipStream_t* streams, int count) {
  hipEvent_t ev = nullptr;
  hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventRecord(ev, after);
  for (int i = 0; i < count && e == hipSuccess; ++i) e = hipStreamWaitEvent(streams[i], ev, 0);
  if (ev) (void)hipEventDestroy(ev);
  return e;
}

// Queries `which` of a batch in groups that share their launches, on streams of
// their own, which start after what `after` holds so far. Those that nothing was
// decided for come back in *left.
int run_bulk_batch(const mlmq_graph* const* graphs, const uint32_t* sources, uint32_t* const* dist_outs,
                   const mlmq_config* conf, const std::vector<int32_t>& which, hipStream_t after,
                   uint32_t timeout_ms, int32_t* status, std::vector<int32_t>* left, uint32_t* left_ms) {
  Deadline deadline(timeout_ms);
  std::vector<int32_t> of[kLanes];
  for (int32_t i : which)
    of[!graphs[i]->tiles ? 0 : (tile_kind(graphs[i]) < kTileLocalBits ? 1 : 2)].push_back(i);
  Streams* streams = nullptr;
  hipError_t e = streams_acquire(&streams);
  if (e != hipSuccess) return hip_fail(e, "batch streams");
  e = start_after(after, streams->s, kLanes);
  if (e != hipSuccess) {
    streams_release(streams);
    return hip_fail(e, "batch streams");
  }
  BulkGroup group[kLanes];
  size_t next[kLanes] = {};
  bool stuck[kLanes] = {};
  for (bool more = true; more;) {
    more = false;
    for (int k = 0; k < kLanes; ++k) {
      if (stuck[k] || (!group[k].busy() && deadline.over())) {
        for (; next[k] < of[k].size(); ++next[k])
          status[of[k][next[k]]] = set_error(MLMQ_ERR_TIMEOUT, "the batch overran its timeout of %u ms", deadline.ms());
      }
      if (!group[k].busy() && next[k] < of[k].size() && resident_waits()) {
        // a server's kernel waits for this batch: the rest goes on beside it
        left->insert(left->end(), of[k].begin() + (long)next[k], of[k].end());
        next[k] = of[k].size();
      }
      if (!group[k].busy() && next[k] < of[k].size())
        group[k].begin(graphs, sources, dist_outs, conf, of[k], &next[k], streams->s[k], &deadline, status, left);
      if (group[k].busy() && group[k].advance()) stuck[k] = !group[k].finish(status, left);
      more = more || group[k].busy() || next[k] < of[k].size();
    }
  }
  if (std::find(stuck, stuck + kLanes, true) == stuck + kLanes) streams_release(streams);
  *left_ms = deadline.left_ms();
  return MLMQ_OK;
}

}  // namespace mlmq
