// Solves that run as a sequence of launches (stepping and tiled), alone or
// several at once.

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

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Solves in flight at once in a batch: one hardware queue each.
constexpr int kLanes = 4;

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

hipError_t BulkSolve::launch(uint32_t i) {
  return g_->tiles ? launch_tiles(tile_, i, blocks_, stream_) : launch_step(step_, i, blocks_, stream_);
}

int BulkSolve::begin(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c, hipStream_t stream,
                     bool unit_weights, bool dev_out, bool timed) {
  *this = BulkSolve();
  g_ = g;
  c_ = c;
  dist_out_ = dist_out;
  stream_ = stream;
  unit_ = unit_weights;
  dev_out_ = dev_out;
  timeout_ms_ = c.timeout_ms ? c.timeout_ms : 60000;
  end_ = std::chrono::steady_clock::now() + std::chrono::milliseconds(timeout_ms_);
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
  if (e_ == hipSuccess) e_ = g->tiles ? launch_tile_init(tile_, stream) : launch_step_init(step_, std::max(64u, blocks_), stream);
  if (e_ == hipSuccess && evw_) e_ = hipEventRecord(evw_, stream);
  return MLMQ_OK;
}

bool BulkSolve::advance() {
  if (no_room_) return true;
  while (e_ == hipSuccess && !__atomic_load_n(state_, __ATOMIC_ACQUIRE)) {
    if (issued_ + 1 < limit_ && issued_ < *begun_ + kAhead) {
      e_ = launch(++issued_);
      continue;
    }
    if ((++spins_ & 1023u) == 0) {
      if (std::chrono::steady_clock::now() > end_) {
        late_ = true;
        return true;
      }
      const hipError_t q = hipStreamQuery(stream_);
      if (q == hipSuccess && issued_ + 1 >= limit_) return true;  // every launch has run
      if (q != hipSuccess && q != hipErrorNotReady) e_ = q;
    }
    return e_ != hipSuccess;
  }
  return true;
}

int BulkSolve::finish(bool* finished) {
  *finished = !no_room_;
  if (no_room_) return MLMQ_OK;
  hipError_t q;
  while ((q = hipStreamQuery(stream_)) == hipErrorNotReady) __builtin_ia32_pause();
  if (e_ == hipSuccess) e_ = q;
  const bool done = e_ == hipSuccess && __atomic_load_n(state_, __ATOMIC_ACQUIRE) == 1;
  int rc = MLMQ_OK;
  if (e_ != hipSuccess)
    rc = hip_fail(e_, "solve");
  else if (done)
    rc = deliver();
  else if (late_)
    rc = set_error(MLMQ_ERR_TIMEOUT, "the solve overran its timeout of %u ms", timeout_ms_);
  else
    *finished = false;  // out of launches, or a list ran over
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
    t.stats[kCtAtomics] = g_->tiles ? s[2] : s[4];
    fill_stats(c_.stats_out, t, ms, wms, g_->tiles ? blocks_ : blocks_ * kStepWaves, 0);
  }
  return rc;
}

bool bulk_solves(const mlmq_graph* g, const mlmq_config& c, bool unit_weights) {
  return (g->tiles || g->step_ready) && is_default_choice(g, c, unit_weights);
}

int run_bulk(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c, bool unit_weights,
             bool dev_out, bool* finished) {
  BulkSolve s;
  const int rc = s.begin(g, source, dist_out, c, reinterpret_cast<hipStream_t>(c.stream), unit_weights, dev_out, true);
  *finished = true;
  if (rc) return rc;
  while (!s.advance()) __builtin_ia32_pause();
  return s.finish(finished);
}

// Queries `which` of a batch, kLanes at a time on streams of their own, which
// start after what `after` (if given) holds so far. Those that nothing was decided for
// come back in *left.
int run_bulk_batch(const mlmq_graph* const* graphs, const uint32_t* sources, uint32_t* const* dist_outs,
                   const mlmq_config* conf, const std::vector<int32_t>& which, hipStream_t after,
                   uint32_t timeout_ms, int32_t* status, std::vector<int32_t>* left) {
  Streams* streams = nullptr;
  hipError_t e = streams_acquire(&streams);
  if (e != hipSuccess) return hip_fail(e, "batch streams");
  if (after) {
    hipEvent_t ev = nullptr;
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(ev, after);
    for (hipStream_t s : streams->s)
      if (e == hipSuccess) e = hipStreamWaitEvent(s, ev, 0);
    if (ev) (void)hipEventDestroy(ev);
    if (e != hipSuccess) {
      streams_release(streams);
      return hip_fail(e, "batch streams");
    }
  }
  BulkSolve lane[kLanes];
  int32_t query[kLanes];
  size_t next = 0;
  int busy = 0;
  for (int32_t& q : query) q = -1;
  do {
    for (int k = 0; k < kLanes; ++k) {
      if (query[k] < 0 && next < which.size()) {
        const int32_t i = which[next++];
        mlmq_config c = conf[i];
        c.timeout_ms = timeout_ms;
        status[i] = lane[k].begin(graphs[i], sources[i], dist_outs[i], c, streams->s[k], false, true, false);
        if (status[i] == MLMQ_OK) {
          query[k] = i;
          ++busy;
        }
      }
      if (query[k] >= 0 && lane[k].advance()) {
        bool finished = true;
        status[query[k]] = lane[k].finish(&finished);
        if (!finished) left->push_back(query[k]);
        query[k] = -1;
        --busy;
      }
    }
  } while (busy || next < which.size());
  streams_release(streams);
  return MLMQ_OK;
}

}  // namespace mlmq
