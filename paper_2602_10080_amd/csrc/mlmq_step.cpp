// Host side of the stepping solve: preparation of a graph's rows, the rules
// that pick the graphs and the calls, and a solve's memory and arguments.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "../../include/mlmq.h"
#include "mlmq_api_internal.h"
#include "mlmq_drive.h"
#include "mlmq_internal.h"
#include "mlmq_shape.h"
#include "mlmq_step.h"

using namespace mlmq;

namespace mlmq {

namespace {

uint32_t class_shift(uint32_t max_w) {
  uint32_t bits = 0;
  while (bits < 32 && (max_w >> bits)) ++bits;
  return bits > 8 ? bits - 8 : 0;
}

struct StepLayout {
  size_t rec, shard, stats, list0, list1, settled, task0, task1, lab, out, bytes;
  uint32_t cap, task_cap;
};

StepLayout step_layout(const mlmq_graph* g, bool own_lab, bool own_out) {
  StepLayout l;
  // A segment takes its share of all vertices and a quarter more, and what
  // the waves' last, partly filled blocks may add.
  l.cap = (uint32_t)((uint64_t)g->n / kStepSegs + (uint64_t)g->n / (4 * kStepSegs) + 8192u);
  // a row above the limit is expanded once per step
  l.task_cap = (uint32_t)(g->m / (kStepChunk / 2) + 64);
  const size_t list = 8ull * kStepSegs * l.cap;
  size_t o = 0;
  auto take = [&o](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  l.rec = take(sizeof(StepRec) * kStepMax);
  l.shard = take(sizeof(StepShard) * kStepSegs);
  l.stats = take(sizeof(StepStats) * kStepSegs);
  l.list0 = take(list);
  l.list1 = take(list);
  l.settled = take(list);
  l.task0 = take(16ull * l.task_cap);
  l.task1 = take(16ull * l.task_cap);
  l.lab = take(own_lab ? 4ull * g->n : 0);
  l.out = take(own_out ? 4ull * g->n : 0);
  l.bytes = o;
  return l;
}

void graph_args(const mlmq_graph* g, StepArgs* a) {
  const bool ordered = g->d_ord_of != nullptr;
  a->off = ordered ? g->d_off_ord : g->d_off;
  a->adj = g->d_sadj;
  a->ioff = g->d_ioff;
  a->iadj = g->d_iadj;
  a->ord_of = ordered ? g->d_ord_of : nullptr;
  a->n = (uint32_t)g->n;
  a->cls_mask = (1u << class_shift(g->max_w)) - 1u;
  a->max_w = g->max_w;
  a->m = (uint64_t)g->m;
  a->phase_cost = 1u << 20;  // three or four launches of 6 us at 50 G edges a second
  // (Both formulas go through the sizes named here; between them they were not
  // measured.) Width of a distance step, as a multiple of the weight below which a vertex
  // has one edge on average. Skewed graphs: wide enough that the vertices most
  // edges end at are settled in the first step and the rest pull (RMAT-23:
  // 1 / 1.5 / 2 / 3 -> 1.13 / 0.98 / 1.14 / 1.32 ms; RMAT-20 0.71 / 0.32 /
  // 0.35 / 0.44). Others: ordering work against the launches of a step
  // (uniform 4 M vertices, 33 M edges: 4 / 8 / 16 / 32 -> 2.04 / 1.70 / 1.71 /
  // 1.72 ms; 150,001 vertices, 0.3 M edges: 8 / 32 / 64 -> 0.69 / 0.46 / 0.39).
  const double deg = std::max(1.0, g->features.avg_deg), m = (double)g->m;
  double f;
  if (g->features.std_deg > g->features.avg_deg)
    f = 1.5 * std::min(3.0, std::max(std::min(1.0, std::max(0.25, deg / 30.0)), std::sqrt(8.4e6 / m)));
  else
    f = 8.0 * std::min(32.0, std::max(1.0, std::sqrt(3.4e7 / m)));
  a->delta = (uint32_t)std::min(1e9, std::max(1.0, f * g->features.avg_w / deg));
}

uint32_t step_blocks(const mlmq_graph* g) {
  // one wave per 64 vertices or 512 edges, up to sixteen waves per CU (with
  // thirty-two the launch and the list counters cost more than the extra loads
  // in flight gain: RMAT-23 1.00 ms against 0.93, uniform 4 M 1.67 against 1.36)
  const uint64_t waves = (uint64_t)g->n / 64 + (uint64_t)g->m / 512;
  return (uint32_t)std::min<uint64_t>(4ull * device_info()->cus, std::max<uint64_t>(16, waves / kStepWaves));
}

}  // namespace

// Whether two configurations ask for the same queues.
static bool same_queues(const mlmq_config& a, const mlmq_config& b) {
  return a.l0_rows == b.l0_rows && a.l1_type == b.l1_type && a.l2_type == b.l2_type && a.relax_mode == b.relax_mode &&
         a.l1_cap == b.l1_cap && a.l1_flush_wb == b.l1_flush_wb && a.delta1 == b.delta1 &&
         a.delta2_log2 == b.delta2_log2 && a.bmax == b.bmax && a.bnum == b.bnum && a.th_v == b.th_v &&
         a.th_hub == b.th_hub && a.hub_chunk == b.hub_chunk && a.wg_size == b.wg_size && a.grid_wgs == b.grid_wgs &&
         a.l2_capacity == b.l2_capacity && a.donate_min == b.donate_min && a.pnum == b.pnum;
}

// The queue configuration of a graph left to the library's choice (the tuned
// one where there is one) is a default, not a request: a solve that carries it
// may run without queues, unless the tuner found queues to be faster. Any other
// configuration gets the queues it describes, and so does a deadline too fine
// for the host to watch (the queue worker's waves watch it themselves).
bool is_default_choice(const mlmq_graph* g, const mlmq_config& c, bool unit_weights) {
  if (c.timeout_ms && c.timeout_ms < 50) return false;
  mlmq_config d;
  {
    std::lock_guard<std::mutex> lk(const_cast<mlmq_graph*>(g)->mu);
    if (g->has_tuned && g->queues_won) return false;
    d = g->has_tuned ? g->tuned : g->sel_config;
  }
  if (unit_weights) {
    d.delta1 = 1;
    d.delta2_log2 = 0;
  }
  return same_queues(c, d);
}

// Whether a graph is shallow enough for steps. A solve takes two to three
// launches a hop, the queue worker a time that grows with the edges too; past
// 320 launches the worker has to begin anew. ms by worker / steps (r: estimated
// radius): triangulated meshes of 64^2 vertices (r 41) 0.39 / 0.51, 128^2 (123)
// 0.98 / 1.22, 384^2 (328) 3.2 / 5.7; a 160^2 mesh with one vertex of degree 40
// (220) 0.91 / 1.49; geometric graphs of 20,000 vertices (90) 0.89 / 1.29 and
// 200,000 (252) 3.5 / 6.2; a ring with few chords (1973) 4.8 / 7.2; but cubes
// with 26 neighbours 64^3 (70) 7.6 / 1.5, uniform graphs (15-60) 0.65 / 0.30 to
// 1.5 / 0.6. Levels need a launch or two a hop: triangulated 64^2 0.44 / 0.45,
// 128^2 1.36 / 1.06, 192^2 (172) 2.1 / 1.75, 384^2 4.1 / 6.7; 160^2 mesh 1.56 / 1.66.
static bool step_suits(uint32_t radius, int64_t m, bool unit) {
  if (radius <= 24) return true;
  return unit ? radius <= 215 && m >= 750ll * radius : radius <= 100 && m >= 4000ll * radius;
}

hipError_t step_prepare(mlmq_graph* g, const int32_t* h_off, const int32_t* h_col) {
  g->step_ready = false;
  // Meshes and road-like graphs (a handful of edges at every vertex) are deep:
  // without the copies at once. Sparse random graphs of a largest degree up to 8 stay on
  // the queue worker too (200,000 vertices, 220,000 edges: 0.58 ms).
  if (g->m == 0 || g->features.max_deg <= 8) return hipSuccess;
  // skewed graphs have hubs that most of the graph is a few hops from
  const bool skewed = g->features.std_deg > g->features.avg_deg;
  const uint32_t radius = skewed ? 0u : estimate_radius(g->n, h_off, h_col);
  for (int unit = 0; unit < 2; ++unit) g->step_for[unit] = step_suits(radius, g->m, unit != 0);
  if (!g->step_for[0] && !g->step_for[1]) return hipSuccess;
  const uint32_t n = (uint32_t)g->n, m = (uint32_t)g->m;
  const bool ordered = g->d_ord_of != nullptr;
  const int32_t* off = ordered ? g->d_off_ord : g->d_off;
  const uint64_t* adj = ordered ? g->d_adj_ord : g->d_adj;
  const uint32_t shift = class_shift(g->max_w);
  // The sorted rows are a copy: the queue worker keeps the caller's edge order
  // (RMAT-20 with bucket queues: 60 ms in that order, 109 over sorted rows,
  // whose runs of equal weight all go to one bucket at a time).
  // One allocation and no temporaries: freeing one would wait for the device
  // to be idle, which beside a resident server kernel it may not be for long. The
  // unsorted in-rows stand where the sorted out-rows come last, and the cursors
  // where the sorted in-rows do.
  const size_t out_bytes = align_up(8ull * m, 256);
  const size_t in_bytes = align_up(std::max(8ull * m, 4ull * (n + 1ull + n / 4096 + 2)), 256);
  hipError_t e = hipMalloc(&g->d_sadj, out_bytes + in_bytes + 4ull * (n + 1ull));
  if (e != hipSuccess) {
    g->d_sadj = nullptr;
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();  // no room for the copies: the graph keeps to the queue worker
    return hipSuccess;
  }
  char* const base = reinterpret_cast<char*>(g->d_sadj);
  g->d_iadj = reinterpret_cast<uint64_t*>(base + out_bytes);
  g->d_ioff = reinterpret_cast<int32_t*>(base + out_bytes + in_bytes);
  e = launch_transpose(off, adj, n, m, g->d_ioff, g->d_sadj, reinterpret_cast<uint32_t*>(g->d_iadj), nullptr);
  if (e == hipSuccess) e = launch_sort_rows(g->d_ioff, g->d_sadj, g->d_iadj, n, shift, nullptr);
  if (e == hipSuccess) e = launch_sort_rows(off, adj, g->d_sadj, n, shift, nullptr);
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  if (e != hipSuccess) return e;
  g->step_ready = true;
  return hipSuccess;
}

size_t step_memory(const mlmq_graph* g, bool own_lab, bool own_out) { return step_layout(g, own_lab, own_out).bytes; }

uint32_t step_arguments(const mlmq_graph* g, char* base, uint32_t source, uint32_t* dist_out, bool dev_out, bool unit,
                        bool stats, StepArgs* a) {
  const bool ordered = g->d_ord_of != nullptr;
  const StepLayout l = step_layout(g, ordered || !dev_out, ordered && !dev_out);
  graph_args(g, a);
  a->lab = ordered || !dev_out ? reinterpret_cast<uint32_t*>(base + l.lab) : dist_out;
  a->out = dev_out ? dist_out : reinterpret_cast<uint32_t*>(base + (ordered ? l.out : l.lab));
  a->rec = reinterpret_cast<StepRec*>(base + l.rec);
  a->shard = reinterpret_cast<StepShard*>(base + l.shard);
  a->stats = stats ? reinterpret_cast<StepStats*>(base + l.stats) : nullptr;
  a->list[0] = reinterpret_cast<uint64_t*>(base + l.list0);
  a->list[1] = reinterpret_cast<uint64_t*>(base + l.list1);
  a->settled = reinterpret_cast<uint64_t*>(base + l.settled);
  a->task[0] = reinterpret_cast<uint64_t*>(base + l.task0);
  a->task[1] = reinterpret_cast<uint64_t*>(base + l.task1);
  a->source = ordered ? g->h_ord_of[source] : source;
  a->cap = l.cap;
  a->task_cap = l.task_cap;
  a->unit_w = unit ? 1u : 0u;
  a->want_max = g->overflow_safe || unit ? 0u : 1u;
  return step_blocks(g);
}

}  // namespace mlmq
