// Host-side internals shared by the C ABI translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/mlmq.h"
#include "mlmq_internal.h"

struct mlmq_tiles;  // tiled copy of a graph (mlmq_tile.cpp)

// Device-resident graph (the opaque mlmq_graph of the C ABI).
struct mlmq_graph {
  int32_t n = 0;
  int64_t m = 0;
  int32_t* d_off = nullptr;   // [n+1]
  uint64_t* d_adj = nullptr;  // [m] col | weight << 32
  // degree-ordered copy (power-law graphs, for plain solves): vertex v is
  // vertex ord_of[v] there; null when the graph keeps its order
  int32_t* d_off_ord = nullptr;
  uint64_t* d_adj_ord = nullptr;
  uint32_t* d_ord_of = nullptr;     // [n] on the device
  std::vector<uint32_t> h_ord_of;   // [n] on the host (sources)
  mlmq_features features{};
  uint64_t deg_hist[33]{};    // bucket k: degrees in [2^(k-1), 2^k), bucket 0: degree 0
  uint32_t max_w = 0;
  uint32_t min_w = 0;
  bool overflow_safe = false;  // (n-1) * max_w < 2^32 - 1
  std::mutex mu;
  bool has_tuned = false;
  mlmq_config tuned{};
  int32_t sel_template = -1;  // the selector's top template (-1: the feature heuristic)
  mlmq_config sel_config{};   // that template as a configuration for this graph
  bool queues_won = false;    // the tuner found queues faster than the bulk solve
  // stepping solve (mlmq_step.cpp): copies in ascending weight class of the
  // out-rows and in-rows of the graph that plain solves run on
  bool step_ready = false;
  bool step_for[2] = {};  // weighted, unit: whether the steps are few (step_suits)
  // Bulk solves that ran out of steps, rounds or lists, by weighted and unit:
  // how many in a row, and how many of the next calls do without one.
  mutable std::atomic<uint32_t> bulk_failed[2] = {}, bulk_skip[2] = {};
  uint64_t* d_sadj = nullptr;  // [m] out-rows, in one allocation with
  int32_t* d_ioff = nullptr;   // [n+1] in-rows
  uint64_t* d_iadj = nullptr;  // [m]
  mlmq_tiles* tiles = nullptr;  // tiled copy (null: the graph does not fall into tiles)
};

namespace mlmq {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct DeviceInfo {
  bool ok = false;
  int device = 0;
  int cus = 0;
  uint64_t ticks_per_ms = 100000;
  size_t lds_per_wg = 65536;
  size_t lds_per_cu = 65536;
  char name[64] = {0};
};

// Byte layout of one query's queue memory inside a slab.
struct QueryPlan {
  uint32_t nrings = 1, nb_log2 = 4, hub_cap = 1, init_words = 0;
  size_t off_ctrl = 0, off_rings = 0, off_hdr = 0, off_data = 0, off_hub_rec = 0, off_hub_cur = 0, off_hub_pub = 0;
  size_t bytes = 0;
};

// A reusable device allocation plus a pinned host staging area.
struct Slab {
  void* dev = nullptr;
  size_t dev_bytes = 0;
  void* host = nullptr;
  size_t host_bytes = 0;
  hipEvent_t done = nullptr;            // marks the last launch of a bulk solve
  hipGraphExec_t graph_exec = nullptr;  // cached captured launch (batch)
  std::vector<uint64_t> graph_key;      // every argument baked into graph_exec
};

struct LaunchShape {
  uint32_t wg = 256, waves = 4, l1_cap = 64, grid = 1, max_grid = 1;
  bool two = false;
  bool stage = false;
  bool pq = false;  // kernel variant with the L2 priority-queue code
  size_t lds = 0;
};

extern thread_local std::string g_last_error;
int set_error(int code, const char* fmt, ...);
int hip_fail(hipError_t e, const char* what);
const DeviceInfo* device_info();
int need_device();
int check_config(const mlmq_config* c);
void default_config(mlmq_config* c);
void heuristic_config(const mlmq_graph* g, mlmq_config* c);
// Candidate template t (-1: the feature heuristic) as a config for g.
int template_config(const mlmq_graph* g, int32_t t, mlmq_config* out);
// The selector's top template for a graph with features f (-1 without a trained model).
int32_t selector_pick(const mlmq_features& f);
const mlmq_config* resolve_config(const mlmq_graph* g, const mlmq_config* cfg, mlmq_config* tmp);
uint64_t count_degree_above(const mlmq_graph* g, uint32_t th);
QueryPlan plan_query(const mlmq_graph* g, const mlmq_config& c, uint32_t extra_nb_log2, uint32_t hub_scale);
QueryDesc make_desc(const mlmq_graph* g, const mlmq_config& c, const QueryPlan& p, char* base, uint32_t* dist,
                    uint32_t source, uint32_t want_wgs);
int slab_acquire(size_t dev_bytes, size_t host_bytes, Slab** out);
void slab_release(Slab* s);
void pool_trim();
int launch_shape(const mlmq_config& c, uint32_t l1_cap, bool two, bool stage, bool pq, LaunchShape* out);
LaunchArgs make_args(const QueryDesc* d_desc, BatchCtrl* d_batch, int nq, const LaunchShape& s, uint32_t timeout_ms,
                     uint32_t* d_beats);
int status_to_code(uint32_t st);
std::string describe_query_state(const QueryDesc& d, const uint32_t* d_beats, uint32_t nbeats);
void fill_stats(mlmq_stats* st, const QueryCtrl& h, double ms, double worker_ms, uint32_t grid, uint32_t retries);
int run_single(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c,
               bool unit_weights = false, bool queues_only = false);
// Whether c is the library's own choice for g (a solve may then run without queues).
bool is_default_choice(const mlmq_graph* g, const mlmq_config& c, bool unit_weights);
// Rows in ascending weight class and a transposed copy, where g suits the stepping solve.
hipError_t step_prepare(mlmq_graph* g, const int32_t* off, const int32_t* col);
// Tiled copy of g (off, col: host CSR): the cut, on the host alone, null where g
// does not fall into tiles; then the copy on the device, which takes the cut over.
mlmq_tiles* tile_cut(const mlmq_graph* g, const int32_t* off, const int32_t* col);
hipError_t tile_prepare(mlmq_graph* g, mlmq_tiles* cut);
void tile_destroy(mlmq_tiles* t);
// Whether a solve on g with c runs as a sequence of launches (stepping or
// tiled) instead of the queue worker.
bool bulk_solves(const mlmq_graph* g, const mlmq_config& c, bool unit_weights);
// Bulk solves and resident server kernels share the device only in turn. A
// resident kernel holds three waves of 160 registers on three SIMDs of a CU
// and two on the fourth; a step's workgroup (four waves of 64 registers) or a
// tile's (eight of 48 and 39 to 131 KB of LDS) would wait for it to leave,
// which under load it does not. So while one is there, or about to be, solves
// take the queue worker, whose one-wave workgroups find room, and a server's
// kernel starts when the bulk solves under way have ended.
class BulkTurn {
 public:
  BulkTurn();
  ~BulkTurn();
  BulkTurn(const BulkTurn&) = delete;
  BulkTurn& operator=(const BulkTurn&) = delete;
  explicit operator bool() const { return mine_; }

 private:
  bool mine_;
};
void resident_begin();         // from here on no bulk solve begins
bool resident_has_room();      // none is under way
bool resident_waits();         // a batch begins no further group
void resident_end();
// Such a solve; *finished = false: nothing was decided, the queue worker must
// solve in the *left_ms that are left of the deadline.
int run_bulk(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c, bool unit_weights,
             bool dev_out, bool* finished, uint32_t* left_ms);
// Makes the streams wait for what `after` (null: the null stream) holds so far.
hipError_t start_after(hipStream_t after, const hipStream_t* streams, int count);
// Several, into device buffers, with one deadline for all; status[i] for each i
// of which, *left: undecided.
int run_bulk_batch(const mlmq_graph* const* graphs, const uint32_t* sources, uint32_t* const* dist_outs,
                   const mlmq_config* conf, const std::vector<int32_t>& which, hipStream_t after,
                   uint32_t timeout_ms, int32_t* status, std::vector<int32_t>* left, uint32_t* left_ms);
// What the host watchdog snapshots when a launch overruns its deadline.
struct WatchdogView {
  const QueryCtrl* d_ctrl = nullptr;  // first query's control block
  const RingCtr* d_rings = nullptr;   // its ring counters
  const uint32_t* d_beats = nullptr;  // per-wave heartbeats
  uint32_t nbeats = 0;
};
// side: the stream that carries the snapshot reads and the cancel store
// (nullptr = a library stream created on first use).
hipError_t wait_with_watchdog(hipStream_t stream, uint32_t timeout_ms, uint32_t* d_cancel, uint32_t* h_one,
                              const WatchdogView& view, hipStream_t side = nullptr);

}  // namespace mlmq
