// Stepping solve: layout shared by its host side and its kernels (not ABI).
//
// Graphs of small diameter (power-law, uniform random) are solved by bulk
// steps instead of the persistent queue worker: every step is one launch of
// the same kernel over the whole device, which first works out from the last
// step's counts what to do now (see mlmq_step.hip). Rows are kept sorted by
// weight class, and a transposed copy lets far vertices pull.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlmq {

constexpr uint32_t kStepSegs = 64;       // segments of a work list, one per lane of a reading wave
constexpr uint32_t kStepMax = 320;       // steps of one solve; a solve that needs more goes to the queue worker
constexpr uint32_t kStepChunk = 2048;    // edges of a task of a row too long for one wave
// Rows above these are cut into tasks: a light sweep of a sorted row ends
// early, a heavy one reads nearly all of it.
constexpr uint32_t kStepLongRow = 32768;
constexpr uint32_t kStepLongHeavy = 8192;
constexpr uint32_t kStepWaves = 4;       // waves of a workgroup (independent of each other)

// What a step does.
enum : uint32_t {
  kOpPush = 1,  // expand the listed vertices: edges that lead below t1
  kOpScan,      // read all labels: list the vertices settled in [t0, t1) and those in [t1, t2), measure the rest
  kOpRescan,    // a list ran over: list every vertex in [t0, t1) again
  kOpHeavy,     // expand the settled list: edges that lead to t1 or above
  kOpPullAll,   // every vertex not below t1 looks at its in-edges
  kOpPull,      // the same for the vertices that the last pull kept
  kOpOut,       // labels back in the caller's order, largest finite label
  kOpDone,
  kOpFail,      // a list ran over while it was rebuilt: the queue worker takes the solve
};

// One step: what it does (its first line, stored by the step itself) and what
// its waves found (the second line; zero before the step).
struct alignas(128) StepRec {
  uint32_t op, t0, t1, t2;
  uint32_t slot;   // counter slot of the list being read; (slot + 1) % 3 is the one being written
  uint32_t par;    // buffer of the list being read; the other one is written
  uint32_t hs;     // set of the settled list and of the scan's sums
  uint32_t low;    // pulls: no in-neighbour of interest is below this
  uint32_t pad0[24];
  uint32_t chunks;    // long-row tasks written for the next step
  uint32_t overflow;  // a list ran over
  uint32_t pad1[30];
};

// Counters of one segment, a line of its own. Reset by the steps themselves.
struct alignas(128) StepShard {
  uint32_t f[3];        // list lengths, by slot
  uint32_t chg_min[3];  // smallest label lowered by the pull that wrote the slot's list
  uint32_t inv_max;     // ~(largest finite label) (kOpOut)
  uint32_t pad;
  // what a scan found, by set
  struct alignas(8) {
    uint32_t h;         // length of the settled list
    uint32_t far_min;   // smallest finite label >= t1
    uint32_t far_cnt;   // unsettled vertices with in-edges
    uint32_t pad;
    uint64_t near_vol;  // out-edges of the newly settled
    uint64_t far_vol;   // in-edges of the unsettled
  } s[3];
};

// Work counters for mlmq_stats, one set per segment.
struct alignas(128) StepStats {
  uint64_t expansions, stale, edges, pushes, atomics;
  uint64_t pad[11];
};

static_assert(sizeof(StepRec) == 256 && sizeof(StepShard) == 128 && sizeof(StepStats) == 128, "lines");

// Words the device writes for the waiting host (pinned, coherent).
struct StepHost {
  uint32_t begun;      // step that has begun
  uint32_t state;      // 0 running, 1 done, 2 failed
  uint32_t max_label;  // with `state`
  uint32_t steps;
  uint64_t stats[5];
};

struct StepArgs {
  const int32_t* off;    // out-rows
  const uint64_t* adj;   // col | weight << 32, rows in ascending weight class
  const int32_t* ioff;   // in-rows, same form
  const uint64_t* iadj;
  uint32_t* lab;         // [n] labels
  const uint32_t* ord_of;  // kOpOut: out[v] = lab[ord_of[v]] (null: lab is the output)
  uint32_t* out;
  StepRec* rec;          // [kStepMax]
  StepShard* shard;      // [kStepSegs]
  StepStats* stats;      // [kStepSegs] or null
  uint64_t* list[2];     // [kStepSegs * cap] vertex | distance << 32
  uint64_t* settled;     // [kStepSegs * cap]
  uint64_t* task[2];     // [2 * task_cap] pairs: first edge | end << 32, distance | vertex << 32 | heavy << 63
  StepHost* host;
  uint32_t n, source;
  uint32_t cap;          // entries of a list segment
  uint32_t task_cap;
  uint32_t delta;        // width of a distance step
  uint32_t phase_cost;   // what a distance step's launches cost, in edges
  uint64_t m;            // edges
  uint32_t cls_mask;     // weights whose bits above this mask agree share a class
  uint32_t max_w;
  uint32_t unit_w;       // 1: every edge weighs 1 (breadth-first levels)
  uint32_t want_max;     // 1: the host needs the largest finite label
};

// Kernel launchers.
hipError_t launch_step_init(const StepArgs& a, uint32_t blocks, hipStream_t s);
hipError_t launch_step(const StepArgs& a, uint32_t step, uint32_t blocks, hipStream_t s);
// One step of `count` solves (arguments in device memory); step 0 is the reset.
hipError_t launch_step_many(const StepArgs* d_args, uint32_t count, uint32_t step, uint32_t blocks, hipStream_t s);

// Rows in ascending weight class: adj_out may not be adj_in. Rows keep their bounds.
hipError_t launch_sort_rows(const int32_t* off, const uint64_t* adj_in, uint64_t* adj_out, uint32_t n, uint32_t shift,
                            hipStream_t s);
// Transposed graph: ioff[n + 1] and iadj[m]; scratch holds n + 1 + (n + 1) / 4096 + 2 words.
hipError_t launch_transpose(const int32_t* off, const uint64_t* adj, uint32_t n, uint32_t m, int32_t* ioff,
                            uint64_t* iadj, uint32_t* scratch, hipStream_t s);

}  // namespace mlmq
