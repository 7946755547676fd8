// Keeping the device a few launches ahead (host side of the stepping and the
// tiled solve), and the two as one kind of solve in flight.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdint>

#include "mlmq_api_internal.h"
#include "mlmq_step.h"
#include "mlmq_tile.h"

namespace mlmq {

// Launches kept ahead of the last one known to have begun: enough that the
// device never waits for the host (a launch costs the host 3 us, the shortest
// one runs 5 us), few enough that those queued past the end cost little (2 us
// each).
constexpr uint32_t kAhead = 5;

// When the host gives a solve up. The time allowed runs from the moment the
// device is seen to begin, as the queue worker's does: work that the stream
// held before is not counted. Past that time and a grace (the same as for the
// queue worker) nothing is waited for, begun or not.
class Deadline {
 public:
  using clk = std::chrono::steady_clock;
  explicit Deadline(uint32_t timeout_ms)
      : ms_(timeout_ms ? timeout_ms : 60000), hard_(clk::now() + std::chrono::milliseconds(ms_ + 3000)) {}
  uint32_t ms() const { return ms_; }
  void begun() {
    if (begun_) return;
    begun_ = true;
    end_ = clk::now() + std::chrono::milliseconds(ms_);
  }
  bool over() const {
    const auto now = clk::now();
    return now > hard_ || (begun_ && now > end_);
  }
  // What is left of the time, for the solver that goes on; 0: nothing.
  uint32_t left_ms() const {
    if (!begun_) return ms_;
    const auto left = std::chrono::duration_cast<std::chrono::milliseconds>(end_ - clk::now()).count();
    return left > 0 ? (uint32_t)left : 0u;
  }
  // The device gets this long to be through with what it was given.
  clk::time_point drained_by() const { return std::max(hard_, clk::now()) + std::chrono::milliseconds(5000); }

 private:
  uint32_t ms_;
  bool begun_ = false;
  clk::time_point hard_, end_{};
};

// Waits until the stream is through with all that was put on it so far (not
// with what other threads put there later); hipErrorNotReady: not by `by`.
hipError_t wait_issued(hipStream_t stream, Slab* slab, Deadline::clk::time_point by);

// One solve on a stream: prepare() takes its memory and lays out its
// arguments, begin() enqueues its first launch, advance() the next ones as the
// device gets to them, finish() waits for the stream and delivers the result.
// One thread at a time; a solve that was prepared must be finished.
class BulkSolve {
 public:
  // timed: fill kernel_ms and worker_ms of c.stats_out.
  int prepare(const mlmq_graph* g, uint32_t source, uint32_t* dist_out, const mlmq_config& c, hipStream_t stream,
              bool unit_weights, bool dev_out, bool timed, Deadline* deadline);
  void begin();
  // True once nothing is left to launch (the end, the deadline or an error).
  bool advance();
  // The solve's status; *finished = false: nothing was decided, the queue
  // worker must solve.
  int finish(bool* finished);
  // The same once the stream has been waited for, with what that wait gave.
  int finish(bool* finished, hipError_t waited);

  bool no_room() const { return no_room_; }
  // For solves that share their launches: what a launch needs and tells.
  const StepArgs& step_args() const { return step_; }
  const TileArgs& tile_args() const { return tile_; }
  uint32_t blocks() const { return blocks_; }
  bool over() const { return __atomic_load_n(state_, __ATOMIC_ACQUIRE) != 0; }
  uint32_t begun() const { return *begun_; }
  void fail(hipError_t e) { e_ = e; }
  void set_late() { late_ = true; }
  Slab* slab() const { return slab_; }

 private:
  hipError_t launch(uint32_t i);
  int deliver();

  const mlmq_graph* g_ = nullptr;
  mlmq_config c_{};
  uint32_t* dist_out_ = nullptr;
  hipStream_t stream_ = nullptr;
  bool unit_ = false, dev_out_ = false, late_ = false, no_room_ = false;
  Slab* slab_ = nullptr;
  StepArgs step_{};
  TileArgs tile_{};
  uint32_t blocks_ = 0, limit_ = 0, issued_ = 0, spins_ = 0;
  Deadline* deadline_ = nullptr;
  // words of the waiting host, and where a result check may put its flag
  volatile uint32_t* begun_ = nullptr;
  uint32_t* state_ = nullptr;
  char* desc_ = nullptr;
  uint32_t* final_ = nullptr;  // the labels in the caller's order, on the device
  hipError_t e_ = hipSuccess;
  hipEvent_t ev0_ = nullptr, evw_ = nullptr, ev1_ = nullptr;
};

// Parts of the two solves.
size_t step_memory(const mlmq_graph* g, bool own_lab, bool own_out);
uint32_t step_arguments(const mlmq_graph* g, char* base, uint32_t source, uint32_t* dist_out, bool dev_out, bool unit,
                        bool stats, StepArgs* a);  // workgroups of a launch
size_t tile_memory(const mlmq_graph* g, bool own_out);
uint32_t tile_arguments(const mlmq_graph* g, char* base, uint32_t source, uint32_t* dist_out, bool dev_out, bool unit,
                        bool stats, TileArgs* a);
hipError_t launch_tiles(const TileArgs& a, uint32_t round, uint32_t blocks, hipStream_t s);
hipError_t launch_tiles_many(const TileArgs* d_args, const TileGraph& like, uint32_t count, uint32_t round,
                             uint32_t blocks, hipStream_t s);
uint32_t tile_kind(const mlmq_graph* g);   // graphs of one kind share a launch
uint32_t tile_count(const mlmq_graph* g);

}  // namespace mlmq
