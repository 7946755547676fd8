// Runs the stepping kernels on the CPU (one host thread per lane) for small
// graphs: the row sort and the transposition, then init and the steps until
// one reports the end. Test infrastructure only.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "sim_step_kernels.inc"

namespace simt {
thread_local unsigned lane;
thread_local Wave* wave;
thread_local Group* group;
thread_local dim3 tidx, bidx, bdim, gdim;
thread_local uint64_t nops;
bool check_stacks = false;
}  // namespace simt

using namespace mlmq;

namespace {

// Device memory and LDS start with whatever was there before.
template <class T>
std::vector<T> garbage(size_t count) {
  std::vector<T> v(count ? count : 1);
  std::memset(static_cast<void*>(v.data()), 0xA5, v.size() * sizeof(T));
  return v;
}

template <class F>
void run_grid(uint32_t blocks, uint32_t block, size_t lds, F f) {
  const uint32_t waves = block / 64;
  std::vector<simt::Wave*> wv;
  std::vector<simt::Group> grp(blocks);
  std::vector<std::barrier<>*> bars;
  std::vector<std::vector<uint64_t>> mem(blocks);
  for (uint32_t g = 0; g < blocks; ++g) {
    bars.push_back(new std::barrier<>(block));
    mem[g] = garbage<uint64_t>(lds / 8 + 1);
    grp[g].bar = bars.back();
    grp[g].lds = reinterpret_cast<uint8_t*>(mem[g].data());
    for (uint32_t w = 0; w < waves; ++w) wv.push_back(new simt::Wave());
  }
  std::vector<std::thread> th;
  for (uint32_t g = 0; g < blocks; ++g)
    for (uint32_t t = 0; t < block; ++t)
      th.emplace_back([&, g, t] {
        simt::lane = t % 64;
        simt::nops = 0;
        simt::wave = wv[g * waves + t / 64];
        simt::group = &grp[g];
        simt::tidx = dim3(t);
        simt::bidx = dim3(g);
        simt::bdim = dim3(block);
        simt::gdim = dim3(blocks);
        f();
      });
  for (auto& t : th) t.join();
  for (auto* p : wv) delete p;
  for (auto* p : bars) delete p;
}

}  // namespace

// in: 8-byte edges of out-rows off; out: rows by weight class.
extern "C" void sim_sort_rows(const int32_t* off, const uint64_t* in, uint64_t* out, uint32_t n, uint32_t shift) {
  run_grid(2, 256, 4 * (256 + 258), [&] { mlmq_sort_rows(off, in, out, n, shift); });
}

extern "C" void sim_transpose(const int32_t* off, const uint64_t* adj, uint32_t n, uint32_t m, int32_t* ioff,
                              uint64_t* iadj) {
  const uint32_t parts = (n + kScanPart - 1u) / kScanPart;
  auto cnt = garbage<uint32_t>(n + 1);
  auto part = garbage<uint32_t>(parts);
  run_grid(1, 256, 0, [&] { mlmq_zero_words(cnt.data(), n); });
  run_grid(2, 256, 0, [&] { mlmq_count_columns(adj, m, cnt.data()); });
  run_grid(parts, 64, 0, [&] { mlmq_scan_parts(cnt.data(), n, ioff, part.data()); });
  run_grid(1, 64, 0, [&] { mlmq_scan_tops(part.data(), parts); });
  run_grid(2, 256, 0, [&] { mlmq_scan_add(part.data(), n, m, ioff, cnt.data()); });
  run_grid(2, 64, 0, [&] { mlmq_transpose_fill(off, adj, n, cnt.data(), iadj); });
}

// One solve; ops (nullable) receives each step's operation, info: steps,
// state (1 done, 2 failed, 0 out of steps), largest label, and the counters.
extern "C" int sim_step(uint32_t n, const int32_t* off, const uint64_t* adj, const int32_t* ioff, const uint64_t* iadj,
                        const uint32_t* ord_of, uint32_t src, uint32_t* dist, uint32_t delta, uint32_t shift,
                        uint32_t max_w, uint32_t unit, uint32_t cap, uint32_t task_cap, uint32_t blocks, uint32_t limit,
                        uint32_t phase_cost, uint8_t* ops, uint64_t* info) {
  auto lab = garbage<uint32_t>(n);
  auto rec = garbage<StepRec>(kStepMax);
  auto shard = garbage<StepShard>(kStepSegs);
  auto stats = garbage<StepStats>(kStepSegs);
  auto l0 = garbage<uint64_t>((size_t)kStepSegs * cap), l1 = l0, l2 = l0;
  auto t0 = garbage<uint64_t>(2ull * task_cap), t1 = t0;
  StepHost host;
  std::memset(&host, 0, sizeof(host));
  StepArgs a;
  std::memset(&a, 0, sizeof(a));
  a.off = off;
  a.adj = adj;
  a.ioff = ioff;
  a.iadj = iadj;
  a.lab = ord_of ? lab.data() : dist;
  a.ord_of = ord_of;
  a.out = dist;
  a.rec = rec.data();
  a.shard = shard.data();
  a.stats = stats.data();
  a.list[0] = l0.data();
  a.list[1] = l1.data();
  a.settled = l2.data();
  a.task[0] = t0.data();
  a.task[1] = t1.data();
  a.host = &host;
  a.n = n;
  a.source = ord_of ? ord_of[src] : src;
  a.cap = cap;
  a.task_cap = task_cap;
  a.delta = delta;
  a.phase_cost = phase_cost;
  a.m = (uint64_t)off[n];
  a.cls_mask = (1u << shift) - 1u;
  a.max_w = max_w;
  a.unit_w = unit;
  a.want_max = 1;
  run_grid(2, 256, 0, [&] { mlmq_step_init(a); });
  uint32_t s = 0;
  while (host.state == 0 && s + 1 < limit && s + 1 < kStepMax) {
    ++s;
    run_grid(blocks, 64 * kStepWaves, kStepLds, [&] { mlmq_step(a, s); });
    if (ops) ops[s] = (uint8_t)rec[s].op;
  }
  info[0] = s;
  info[1] = host.state;
  info[2] = host.max_label;
  for (int i = 0; i < 5; ++i) info[3 + i] = host.stats[i];
  return 0;
}
