// Runs the tiled solve's kernels on the CPU (one host thread per lane) for
// small graphs: the build of the tiled copy, then rounds until one reports the
// end. Test infrastructure only.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "hip/hip_runtime.h"

#include "sim_tile_kernels.inc"

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

// id_of, inv, verts: a cut into tiles; info: state, rounds, largest label and
// the counters.
extern "C" void sim_tiles(uint32_t n, const int32_t* off, const uint64_t* adj, const uint32_t* id_of,
                          const uint32_t* inv, const uint32_t* verts, uint32_t tiles, uint32_t sbits, uint32_t xcap,
                          uint32_t src, uint32_t* dist, uint32_t width, uint32_t unit,
                          uint32_t blocks, uint32_t threads, uint32_t limit, uint64_t* info) {
  const uint32_t S = 1u << sbits;
  const uint64_t ids = (uint64_t)tiles << sbits, m = (uint64_t)off[n];
  auto n_extra = garbage<uint32_t>(ids), n_cut = garbage<uint32_t>(ids);
  auto xb = garbage<uint32_t>(tiles + 1), cb = garbage<uint32_t>(tiles + 1);
  auto xoff = garbage<uint16_t>((size_t)tiles * (S + 8));
  auto edge = garbage<uint32_t>(4 * ids), extra = garbage<uint32_t>(m);
  auto cut = garbage<uint64_t>(m);
  TileBuild b;
  std::memset(&b, 0, sizeof(b));
  b.off = off;
  b.adj = adj;
  b.inv = const_cast<uint32_t*>(inv);
  b.id_of = id_of;
  b.n_extra = n_extra.data();
  b.n_cut = n_cut.data();
  b.xbase = xb.data();
  b.cbase = cb.data();
  b.xoff = xoff.data();
  b.edge = edge.data();
  b.extra = extra.data();
  b.cut = cut.data();
  b.tiles = tiles;
  b.sbits = sbits;
  run_grid(1, 256, 0, [&] { mlmq_tile_degrees(b); });
  run_grid(tiles, 64, 0, [&] { mlmq_tile_places(b); });
  run_grid(1, 64, 0, [&] { mlmq_tile_bases(b); });
  run_grid(1, 256, 0, [&] { mlmq_tile_edges(b); });
  auto lab = garbage<uint32_t>(ids), done = lab;
  auto k0 = garbage<uint32_t>(tiles), k1 = k0, k2 = k0;
  auto active = garbage<uint32_t>(kTileRounds + 2);
  auto stats = garbage<TileStats>(kTileSegs);
  TileHost host;
  std::memset(&host, 0, sizeof(host));
  TileArgs a;
  std::memset(&a, 0, sizeof(a));
  a.g.verts = verts;
  a.g.xbase = xb.data();
  a.g.extra = extra.data();
  a.g.xoff = xoff.data();
  a.g.cbase = cb.data();
  a.g.edge = edge.data();
  a.g.cut = cut.data();
  a.g.id_of = id_of;
  a.g.n = n;
  a.g.tiles = tiles;
  a.g.sbits = sbits;
  a.g.xcap = xcap;
  a.lab = lab.data();
  a.done = done.data();
  a.key[0] = k0.data();
  a.key[1] = k1.data();
  a.key[2] = k2.data();
  a.active = active.data();
  a.stats = stats.data();
  a.out = dist;
  a.host = &host;
  a.source = id_of[src];
  a.width = width;
  a.unit_w = unit;
  a.count_work = 1;
  run_grid(1, 256, 0, [&] { mlmq_tile_init(a); });
  const size_t lds = tile_lds_bytes(sbits, xcap, threads);
  for (uint32_t r = 1; r < limit && host.state == 0; ++r) run_grid(blocks, threads, lds, [&] { mlmq_tile_round(a, r); });
  info[0] = host.state;
  info[1] = host.rounds;
  info[2] = host.max_label;
  for (int i = 0; i < 4; ++i) info[3 + i] = host.stats[i];
}
