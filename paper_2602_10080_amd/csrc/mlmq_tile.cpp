// Host side of the tiled solve: which graphs are cut, their copy on the device,
// and a solve's memory and arguments.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <vector>

#include "../../include/mlmq.h"
#include "mlmq_api_internal.h"
#include "mlmq_cut.h"
#include "mlmq_drive.h"
#include "mlmq_internal.h"
#include "mlmq_tile.h"

using namespace mlmq;

struct mlmq_tiles {
  TileGraph g{};
  TileCut cut;                  // ids on the host (sources)
  void* mem = nullptr;          // one allocation behind g's arrays
  uint32_t blocks = 0;          // workgroups that fit on the device at once
};

namespace mlmq {

namespace {

constexpr uint32_t kThreads = 512;  // of a workgroup: eight waves, two a SIMD
constexpr uint32_t kCutThreads = 16;

}  // namespace

void tile_destroy(mlmq_tiles* t) {
  if (!t) return;
  (void)hipFree(t->mem);
  delete t;
}

namespace {

// 1024 vertices a tile: four tiles fit a CU, loading one is short, and a round
// ends with its slowest tile (2048 x 2048 road-like grid: 1024 / 2048 / 4096
// vertices 7.0 / 7.2 / 8.0 ms; 611 x 1379 with detours 3.3 / 3.6 / 4.3). A
// graph that fits the largest tile is one tile: nothing is cut, and one round
// solves it.
struct TileSize {
  uint32_t sbits, xcap;
};
TileSize tile_size(const mlmq_graph* g) {
  return (uint32_t)g->n <= (1u << kTileLocalBits) ? TileSize{kTileLocalBits, 4096u} : TileSize{10u, 1024u};
}

}  // namespace

mlmq_tiles* tile_cut(const mlmq_graph* g, const int32_t* off, const int32_t* col) {
  const TileSize z = tile_size(g);
  if (g->m == 0 || g->max_w > kTileMaxWeight || (uint32_t)g->n > kTileMostVertices) return nullptr;
  // Few edges at every vertex, or a graph that is one tile. The lines are on the
  // safe side, not where tiles stop paying: with 9.0, 500 and half of the edges
  // cut, ms by the queue worker / by tiles were 6.5 / 3.5 (512^2, eight
  // neighbours), 4.6 / 1.9 (512^2 triangulated), 2.6 / 1.8 (64^3, six neighbours),
  // 3.5 / 2.6 (geometric graph of 200,000 vertices, degree 8), 3.1 / 1.6 (512^2 mesh
  // with one vertex of degree 40) and 9.9 / 2.9 (1024^2 with one of 400); against
  // that stands the time of a cut that is then refused (making a uniform graph of
  // 150,001 vertices 1.7 ms -> 5.3).
  if (z.sbits == kTileLocalBits) {
    if (g->m > (int64_t)z.xcap + (4ll << z.sbits)) return nullptr;
  } else {
    if ((double)g->m / g->n > 4.8) return nullptr;
    for (int32_t v = 0; v < g->n; ++v)
      if (off[v + 1] - off[v] > 32) return nullptr;
  }
  if (tile_lds_bytes(z.sbits, z.xcap, kThreads) > device_info()->lds_per_wg) return nullptr;
  std::unique_ptr<mlmq_tiles> t(new mlmq_tiles());
  return cut_into_tiles(g->n, off, col, z.sbits, z.xcap, kTileMost, kCutThreads, &t->cut) ? t.release() : nullptr;
}

hipError_t tile_prepare(mlmq_graph* g, mlmq_tiles* of) {
  std::unique_ptr<mlmq_tiles> t(of);
  if (!t) return hipSuccess;
  const TileCut& c = t->cut;
  const uint32_t sbits = tile_size(g).sbits, xcap = tile_size(g).xcap, S = 1u << sbits;
  const DeviceInfo* di = device_info();
  const size_t lds = tile_lds_bytes(sbits, xcap, kThreads);
  const uint32_t tiles = (uint32_t)c.verts.size();
  const uint64_t ids = (uint64_t)tiles << sbits;
  const uint32_t per_cu = std::max<uint32_t>(1, std::min<uint32_t>(4, (uint32_t)(di->lds_per_cu / lds)));
  t->blocks = std::min<uint32_t>(tiles, per_cu * (uint32_t)di->cus);
  if (tiles > kTileVisits * t->blocks) return hipSuccess;
  size_t o = 0;
  auto take = [&o](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  const size_t o_verts = take(4ull * tiles), o_id = take(4ull * g->n), o_xb = take(4ull * (tiles + 1)), o_cb = take(4ull * (tiles + 1));
  const size_t o_xoff = take(2ull * tiles * (S + 8)), o_edge = take(16ull * ids);
  const size_t o_extra = take(4ull * c.extra), o_cut = take(8ull * c.cut);
  // Scratch from the solves' pool: freeing memory would wait for the device to
  // be idle. No room for it or the copy: the graph keeps to the queue worker.
  Slab* slab = nullptr;
  if (slab_acquire(12ull * ids, 0, &slab) != MLMQ_OK) return hipSuccess;
  void* const tmp = slab->dev;
  hipError_t e = hipMalloc(&t->mem, o);
  if (e == hipErrorOutOfMemory) {
    (void)hipGetLastError();
    slab_release(slab);
    return hipSuccess;
  }
  if (e == hipSuccess) {
    char* const base = static_cast<char*>(t->mem);
    TileBuild b;
    std::memset(&b, 0, sizeof(b));
    b.off = g->d_off;
    b.adj = g->d_adj;
    b.inv = static_cast<uint32_t*>(tmp);
    b.n_extra = static_cast<uint32_t*>(tmp) + ids;
    b.n_cut = static_cast<uint32_t*>(tmp) + 2 * ids;
    b.id_of = reinterpret_cast<uint32_t*>(base + o_id);
    b.xbase = reinterpret_cast<uint32_t*>(base + o_xb);
    b.cbase = reinterpret_cast<uint32_t*>(base + o_cb);
    b.xoff = reinterpret_cast<uint16_t*>(base + o_xoff);
    b.extra = reinterpret_cast<uint32_t*>(base + o_extra);
    b.edge = reinterpret_cast<uint32_t*>(base + o_edge);
    b.cut = reinterpret_cast<uint64_t*>(base + o_cut);
    b.tiles = tiles;
    b.sbits = sbits;
    if (g->n <= 65536) {  // one copy for both: a copy takes longer than its bytes
      std::vector<uint32_t> both(o_id / 4 + (size_t)g->n);
      std::copy(c.verts.begin(), c.verts.end(), both.begin());
      std::copy(c.id_of.begin(), c.id_of.end(), both.begin() + (long)(o_id / 4));
      e = hipMemcpy(base, both.data(), 4ull * both.size(), hipMemcpyHostToDevice);
    } else {
      e = hipMemcpy(base + o_verts, c.verts.data(), 4ull * tiles, hipMemcpyHostToDevice);
      if (e == hipSuccess) e = hipMemcpy(base + o_id, c.id_of.data(), 4ull * g->n, hipMemcpyHostToDevice);
    }
    b.n = (uint32_t)g->n;
    if (e == hipSuccess) e = launch_tile_ids(b, nullptr);
    if (e == hipSuccess) e = launch_tile_count(b, nullptr);
    if (e == hipSuccess) e = launch_tile_fill(b, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    t->g.verts = reinterpret_cast<uint32_t*>(base + o_verts);
    t->g.xbase = b.xbase;
    t->g.extra = b.extra;
    t->g.cbase = b.cbase;
    t->g.xoff = b.xoff;
    t->g.edge = b.edge;
    t->g.cut = b.cut;
    t->g.id_of = b.id_of;
    t->g.n = (uint32_t)g->n;
    t->g.tiles = tiles;
    t->g.sbits = sbits;
    t->g.xcap = xcap;
  }
  slab_release(slab);
  // the same bound for every graph: a smaller one never lowers a larger one's
  if (e == hipSuccess) e = tile_set_lds(di->lds_per_wg);
  g->tiles = t.release();  // freed with the graph, on failure too
  return e;
}

namespace {

struct TileLayout {
  size_t lab, done, key0, key1, key2, active, stats, out, bytes;
};

TileLayout tile_layout(const mlmq_graph* g, bool own_out) {
  const TileGraph& t = g->tiles->g;
  const uint64_t ids = (uint64_t)t.tiles << t.sbits;
  TileLayout l;
  size_t o = 0;
  auto take = [&o](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes, 256);
    return at;
  };
  l.lab = take(4 * ids);
  l.done = take(4 * ids);
  l.key0 = take(4ull * t.tiles);
  l.key1 = take(4ull * t.tiles);
  l.key2 = take(4ull * t.tiles);
  l.active = take(4ull * (kTileRounds + 2));
  l.stats = take(sizeof(TileStats) * kTileSegs);
  l.out = take(own_out ? 4ull * g->n : 0);
  l.bytes = o;
  return l;
}

}  // namespace

size_t tile_memory(const mlmq_graph* g, bool own_out) { return tile_layout(g, own_out).bytes; }

uint32_t tile_arguments(const mlmq_graph* g, char* base, uint32_t source, uint32_t* dist_out, bool dev_out, bool unit,
                        bool stats, TileArgs* a) {
  const mlmq_tiles* t = g->tiles;
  const TileLayout l = tile_layout(g, !dev_out);
  a->g = t->g;
  a->lab = reinterpret_cast<uint32_t*>(base + l.lab);
  a->done = reinterpret_cast<uint32_t*>(base + l.done);
  a->key[0] = reinterpret_cast<uint32_t*>(base + l.key0);
  a->key[1] = reinterpret_cast<uint32_t*>(base + l.key1);
  a->key[2] = reinterpret_cast<uint32_t*>(base + l.key2);
  a->active = reinterpret_cast<uint32_t*>(base + l.active);
  a->stats = reinterpret_cast<TileStats*>(base + l.stats);
  a->out = dev_out ? dist_out : reinterpret_cast<uint32_t*>(base + l.out);
  a->source = t->cut.id_of[source];
  // Width of a round: about a dozen hops of a mesh (light edges are taken, so a
  // hop is half a mean weight long). Wider, corrections that cross borders have
  // further to go; narrower, the launches count (2048 x 2048: 2 / 4 / 8 / 16
  // mean weights 11.4 / 8.7 / 7.0 / 10.4 ms). Levels need no correction within
  // a tile: 16 / 64 of them a round 3.8 / 2.8 ms.
  const double w = t->g.tiles == 1 ? 4e9 : (unit ? 64.0 : 8.0 * g->features.avg_w);
  a->width = (uint32_t)std::min(4e9, std::max(1.0, w));
  a->unit_w = unit ? 1u : 0u;
  a->count_work = stats ? 1u : 0u;
  return t->blocks;
}

hipError_t launch_tiles(const TileArgs& a, uint32_t round, uint32_t blocks, hipStream_t s) {
  return launch_tile_round(a, round, blocks, kThreads, s);
}

hipError_t launch_tiles_many(const TileArgs* d_args, const TileGraph& like, uint32_t count, uint32_t round,
                             uint32_t blocks, hipStream_t s) {
  return launch_tile_many(d_args, count, round, blocks, kThreads, tile_lds_bytes(like.sbits, like.xcap, kThreads), s);
}

uint32_t tile_kind(const mlmq_graph* g) { return g->tiles->g.sbits; }
uint32_t tile_count(const mlmq_graph* g) { return g->tiles->g.tiles; }

}  // namespace mlmq
