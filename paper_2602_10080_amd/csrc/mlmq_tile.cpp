// Host side of the tiled solve: cutting a graph into tiles, and the rounds.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <memory>
#include <vector>

#include "../../include/mlmq.h"
#include "mlmq_api_internal.h"
#include "mlmq_drive.h"
#include "mlmq_internal.h"
#include "mlmq_tile.h"

using namespace mlmq;

struct mlmq_tiles {
  TileGraph g{};
  std::vector<uint32_t> id_of;  // [n] on the host (sources)
  void* mem = nullptr;          // one allocation behind g's arrays
  uint32_t blocks = 0;          // workgroups that fit on the device at once
};

namespace mlmq {

namespace {

constexpr uint32_t kThreads = 512;  // of a workgroup: eight waves, two a SIMD

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Tiles grown breadth-first, each from a vertex on the border of the ones
// before, so that they are compact: a tile's vertices, the vertices' ids, and
// how many edges are cut or stand past a vertex's fourth inside its tile. False
// when the graph does not fall into such pieces: more than a quarter of the
// edges would be cut, or more tiles than a solve takes.
bool cut_into_tiles(int32_t n, const int32_t* off, const int32_t* col, uint32_t sbits, uint32_t xcap,
                    std::vector<uint32_t>* id_of, std::vector<uint32_t>* inv, std::vector<uint32_t>* verts,
                    uint64_t* cut_edges, uint64_t* extra_edges) {
  const uint32_t S = 1u << sbits;
  id_of->assign((size_t)n, kInf);
  inv->clear();
  verts->clear();
  std::vector<uint32_t> seen((size_t)n, 0u);  // tile + 1 whose queue a vertex was put in last
  std::vector<uint32_t> border, queue;
  size_t bh = 0;
  int32_t next = 0, left = n;
  uint64_t edges = 0, cut = 0, extra = 0;
  while (left > 0) {
    if (verts->size() == kTileMost) return false;
    const uint32_t t = (uint32_t)verts->size();
    const uint32_t base = t << sbits;
    uint32_t place = 0, ne = 0, nx = 0;
    inv->resize((size_t)base + S, kInf);
    bool full = false;
    while (!full && left > 0 && place < S - S / 4) {
      int32_t seed = -1;
      while (bh < border.size() && seed < 0) {
        const uint32_t b = border[bh++];
        if ((*id_of)[b] == kInf) seed = (int32_t)b;
      }
      if (seed < 0) {
        while ((*id_of)[next] != kInf) ++next;
        seed = next;
      }
      queue.clear();
      queue.push_back((uint32_t)seed);
      seen[seed] = t + 1u;
      size_t qh = 0;
      for (; qh < queue.size(); ++qh) {
        const uint32_t v = queue[qh];
        const uint32_t deg = (uint32_t)(off[v + 1] - off[v]);
        const uint32_t over = deg > 4u ? deg - 4u : 0u;
        if (place == S || nx + over > xcap) {
          full = true;
          break;
        }
        (*id_of)[v] = base + place;
        (*inv)[(size_t)base + place] = v;
        ++place;
        --left;
        ne += deg;
        nx += over;
        for (int32_t e = off[v]; e < off[v + 1]; ++e) {
          const uint32_t u = (uint32_t)col[e];
          if ((*id_of)[u] == kInf && seen[u] != t + 1u) {
            seen[u] = t + 1u;
            queue.push_back(u);
          }
        }
      }
      border.insert(border.end(), queue.begin() + (long)qh, queue.end());
    }
    verts->push_back(place);
    for (uint32_t i = 0; i < place; ++i) {
      const uint32_t v = (*inv)[(size_t)base + i];
      uint32_t inside = 0;  // loops are left out
      for (int32_t e = off[v]; e < off[v + 1]; ++e) {
        const uint32_t u = (uint32_t)col[e];
        if (((*id_of)[u] >> sbits) != t)
          ++cut;
        else if (u != v)
          ++inside;
      }
      extra += inside > 4u ? inside - 4u : 0u;
    }
    edges += ne;
    // a graph without such pieces shows it at once
    if ((verts->size() >= 8 || left == 0) && 4 * cut > edges) return false;
    if (place == 0) return false;  // a row that fits no tile
  }
  *cut_edges = cut;
  *extra_edges = extra;
  return true;
}

}  // namespace

void tile_destroy(mlmq_tiles* t) {
  if (!t) return;
  (void)hipFree(t->mem);
  delete t;
}

hipError_t tile_prepare(mlmq_graph* g, const int32_t* off, const int32_t* col) {
  const mlmq_features& f = g->features;
  // 1024 vertices a tile: four tiles fit a CU, loading one is short, and a round
  // ends with its slowest tile (2048 x 2048 road-like grid: 1024 / 2048 / 4096
  // vertices 7.0 / 7.2 / 8.0 ms; 611 x 1379 with detours 3.3 / 3.6 / 4.3). A
  // graph that fits the largest tile is one tile: nothing is cut, and one round
  // solves it.
  const bool small = (uint32_t)g->n <= (1u << kTileLocalBits);
  const uint32_t sbits = small ? kTileLocalBits : 10u, xcap = small ? 4096u : 1024u;
  const uint32_t S = 1u << sbits;
  if (g->m == 0 || g->max_w > kTileMaxWeight || (uint32_t)g->n > kTileMostVertices) return hipSuccess;
  // few edges at every vertex, or a graph that is one tile
  if (small ? g->m > (int64_t)xcap + 4 * S : f.avg_deg > 4.8 || f.max_deg > 32) return hipSuccess;
  const size_t lds = tile_lds_bytes(sbits, xcap, kThreads);
  const DeviceInfo* di = device_info();
  if (lds > di->lds_per_wg) return hipSuccess;
  std::vector<uint32_t> inv, verts;
  uint64_t cut = 0, extra = 0;
  std::unique_ptr<mlmq_tiles> t(new mlmq_tiles());
  if (!cut_into_tiles(g->n, off, col, sbits, xcap, &t->id_of, &inv, &verts, &cut, &extra)) return hipSuccess;
  const uint32_t tiles = (uint32_t)verts.size();
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
  const size_t o_verts = take(4ull * tiles), o_xb = take(4ull * (tiles + 1)), o_cb = take(4ull * (tiles + 1));
  const size_t o_xoff = take(2ull * tiles * (S + 8)), o_id = take(4ull * g->n), o_edge = take(16ull * ids);
  const size_t o_extra = take(4ull * extra), o_cut = take(8ull * cut);
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
    e = hipMemcpy(base + o_verts, verts.data(), 4ull * tiles, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(base + o_id, t->id_of.data(), 4ull * g->n, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(tmp, inv.data(), 4ull * ids, hipMemcpyHostToDevice);
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
  a->source = t->id_of[source];
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
