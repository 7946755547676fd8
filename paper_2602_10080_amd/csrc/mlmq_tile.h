// Tiled solve: layout shared by its host side and its kernels (not ABI).
//
// Meshes and road-like graphs (few edges at every vertex, deep, and easily cut
// into pieces with few edges between them) are cut into tiles of up to
// 2^sbits vertices that fit a workgroup's LDS with all their edges. A solve is
// a sequence of launches; in each, every active tile is loaded into LDS and
// relaxed there until nothing inside changes, then pushes over its cut edges
// (see mlmq_tile.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mlmq {

constexpr uint32_t kTileLocalBits = 12;  // a packed edge: target in the tile, weight above it
constexpr uint32_t kTileMaxWeight = (1u << 20) - 1u;
constexpr uint32_t kTileRounds = 8192;   // launches of one solve
constexpr uint32_t kTileMostVertices = 1u << 24;  // of a graph
constexpr uint32_t kTileMost = 17408;    // tiles of a graph: those vertices in tiles that are 94% full
constexpr uint32_t kTileQueue = 512;     // vertices of a wave's frontier
constexpr uint32_t kTileVisits = 64;     // most tiles that a workgroup visits in a round

// Words the device writes for the waiting host (pinned, coherent).
struct TileHost {
  uint32_t begun;      // round that has begun
  uint32_t state;      // 0 running, 1 done
  uint32_t max_label;  // largest finite label, with `state`
  uint32_t rounds;
  uint64_t stats[4];   // expansions, edges, pushes, atomics
};

// Work counters for mlmq_stats, one set per segment.
struct alignas(128) TileStats {
  uint64_t expansions, edges, pushes, atomics;
  uint32_t inv_max;  // ~(largest finite label)
  uint32_t pad[23];
};
constexpr uint32_t kTileSegs = 64;

// Vertex ids of the tiled copy: tile << sbits | place in the tile. A vertex's
// first four edges inside its tile stand in one 16-byte record (missing ones
// lead back to the vertex at weight 0), further ones in the tile's extra list.
struct TileGraph {
  const uint32_t* verts;   // [tiles] vertices of a tile
  const uint32_t* edge;    // [tiles << sbits][4] place in the tile | weight << 12
  const uint32_t* xbase;   // [tiles + 1] first extra edge
  const uint32_t* extra;   // the same form
  const uint16_t* xoff;    // [tiles][2^sbits + 8] first extra edge of a vertex within its tile
  const uint32_t* cbase;   // [tiles + 1] first cut edge
  const uint64_t* cut;     // target id | weight << 32 | place of the source << 52
  const uint32_t* id_of;   // [n] caller's vertex -> id
  uint32_t n, tiles, sbits;
  uint32_t xcap;           // most extra edges of a tile
};

struct TileArgs {
  TileGraph g;
  uint32_t* lab;       // [tiles << sbits] labels
  uint32_t* done;      // [tiles << sbits] label a vertex was last expanded at; pending: lab < done
  uint32_t* key[3];    // [tiles] smallest pending label of a tile: read, written, cleared in turn
  uint32_t* active;    // [kTileRounds + 2] whether a round had a tile to visit
  TileStats* stats;    // [kTileSegs]
  uint32_t* out;       // [n] caller's order
  TileHost* host;
  uint32_t source;     // id
  uint32_t width;      // a round's limit lies that much further than the last one's
  uint32_t unit_w;     // 1: every edge weighs 1 (breadth-first levels)
  uint32_t count_work; // 1: keep the counters
};

// LDS bytes of a workgroup.
size_t tile_lds_bytes(uint32_t sbits, uint32_t xcap, uint32_t threads);
hipError_t launch_tile_init(const TileArgs& a, hipStream_t s);
hipError_t launch_tile_round(const TileArgs& a, uint32_t round, uint32_t blocks, uint32_t threads, hipStream_t s);
// One round of `count` solves (arguments in device memory); round 0 is the reset.
hipError_t launch_tile_many(const TileArgs* d_args, uint32_t count, uint32_t round, uint32_t blocks, uint32_t threads,
                            size_t lds, hipStream_t s);
// Dynamic LDS that the round kernels may use.
hipError_t tile_set_lds(size_t bytes);

// Building the tiled copy. inv: [tiles << sbits] caller's vertex of an id (kInf: none).
struct TileBuild {
  const int32_t* off;
  const uint64_t* adj;
  uint32_t* inv;
  const uint32_t* id_of;
  uint32_t* n_extra;  // [tiles << sbits] extra edges of a vertex, then their first place
  uint32_t* n_cut;    // the same for edges that leave the tile
  uint32_t* xbase;    // [tiles + 1]
  uint32_t* cbase;    // [tiles + 1]
  uint16_t* xoff;
  uint32_t* edge;
  uint32_t* extra;
  uint64_t* cut;
  uint32_t tiles, sbits, n;
};
hipError_t launch_tile_ids(const TileBuild& b, hipStream_t s);  // inv from id_of
hipError_t launch_tile_count(const TileBuild& b, hipStream_t s);  // counts, places in the tile, bases
hipError_t launch_tile_fill(const TileBuild& b, hipStream_t s);

}  // namespace mlmq
