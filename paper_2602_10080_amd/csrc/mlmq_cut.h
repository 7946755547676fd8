// Cutting a graph into tiles, from its rows on the host (not ABI; no device).
#pragma once

#include <cstdint>
#include <vector>

namespace mlmq {

struct TileCut {
  std::vector<uint32_t> id_of;  // [n] tile << sbits | place in the tile
  std::vector<uint32_t> verts;  // [tiles] vertices of a tile
  uint64_t cut = 0;             // edges that leave their tile
  uint64_t extra = 0;           // edges inside it past a vertex's fourth (loops left out)
};

// Tiles of up to 2^sbits vertices and xcap edges past the vertices' fourth,
// grown breadth-first, each from a vertex on the border of the ones before, so
// that they are compact. False when the graph does not fall into such pieces:
// more than a quarter of the edges would be cut, or more than `most` tiles.
// The edges of the finished tiles are counted by up to max_threads threads.
bool cut_into_tiles(int32_t n, const int32_t* off, const int32_t* col, uint32_t sbits, uint32_t xcap, uint32_t most,
                    uint32_t max_threads, TileCut* out);

}  // namespace mlmq
