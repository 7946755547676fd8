// What a graph looks like, from its rows on the host (not ABI; no device).
#pragma once

#include <cstdint>

namespace mlmq {

// About how many hops the whole of the graph lies from a vertex of it: searches
// of 2048 vertices (a quarter of a small graph) from four places of sixteen,
// those that do not end among fewer vertices, each continued at the power of
// the radius by which it last grew. The largest of them; 0 when all end early.
uint32_t estimate_radius(int32_t n, const int32_t* off, const int32_t* col);

}  // namespace mlmq
