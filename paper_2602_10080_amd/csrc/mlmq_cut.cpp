#include "mlmq_cut.h"

#include <algorithm>
#include <thread>

namespace mlmq {

namespace {

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr uint32_t kFirstTiles = 16;  // a graph that does not fall into tiles shows it in these, or
constexpr uint32_t kSomeTiles = 16;   // in one of every so many later ones

// One pass grows the tiles, 16-21 ns a vertex (611 x 1379 and 2048 x 2048
// road-like grids 17 and 85 ms with the counting of edges inside it). Several
// tiles grown at once, each from a border of its own, took a third of that, but
// where their regions met the tiles came out in pieces and solves took 6% longer.
struct Cutter {
  int32_t n;
  const int32_t* off;
  const int32_t* col;
  uint32_t sbits, xcap;
  TileCut* out;
  std::vector<uint32_t> queue;  // all that the tile's searches have met, in order; `met` of it are in use
  std::vector<uint64_t> seen;   // a bit for each of them (and for some that are in tiles)
  std::vector<uint64_t> taken;  // a bit for every vertex that is in a tile
  size_t met = 0;
  uint64_t edges = 0, cut = 0, extra = 0;

  // Puts u into the queue if this tile has not met it; without a branch, as
  // half of a search's edges lead back and which ones cannot be foreseen.
  void meet(uint32_t u) {
    uint64_t& word = seen[u >> 6];
    const uint64_t bit = 1ull << (u & 63u);
    queue[met] = u;
    met += ((word | taken[u >> 6]) & bit) == 0;
    word |= bit;
  }
  void room(size_t more) {
    if (queue.size() < met + more) queue.resize(2 * (met + more));
  }
  void forget() {
    for (size_t i = 0; i < met; ++i) seen[queue[i] >> 6] = 0;
    met = 0;
  }
  // The neighbours of v.
  void meet_row(uint32_t v) {
    const uint32_t o = (uint32_t)off[v], deg = (uint32_t)off[v + 1] - o, last = (uint32_t)(off[n] - 1);
    room(deg + 5);
    if (!deg) return;
    const uint32_t u0 = (uint32_t)col[o], u1 = (uint32_t)col[std::min(o + 1u, last)];
    const uint32_t u2 = (uint32_t)col[std::min(o + 2u, last)], u3 = (uint32_t)col[std::min(o + 3u, last)];
    for (uint32_t u : {u0, deg > 1u ? u1 : u0, deg > 2u ? u2 : u0, deg > 3u ? u3 : u0}) meet(u);
    for (uint32_t k = 4; k < deg; ++k) meet((uint32_t)col[o + k]);
  }

  // Where to begin: at a vertex that reaches some hundred others if a few looks
  // find one. (Begun among small pieces, a graph whose one large piece does not
  // fall into tiles shows it at the end only.)
  int32_t start() {
    for (int64_t i = 0; i < 16; ++i) {
      const int32_t at = (int32_t)(i * n / 16);
      room(1);
      meet((uint32_t)at);
      for (size_t qh = 0; qh < met && met < 256; ++qh) meet_row(queue[qh]);
      const bool large = met >= 256;
      forget();
      if (large) return at;
    }
    return 0;
  }

  // What the edges of vertices [from, to) come to.
  void count(int32_t from, int32_t to, uint64_t* cut_edges, uint64_t* extra_edges) const {
    const uint32_t* const id_of = out->id_of.data();
    uint64_t c = 0, x = 0;
    for (int32_t v = from; v < to; ++v) {
      const uint32_t t = id_of[v] >> sbits;
      uint32_t inside = 0, loops = 0;
      for (int32_t e = off[v]; e < off[v + 1]; ++e) {
        inside += (id_of[(uint32_t)col[e]] >> sbits) == t;
        loops += col[e] == v;
      }
      c += (uint32_t)(off[v + 1] - off[v]) - inside;
      inside -= loops;
      x += inside > 4u ? inside - 4u : 0u;
    }
    *cut_edges = c;
    *extra_edges = x;
  }

  bool grow(uint32_t most) {
    const uint32_t S = 1u << sbits;
    std::vector<uint32_t> border;
    size_t bh = 0;
    int32_t next = start(), scanned = 0, left = n;
    uint64_t edges = 0, cut = 0;  // of the first tiles
    while (left > 0) {
      const uint32_t t = (uint32_t)out->verts.size(), base = t << sbits;
      if (t == most) return false;
      uint32_t place = 0, nx = 0;
      bool full = false;
      forget();
      while (!full && left > 0 && place < S - S / 4) {
        size_t qh = met;
        room(1);
        while (bh < border.size() && met == qh) meet(border[bh++]);
        while (met == qh && scanned < n) {
          if ((next & 63) == 0 && taken[next >> 6] == ~0ull) {  // 64 vertices that are all placed
            next += 64;
            scanned += 64;
          } else {
            meet((uint32_t)next);
            ++next;
            ++scanned;
          }
          if (next >= n) next = 0;
        }
        if (met == qh) break;
        for (; qh < met; ++qh) {
          const uint32_t v = queue[qh];
          const uint32_t deg = (uint32_t)(off[v + 1] - off[v]), over = deg > 4u ? deg - 4u : 0u;
          if (place == S || nx + over > xcap) {
            full = true;
            break;
          }
          out->id_of[v] = base + place++;
          taken[v >> 6] |= 1ull << (v & 63u);
          --left;
          nx += over;
          meet_row(v);
          // rows that come up soon: most of a large graph is in no cache
          if (qh + 16 < met) __builtin_prefetch(col + off[queue[qh + 16]]);
          if (met) __builtin_prefetch(off + queue[met - 1]);
        }
        border.insert(border.end(), queue.begin() + (long)qh, queue.begin() + (long)met);
      }
      if (place == 0) return false;  // a row that fits no tile
      out->verts.push_back(place);
      if (t < kFirstTiles || t % kSomeTiles == 0) {
        for (size_t i = 0; i < met; ++i) {
          const uint32_t v = queue[i];
          if ((out->id_of[v] >> sbits) != t || out->id_of[v] == kNone) continue;
          for (int32_t e = off[v]; e < off[v + 1]; ++e) cut += (out->id_of[(uint32_t)col[e]] >> sbits) != t;
          edges += (uint32_t)(off[v + 1] - off[v]);
        }
        if (t >= 7 && (t < kFirstTiles ? 4 * cut > edges : 100 * cut > 27 * edges)) return false;
      }
    }
    return true;
  }
};

}  // namespace

bool cut_into_tiles(int32_t n, const int32_t* off, const int32_t* col, uint32_t sbits, uint32_t xcap, uint32_t most,
                    uint32_t max_threads, TileCut* out) {
  Cutter c{n, off, col, sbits, xcap, out};
  out->id_of.assign((size_t)n, kNone);
  out->verts.clear();
  c.taken.assign((size_t)n / 64 + 1, 0ull);
  c.seen.assign((size_t)n / 64 + 1, 0ull);
  c.queue.resize(4u << sbits);
  if (!c.grow(most)) return false;
  // one thread for every 131072 vertices
  const uint32_t parts = std::min({max_threads, std::max(1u, std::thread::hardware_concurrency()), (uint32_t)n / 131072u + 1u});
  std::vector<uint64_t> sums(2 * parts, 0ull);
  std::vector<std::thread> helpers;
  auto part = [&](uint32_t i) {
    c.count((int32_t)((int64_t)n * i / parts), (int32_t)((int64_t)n * (i + 1) / parts), &sums[2 * i], &sums[2 * i + 1]);
  };
  uint32_t started = 1;
  try {
    for (; started < parts; ++started) helpers.emplace_back(part, started);
  } catch (...) {  // fewer threads: the rest is counted here
  }
  part(0);
  for (uint32_t i = started; i < parts; ++i) part(i);
  for (std::thread& t : helpers) t.join();
  out->cut = out->extra = 0;
  for (uint32_t i = 0; i < parts; ++i) {
    out->cut += sums[2 * i];
    out->extra += sums[2 * i + 1];
  }
  return 4 * out->cut <= (uint64_t)off[n];
}

}  // namespace mlmq
