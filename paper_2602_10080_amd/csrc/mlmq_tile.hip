// Tiled SSSP kernels for CDNA4 (gfx950): meshes and road-like graphs.
//
// A shortest path on such a graph is thousands of hops long, and through
// queues in memory every hop costs the round trips of a label, a row, an edge
// and a device-wide atomic (8 us of wall time on a 2048 x 2048 road-like
// grid). A tile of vertices with its edges fits the 160 KB of a CU's LDS,
// where the same hop is a few hundred cycles. One launch (a round) takes the
// smallest pending label of all tiles and gives every tile that has a label
// pending below that + width to a workgroup:
//   - labels, the labels at which vertices were last expanded, and packed
//     4-byte edges are loaded into LDS;
//   - every wave expands the vertices of a frontier of its own, one a lane, and
//     those they improve, with LDS atomics, until no vertex below the round's
//     limit is pending;
//   - changed labels are written back, the tile's cut edges push over its
//     border with device-wide atomicMin, and the tiles' smallest pending
//     labels are noted for the next round.
// What bounds it: the chain of LDS round trips. A hop costs 0.45 us (ring entry;
// label, last expansion and edges; atomics); with the waves in lockstep, a
// barrier and a shared frontier a hop, it took 1.0 us. The rest of a round is
// the launch, the load (1.3 us for 1024 vertices), the write-back (1.6 us) and
// the slowest tile.
// No workgroup waits for another, so a round makes progress whatever else the
// device runs; the launch boundary makes one round's writes visible to the
// next. A label may be improved from outside while its tile is in LDS: the
// write-back is an atomicMin, the vertex stays pending (its label is below
// the one it was expanded at), and the improvement has noted the tile's key.

#include "mlmq_tile.h"

namespace mlmq {
namespace {

constexpr uint32_t kInf32 = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t lane() { return __lane_id(); }
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ uint32_t popc(uint64_t m) { return (uint32_t)__popcll(m); }
__device__ __forceinline__ uint32_t first_lane(uint64_t m) { return (uint32_t)__ffsll((long long)m) - 1; }
__device__ __forceinline__ uint32_t rank_of(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ uint32_t uni(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t lane_val(uint32_t x, uint32_t l) { return __builtin_amdgcn_readlane(x, l); }
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) x = min(x, (uint32_t)__shfl_xor(x, o));
  return uni(x);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) x += __shfl_xor(x, o);
  return uni(x);
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o);
    if (lane() >= (uint32_t)o) x += y;
  }
  return x;
}
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) { return a > kInf32 - b ? kInf32 : a + b; }

// LDS (workgroup scope) and device memory (agent scope).
__device__ __forceinline__ uint32_t l_ld(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void l_st(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t l_add(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t l_min(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t g_min(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t g_add(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A workgroup's LDS: control words, then the tile.
struct Lds {
  uint32_t* ctl;    // [kCtlWords]
  uint32_t* lab;    // [S]
  uint32_t* done;   // [S]
  uint32_t* edge;   // [S][4]
  uint32_t* extra;  // [xcap]
  uint16_t* xoff;   // [S + 8]
  uint16_t* q;      // [waves][kTileQueue] frontiers, one ring a wave
};
// ctl: the smallest pending label, how many active tiles each wave counted, the
// tiles that the workgroup visits.
constexpr uint32_t kCtlMin = 0, kCtlCount = 8, kCtlMine = kCtlCount + 16u;
constexpr uint32_t kCtlWords = kCtlMine + kTileVisits;

__device__ __forceinline__ Lds carve(uint64_t* smem, uint32_t sbits, uint32_t xcap) {
  const uint32_t S = 1u << sbits;
  Lds l;
  uint32_t* p = reinterpret_cast<uint32_t*>(smem);
  l.ctl = p;
  p += kCtlWords;
  l.lab = p;
  p += S;
  l.done = p;
  p += S;
  l.edge = p;
  p += 4u * S;
  l.extra = p;
  p += xcap;
  l.xoff = reinterpret_cast<uint16_t*>(p);
  p += (S + 8u) / 2u;
  l.q = reinterpret_cast<uint16_t*>(p);
  return l;
}

// Appends the lanes' vertices with ok to the wave's ring; one that does not
// fit stays pending and is found when the ring has run empty.
__device__ __forceinline__ void enqueue(uint16_t* q, uint32_t head, uint32_t& tail, uint32_t v, bool ok) {
  const uint64_t m = ballot(ok);
  const uint32_t at = tail + rank_of(m);
  if (ok && at - head < kTileQueue) q[at & (kTileQueue - 1u)] = (uint16_t)v;
  tail = min(tail + popc(m), head + kTileQueue);
}

// Smallest pending label of the tile in LDS (a barrier before and after).
__device__ __forceinline__ uint32_t pending_min(const Lds& l, uint32_t nv) {
  uint32_t mn = kInf32;
  for (uint32_t i = threadIdx.x; i < nv; i += blockDim.x) {
    const uint32_t d = l.lab[i];
    if (d < l.done[i]) mn = min(mn, d);
  }
  mn = wave_min(mn);
  if (lane() == 0 && mn != kInf32) (void)l_min(l.ctl + kCtlMin, mn);
  __syncthreads();
  mn = uni(l_ld(l.ctl + kCtlMin));
  __syncthreads();
  if (threadIdx.x == 0) l_st(l.ctl + kCtlMin, kInf32);
  return mn;
}

struct alignas(16) Quad {
  uint32_t x, y, z, w;
};

// Counters of a lane.
struct Work {
  uint32_t exp, edge, push, atom;
};

// One visit of tile t: everything pending below limit.
__device__ __forceinline__ void visit(const TileArgs& a, const Lds& l, uint32_t t, uint32_t limit, uint32_t* key,
                                      Work& work) {
  // (in a group of solves the arguments are in memory: read once)
  const bool unit = uni(a.unit_w) != 0u, count = uni(a.count_work) != 0u;
  const uint32_t S = 1u << a.g.sbits, tid = threadIdx.x, nt = blockDim.x;
  const uint32_t nv = uni(a.g.verts[t]);
  const uint64_t vb = (uint64_t)t << a.g.sbits;
  const uint32_t xb = uni(a.g.xbase[t]), nx = uni(a.g.xbase[t + 1u]) - xb;
  {
    const Quad* ge = reinterpret_cast<const Quad*>(a.g.edge + 4u * vb);
    Quad* le = reinterpret_cast<Quad*>(l.edge);
    for (uint32_t i = tid; i < nv; i += nt) {
      const uint32_t d = a.lab[vb + i], x = a.done[vb + i];
      const Quad e = ge[i];
      l.lab[i] = d;
      l.done[i] = x;
      le[i] = e;
    }
    for (uint32_t i = tid; i < nx; i += nt) l.extra[i] = a.g.extra[xb + i];
    if (nx) {
      const uint32_t* go = reinterpret_cast<const uint32_t*>(a.g.xoff + (uint64_t)t * (S + 8u));
      uint32_t* lo = reinterpret_cast<uint32_t*>(l.xoff);
      for (uint32_t i = tid; i < (nv + 2u) / 2u; i += nt) lo[i] = go[i];
    }
    if (tid == 0u) l_st(l.ctl + kCtlMin, kInf32);
  }
  __syncthreads();
  uint32_t left;
  uint16_t* const q = l.q + (tid >> 6) * kTileQueue;
  const Quad* const quad = reinterpret_cast<const Quad*>(l.edge);
  const uint32_t place = (1u << kTileLocalBits) - 1u;
  do {
    uint32_t head = 0, tail = 0;
    for (uint32_t b = tid & ~63u; b < nv; b += nt) {
      const uint32_t i = b + lane();
      bool in = i < nv;
      if (in) {
        const uint32_t d = l.lab[i];
        in = d < limit && d < l.done[i];
      }
      enqueue(q, head, tail, i, in);
    }
    compiler_fence();
    // Until the ring is empty, no wave waits for another: a hop costs the ring
    // entry, the vertex and its edges, and the atomics, three LDS round trips.
    while (head != tail) {
      const bool in = lane() < tail - head;
      const uint32_t v = q[(head + (in ? lane() : 0u)) & (kTileQueue - 1u)];
      head += min(tail - head, 64u);
      const uint32_t d = l_ld(l.lab + v), x = l_ld(l.done + v);
      const Quad e = quad[v];
      const bool go = in && d < x;  // otherwise expanded at this label before
      const uint32_t u0 = e.x & place, u1 = e.y & place, u2 = e.z & place, u3 = e.w & place;
      const uint32_t n0 = sat_add(d, unit ? 1u : e.x >> kTileLocalBits);
      const uint32_t n1 = sat_add(d, unit ? 1u : e.y >> kTileLocalBits);
      const uint32_t n2 = sat_add(d, unit ? 1u : e.z >> kTileLocalBits);
      const uint32_t n3 = sat_add(d, unit ? 1u : e.w >> kTileLocalBits);
      uint32_t o0 = 0, o1 = 0, o2 = 0, o3 = 0;
      if (go) {
        l_st(l.done + v, d);
        o0 = l_min(l.lab + u0, n0);
        o1 = l_min(l.lab + u1, n1);
        o2 = l_min(l.lab + u2, n2);
        o3 = l_min(l.lab + u3, n3);
      }
      compiler_fence();
      enqueue(q, head, tail, u0, n0 < min(o0, limit));
      enqueue(q, head, tail, u1, n1 < min(o1, limit));
      enqueue(q, head, tail, u2, n2 < min(o2, limit));
      enqueue(q, head, tail, u3, n3 < min(o3, limit));
      if (nx) {
        const uint32_t x1 = go ? l.xoff[v + 1u] : 0u;
        for (uint32_t k = go ? l.xoff[v] : 0u; ballot(k < x1); ++k) {
          uint32_t u = 0, nd = 0, old = 0;
          if (k < x1) {
            const uint32_t ex = l.extra[k];
            u = ex & place;
            nd = sat_add(d, unit ? 1u : ex >> kTileLocalBits);
            old = l_min(l.lab + u, nd);
            if (count) {
              work.edge += 1u;
              work.atom += 1u;
              work.push += nd < old ? 1u : 0u;
            }
          }
          enqueue(q, head, tail, u, nd < min(old, limit));
        }
      }
      if (count && go) {
        // entries that lead back to the vertex fill its record up
        const uint32_t edges = (u0 != v) + (u1 != v) + (u2 != v) + (u3 != v);
        work.exp += 1u;
        work.edge += edges;
        work.atom += edges;
        work.push += (n0 < o0) + (n1 < o1) + (n2 < o2) + (n3 < o3);
      }
      compiler_fence();
    }
    __syncthreads();
    left = pending_min(l, nv);
  } while (left < limit);
  // labels back; over the border
  for (uint32_t i = tid; i < nv; i += nt) {
    const uint32_t d = l.lab[i];
    if (d < a.lab[vb + i]) (void)g_min(a.lab + vb + i, d);
    const uint32_t x = l.done[i];
    if (x != a.done[vb + i]) a.done[vb + i] = x;
  }
  const uint32_t ce = uni(a.g.cbase[t + 1u]);
  for (uint32_t i = uni(a.g.cbase[t]) + tid; i < ce; i += nt) {
    const uint64_t c = a.g.cut[i];
    const uint32_t d = l.done[(uint32_t)(c >> 52)];
    const uint32_t dst = (uint32_t)c;
    const uint32_t nd = sat_add(d, unit ? 1u : (uint32_t)(c >> 32) & kTileMaxWeight);
    if (count) work.edge += d != kInf32 ? 1u : 0u;
    if (nd >= a.lab[dst]) continue;
    if (count) work.atom += 1u;
    if (nd >= g_min(a.lab + dst, nd)) continue;
    if (count) work.push += 1u;
    (void)g_min(key + (dst >> a.g.sbits), nd);
  }
  if (tid == 0u && left != kInf32) (void)g_min(key + t, left);
  __syncthreads();  // LDS is reused by the next tile
}

}  // namespace

// A wave's stretch of the keys: kKeys times 64 consecutive tiles, all loads in
// flight at once.
constexpr uint32_t kKeys = 8;
__device__ __forceinline__ uint32_t key_tile(uint32_t b, uint32_t j) {
  return b + ((threadIdx.x & ~63u) * kKeys) + 64u * j + lane();
}
__device__ __forceinline__ void load_keys(uint32_t (&k)[kKeys], const uint32_t* key, uint32_t b, uint32_t tiles) {
#pragma unroll
  for (uint32_t j = 0; j < kKeys; ++j) {
    const uint32_t t = key_tile(b, j);
    k[j] = t < tiles ? key[t] : kInf32;
  }
}

__device__ __forceinline__ void add_work(uint64_t* to, uint32_t mine) {
  const uint32_t x = wave_sum(mine);
  if (lane() == 0 && x) (void)__hip_atomic_fetch_add(to, (uint64_t)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One round: the tiles with a label pending below the limit, or, when nothing
// is pending, the labels in the caller's order, then the report to the host.
__device__ __forceinline__ void tile_round_body(const TileArgs& a, uint32_t round) {
  extern __shared__ uint64_t smem[];
  const Lds l = carve(smem, a.g.sbits, a.g.xcap);
  const uint32_t tid = threadIdx.x, nt = blockDim.x;
  uint32_t* const k0 = a.key[0];
  uint32_t* const k1 = a.key[1];
  uint32_t* const k2 = a.key[2];
  const uint32_t r3 = round % 3u;
  const uint32_t* const key = r3 == 0u ? k0 : (r3 == 1u ? k1 : k2);
  uint32_t* const next = r3 == 0u ? k1 : (r3 == 1u ? k2 : k0);
  uint32_t* const clear = r3 == 0u ? k2 : (r3 == 1u ? k0 : k1);
  if (blockIdx.x == 0 && tid == 0u)
    __hip_atomic_store(&a.host->begun, round, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  // smallest pending label of all
  if (tid == 0u) l_st(l.ctl + kCtlMin, kInf32);
  __syncthreads();
  uint32_t mn = kInf32;
  for (uint32_t b = 0; b < a.g.tiles; b += kKeys * nt) {
    uint32_t k[kKeys];
    load_keys(k, key, b, a.g.tiles);
#pragma unroll
    for (uint32_t j = 0; j < kKeys; ++j) mn = min(mn, k[j]);
  }
  mn = wave_min(mn);
  if (lane() == 0 && mn != kInf32) (void)l_min(l.ctl + kCtlMin, mn);
  __syncthreads();
  mn = uni(l_ld(l.ctl + kCtlMin));
  if (mn == kInf32) {
    if (uni(a.active[round - 1u]) != 0u) {
      uint32_t inv = kInf32;
      for (uint64_t v = (uint64_t)blockIdx.x * nt + tid; v < a.g.n; v += (uint64_t)gridDim.x * nt) {
        const uint32_t d = a.lab[a.g.id_of[v]];
        a.out[v] = d;
        if (d != kInf32) inv = min(inv, ~d);
      }
      inv = wave_min(inv);
      if (lane() == 0 && inv != kInf32) (void)g_min(&a.stats[blockIdx.x & (kTileSegs - 1u)].inv_max, inv);
    } else if (blockIdx.x == 0 && tid < 64u && uni(a.active[round - 2u]) != 0u) {
      const TileStats* s = a.stats + lane();
      const uint32_t inv = wave_min(s->inv_max);
      uint64_t st[4] = {s->expansions, s->edges, s->pushes, s->atomics};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int o = 32; o; o >>= 1) {
          const uint32_t lo = __shfl_xor((uint32_t)st[i], o), hi = __shfl_xor((uint32_t)(st[i] >> 32), o);
          st[i] += (uint64_t)lo | ((uint64_t)hi << 32);
        }
      }
      if (tid == 0u) {
        TileHost* h = a.host;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          __hip_atomic_store(&h->stats[i], st[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h->max_label, ~inv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h->rounds, round - 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h->state, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
    return;
  }
  if (blockIdx.x == 0 && tid == 0u) a.active[round] = 1u;
  // the workgroup's share of the others' keys goes on to the next round
  // The limit moves on by width a round whether or not every label below the
  // last one is settled: a path that crosses a border is a round late, and
  // holding everything back for the latest one took twice as many rounds
  // (2048 x 2048 road-like grid: 12.6 ms against 7.2).
  // From half of the rounds on sixteen times as fast: a path of 100,000 vertices
  // ran out of rounds at 65,000 hops, after 90 ms that the queue worker then
  // added its 256 to.
  const uint64_t pace = round + (round > kTileRounds / 2u ? 15ull * (round - kTileRounds / 2u) : 0ull);
  const uint64_t steady = pace * a.width;
  uint32_t limit = sat_add(mn, a.width);
  if (steady > limit) limit = steady < kInf32 ? (uint32_t)steady : kInf32;
  for (uint32_t t = blockIdx.x * nt + tid; t < a.g.tiles; t += gridDim.x * nt) {
    const uint32_t k = key[t];
    clear[t] = kInf32;
    if (k >= limit && k != kInf32) (void)g_min(next + t, k);
  }
  // Active tiles in order: workgroup b takes the b-th, the (b + grid)-th, ...;
  // all workgroups count the same keys, each wave a stretch of them.
  uint32_t total = 0;
  for (uint32_t b = 0; b < a.g.tiles; b += kKeys * nt) {
    uint32_t k[kKeys], at = 0;
    load_keys(k, key, b, a.g.tiles);
#pragma unroll
    for (uint32_t j = 0; j < kKeys; ++j) at += popc(ballot(k[j] < limit));
    if (lane() == 0) l.ctl[kCtlCount + (tid >> 6)] = at;
    __syncthreads();
    const uint32_t x = lane() < nt / 64u ? l.ctl[kCtlCount + lane()] : 0u;
    const uint32_t incl = wave_incl_scan(x);
    uint32_t rank = total + lane_val(incl - x, uni(tid >> 6));
    total += lane_val(incl, 63);
#pragma unroll
    for (uint32_t j = 0; j < kKeys; ++j) {
      const uint64_t m = ballot(k[j] < limit);
      const uint32_t r = rank + rank_of(m);
      if (k[j] < limit && r % gridDim.x == blockIdx.x) l.ctl[kCtlMine + r / gridDim.x] = key_tile(b, j);
      rank += popc(m);
    }
    __syncthreads();
  }
  Work work = {0, 0, 0, 0};
  for (uint32_t i = blockIdx.x, k = 0; i < total; i += gridDim.x, ++k)
    visit(a, l, uni(l.ctl[kCtlMine + k]), limit, next, work);
  if (a.count_work) {
    TileStats* s = a.stats + (blockIdx.x & (kTileSegs - 1u));
    add_work(&s->expansions, work.exp);
    add_work(&s->edges, work.edge);
    add_work(&s->pushes, work.push);
    add_work(&s->atomics, work.atom);
  }
}

__global__ void __launch_bounds__(1024) mlmq_tile_round(TileArgs a, uint32_t round) { tile_round_body(a, round); }
// The same round of several solves, one a grid row.
__global__ void __launch_bounds__(1024) mlmq_tile_round_many(const TileArgs* all, uint32_t round) {
  tile_round_body(all[blockIdx.y], round);
}

// Round 0: labels unreachable and nothing expanded, the source pending at 0.
__device__ __forceinline__ void tile_init_body(const TileArgs& a) {
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t ids = (uint64_t)a.g.tiles << a.g.sbits;
  for (uint64_t i = tid; i < ids; i += stride) {
    a.lab[i] = i == a.source ? 0u : kInf32;
    a.done[i] = kInf32;
  }
  for (uint64_t i = tid; i < kTileRounds + 2u; i += stride) a.active[i] = i == 0u ? 1u : 0u;
  for (uint64_t i = tid; i < a.g.tiles; i += stride) {
    a.key[0][i] = a.key[2][i] = kInf32;
    a.key[1][i] = i == a.source >> a.g.sbits ? 0u : kInf32;
  }
  for (uint64_t i = tid; i < kTileSegs; i += stride) {
    TileStats* s = a.stats + i;
    s->expansions = s->edges = s->pushes = s->atomics = 0ull;
    s->inv_max = kInf32;
  }
}

__global__ void __launch_bounds__(256) mlmq_tile_init(TileArgs a) { tile_init_body(a); }
__global__ void __launch_bounds__(256) mlmq_tile_init_many(const TileArgs* all) { tile_init_body(all[blockIdx.y]); }

// ------------------------------------------------------------ building the tiled copy

// inv[id] = vertex of every id, kInf where a tile has none (it is filled first).
__global__ void __launch_bounds__(256) mlmq_tile_blank(TileBuild b) {
  const uint64_t ids = (uint64_t)b.tiles << b.sbits;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ids; i += (uint64_t)gridDim.x * blockDim.x)
    b.inv[i] = kInf32;
}
__global__ void __launch_bounds__(256) mlmq_tile_ids(TileBuild b) {
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < b.n; v += (uint64_t)gridDim.x * blockDim.x)
    b.inv[b.id_of[v]] = (uint32_t)v;
}
// Edges of every vertex inside its tile past the first four, and across its
// border (self-loops never improve a label and are left out).
__global__ void __launch_bounds__(256) mlmq_tile_degrees(TileBuild b) {
  const uint64_t ids = (uint64_t)b.tiles << b.sbits;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ids; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t v = b.inv[i];
    uint32_t loc = 0, cut = 0;
    if (v != kInf32)
      for (int32_t e = b.off[v]; e < b.off[v + 1u]; ++e) {
        const uint32_t w = (uint32_t)b.adj[e];
        if (w == v) continue;
        if ((b.id_of[w] >> b.sbits) == (uint32_t)(i >> b.sbits)) ++loc; else ++cut;
      }
    b.n_extra[i] = loc > 4u ? loc - 4u : 0u;
    b.n_cut[i] = cut;
  }
}
// One wave per tile: places of its vertices' extra and cut edges, and its totals.
__global__ void __launch_bounds__(64) mlmq_tile_places(TileBuild b) {
  const uint32_t S = 1u << b.sbits, t = blockIdx.x;
  const uint64_t base = (uint64_t)t << b.sbits;
  uint32_t rx = 0, rc = 0;
  for (uint32_t k = 0; k < S; k += 64u) {
    const uint64_t i = base + k + lane();
    const uint32_t x = b.n_extra[i], y = b.n_cut[i];
    const uint32_t ix = wave_incl_scan(x), iy = wave_incl_scan(y);
    b.n_extra[i] = rx + ix - x;
    b.n_cut[i] = rc + iy - y;
    b.xoff[(uint64_t)t * (S + 8u) + k + lane()] = (uint16_t)(rx + ix - x);
    rx += lane_val(ix, 63);
    rc += lane_val(iy, 63);
  }
  if (lane() < 8u) b.xoff[(uint64_t)t * (S + 8u) + S + lane()] = (uint16_t)rx;
  if (lane() == 0) {
    b.xbase[t + 1u] = rx;
    b.cbase[t + 1u] = rc;
  }
}
__global__ void __launch_bounds__(64) mlmq_tile_bases(TileBuild b) {
  uint32_t rx = 0, rc = 0;
  for (uint32_t k = 0; k < b.tiles; k += 64u) {
    const uint32_t i = k + lane();
    const uint32_t x = i < b.tiles ? b.xbase[i + 1u] : 0u, y = i < b.tiles ? b.cbase[i + 1u] : 0u;
    const uint32_t ix = wave_incl_scan(x), iy = wave_incl_scan(y);
    if (i < b.tiles) {
      b.xbase[i + 1u] = rx + ix;
      b.cbase[i + 1u] = rc + iy;
    }
    rx += lane_val(ix, 63);
    rc += lane_val(iy, 63);
  }
  if (lane() == 0) b.xbase[0] = b.cbase[0] = 0u;
}
__global__ void __launch_bounds__(256) mlmq_tile_edges(TileBuild b) {
  const uint64_t ids = (uint64_t)b.tiles << b.sbits;
  const uint32_t low = (1u << b.sbits) - 1u;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < ids; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t v = b.inv[i];
    const uint32_t t = (uint32_t)(i >> b.sbits), place = (uint32_t)i & low;
    uint32_t k = 0;
    if (v != kInf32) {
      uint32_t x = b.xbase[t] + b.n_extra[i], y = b.cbase[t] + b.n_cut[i];
      for (int32_t e = b.off[v]; e < b.off[v + 1u]; ++e) {
        const uint64_t a = b.adj[e];
        if ((uint32_t)a == v) continue;
        const uint32_t id = b.id_of[(uint32_t)a];
        const uint32_t w = (uint32_t)(a >> 32);
        const uint32_t word = (id & low) | (w << kTileLocalBits);
        if ((id >> b.sbits) != t)
          b.cut[y++] = (uint64_t)id | ((uint64_t)w << 32) | ((uint64_t)place << 52);
        else if (k < 4u)
          b.edge[4u * i + k++] = word;
        else
          b.extra[x++] = word;
      }
    }
    for (; k < 4u; ++k) b.edge[4u * i + k] = place;
  }
}

// ------------------------------------------------------------ launchers

size_t tile_lds_bytes(uint32_t sbits, uint32_t xcap, uint32_t threads) {
  const size_t S = 1ull << sbits;
  return 4ull * (kCtlWords + 6u * S + xcap + (S + 8u) / 2u + threads / 64u * kTileQueue / 2u);
}

hipError_t tile_set_lds(size_t bytes) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(mlmq_tile_round),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(mlmq_tile_round_many),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  return e;
}

hipError_t launch_tile_init(const TileArgs& a, hipStream_t s) {
  const uint64_t blocks = ((uint64_t)a.g.tiles << a.g.sbits) / 1024u + 8u;
  hipLaunchKernelGGL(mlmq_tile_init, dim3((uint32_t)(blocks < 2048u ? blocks : 2048u)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_tile_round(const TileArgs& a, uint32_t round, uint32_t blocks, uint32_t threads, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_tile_round, dim3(blocks), dim3(threads), tile_lds_bytes(a.g.sbits, a.g.xcap, threads), s, a, round);
  return hipGetLastError();
}

hipError_t launch_tile_many(const TileArgs* d_args, uint32_t count, uint32_t round, uint32_t blocks, uint32_t threads,
                            size_t lds, hipStream_t s) {
  if (round == 0u)
    hipLaunchKernelGGL(mlmq_tile_init_many, dim3(256, count), dim3(256), 0, s, d_args);
  else
    hipLaunchKernelGGL(mlmq_tile_round_many, dim3(blocks, count), dim3(threads), lds, s, d_args, round);
  return hipGetLastError();
}

hipError_t launch_tile_ids(const TileBuild& b, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_tile_blank, dim3(1024), dim3(256), 0, s, b);
  hipLaunchKernelGGL(mlmq_tile_ids, dim3(1024), dim3(256), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_tile_count(const TileBuild& b, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_tile_degrees, dim3(2048), dim3(256), 0, s, b);
  hipLaunchKernelGGL(mlmq_tile_places, dim3(b.tiles), dim3(64), 0, s, b);
  hipLaunchKernelGGL(mlmq_tile_bases, dim3(1), dim3(64), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_tile_fill(const TileBuild& b, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_tile_edges, dim3(2048), dim3(256), 0, s, b);
  return hipGetLastError();
}

}  // namespace mlmq
