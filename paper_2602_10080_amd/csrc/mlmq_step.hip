// Stepping SSSP kernels for CDNA4 (gfx950): graphs of small diameter.
//
// The persistent queue worker finds work through queues and orders it only
// within a wave, so on power-law and uniform graphs it scans every edge two
// to many times. Here a solve is a sequence of launches of one kernel, one
// bulk step each, over labels in device memory:
//   - distances are settled in steps of width delta: inside a step [t0, t1)
//     vertices push only the edges that lead below t1 (rows are sorted by
//     weight class, so the others are not even read), until nothing changes;
//     then labels below t1 are final;
//   - a scan of all labels (4 bytes a vertex, the cheapest pass there is)
//     finds the newly settled vertices, the next step's first ones and how
//     many edges lie on either side;
//   - if the settled side still holds many edges that lead to t1 or above and
//     few vertices are left, those vertices pull instead: each reads its
//     in-edges in ascending weight until none can improve it, a cache line or
//     two per vertex on a power-law graph, whose heavy vertices are the
//     settled ones; otherwise the settled vertices push the rest of their
//     rows and the next step begins.
// Every step derives what it does from the counts its predecessor left, the
// same in every wave; there is no wait inside a kernel and no barrier, so a
// launch makes progress whatever else the device runs. The host keeps a few
// launches ahead of the device and stops when a step reports the end.
//
// Labels only fall, by atomicMin while vertices push and by their one owner
// while they pull, so a plain load of a label is at worst too large: the
// result is the fixed point, the same vector whatever the order.

#include "mlmq_step.h"

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
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) x += __shfl_xor(x, o);
  return uni(x);
}
__device__ __forceinline__ uint64_t wave_sum64(uint64_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) {
    const uint32_t lo = __shfl_xor((uint32_t)x, o), hi = __shfl_xor((uint32_t)(x >> 32), o);
    x += (uint64_t)lo | ((uint64_t)hi << 32);
  }
  return x;
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
#pragma unroll
  for (int o = 32; o; o >>= 1) x = min(x, (uint32_t)__shfl_xor(x, o));
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
__device__ __forceinline__ uint32_t ld32(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld64(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st32(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t add32(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void add64(uint64_t* p, uint64_t v) {
  (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Plain cached load of a label (may be stale, i.e. too large).
__device__ __forceinline__ uint32_t ld_label(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void wave_fence() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) { return a > kInf32 - b ? kInf32 : a + b; }
__device__ __forceinline__ uint64_t make_elem(uint32_t v, uint32_t d) { return (uint64_t)v | ((uint64_t)d << 32); }

// One of two buffers (selected, so that the pair is never addressed through memory).
__device__ __forceinline__ uint64_t* pick(uint64_t* const (&p)[2], uint32_t i) {
  uint64_t* const even = p[0];
  uint64_t* const odd = p[1];
  return i & 1u ? odd : even;
}

// ------------------------------------------------------------ a wave's state

// A list being written: 128 entries in LDS, sent out 64 at a time (one
// counter atomic and one 512-byte store per block), each block to the next
// segment in turn, so that the segments stay even.
struct Out {
  uint64_t* buf;   // LDS, 128 entries
  uint64_t* list;
  uint32_t n, seg;
};

struct Wave {
  StepArgs a;
  uint32_t step, w, nw;  // this launch, this wave, waves of the launch
  uint32_t op, t0, t1, t2, slot, par, hs, low;
  uint32_t* order;       // LDS, 64 words
  Out f, h;              // next list, settled list
  uint32_t tasks;        // long-row tasks of the last step
  uint32_t chg_min;      // per lane: smallest label it lowered (pulls)
  uint32_t n_exp, n_stale, n_edges, n_push, n_atom;  // per lane
};

__device__ __forceinline__ uint32_t* f_counter(const Wave& c, uint32_t seg) {
  return &c.a.shard[seg].f[c.slot + 1u >= 3u ? c.slot - 2u : c.slot + 1u];
}
__device__ __forceinline__ uint32_t* h_counter(const Wave& c, uint32_t seg) { return &c.a.shard[seg].s[c.hs].h; }

// Sends the first k <= 64 entries of o out and moves the rest to the front.
__device__ __forceinline__ void out_flush(Wave& c, Out& o, bool settled, uint32_t k) {
  uint32_t base = 0;
  if (lane() == 0) base = add32(settled ? h_counter(c, o.seg) : f_counter(c, o.seg), k);
  base = lane_val(base, 0);
  const uint64_t e = lane() < k ? o.buf[lane()] : 0;
  const uint32_t room = base < c.a.cap ? c.a.cap - base : 0u;
  if (lane() < min(k, room)) o.list[(uint64_t)o.seg * c.a.cap + base + lane()] = e;
  if (k > room && lane() == 0) st32(&c.a.rec[c.step].overflow, 1u);
  const uint32_t left = o.n - k;
  const uint64_t x = lane() < left ? o.buf[64u + lane()] : 0;
  wave_fence();
  if (lane() < left) o.buf[lane()] = x;
  wave_fence();
  o.n = left;
  o.seg = (o.seg + 1u) & (kStepSegs - 1u);
}
__device__ __forceinline__ void append(Wave& c, Out& o, bool settled, uint64_t e, bool ok) {
  const uint64_t m = ballot(ok);
  if (!m) return;
  if (ok) o.buf[o.n + rank_of(m)] = e;
  wave_fence();
  o.n += popc(m);
  if (o.n >= 64u) out_flush(c, o, settled, 64u);
}
__device__ __forceinline__ void out_finish(Wave& c, Out& o, bool settled) {
  if (o.n) out_flush(c, o, settled, o.n);
}

// ------------------------------------------------------------ what to do now

// The step's operation and thresholds, from the last step's record and the
// segments' counters (lane i reads segment i): the same in every workgroup.
// Plain loads: the launch boundary has made the last step's writes visible,
// and a workgroup's reads of these lines hit its XCD's L2 (agent-scope loads
// here, by every wave, made an empty step take 7.5 us instead of 2.1).
__device__ __forceinline__ void decide(Wave& c) {
  const StepRec* p = c.a.rec + (c.step - 1u);
  const StepShard* s = c.a.shard + lane();
  const uint32_t op = uni(p->op);
  c.t0 = uni(p->t0);
  c.t1 = uni(p->t1);
  c.t2 = uni(p->t2);
  c.slot = uni(p->slot);
  c.par = uni(p->par);
  c.hs = uni(p->hs);
  c.low = uni(p->low);
  const uint32_t chunks = uni(p->chunks);
  const bool over = uni(p->overflow) != 0u;
  const uint32_t f0 = s->f[0], f1 = s->f[1], f2 = s->f[2];
  c.tasks = 0;
  if (op == kOpDone || op == kOpFail) {
    c.op = op;
    return;
  }
  if (op == kOpOut) {
    c.op = kOpDone;
    return;
  }
  const uint32_t out = c.slot + 1u >= 3u ? c.slot - 2u : c.slot + 1u;
  const uint32_t listed = wave_sum(min(out == 0u ? f0 : (out == 1u ? f1 : f2), c.a.cap));
  bool next_list = true;  // go on to the list that was written
  if (op == kOpPush) {
    if (over) {
      c.op = kOpRescan;
    } else if ((!c.a.unit_w && listed) || chunks) {
      c.op = kOpPush;
      c.tasks = min(chunks, c.a.task_cap);
    } else {
      c.op = kOpScan;
    }
  } else if (op == kOpRescan) {
    c.op = over ? kOpFail : kOpPush;
  } else if (op == kOpHeavy) {
    c.t0 = c.t1;
    c.t1 = c.a.unit_w ? sat_add(c.t0, 1u) : c.t2;
    if (over) {
      c.op = chunks ? kOpFail : kOpRescan;
    } else if ((!c.a.unit_w && listed) || chunks) {
      c.op = kOpPush;
      c.tasks = min(chunks, c.a.task_cap);
    } else {
      c.op = kOpScan;
    }
  } else if (op == kOpScan) {
    const uint64_t near_vol = wave_sum64(s->s[c.hs].near_vol);
    const uint64_t far_vol = wave_sum64(s->s[c.hs].far_vol);
    const uint32_t far_cnt = wave_sum(s->s[c.hs].far_cnt);
    const uint32_t far_min = wave_min(s->s[c.hs].far_min);
    if (over) {
      c.op = kOpFail;
    } else if (near_vol == 0u && far_min == kInf32) {
      c.op = c.a.ord_of || c.a.want_max ? kOpOut : kOpDone;
    } else if (near_vol == 0u) {
      if (listed) {  // nothing new was settled, but the next step has vertices
        c.t0 = c.t1;
        c.t1 = c.t2;
        c.op = kOpPush;
      } else {
        // An empty stretch: on to the smallest label. The list that the last
        // scan wrote is empty too, and this one writes the next: were it the
        // same, a workgroup that starts late would find it no longer empty
        // and push from it while it is being written.
        c.t0 = far_min;
        c.t1 = c.a.unit_w ? far_min + 1u : far_min;
        c.op = kOpScan;
      }
    } else {
      // Pulling costs about three cache lines per vertex left (its bounds, a
      // line of edges, their labels) and the share of its row that lies below
      // its label, the more the fewer of the in-neighbours are settled yet
      // (with one hub settled, levels on RMAT-23 took 15 ms by pulling at
      // once, 0.5 ms when the hub pushes first). Pushing costs the settled
      // vertices' edges now, many of them with an atomic, and the remaining
      // ones' later, and the launches of at least one more distance step.
      const uint64_t frac = c.a.unit_w ? 42u : min((uint64_t)256u, ((uint64_t)c.t1 * 512u) / ((uint64_t)c.a.max_w + 1u));
      const uint64_t settled = c.a.m > far_vol ? c.a.m - far_vol : 1u;
      const uint64_t probes = min((uint64_t)1u << 18, (c.a.m << 8) / settled);  // in-edges read per settled one, x 256
      const uint64_t pull = 24ull * far_cnt + 3u * frac * (probes * (far_vol >> 8) >> 8);
      if (pull < 3u * near_vol + far_vol + c.a.phase_cost) {
        c.op = kOpPullAll;
        c.low = 0;
      } else {
        c.op = kOpHeavy;
        next_list = false;
      }
    }
  } else {  // a pull
    const uint32_t low = wave_min(s->chg_min[out]);  // smallest label that the sweep lowered
    if (low == kInf32 || (listed == 0u && !over)) {
      c.op = c.a.ord_of || c.a.want_max ? kOpOut : kOpDone;
    } else if (over) {
      c.op = kOpPullAll;
      c.low = 0;
    } else {
      c.op = kOpPull;
      c.low = low;
    }
  }
  if (next_list) {
    c.slot = out;
    c.par ^= 1u;
  }
  if (c.op == kOpScan) {
    c.t2 = sat_add(c.t1, c.a.delta);
    c.hs = c.hs == 2u ? 0u : c.hs + 1u;
  }
  // every lane holds the same values: into scalar registers
  c.op = uni(c.op);
  c.t0 = uni(c.t0);
  c.t1 = uni(c.t1);
  c.t2 = uni(c.t2);
  c.slot = uni(c.slot);
  c.par = uni(c.par);
  c.hs = uni(c.hs);
  c.low = uni(c.low);
  c.tasks = uni(c.tasks);
}

// The first wave records the step, clears the counters that the next step may
// write, and tells the host.
__device__ __forceinline__ void record(const Wave& c) {
  StepRec* r = c.a.rec + c.step;
  StepShard* s = c.a.shard + lane();
  const uint32_t clr = c.slot == 0u ? 2u : c.slot - 1u;  // (slot + 2) % 3
  const uint32_t nh = c.hs == 2u ? 0u : c.hs + 1u;
  st32(&s->f[clr], 0u);
  st32(&s->chg_min[clr], kInf32);
  st32(&s->s[nh].h, 0u);
  st32(&s->s[nh].far_min, kInf32);
  st32(&s->s[nh].far_cnt, 0u);
  __hip_atomic_store(&s->s[nh].near_vol, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&s->s[nh].far_vol, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (lane() == 0) {
    st32(&r->op, c.op);
    st32(&r->t0, c.t0);
    st32(&r->t1, c.t1);
    st32(&r->t2, c.t2);
    st32(&r->slot, c.slot);
    st32(&r->par, c.par);
    st32(&r->hs, c.hs);
    st32(&r->low, c.low);
    __hip_atomic_store(&c.a.host->begun, c.step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// ------------------------------------------------------------ pushing

__device__ __forceinline__ uint32_t weight_of(const Wave& c, uint64_t e) {
  return c.a.unit_w ? 1u : (uint32_t)(e >> 32);
}

// Relaxes U edges per lane at distance d[u], those whose candidate lies in
// [lo, hi); improved vertices below enq join the next list. All label loads
// go out before the first atomic.
template <int U>
__device__ __forceinline__ void relax(Wave& c, const bool (&has)[U], const uint64_t (&e)[U], const uint32_t (&d)[U],
                                      uint32_t lo, uint32_t hi, uint32_t enq) {
  uint32_t nd[U], lab[U];
  bool cand[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint64_t sum = (uint64_t)d[u] + weight_of(c, e[u]);
    cand[u] = has[u] && sum >= lo && sum < hi;
    nd[u] = (uint32_t)sum;
    lab[u] = 0;
    if (cand[u]) lab[u] = ld_label(c.a.lab + (uint32_t)e[u]);
    c.n_edges += has[u] ? 1u : 0u;
  }
  bool imp[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    imp[u] = false;
    if (cand[u] && nd[u] < lab[u]) {
      const uint32_t old = __hip_atomic_fetch_min(c.a.lab + (uint32_t)e[u], nd[u], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
      imp[u] = nd[u] < old;
      c.n_atom += 1u;
      c.n_push += imp[u] ? 1u : 0u;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) append(c, c.f, false, make_elem((uint32_t)e[u], nd[u]), imp[u] && nd[u] < enq);
}

// Whether a row part whose first edge is e holds nothing below hi for a
// vertex at distance d.
__device__ __forceinline__ bool beyond(const Wave& c, uint64_t e, uint32_t d, uint32_t hi) {
  const uint32_t w = c.a.unit_w ? 1u : ((uint32_t)(e >> 32) & ~c.a.cls_mask);
  return hi != kInf32 && (uint64_t)d + w >= hi;
}

// Whole wave sweeps the edges [x, end) of a vertex at distance d; the next
// 256 edges are loaded before the current ones are relaxed.
__device__ __forceinline__ void sweep(Wave& c, uint32_t d, uint32_t x, uint32_t end, uint32_t lo, uint32_t hi,
                                      uint32_t enq) {
  constexpr int U = 4;
  uint64_t nx[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = x + 64u * u + lane();
    nx[u] = i < end ? c.a.adj[i] : 0ull;
  }
  while (x < end) {
    uint64_t e[U];
    bool has[U];
    uint32_t dd[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      e[u] = nx[u];
      has[u] = x + 64u * u + lane() < end;
      dd[u] = d;
    }
    const uint64_t first = (uint64_t)lane_val((uint32_t)e[0], 0) | ((uint64_t)lane_val((uint32_t)(e[0] >> 32), 0) << 32);
    if (beyond(c, first, d, hi)) return;
    x += 64u * U;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = x + 64u * u + lane();
      nx[u] = i < end ? c.a.adj[i] : 0ull;
    }
    relax<U>(c, has, e, dd, lo, hi, enq);
  }
}

// Expands the lanes' vertices (those with ok): eight lanes to a row, one
// 64-byte line of edges at a time; rows that go on past 64 edges are finished
// by the whole wave, and rows above kStepLongRow are cut into tasks that the
// waves of the next step share.
__device__ __forceinline__ void expand(Wave& c, uint32_t v, uint32_t d, uint32_t beg, uint32_t end, bool ok, uint32_t lo,
                                       uint32_t hi, uint32_t enq, bool heavy) {
  c.n_exp += ok ? 1u : 0u;
  const bool big = ok && end - beg > (heavy ? kStepLongHeavy : kStepLongRow);
  uint64_t mb = ballot(big);
  uint32_t first = 0, mine = 0;
  if (mb) {  // one counter atomic for all of the wave's long rows
    mine = big ? (end - beg + kStepChunk - 1u) / kStepChunk : 0u;
    const uint32_t incl = wave_incl_scan(mine);
    const uint32_t all = lane_val(incl, 63);
    if (lane() == 0) first = add32(&c.a.rec[c.step].chunks, all);
    first = lane_val(first, 0) + incl - mine;
  }
  for (; mb; mb &= mb - 1) {
    const uint32_t j = first_lane(mb);
    const uint32_t bv = lane_val(v, j), bd = lane_val(d, j), bb = lane_val(beg, j), be = lane_val(end, j);
    const uint32_t nch = lane_val(mine, j), base = lane_val(first, j);
    uint64_t* const out = pick(c.a.task, c.step);
    for (uint32_t i = lane(); i < nch; i += 64u) {
      if (base + i >= c.a.task_cap) {
        st32(&c.a.rec[c.step].overflow, 1u);
        break;
      }
      const uint32_t x = bb + i * kStepChunk;
      out[2ull * (base + i)] = (uint64_t)x | ((uint64_t)min(be, x + kStepChunk) << 32);
      out[2ull * (base + i) + 1u] = (uint64_t)bd | ((uint64_t)(bv | (heavy ? 0x80000000u : 0u)) << 32);
    }
  }
  ok = ok && !big && end > beg;
  const uint64_t m = ballot(ok);
  if (!m) return;
  if (ok) c.order[rank_of(m)] = lane();
  wave_fence();
  const uint32_t cnt = popc(m);
  const uint32_t sub = lane() & 7u, grp = lane() >> 3;
  for (uint32_t k = 0; k < cnt; k += 8u) {
    const bool in = k + grp < cnt;
    const uint32_t src = c.order[in ? k + grp : 0u];
    const uint32_t gd = __shfl(d, (int)src), gb = __shfl(beg, (int)src), ge = __shfl(end, (int)src);
    uint32_t x = gb;  // the group's place in its row
    bool act = in;
    uint64_t nx = act && x + sub < ge ? c.a.adj[x + sub] : 0ull;
    uint32_t r = 0;
    for (;; ++r) {
      const uint64_t e[1] = {nx};
      const uint32_t fw = __shfl((uint32_t)(e[0] >> 32), (int)(lane() & 56u));
      act = act && x < ge && !beyond(c, (uint64_t)fw << 32, gd, hi);
      if (r == 8u || !ballot(act)) break;
      const bool has[1] = {act && x + sub < ge};
      const uint32_t dd[1] = {gd};
      x += 8u;
      nx = act && x + sub < ge ? c.a.adj[x + sub] : 0ull;
      relax<1>(c, has, e, dd, lo, hi, enq);
    }
    for (uint64_t ml = ballot(act && sub == 0u); ml; ml &= ml - 1) {
      const uint32_t j = first_lane(ml);
      sweep(c, lane_val(gd, j), lane_val(x, j), lane_val(ge, j), lo, hi, enq);
    }
  }
  wave_fence();
}

// Entries of a list that one wave takes at a time: few when the list is
// short, so that it spreads over the device.
__device__ __forceinline__ uint32_t share_of(uint32_t total, uint32_t nw) {
  const uint32_t per = (total + nw - 1u) / nw;
  return per >= 64u ? 64u : (per <= 8u ? 8u : (per + 7u) & ~7u);
}

// Entry idx of a list whose segments hold cnt entries each (lane i: segment
// i; incl: inclusive scan of cnt).
__device__ __forceinline__ uint64_t list_get(const uint64_t* list, uint32_t cap, uint32_t incl, uint32_t cnt,
                                             uint32_t idx, bool in) {
  uint32_t j = 0;
#pragma unroll
  for (uint32_t st = 32; st; st >>= 1)
    if (__shfl(incl, (int)(j + st - 1u)) <= idx) j += st;
  const uint32_t excl = __shfl(incl - cnt, (int)j);
  return in ? list[(uint64_t)j * cap + (idx - excl)] : 0ull;
}

// Expands a list's entries that still hold their vertex's label.
__device__ __forceinline__ void push_list(Wave& c, const uint64_t* list, uint32_t cnt, uint32_t lo, uint32_t hi,
                                          uint32_t enq, bool heavy) {
  const uint32_t incl = wave_incl_scan(cnt);
  const uint32_t total = lane_val(incl, 63);
  const uint32_t per = share_of(total, c.nw);
  for (uint64_t base = (uint64_t)c.w * per; base < total; base += (uint64_t)c.nw * per) {
    const uint32_t idx = (uint32_t)base + lane();
    const bool in = lane() < per && idx < total;
    const uint64_t e = list_get(list, c.a.cap, incl, cnt, in ? idx : 0u, in);
    const uint32_t v = (uint32_t)e, d = (uint32_t)(e >> 32);
    const uint32_t lab = ld_label(c.a.lab + v);
    const uint32_t beg = (uint32_t)c.a.off[v], end = (uint32_t)c.a.off[v + 1u];
    const bool ok = in && d <= lab;
    c.n_stale += in && !ok ? 1u : 0u;
    expand(c, v, d, beg, end, ok, lo, hi, enq, heavy);
  }
}

__device__ __forceinline__ void do_push(Wave& c) {
  const uint64_t* const in = pick(c.a.task, c.step - 1u);
  for (uint32_t t = c.w; t < c.tasks; t += c.nw) {
    const uint64_t r = in[2ull * t], x = in[2ull * t + 1u];
    const uint32_t rb = uni((uint32_t)r), re = uni((uint32_t)(r >> 32));
    const uint32_t d = uni((uint32_t)x), vf = uni((uint32_t)(x >> 32));
    if (uni(ld_label(c.a.lab + (vf & 0x7FFFFFFFu))) < d) continue;
    // a heavy task belongs to the step that ended at t0
    if (vf >> 31)
      sweep(c, d, rb, re, c.t0, kInf32, c.a.unit_w ? 0u : c.t1);
    else
      sweep(c, d, rb, re, 0u, c.t1, c.t1);
  }
  const uint32_t cnt = c.a.unit_w ? 0u : min(c.a.shard[lane()].f[c.slot], c.a.cap);
  push_list(c, pick(c.a.list, c.par), cnt, 0u, c.t1, c.t1, false);
}

__device__ __forceinline__ void do_heavy(Wave& c) {
  const uint32_t cnt = min(*h_counter(c, lane()), c.a.cap);
  push_list(c, c.a.settled, cnt, c.t1, kInf32, c.a.unit_w ? 0u : c.t2, true);
}

// ------------------------------------------------------------ scanning

// Sums of a workgroup's waves, kept in LDS until its first wave adds them to
// a segment's counters: a wave's own atomics (thousands of waves on 64 lines)
// took longer than reading the labels.
struct ScanSum {
  uint64_t near_vol, far_vol;
  uint32_t far_cnt, far_min;
};

// A wave takes 512 consecutive vertices at a time, all their label loads in
// flight at once.
__device__ __forceinline__ void do_scan(Wave& c, ScanSum* sums, uint32_t wl) {
  constexpr int U = 8;
  uint64_t near_vol = 0, far_vol = 0;
  uint32_t far_cnt = 0, far_min = kInf32;
  for (uint64_t base = (uint64_t)c.w * 64u * U; base < c.a.n; base += (uint64_t)c.nw * 64u * U) {
    uint32_t lab[U], deg[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t v = base + 64u * u + lane();
      lab[u] = v < c.a.n ? ld_label(c.a.lab + v) : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t v = base + 64u * u + lane();
      deg[u] = 0;
      if (v < c.a.n && lab[u] >= c.t0) {
        const int32_t* const o = lab[u] < c.t1 ? c.a.off : c.a.ioff;
        deg[u] = (uint32_t)(o[v + 1u] - o[v]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint64_t v = base + 64u * u + lane();
      const bool in = v < c.a.n;
      const bool near = in && lab[u] >= c.t0 && lab[u] < c.t1;
      const bool far = in && lab[u] >= c.t1;
      near_vol += near ? deg[u] : 0u;
      far_vol += far ? deg[u] : 0u;
      far_cnt += far && deg[u] ? 1u : 0u;
      far_min = far ? min(far_min, lab[u]) : far_min;
      append(c, c.h, true, make_elem((uint32_t)v, lab[u]), near && deg[u] != 0u);
      append(c, c.f, false, make_elem((uint32_t)v, lab[u]), far && lab[u] < c.t2 && !c.a.unit_w);
    }
  }
  near_vol = wave_sum64(near_vol);
  far_vol = wave_sum64(far_vol);
  far_cnt = wave_sum(far_cnt);
  far_min = wave_min(far_min);
  if (lane() == 0) sums[wl] = {near_vol, far_vol, far_cnt, far_min};
}

__device__ __forceinline__ void add_scan(const Wave& c, const ScanSum* sums) {
  ScanSum t = sums[0];
  for (uint32_t i = 1; i < kStepWaves; ++i) {
    t.near_vol += sums[i].near_vol;
    t.far_vol += sums[i].far_vol;
    t.far_cnt += sums[i].far_cnt;
    t.far_min = min(t.far_min, sums[i].far_min);
  }
  auto* s = &c.a.shard[blockIdx.x & (kStepSegs - 1u)].s[c.hs];
  if (lane() == 0) {
    if (t.near_vol) add64(&s->near_vol, t.near_vol);
    if (t.far_vol) add64(&s->far_vol, t.far_vol);
    if (t.far_cnt) add32(&s->far_cnt, t.far_cnt);
    if (t.far_min != kInf32)
      (void)__hip_atomic_fetch_min(&s->far_min, t.far_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__device__ __forceinline__ void do_rescan(Wave& c) {
  for (uint64_t base = (uint64_t)c.w * 64u; base < c.a.n; base += (uint64_t)c.nw * 64u) {
    const uint32_t v = (uint32_t)base + lane();
    const uint32_t lab = v < c.a.n ? ld_label(c.a.lab + v) : kInf32;
    append(c, c.f, false, make_elem(v, lab), v < c.a.n && lab >= c.t0 && lab < c.t1);
  }
}

// ------------------------------------------------------------ pulling

// Candidate through in-edge e, if it could beat best.
__device__ __forceinline__ uint32_t pull_edge(Wave& c, uint64_t e, bool has, uint32_t best) {
  const uint32_t w = weight_of(c, e);
  uint32_t cand = kInf32;
  if (has && (uint64_t)w + c.low < best) {
    const uint32_t lu = ld_label(c.a.lab + (uint32_t)e);
    const uint64_t sum = (uint64_t)lu + w;
    if (sum < kInf32) cand = (uint32_t)sum;
  }
  c.n_edges += has ? 1u : 0u;
  return cand;
}

// The lanes' vertices (those with ok, label lab >= t1) take the best of their
// in-edges: eight lanes to a row, ascending weight classes, until no further
// edge can improve the label. Every in-neighbour that may still fall stays at
// t1 or above, so a vertex is final once its label is at most t1 plus its
// lightest in-edge; the others join the next list.
__device__ __forceinline__ void pull(Wave& c, uint32_t v, uint32_t lab, uint32_t beg, uint32_t end, bool ok) {
  const uint64_t m = ballot(ok);
  if (!m) return;
  if (ok) c.order[rank_of(m)] = lane();
  wave_fence();
  const uint32_t cnt = popc(m);
  const uint32_t sub = lane() & 7u, grp = lane() >> 3;
  for (uint32_t k = 0; k < cnt; k += 8u) {
    const bool in = k + grp < cnt;
    const uint32_t src = c.order[in ? k + grp : 0u];
    const uint32_t gv = __shfl(v, (int)src), gl = __shfl(lab, (int)src);
    const uint32_t gb = __shfl(beg, (int)src), ge = __shfl(end, (int)src);
    uint32_t x = gb, best = gl, wmin = 0;
    bool act = in;
    uint64_t nx = act && x + sub < ge ? c.a.iadj[x + sub] : 0ull;
    for (uint32_t r = 0;; ++r) {
      const uint64_t e = nx;
      uint32_t fw = __shfl((uint32_t)(e >> 32), (int)(lane() & 56u));
      fw = c.a.unit_w ? 1u : (fw & ~c.a.cls_mask);
      if (r == 0u) wmin = fw;
      act = act && x < ge && (uint64_t)fw + c.low < best && best > c.t1;
      if (r == 16u || !ballot(act)) break;
      const bool has = act && x + sub < ge;
      x += 8u;
      nx = act && x + sub < ge ? c.a.iadj[x + sub] : 0ull;
      uint32_t cand = pull_edge(c, e, has, best);
      cand = min(cand, (uint32_t)__shfl_xor(cand, 1));
      cand = min(cand, (uint32_t)__shfl_xor(cand, 2));
      cand = min(cand, (uint32_t)__shfl_xor(cand, 4));
      best = min(best, cand);
    }
    // long rows: the whole wave goes on, 256 edges at a time
    for (uint64_t ml = ballot(act && sub == 0u); ml; ml &= ml - 1) {
      const uint32_t j = first_lane(ml);
      uint32_t b = lane_val(best, j);
      const uint32_t re = lane_val(ge, j);
      for (uint32_t y = lane_val(x, j); y < re; y += 256u) {
        uint64_t e[4];
        uint32_t cand = kInf32;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t i = y + 64u * u + lane();
          e[u] = i < re ? c.a.iadj[i] : 0ull;
        }
        uint32_t fw = lane_val((uint32_t)(e[0] >> 32), 0);
        fw = c.a.unit_w ? 1u : (fw & ~c.a.cls_mask);
        if ((uint64_t)fw + c.low >= b || b <= c.t1) break;
#pragma unroll
        for (int u = 0; u < 4; ++u) cand = min(cand, pull_edge(c, e[u], y + 64u * u + lane() < re, b));
        b = min(b, wave_min(cand));
      }
      if ((lane() & 56u) == (j & 56u)) best = b;
    }
    const bool mine = in && sub == 0u;
    c.n_exp += mine ? 1u : 0u;
    if (mine && best < gl) {
      st32(c.a.lab + gv, best);
      c.chg_min = min(c.chg_min, best);
      c.n_push += 1u;
    }
    // room: how small a neighbour's label must be to lower this one
    const uint32_t room = best == kInf32 ? kInf32 : (best > wmin ? best - wmin : 0u);
    append(c, c.f, false, make_elem(gv, room), mine && room > c.t1);
  }
  wave_fence();
}

__device__ __forceinline__ void do_pull_all(Wave& c) {
  for (uint64_t base = (uint64_t)c.w * 64u; base < c.a.n; base += (uint64_t)c.nw * 64u) {
    const uint32_t v = (uint32_t)base + lane();
    const uint32_t lab = v < c.a.n ? ld_label(c.a.lab + v) : 0u;
    const bool far = v < c.a.n && lab >= c.t1;
    uint32_t beg = 0, end = 0;
    if (far) {
      beg = (uint32_t)c.a.ioff[v];
      end = (uint32_t)c.a.ioff[v + 1u];
    }
    pull(c, v, lab, beg, end, far && end > beg);
  }
}

// What changes a label in this sweep is a label that the last one lowered (or
// this one does, from such a label): none of them is below c.low, so vertices
// without room for that leave for good, their rows unread (on RMAT-23 the
// sweeps after the first took 42-48 us each when every listed row was read).
__device__ __forceinline__ void do_pull(Wave& c) {
  const uint64_t* const list = pick(c.a.list, c.par);
  const uint32_t cnt = min(c.a.shard[lane()].f[c.slot], c.a.cap);
  const uint32_t incl = wave_incl_scan(cnt);
  const uint32_t total = lane_val(incl, 63);
  const uint32_t per = share_of(total, c.nw);
  for (uint64_t base = (uint64_t)c.w * per; base < total; base += (uint64_t)c.nw * per) {
    const uint32_t idx = (uint32_t)base + lane();
    const bool in = lane() < per && idx < total;
    const uint64_t e = list_get(list, c.a.cap, incl, cnt, in ? idx : 0u, in);
    const uint32_t v = (uint32_t)e;
    const bool ok = in && (uint32_t)(e >> 32) > c.low;
    uint32_t lab = 0, beg = 0, end = 0;
    if (ok) {
      lab = ld_label(c.a.lab + v);
      beg = (uint32_t)c.a.ioff[v];
      end = (uint32_t)c.a.ioff[v + 1u];
    }
    pull(c, v, lab, beg, end, ok && end > beg);
  }
}

// ------------------------------------------------------------ the end

__device__ __forceinline__ void do_out(Wave& c) {
  uint32_t inv = kInf32;
  for (uint64_t base = (uint64_t)c.w * 64u; base < c.a.n; base += (uint64_t)c.nw * 64u) {
    const uint32_t v = (uint32_t)base + lane();
    if (v < c.a.n) {
      const uint32_t d = ld_label(c.a.lab + (c.a.ord_of ? c.a.ord_of[v] : v));
      if (c.a.ord_of) c.a.out[v] = d;
      if (d != kInf32) inv = min(inv, ~d);
    }
  }
  inv = wave_min(inv);
  if (lane() == 0 && inv != kInf32)
    (void)__hip_atomic_fetch_min(&c.a.shard[c.w & (kStepSegs - 1u)].inv_max, inv, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
}

// First step after the end: the outcome goes to the host.
__device__ __forceinline__ void do_done(const Wave& c) {
  const uint32_t inv = wave_min(ld32(&c.a.shard[lane()].inv_max));
  uint64_t st[5] = {0, 0, 0, 0, 0};
  if (c.a.stats) {
    const StepStats* s = c.a.stats + lane();
    st[0] = wave_sum64(ld64(&s->expansions));
    st[1] = wave_sum64(ld64(&s->stale));
    st[2] = wave_sum64(ld64(&s->edges));
    st[3] = wave_sum64(ld64(&s->pushes));
    st[4] = wave_sum64(ld64(&s->atomics));
  }
  if (lane() == 0) {
    StepHost* h = c.a.host;
#pragma unroll
    for (int i = 0; i < 5; ++i) __hip_atomic_store(&h->stats[i], st[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&h->max_label, ~inv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&h->steps, c.step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&h->state, c.op == kOpDone ? 1u : 2u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__device__ __forceinline__ void add_stats(const Wave& c) {
  StepStats* s = c.a.stats + (c.w & (kStepSegs - 1u));
  const uint32_t x[5] = {wave_sum(c.n_exp), wave_sum(c.n_stale), wave_sum(c.n_edges), wave_sum(c.n_push),
                         wave_sum(c.n_atom)};
  if (lane() == 0) {
    if (x[0]) add64(&s->expansions, x[0]);
    if (x[1]) add64(&s->stale, x[1]);
    if (x[2]) add64(&s->edges, x[2]);
    if (x[3]) add64(&s->pushes, x[3]);
    if (x[4]) add64(&s->atomics, x[4]);
  }
}

}  // namespace

// LDS: the step's decision and the waves' sums, then for each wave two
// outgoing lists of 128 entries and the lane order (8-byte words).
constexpr uint32_t kStepHeadLds = 8u + 3u * kStepWaves + kStepWaves;
constexpr uint32_t kStepWaveLds = 2u * 128u + 32u;
constexpr uint32_t kStepLds = 8u * (kStepHeadLds + kStepWaves * kStepWaveLds);

__device__ __forceinline__ void step_body(const StepArgs& a, uint32_t step) {
  extern __shared__ uint64_t smem[];
  uint32_t* const dec = reinterpret_cast<uint32_t*>(smem);
  ScanSum* const sums = reinterpret_cast<ScanSum*>(smem + 8);
  uint32_t* const flag = reinterpret_cast<uint32_t*>(smem + 8 + 3 * kStepWaves);
  Wave c;
  c.a = a;
  c.step = step;
  const uint32_t wl = uni(threadIdx.x >> 6);
  c.w = blockIdx.x * kStepWaves + wl;
  c.nw = gridDim.x * kStepWaves;
  uint64_t* const mine = smem + kStepHeadLds + wl * kStepWaveLds;
  c.order = reinterpret_cast<uint32_t*>(mine + 256);
  c.n_exp = c.n_stale = c.n_edges = c.n_push = c.n_atom = 0;
  c.chg_min = kInf32;
  if (wl == 0u) {
    decide(c);
    if (lane() == 0) {
      dec[0] = c.op;
      dec[1] = c.t0;
      dec[2] = c.t1;
      dec[3] = c.t2;
      dec[4] = c.slot;
      dec[5] = c.par;
      dec[6] = c.hs;
      dec[7] = c.low;
      dec[8] = c.tasks;
    }
    if (blockIdx.x == 0) record(c);
  }
  __syncthreads();
  c.op = uni(dec[0]);
  c.t0 = uni(dec[1]);
  c.t1 = uni(dec[2]);
  c.t2 = uni(dec[3]);
  c.slot = uni(dec[4]);
  c.par = uni(dec[5]);
  c.hs = uni(dec[6]);
  c.low = uni(dec[7]);
  c.tasks = uni(dec[8]);
  if (c.op == kOpDone || c.op == kOpFail) {
    if (c.w == 0u && uni(a.rec[step - 1u].op) != c.op) do_done(c);
    return;
  }
  c.f = {mine, pick(a.list, c.par + 1u), 0u, c.w & (kStepSegs - 1u)};
  c.h = {mine + 128, a.settled, 0u, c.w & (kStepSegs - 1u)};
  switch (c.op) {
    case kOpPush: do_push(c); break;
    case kOpScan: do_scan(c, sums, wl); break;
    case kOpRescan: do_rescan(c); break;
    case kOpHeavy: do_heavy(c); break;
    case kOpPullAll: do_pull_all(c); break;
    case kOpPull: do_pull(c); break;
    default: do_out(c); break;
  }
  out_finish(c, c.f, false);
  out_finish(c, c.h, true);
  if (a.stats) add_stats(c);
  if (c.op == kOpScan || c.op == kOpPullAll || c.op == kOpPull) {
    const uint32_t low = wave_min(c.chg_min);
    if (lane() == 0) flag[wl] = low;
    __syncthreads();
    if (wl == 0u) {
      if (c.op == kOpScan) {
        add_scan(c, sums);
      } else {
        const uint32_t all = wave_min(lane() < kStepWaves ? flag[lane()] : kInf32);
        StepShard* s = c.a.shard + (blockIdx.x & (kStepSegs - 1u));
        if (lane() == 0 && all != kInf32)
          (void)__hip_atomic_fetch_min(&s->chg_min[c.slot + 1u >= 3u ? c.slot - 2u : c.slot + 1u], all, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

__global__ void __launch_bounds__(64 * kStepWaves) mlmq_step(StepArgs a, uint32_t step) { step_body(a, step); }
// The same step of several solves, one a grid row: the launches and the steps
// with little to do are shared.
__global__ void __launch_bounds__(64 * kStepWaves) mlmq_step_many(const StepArgs* all, uint32_t step) {
  step_body(all[blockIdx.y], step);
}

// Step 0: labels unreachable but the source's, counters zero, the source in
// the first list, thresholds of the first distance step.
__device__ __forceinline__ void step_init_body(const StepArgs& a) {
  const uint32_t tid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
  for (uint64_t i = tid; i < a.n; i += stride) a.lab[i] = i == a.source ? 0u : kInf32;
  uint32_t* const rec = reinterpret_cast<uint32_t*>(a.rec);
  constexpr uint32_t kRecWords = sizeof(StepRec) / 4;
  for (uint32_t i = tid; i < kStepMax * kRecWords; i += stride) {
    uint32_t x = 0;
    // record 0: a push that wrote slot 0 and buffer 0 and settles [0, first step)
    if (i == 0u) x = kOpPush;
    if (i == 2u) x = a.unit_w ? 1u : a.delta;
    if (i == 4u) x = 2u;
    if (i == 5u) x = 1u;
    rec[i] = x;
  }
  for (uint32_t i = tid; i < kStepSegs; i += stride) {
    StepShard* s = a.shard + i;
    s->f[0] = i == 0u ? 1u : 0u;
    s->f[1] = s->f[2] = 0u;
    s->chg_min[0] = s->chg_min[1] = s->chg_min[2] = kInf32;
    s->inv_max = kInf32;
    for (int k = 0; k < 3; ++k) {
      s->s[k].h = s->s[k].far_cnt = 0u;
      s->s[k].far_min = kInf32;
      s->s[k].near_vol = s->s[k].far_vol = 0ull;
    }
    if (a.stats) {
      StepStats* t = a.stats + i;
      t->expansions = t->stale = t->edges = t->pushes = t->atomics = 0ull;
    }
  }
  if (tid == 0u) a.list[0][0] = make_elem(a.source, 0u);
}

__global__ void __launch_bounds__(256) mlmq_step_init(StepArgs a) { step_init_body(a); }
__global__ void __launch_bounds__(256) mlmq_step_init_many(const StepArgs* all) { step_init_body(all[blockIdx.y]); }

// ------------------------------------------------------------ graph preparation

namespace {

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t x, uint32_t m) {
  const uint32_t lo = (uint32_t)__shfl_xor((uint32_t)x, (int)m), hi = (uint32_t)__shfl_xor((uint32_t)(x >> 32), (int)m);
  return (uint64_t)lo | ((uint64_t)hi << 32);
}
// Ascending bitonic sort of the wave's 64 keys.
__device__ __forceinline__ uint64_t sort64(uint64_t x) {
#pragma unroll
  for (uint32_t k = 2; k <= 64; k <<= 1) {
#pragma unroll
    for (uint32_t j = k >> 1; j; j >>= 1) {
      const uint64_t y = shfl_xor64(x, j);
      const bool up = (lane() & k) == 0u || k == 64u;
      const bool low = (lane() & j) == 0u;
      const bool take_min = low == up;
      x = take_min == (x < y) ? x : y;
    }
  }
  return x;
}

constexpr uint32_t kScanPart = 4096;  // counts one wave scans

}  // namespace

// Rows in ascending weight class (weight >> shift, at most 256 classes): rows
// of up to 64 edges are sorted by one wave in registers, longer ones by a
// counting sort of the whole workgroup (histogram and cursors in LDS).
__global__ void __launch_bounds__(256) mlmq_sort_rows(const int32_t* off, const uint64_t* in, uint64_t* out, uint32_t n,
                                                      uint32_t shift) {
  extern __shared__ uint64_t smem[];
  uint32_t* const hist = reinterpret_cast<uint32_t*>(smem);  // [256]
  uint32_t* const bound = hist + 256;                        // [257]
  const uint32_t t = threadIdx.x, wl = uni(t >> 6);
  for (uint64_t r0 = (uint64_t)blockIdx.x * 256u; r0 < n; r0 += (uint64_t)gridDim.x * 256u) {
    const uint32_t rows = (uint32_t)min((uint64_t)256u, (uint64_t)n - r0);
    if (t < rows) bound[t] = (uint32_t)off[r0 + t];
    if (t == 0u) bound[rows] = (uint32_t)off[r0 + rows];
    __syncthreads();
    for (uint32_t j = wl; j < rows; j += 4u) {
      const uint32_t b = uni(bound[j]), deg = uni(bound[j + 1u]) - b;
      if (deg == 0u || deg > 64u) continue;
      uint64_t x = lane() < deg ? in[b + lane()] : ~0ull;
      if (deg > 1u) x = sort64(x);  // the weight is the word's high half
      if (lane() < deg) out[b + lane()] = x;
    }
    for (uint32_t j = 0; j < rows; ++j) {
      const uint32_t b = uni(bound[j]), e = uni(bound[j + 1u]);
      if (e - b <= 64u) continue;
      __syncthreads();
      hist[t] = 0u;
      __syncthreads();
      for (uint32_t i = b + t; i < e; i += 256u)
        (void)__hip_atomic_fetch_add(&hist[(uint32_t)(in[i] >> 32) >> shift], 1u, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
      __syncthreads();
      if (wl == 0u) {
        uint32_t run = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
          const uint32_t x = hist[64u * k + lane()];
          const uint32_t incl = wave_incl_scan(x);
          hist[64u * k + lane()] = run + incl - x;
          run += lane_val(incl, 63);
        }
      }
      __syncthreads();
      for (uint32_t i = b + t; i < e; i += 256u) {
        const uint64_t x = in[i];
        const uint32_t p = __hip_atomic_fetch_add(&hist[(uint32_t)(x >> 32) >> shift], 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        out[b + p] = x;
      }
    }
    __syncthreads();
  }
}

// In-degrees, their prefix sums, then every edge at its column's cursor.
__global__ void __launch_bounds__(256) mlmq_zero_words(uint32_t* p, uint32_t n) {
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = 0u;
}
// Lanes that meet the same column as the wave's first one share an atomic: rows
// of one edge to a hub follow each other (making a star of 100,000 leaves took
// 4.7 ms with an atomic an edge, 3.0 so; most of it now sorts the one long row).
__global__ void __launch_bounds__(256) mlmq_count_columns(const uint64_t* adj, uint32_t m, uint32_t* cnt) {
  const uint64_t first = (uint64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u);
  for (uint64_t base = first; base < m; base += (uint64_t)gridDim.x * blockDim.x) {
    const bool in = base + lane() < m;
    const uint32_t c = in ? (uint32_t)adj[base + lane()] : 0u;
    const uint32_t c0 = lane_val(c, 0);
    const uint64_t same = ballot(in && c == c0);
    if (lane() == 0)
      (void)add32(cnt + c, popc(same));
    else if (in && !(same >> lane() & 1u))
      (void)add32(cnt + c, 1u);
  }
}
__global__ void __launch_bounds__(64) mlmq_scan_parts(const uint32_t* cnt, uint32_t n, int32_t* ioff, uint32_t* part) {
  const uint64_t b = (uint64_t)blockIdx.x * kScanPart;
  uint32_t run = 0;
  for (uint32_t k = 0; k < kScanPart; k += 64u) {
    const uint64_t i = b + k + lane();
    const uint32_t x = i < n ? cnt[i] : 0u;
    const uint32_t incl = wave_incl_scan(x);
    if (i < n) ioff[i] = (int32_t)(run + incl - x);
    run += lane_val(incl, 63);
  }
  if (lane() == 0) part[blockIdx.x] = run;
}
__global__ void __launch_bounds__(64) mlmq_scan_tops(uint32_t* part, uint32_t parts) {
  uint32_t run = 0;
  for (uint32_t k = 0; k < parts; k += 64u) {
    const uint32_t i = k + lane();
    const uint32_t x = i < parts ? part[i] : 0u;
    const uint32_t incl = wave_incl_scan(x);
    if (i < parts) part[i] = run + incl - x;
    run += lane_val(incl, 63);
  }
}
__global__ void __launch_bounds__(256) mlmq_scan_add(const uint32_t* part, uint32_t n, uint32_t m, int32_t* ioff,
                                                     uint32_t* cursor) {
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += (uint64_t)gridDim.x * blockDim.x) {
    if (i == n) {
      ioff[n] = (int32_t)m;
      continue;
    }
    const uint32_t x = (uint32_t)ioff[i] + part[i / kScanPart];
    ioff[i] = (int32_t)x;
    cursor[i] = x;
  }
}
// A wave takes 64 rows at a time and spreads their edges over its lanes.
__global__ void __launch_bounds__(64) mlmq_transpose_fill(const int32_t* off, const uint64_t* adj, uint32_t n,
                                                          uint32_t* cursor, uint64_t* iadj) {
  for (uint64_t r0 = (uint64_t)blockIdx.x * 64u; r0 < n; r0 += (uint64_t)gridDim.x * 64u) {
    const uint64_t v = r0 + lane();
    const uint32_t beg = v < n ? (uint32_t)off[v] : 0u;
    const uint32_t deg = v < n ? (uint32_t)off[v + 1u] - beg : 0u;
    const uint32_t incl = wave_incl_scan(deg);
    const uint32_t total = lane_val(incl, 63);
    const uint32_t first = lane_val(beg, 0);  // the 64 rows are consecutive in adj
    for (uint32_t x = 0; x < total; x += 64u) {
      const uint32_t i = x + lane();
      uint32_t j = 0;
#pragma unroll
      for (uint32_t st = 32; st; st >>= 1)
        if (__shfl(incl, (int)(j + st - 1u)) <= i) j += st;
      const bool in = i < total;
      const uint64_t e = in ? adj[first + i] : 0ull;
      const uint32_t c = (uint32_t)e;
      const uint32_t c0 = lane_val(c, 0);
      const uint64_t same = ballot(in && c == c0);
      const bool shared = (same >> lane() & 1u) != 0u;
      uint32_t at = 0;
      if (lane() == 0)
        at = add32(cursor + c, popc(same));
      else if (in && !shared)
        at = add32(cursor + c, 1u);
      const uint32_t at0 = lane_val(at, 0);
      at = shared ? at0 + rank_of(same) : at;
      if (in) iadj[at] = (r0 + j) | (e & 0xFFFFFFFF00000000ull);
    }
  }
}

// ------------------------------------------------------------ launchers

hipError_t launch_step_init(const StepArgs& a, uint32_t blocks, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_step_init, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_step(const StepArgs& a, uint32_t step, uint32_t blocks, hipStream_t s) {
  hipLaunchKernelGGL(mlmq_step, dim3(blocks), dim3(64 * kStepWaves), kStepLds, s, a, step);
  return hipGetLastError();
}

hipError_t launch_step_many(const StepArgs* d_args, uint32_t count, uint32_t step, uint32_t blocks, hipStream_t s) {
  if (step == 0u)
    hipLaunchKernelGGL(mlmq_step_init_many, dim3(blocks < 64u ? 64u : blocks, count), dim3(256), 0, s, d_args);
  else
    hipLaunchKernelGGL(mlmq_step_many, dim3(blocks, count), dim3(64 * kStepWaves), kStepLds, s, d_args, step);
  return hipGetLastError();
}

hipError_t launch_sort_rows(const int32_t* off, const uint64_t* adj_in, uint64_t* adj_out, uint32_t n, uint32_t shift,
                            hipStream_t s) {
  const uint32_t blocks = n / 256u + 1u < 4096u ? n / 256u + 1u : 4096u;
  hipLaunchKernelGGL(mlmq_sort_rows, dim3(blocks), dim3(256), 4u * (256u + 258u), s, off, adj_in, adj_out, n, shift);
  return hipGetLastError();
}

hipError_t launch_transpose(const int32_t* off, const uint64_t* adj, uint32_t n, uint32_t m, int32_t* ioff,
                            uint64_t* iadj, uint32_t* scratch, hipStream_t s) {
  const uint32_t parts = (n + kScanPart - 1u) / kScanPart;
  uint32_t* const cnt = scratch;
  uint32_t* const part = scratch + n + 1u;
  hipLaunchKernelGGL(mlmq_zero_words, dim3(1024), dim3(256), 0, s, cnt, n);
  hipLaunchKernelGGL(mlmq_count_columns, dim3(4096), dim3(256), 0, s, adj, m, cnt);
  hipLaunchKernelGGL(mlmq_scan_parts, dim3(parts), dim3(64), 0, s, cnt, n, ioff, part);
  hipLaunchKernelGGL(mlmq_scan_tops, dim3(1), dim3(64), 0, s, part, parts);
  hipLaunchKernelGGL(mlmq_scan_add, dim3(1024), dim3(256), 0, s, part, n, m, ioff, cnt);
  hipLaunchKernelGGL(mlmq_transpose_fill, dim3(8192), dim3(64), 0, s, off, adj, n, cnt, iadj);
  return hipGetLastError();
}

}  // namespace mlmq
