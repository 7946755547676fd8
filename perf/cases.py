"""The shortest-path work whose speed matters to a user of this library.

Every case builds a seeded synthetic graph on the GPU (the shapes of the
repository's benchmark, selector corpus and tests: road-like grids and meshes,
RMAT power-law graphs, uniform random graphs), uploads it once as a
``Graph`` handle, as a program that asks for many paths on one map does, and a
pass is one public call: ``sssp``, ``bfs`` or ``sssp_batch``.
"""
import math

import numpy as np
import torch

import paper_2602_10080_amd as mlmq

INF = 0xFFFFFFFF

# A user's own queue choice instead of the library's default: a near-far L1
# over bucketed L2 rings.
QUEUES = {"near-far over buckets": dict(l0_rows=1, l1_type=2, l2_type=1, bmax=32, bnum=4, delta2_log2=7, delta1=128,
                                        l1_cap=256, th_hub=0)}


def listed():
    return [
        # the smallest call: a neighbourhood map, a few hundred vertices; call overhead and launches count
        dict(name="mesh 24x37", op="sssp", graph="grid", rows=24, cols=37, p_drop=0.0, wmax=255, source="seeded"),
        # the benchmark's small mesh, solved from a corner (latency-bound)
        dict(name="mesh 256x256", op="sssp", graph="grid", rows=256, cols=256, p_drop=0.0, wmax=255, source="corner"),
        # an irregular road map of odd size with many missing streets and wide weights
        dict(name="road 611x1379", op="sssp", graph="grid", rows=611, cols=1379, p_drop=0.2, wmax=65535, source="seeded"),
        # the benchmark's large road-like map, solved from its centre
        dict(name="road 2048x2048", op="sssp", graph="grid", rows=2048, cols=2048, p_drop=0.05, wmax=255, source="centre"),
        # a small social-network-like graph
        dict(name="rmat 14", op="sssp", graph="rmat", scale=14, ef=16, wmax=255, source="hub"),
        # the serving workload's power-law graph, read back into host memory as a service does
        dict(name="rmat 20 to host", op="sssp", graph="rmat", scale=20, ef=16, wmax=255, source="hub", out="host"),
        # the headline benchmark: the largest graph
        dict(name="rmat 23", op="sssp", graph="rmat", scale=23, ef=16, wmax=255, source="hub"),
        # a mid-sized sparse random graph of odd size
        dict(name="uniform 150001", op="sssp", graph="uniform", n=150001, pairs=300000, wmax=255, source="seeded"),
        # the serving workload's uniform graph, weights wide enough that distances might overflow 32 bits
        dict(name="uniform 4M wide", op="sssp", graph="uniform", n=1 << 22, pairs=1 << 25, wmax=65535, source="seeded"),
        # breadth-first levels of a power-law graph
        dict(name="bfs rmat 21", op="bfs", graph="rmat", scale=21, ef=16, wmax=255, source="hub"),
        # a user's explicit queue configuration on a road-like map
        dict(name="road 512 queues", op="sssp", graph="grid", rows=512, cols=512, p_drop=0.05, wmax=255, source="centre",
             queues="near-far over buckets"),
        # the batch workload: many sources on two resident graphs in one call
        dict(name="batch 16+8", op="batch", scale=20, ef=16, side=1024, nrmat=16, ngrid=8, p_drop=0.05, wmax=255),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    wmax = rng.choice((16, 255, 65535))
    kind = rng.choice(("grid", "grid", "rmat", "rmat", "uniform", "batch"))
    if kind == "batch":
        return dict(op="batch", scale=rng.randint(12, 20), ef=rng.choice((4, 8, 16)), side=_log_int(rng, 64, 1024),
                    nrmat=rng.randint(1, 16), ngrid=rng.randint(1, 8), p_drop=rng.choice((0.0, 0.05, 0.2)), wmax=255)
    case = dict(op="bfs" if rng.random() < 0.2 else "sssp", graph=kind, wmax=wmax)
    if kind == "grid":
        case.update(rows=_log_int(rng, 16, 2048), cols=_log_int(rng, 16, 2048), p_drop=rng.choice((0.0, 0.05, 0.2)),
                    source=rng.choice(("corner", "centre", "seeded")))
    elif kind == "rmat":
        case.update(scale=rng.randint(10, 22), ef=rng.choice((4, 8, 16)), source=rng.choice(("hub", "seeded")))
    else:
        n = _log_int(rng, 1 << 10, 1 << 22)
        case.update(n=n, pairs=int(n * rng.choice((2, 4, 8))), source="seeded")
    if rng.random() < 0.15:
        case["out"] = "host"
    elif case["op"] == "sssp" and kind != "uniform" and rng.random() < 0.1:
        case["queues"] = "near-far over buckets"
    return case


# ---------------------------------------------------------------- graphs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _csr(n, u, v, wmax, gen):
    """CSR (off int32, col int32, w int32 holding uint32) of the undirected
    pairs u < v, both directions with one weight, rows sorted by column."""
    w = torch.randint(1, wmax + 1, (u.numel(),), generator=gen, device="cuda", dtype=torch.int32)
    key, order = torch.sort(torch.cat((u * n + v, v * n + u)))
    w = torch.cat((w, w))[order]
    row = torch.div(key, n, rounding_mode="floor")
    off = torch.searchsorted(row, torch.arange(n + 1, device="cuda")).to(torch.int32)
    return n, off, (key - row * n).to(torch.int32), w


def _grid(rows, cols, p_drop, wmax, gen):
    vid = torch.arange(rows * cols, device="cuda").view(rows, cols)
    u = torch.cat((vid[:, :-1].reshape(-1), vid[:-1].reshape(-1)))
    v = torch.cat((vid[:, 1:].reshape(-1), vid[1:].reshape(-1)))
    if p_drop:
        keep = torch.rand(u.numel(), generator=gen, device="cuda") >= p_drop
        u, v = u[keep], v[keep]
    return _csr(rows * cols, u, v, wmax, gen)


def _pairs(n, u, v):
    """The distinct pairs u < v, without loops."""
    lo, hi = torch.minimum(u, v), torch.maximum(u, v)
    key = torch.unique((lo * n + hi)[lo != hi])
    lo = torch.div(key, n, rounding_mode="floor")
    return lo, key - lo * n


def _rmat(scale, ef, wmax, gen):
    n, m = 1 << scale, ef << scale
    u = torch.zeros(m, dtype=torch.int64, device="cuda")
    v = torch.zeros(m, dtype=torch.int64, device="cuda")
    for _ in range(scale):  # quadrants 0.57, 0.19, 0.19, 0.05
        r = torch.rand(m, generator=gen, device="cuda")
        u = 2 * u + (r >= 0.76).long()
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).long()
    perm = torch.randperm(n, generator=gen, device="cuda")
    return _csr(n, *_pairs(n, perm[u], perm[v]), wmax, gen)


def _uniform(n, pairs, wmax, gen):
    u = torch.randint(0, n, (pairs,), generator=gen, device="cuda")
    v = torch.randint(0, n, (pairs,), generator=gen, device="cuda")
    return _csr(n, *_pairs(n, u, v), wmax, gen)


def _build(case, gen):
    if case["graph"] == "grid":
        return _grid(case["rows"], case["cols"], case["p_drop"], case["wmax"], gen)
    if case["graph"] == "rmat":
        return _rmat(case["scale"], case["ef"], case["wmax"], gen)
    return _uniform(case["n"], case["pairs"], case["wmax"], gen)


def _seeded_source(csr, gen, k=1):
    """k sources drawn among the vertices that have edges."""
    n, off = csr[0], csr[1]
    cand = torch.nonzero(off[1:] > off[:-1]).view(-1)
    return cand[torch.randint(0, cand.numel(), (k,), generator=gen, device="cuda")].tolist()


def _source(case, csr, gen):
    if case["source"] == "corner":
        return 0
    if case["source"] == "centre":
        return case["rows"] // 2 * case["cols"] + case["cols"] // 2
    if case["source"] == "hub":
        return int(torch.argmax(csr[1][1:] - csr[1][:-1]))
    return _seeded_source(csr, gen)[0]


def _inputs(case, seed):
    """[(graph number, source)] and the CSR graphs of a case."""
    gen = _gen(seed)
    if case["op"] == "batch":
        rm = _rmat(case["scale"], case["ef"], case["wmax"], gen)
        gr = _grid(case["side"], case["side"], case["p_drop"], case["wmax"], gen)
        queries = [(0, s) for s in _seeded_source(rm, gen, case["nrmat"])]
        queries += [(1, s) for s in _seeded_source(gr, gen, case["ngrid"])]
        return [rm, gr], queries
    csr = _build(case, gen)
    return [csr], [(0, _source(case, csr, gen))]


def prepare(case, seed):
    csrs, queries = _inputs(case, seed)
    graphs = [mlmq.Graph(*c) for c in csrs]
    if case.get("out") == "host":
        outs = [np.empty(graphs[k].n, dtype=np.uint32) for k, _ in queries]
    else:
        outs = [mlmq.new_dist(graphs[k].n) for k, _ in queries]
    config = mlmq.default_config(**QUEUES[case["queues"]]) if case.get("queues") else None
    return dict(op=case["op"], graphs=graphs, queries=queries, outs=outs, config=config)


# ---------------------------------------------------------------- a pass

def run(state):
    graphs, queries, outs = state["graphs"], state["queries"], state["outs"]
    if state["op"] == "batch":
        _, status = mlmq.sssp_batch([graphs[k] for k, _ in queries], [s for _, s in queries], outs=outs)
        return [*outs, *status]
    call = mlmq.bfs if state["op"] == "bfs" else mlmq.sssp
    out = call(graphs[0], queries[0][1], out=outs[0], config=state["config"])
    return out.view(np.int32) if isinstance(out, np.ndarray) else out


# ---------------------------------------------------------------- work and exact values

def _size(kind, case):
    """Vertices and directed edges (about: duplicates of RMAT and uniform draws are not counted out)."""
    if kind == "grid":
        r, c = case["rows"], case["cols"]
        return r * c, int(2 * (2 * r * c - r - c) * (1.0 - case["p_drop"]))
    if kind == "rmat":
        return 1 << case["scale"], 2 * case["ef"] << case["scale"]
    return case["n"], 2 * case["pairs"]


def work(case):
    """Every row offset, edge and weight read once, every distance written
    once; one addition and one comparison per edge. A batch reads each graph
    once per query (the queries share no result)."""
    if case["op"] == "batch":
        parts = [(_size("rmat", case), case["nrmat"]),
                 (_size("grid", dict(case, rows=case["side"], cols=case["side"])), case["ngrid"])]
    else:
        parts = [(_size(case["graph"], case), 1)]
    return dict(bytes=sum(k * (4 * n + 8 * m + 4 * n) for (n, m), k in parts),
                flops=sum(k * 2 * m for (_, m), k in parts))


def _relax(csr, source, unit):
    """Distances by rounds of relaxation in 64-bit integers, each round over
    the edges of the vertices that changed in the last one."""
    n, off, col, w = csr
    off = off.long()
    dist = torch.full((n,), 1 << 40, dtype=torch.int64, device="cuda")
    dist[source] = 0
    front = torch.tensor([source], device="cuda")
    while front.numel():
        deg = off[front + 1] - off[front]
        start = torch.cumsum(deg, 0) - deg
        total = int(deg.sum())
        if not total:
            break
        edge = torch.arange(total, device="cuda") + torch.repeat_interleave(off[front] - start, deg)
        to = col[edge].long()
        cost = 1 if unit else w[edge].long() & INF
        old = dist[to]
        dist.scatter_reduce_(0, to, torch.repeat_interleave(dist[front], deg) + cost, "amin")
        front = torch.unique(to[dist[to] < old])
    return torch.where(dist < (1 << 40), dist, torch.full_like(dist, -1)).to(torch.int32)


def exact(case, seed):
    csrs, queries = _inputs(case, seed)
    outs = [_relax(csrs[k], s, case["op"] == "bfs") for k, s in queries]
    if case["op"] == "batch":
        return [*outs, *([0] * len(outs))]
    return outs[0]
