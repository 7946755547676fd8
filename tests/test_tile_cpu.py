"""The tiled solve's kernels executed on the CPU (one host thread per lane;
see tests/simt) against the oracle, on cuts of every kind: many small tiles,
one tile, scattered vertices, wide and narrow rounds.
Integer arithmetic: every comparison is exact."""
import ctypes
import os
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
INF = 0xFFFFFFFF


@pytest.fixture(scope="module")
def sim():
    sys.path.insert(0, os.path.join(HERE, "simt"))
    import build_tile_sim
    return ctypes.CDLL(build_tile_sim.build(os.path.join(ROOT, "_build", "simt")))


def _cut(n, sbits, fill, rng):
    """Vertices in id order (rng None) or scattered, `fill` to a tile."""
    order = np.arange(n) if rng is None else rng.permutation(n)
    place = np.arange(n)
    ids = ((place // fill) << sbits) + place % fill
    tiles = (n + fill - 1) // fill
    id_of, inv = np.zeros(n, np.uint32), np.full(tiles << sbits, INF, np.uint32)
    id_of[order] = ids
    inv[ids] = order
    verts = np.full(tiles, fill, np.uint32)
    verts[-1] = n - (tiles - 1) * fill
    return id_of, inv, verts


def _solve(sim, csr, src, cut, sbits, width, unit=0, blocks=2, threads=128, limit=2000):
    id_of, inv, verts = cut
    adj = csr.col.astype(np.uint64) | (csr.w.astype(np.uint64) << np.uint64(32))
    if not csr.m:
        adj = np.zeros(1, np.uint64)
    off = csr.off32()
    extra = np.bincount(id_of >> sbits, weights=np.maximum(csr.degrees() - 4, 0), minlength=len(verts))
    xcap = int(extra.max()) + 4
    dist, info = np.zeros(csr.n, np.uint32), np.zeros(8, np.uint64)
    p = lambda x: ctypes.c_void_p(x.ctypes.data)  # noqa: E731
    u = lambda x: ctypes.c_uint32(int(x))  # noqa: E731
    sim.sim_tiles(u(csr.n), p(off), p(adj), p(id_of), p(inv), p(verts), u(len(verts)), u(sbits), u(xcap), u(src),
                  p(dist), u(width), u(unit), u(blocks), u(threads), u(limit), p(info))
    return dist, info


def _graphs():
    rng = np.random.default_rng(5)
    out = {"road": (gg.grid(20, 23, 0.1, seed=2), 231), "mesh": (gg.grid(16, 16, 0.0, wmax=65535, seed=3), 0),
           "sparse": (gg.uniform(300, 330, wmax=255, seed=6), 3),
           "multi": (gg.random_small(200, 900, 9, rng, wmin=0), 3),  # directed, loops, parallel edges, zero weights
           "one": (gg.from_edges(1, [], [], []), 0),
           "isolated": (gg.from_edges(70, np.arange(1, 69), np.arange(2, 70), np.ones(68)), 0),
           "path": (gg.from_edges(200, np.arange(199), np.arange(1, 200), rng.integers(0, 300, 199)), 0)}
    star = np.arange(1, 150)
    out["star"] = (gg.from_edges(150, np.zeros(149, int), star, rng.integers(1, 99, 149)), 0)
    return out


GRAPHS = _graphs()


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("kind", ["strips", "scattered", "single", "narrow"])
def test_tiles_match_oracle(sim, name, kind):
    csr, src = GRAPHS[name]
    mean = max(1, int(csr.w.astype(np.float64).mean()) if csr.m else 1)
    sbits, fill, width, kw, rng = 7, 101, 8 * mean, {}, None
    if kind == "scattered":  # every tile pushes to most others, everything at once
        sbits, fill, rng, width = 6, 64, np.random.default_rng(1), 2**32 - 1
    elif kind == "single":
        sbits, fill, width, kw = 9, 512, 2**32 - 1, dict(blocks=1, threads=256)
    elif kind == "narrow":
        width, kw = max(1, mean // 2), dict(threads=64)
    cut = _cut(csr.n, sbits, fill, rng)
    dist, info = _solve(sim, csr, src, cut, sbits, width, **kw)
    want = oracle.dijkstra(csr, src)
    assert info[0] == 1 and np.array_equal(dist, want), (np.nonzero(dist != want)[0][:5], info)
    assert info[2] == want[want != oracle.UNREACHABLE].max()
    if kind in ("strips", "single"):
        dist, info = _solve(sim, csr, src, cut, sbits, 8, unit=1, **kw)
        assert info[0] == 1 and np.array_equal(dist, oracle.bfs(csr, src))


def test_saturating_candidates(sim):
    """Sums past the largest distance are dropped, not wrapped around."""
    w = (1 << 20) - 1
    n = 4200
    csr = gg.from_edges(n, np.concatenate([np.arange(n - 1), [0]]), np.concatenate([np.arange(1, n), [n - 1]]),
                        np.concatenate([np.full(n - 1, w), [7]]))
    cut = _cut(n, 11, 2048, None)
    dist, info = _solve(sim, csr, 0, cut, 11, 400 * w, threads=64, blocks=1, limit=60)
    fits = np.arange(n, dtype=np.uint64) * np.uint64(w)
    want = np.where(fits < INF, fits, INF).astype(np.uint32)
    want[n - 1] = 7
    assert info[0] == 1 and np.array_equal(dist, want)


@pytest.mark.parametrize("name", ["road", "multi", "star", "path"])
def test_work_counters(sim, name):
    """Edges that were looked at, not places of records: from one tile in one
    round by one wave each vertex is expanded at least once, its edges counted
    each time; a path has as many improvements as reached vertices."""
    csr, src = GRAPHS[name]
    cut = _cut(csr.n, 9, 512, None)
    dist, info = _solve(sim, csr, src, cut, 9, 2**32 - 1, blocks=1, threads=64)
    assert info[0] == 1
    exp, edges, pushes, atomics = (int(x) for x in info[3:7])
    reached = dist != INF
    row = np.repeat(np.arange(csr.n), csr.degrees())
    real = int((reached[row] & (csr.col != row)).sum())  # loops are not kept
    assert exp >= reached.sum() and edges >= real and pushes >= reached.sum() - 1
    assert edges == atomics  # inside a tile every candidate is an atomic
    if name in ("star", "path"):  # nothing is expanded twice
        assert exp == reached.sum() and edges == real and pushes == reached.sum() - 1
    many, info = _solve(sim, csr, src, _cut(csr.n, 6, 64, None), 6, 2**32 - 1, threads=64)
    exp, edges, pushes, atomics = (int(x) for x in info[3:7])
    assert edges >= real and atomics <= edges and pushes <= atomics and pushes >= reached.sum() - 1
