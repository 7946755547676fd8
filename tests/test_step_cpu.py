"""The stepping kernels executed on the CPU (one host thread per lane; see
tests/simt) against the oracle: every shape of graph the solve accepts, list
sizes that run over, long rows that become tasks, one step per level and few
wide steps, with and without a renumbering, shortest paths and breadth-first
levels. Integer arithmetic: every comparison is exact."""
import ctypes
import os
import sys

import numpy as np
import pytest

import graphgen as gg
import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PUSH, SCAN, RESCAN, HEAVY, PULL_ALL, PULL = 1, 2, 3, 4, 5, 6


@pytest.fixture(scope="module")
def sim():
    sys.path.insert(0, os.path.join(HERE, "simt"))
    import build_step_sim
    return ctypes.CDLL(build_step_sim.build(os.path.join(ROOT, "_build", "simt")))


def _p(x):
    return ctypes.c_void_p(x.ctypes.data if x is not None else None)


def _u(x):
    return ctypes.c_uint32(int(x))


def _shift(csr):
    return max(0, int(csr.w.max() if csr.m else 0).bit_length() - 8)


def _prepared(sim, csr):
    """Sorted out-rows and sorted in-rows, by the library's own kernels."""
    off = csr.off32()
    adj = csr.col.astype(np.uint64) | (csr.w.astype(np.uint64) << np.uint64(32))
    srt, ioff, tmp = np.zeros_like(adj), np.zeros(csr.n + 1, np.int32), np.zeros_like(adj)
    iadj = np.zeros_like(adj)
    sh = _u(_shift(csr))
    sim.sim_sort_rows(_p(off), _p(adj), _p(srt), _u(csr.n), sh)
    sim.sim_transpose(_p(off), _p(srt), _u(csr.n), _u(csr.m), _p(ioff), _p(tmp))
    sim.sim_sort_rows(_p(ioff), _p(tmp), _p(iadj), _u(csr.n), sh)
    return off, adj, srt, ioff, iadj


def _solve(sim, csr, prep, src, delta, unit=0, ord_of=None, cap=None, task_cap=None, blocks=2, limit=320, phase_cost=0):
    off, _, srt, ioff, iadj = prep
    dist = np.zeros(csr.n, np.uint32)
    ops, info = np.zeros(512, np.uint8), np.zeros(8, np.uint64)
    sim.sim_step(_u(csr.n), _p(off), _p(srt), _p(ioff), _p(iadj), _p(ord_of), _u(src), _p(dist), _u(delta),
                 _u(_shift(csr)), _u(csr.w.max() if csr.m else 0), _u(unit), _u(cap or csr.n + 512),
                 _u(task_cap or csr.m // 1024 + 64), _u(blocks), _u(limit), _u(phase_cost), _p(ops), _p(info))
    return dist, ops[1:int(info[0]) + 1].tolist(), info


def _hubs(k, half):
    """Two joined hubs of k and half leaves (rows too long for eight lanes)."""
    rng = np.random.default_rng(7)
    leaves = np.arange(2, k + 2)
    src = np.concatenate([np.zeros(k, int), leaves, np.ones(half, int), leaves[:half], [0, 1], leaves[:k // 4]])
    dst = np.concatenate([leaves, np.zeros(k, int), leaves[:half], np.ones(half, int), [1, 0], leaves[-(k // 4):]])
    return gg.from_edges(k + 2, src, dst, rng.integers(1, 256, src.size))


def _graphs():
    rng = np.random.default_rng(5)
    out = {"rmat9": (g := gg.rmat(9, 8, seed=3), gg.max_degree_vertex(g)),
           "rmat8-wide": (g := gg.rmat(8, 16, wmax=65535, seed=4), gg.max_degree_vertex(g)),
           "uniform": (gg.uniform(700, 3000, wmax=65535, seed=4), 17),
           "sparse": (gg.uniform(601, 900, wmax=255, seed=6), 3),
           "grid": (gg.grid(12, 11, 0.1, seed=2), 7),
           "hubs": (_hubs(700, 400), 5),
           "multi": (gg.random_small(300, 4000, 9, rng, wmin=0), 3),  # directed, loops, parallel edges, zero weights
           "directed": (gg.random_small(900, 2000, 255, rng, wmin=1), 11),
           "one": (gg.from_edges(1, [], [], []), 0),
           "isolated": (gg.from_edges(70, np.arange(1, 69), np.arange(2, 70), np.ones(68)), 0)}
    z = gg.rmat(7, 8, seed=6)
    z.w[:] = 0
    out["zero"] = (z, gg.max_degree_vertex(z))
    # candidates at and past the largest distance, beside shorter ways round them
    out["saturating"] = (gg.from_edges(6, [0, 1, 0, 3, 4, 2], [1, 2, 2, 4, 0, 3],
                                       [2**31, 2**31, 5, 2**32 - 8, 2**32 - 1, 1]), 0)
    return out


GRAPHS = _graphs()


@pytest.mark.parametrize("name", list(GRAPHS))
def test_rows_and_transpose(sim, name):
    """The prepared rows hold the same edges; weight classes ascend in each."""
    csr, _ = GRAPHS[name]
    off, adj, srt, ioff, iadj = _prepared(sim, csr)
    row = np.repeat(np.arange(csr.n, dtype=np.uint64), csr.degrees())
    sh = np.uint64(32 + _shift(csr))
    for o, a, want in ((off, srt, np.stack([row, adj])),
                       (ioff, iadj, np.stack([adj & np.uint64(0xFFFFFFFF), row | (adj >> np.uint64(32) << np.uint64(32))]))):
        r = np.repeat(np.arange(csr.n, dtype=np.uint64), np.diff(o))
        got = np.stack([r, a])
        assert np.array_equal(got[:, np.lexsort(got)], want[:, np.lexsort(want)])
        assert ((np.diff((a >> sh).astype(np.int64)) >= 0) | (np.diff(r.astype(np.int64)) > 0)).all()


@pytest.mark.parametrize("name", list(GRAPHS))
def test_steps_match_oracle(sim, name):
    csr, src = GRAPHS[name]
    prep = _prepared(sim, csr)
    want, levels = oracle.dijkstra(csr, src), oracle.bfs(csr, src)
    mean = max(1, int(csr.w.astype(np.float64).mean()) if csr.m else 1)
    seen = set()
    for delta in sorted({max(1, mean // 8), 2 * mean, 2**32 - 1}):
        dist, ops, info = _solve(sim, csr, prep, src, delta, blocks=1 + delta % 2, limit=150)
        if info[1] == 0:  # out of steps: the queue worker would take over
            assert len(ops) == 149 and delta < mean
            continue
        assert info[1] == 1 and np.array_equal(dist, want), (delta, ops)
        fin = want[want != oracle.UNREACHABLE]
        assert info[2] == fin.max()
        seen |= set(ops)
    dist, ops, info = _solve(sim, csr, prep, src, 1, unit=1)
    assert info[1] == 1 and np.array_equal(dist, levels), ops
    if name == "rmat9":
        dist, ops, info = _solve(sim, csr, prep, src, 12, blocks=1, phase_cost=1 << 20)
        assert info[1] == 1 and np.array_equal(dist, want), ops
        assert {PUSH, SCAN, HEAVY, PULL_ALL, PULL} <= seen | set(ops)


def test_rows_cut_into_tasks(sim):
    """Rows above the limits of a heavy and of a light sweep, from a leaf (the
    hubs are reached) and from a hub (the first row is the longest)."""
    csr = _hubs(33000, 9000)
    prep = _prepared(sim, csr)
    for src, delta, unit in ((5, 20, 0), (0, 2**32 - 1, 0)):
        dist, ops, info = _solve(sim, csr, prep, src, delta, unit=unit, limit=100)
        want = oracle.bfs(csr, src) if unit else oracle.dijkstra(csr, src)
        assert info[1] == 1 and np.array_equal(dist, want), (src, ops)


def test_renumbered_labels_come_back(sim):
    """Solved on renumbered vertices, returned in the caller's order."""
    csr, src = GRAPHS["rmat9"]
    perm = np.random.default_rng(1).permutation(csr.n).astype(np.uint32)
    row = np.repeat(np.arange(csr.n), csr.degrees())
    ren = gg.from_edges(csr.n, perm[row], perm[csr.col], csr.w)
    dist, _, info = _solve(sim, ren, _prepared(sim, ren), src, 16, ord_of=perm)
    assert info[1] == 1 and np.array_equal(dist, oracle.dijkstra(csr, src))


@pytest.mark.parametrize("cap,task_cap", [(12, 4096), (17, 4096)])
def test_lists_that_run_over(sim, cap, task_cap):
    """Segments or task tables too small: the lists are rebuilt from the
    labels, or the solve gives up; an answer that comes back is the right one."""
    for name in ("rmat9", "hubs", "uniform"):
        csr, src = GRAPHS[name]
        if cap * 64 < csr.n:
            continue
        prep, want = _prepared(sim, csr), oracle.dijkstra(csr, src)
        for delta in (64, 2**32 - 1):
            dist, ops, info = _solve(sim, csr, prep, src, delta, cap=cap, task_cap=task_cap, limit=60)
            if info[1] == 1:
                assert np.array_equal(dist, want), (name, delta, ops)


def test_out_of_steps_is_reported(sim):
    csr = gg.from_edges(90, np.arange(89), np.arange(1, 90), np.ones(89))
    dist, ops, info = _solve(sim, csr, _prepared(sim, csr), 0, 1, limit=40, blocks=1)
    assert info[1] == 0 and len(ops) == 39


def test_transpose_of_hub_rows(sim):
    """Whole waves of edges to one column, beside others, and partly filled."""
    for leaves in (1, 63, 64, 65, 1000):
        k = np.arange(1, leaves + 1)
        csr = gg.from_edges(leaves + 3, np.concatenate([k, k[::3], [0], k[:5]]),
                            np.concatenate([0 * k, 0 * k[::3] + leaves + 1, [leaves + 2], k[::-1][:5]]),
                            np.arange(1, leaves + len(k[::3]) + 2 + len(k[:5])))
        off, adj, srt, ioff, iadj = _prepared(sim, csr)
        row = np.repeat(np.arange(csr.n, dtype=np.uint64), csr.degrees())
        col = adj & np.uint64(0xFFFFFFFF)
        want = np.stack([col, row | (adj >> np.uint64(32) << np.uint64(32))])
        got = np.stack([np.repeat(np.arange(csr.n, dtype=np.uint64), np.diff(ioff)), iadj])
        assert np.array_equal(got[:, np.lexsort(got)], want[:, np.lexsort(want)])


@pytest.mark.parametrize("name,cap,phase_cost", [("rmat9", 64, 0), ("rmat9", 65, 0), ("rmat9", 96, 0), ("multi", 64, 0),
                                                 ("multi", 65, 0), ("multi", 96, 0)])
def test_an_overrun_list_is_rebuilt(sim, name, cap, phase_cost):
    """A push that fills a segment of its list: the step's vertices are listed
    again from the labels and the solve ends with the right ones."""
    csr, src = GRAPHS[name]
    prep, want = _prepared(sim, csr), oracle.dijkstra(csr, src)
    seen = set()
    for delta in (64, 256, 2**32 - 1):
        for blocks in (1, 2):
            dist, ops, info = _solve(sim, csr, prep, src, delta, cap=cap, blocks=blocks, limit=150, phase_cost=phase_cost)
            if info[1] == 1:
                assert np.array_equal(dist, want), (delta, ops)
                seen |= set(ops)
    assert RESCAN in seen


def test_lists_too_small_to_rebuild_are_reported(sim):
    csr, src = GRAPHS["rmat9"]
    prep = _prepared(sim, csr)
    for cap in (12, 17):
        dist, ops, info = _solve(sim, csr, prep, src, 2**32 - 1, cap=cap, limit=60)
        assert info[1] == 2, ops


def test_a_task_table_that_runs_over(sim):
    """A long row whose tasks do not fit: the solve reports that it cannot go
    on; with room for them it ends."""
    csr = _hubs(8500, 200)
    prep = _prepared(sim, csr)
    for task_cap, state in ((2, 2), (64, 1)):
        dist, ops, info = _solve(sim, csr, prep, 5, 200, task_cap=task_cap, limit=150)
        assert info[1] == state, ops
    assert np.array_equal(dist, oracle.dijkstra(csr, 5))
