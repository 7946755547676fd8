"""The library's host code on the CPU, over a stand-in device (tests/simt/host):
the order of work on streams, waits and deadlines, memory that runs out, and
which solver a call takes. Distances are whole numbers: every comparison is
exact."""
import ctypes
import os
import sys
import threading
import time

import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2602_10080_amd as mlmq

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Sim:
    """The host code with its device, through the C ABI."""

    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        mlmq._declare(self.lib)
        self.lib.sim_alloc.restype = self.lib.sim_stream.restype = ctypes.c_void_p
        self.lib.sim_alloc.argtypes = [ctypes.c_size_t]
        self.lib.sim_hold.argtypes = [ctypes.c_void_p, ctypes.c_int]
        self.lib.sim_fill.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32]
        self.lib.sim_wait.argtypes = [ctypes.c_void_p, ctypes.c_double]
        self.lib.sim_set.argtypes = [ctypes.c_char_p, ctypes.c_double]
        self.lib.sim_get.argtypes = [ctypes.c_char_p]
        self.lib.sim_get.restype = ctypes.c_double

    def set(self, **kw):
        for k, v in kw.items():
            self.lib.sim_set(k.encode(), float(v))

    def count(self, what):
        return int(self.lib.sim_get(what.encode()))

    def graph(self, csr, flags=0):
        h = ctypes.c_void_p()
        off = csr.off32()
        rc = self.lib.mlmq_graph_create(csr.n, csr.m, off.ctypes.data, csr.col.ctypes.data, csr.w.ctypes.data, flags,
                                        ctypes.byref(h))
        assert rc == 0, self.error()
        return h

    def error(self):
        return self.lib.mlmq_last_error().decode()

    def config(self, g, **kw):
        c = mlmq.Config()
        c.struct_size = ctypes.sizeof(c)
        assert self.lib.mlmq_graph_config(g, ctypes.byref(c)) == 0
        return c.copy(**kw)

    def buffer(self, n):
        """A device buffer and its contents as an array."""
        p = self.lib.sim_alloc(4 * n)
        return p, np.ctypeslib.as_array((ctypes.c_uint32 * n).from_address(p))

    def sssp(self, g, src, out, cfg=None, bfs=False):
        f = self.lib.mlmq_bfs if bfs else self.lib.mlmq_sssp
        return f(g, src, out, ctypes.byref(cfg) if cfg is not None else None)

    def batch(self, queries, cfgs=None):
        """queries: (graph, source, buffer address); the call's status and each query's."""
        n = len(queries)
        st = (ctypes.c_int32 * n)(*[99] * n)
        rc = self.lib.mlmq_sssp_batch((ctypes.c_void_p * n)(*[q[0].value for q in queries]),
                                      (ctypes.c_uint32 * n)(*[q[1] for q in queries]),
                                      (ctypes.c_void_p * n)(*[q[2] for q in queries]), n,
                                      (ctypes.c_void_p * n)(*[ctypes.addressof(c) for c in cfgs]) if cfgs else None, st)
        return rc, list(st)


@pytest.fixture(scope="module")
def _sim():
    sys.path.insert(0, os.path.join(HERE, "simt"))
    import build_host_sim
    return Sim(build_host_sim.build(os.path.join(ROOT, "_build", "simt")))


@pytest.fixture
def sim(_sim):
    _sim.set(steps=6, worker_ms=0, worker_more=0, served_ms=0, step_ms=0, room=-1, largest=-1, reset=1)
    yield _sim
    _sim.set(steps=6, worker_ms=0, worker_more=0, served_ms=0, step_ms=0, room=-1, largest=-1)


ROAD = gg.grid(70, 80, 0.05, seed=1)      # several tiles
MESH = gg.grid(20, 30, 0.0, seed=2)       # one tile
SKEWED = gg.rmat(12, 8, seed=3)           # steps
QUEUES = dict(l0_rows=1, l1_type=2, l2_type=1, bmax=32, bnum=4, delta2_log2=7, delta1=128, l1_cap=256, th_hub=0)


def test_routes_and_results(sim):
    for csr, kernel in ((ROAD, "tile"), (MESH, "tile"), (SKEWED, "step")):
        g = sim.graph(csr)
        p, out = sim.buffer(csr.n)
        host = np.zeros(csr.n, np.uint32)
        for how, bulk in ((None, True), (sim.config(g), True), (sim.config(g, **QUEUES), False)):
            sim.set(reset=1)
            assert sim.sssp(g, 5, p, how) == 0
            np.testing.assert_array_equal(out, oracle.dijkstra(csr, 5))
            assert (sim.count(kernel) > 0, sim.count("worker") > 0) == (bulk, not bulk)
        assert sim.sssp(g, 5, host.ctypes.data) == 0 and sim.sssp(g, 7, p, bfs=True) == 0
        np.testing.assert_array_equal(host, oracle.dijkstra(csr, 5))
        np.testing.assert_array_equal(out, oracle.bfs(csr, 7))


def test_calls_without_a_configuration(sim):
    """A NULL configuration has no stream and no place for counters, whatever
    the stack held before; in a batch too."""
    for csr in (ROAD, MESH, SKEWED):
        g = sim.graph(csr)
        p, out = sim.buffer(csr.n)
        for call in (lambda: sim.sssp(g, 5, p), lambda: sim.sssp(g, 5, p, bfs=True),
                     lambda: sim.lib.mlmq_sssp_noalloc(g, 5, p, None), lambda: sim.batch([(g, 5, p)])[0]):
            sim.lib.sim_dirty_stack()
            assert call() == 0, sim.error()
        np.testing.assert_array_equal(out, oracle.dijkstra(csr, 5))


@pytest.mark.parametrize("queues", [False, True])
def test_batch_starts_after_work_on_the_null_stream(sim, queues):
    """A fill of the output buffers that still waits on the null stream comes
    before the batch's solves, whichever solver they take."""
    work = [(ROAD, sim.graph(ROAD)), (SKEWED, sim.graph(SKEWED)), (MESH, sim.graph(MESH))]
    outs = [sim.buffer(c.n) for c, _ in work]
    cfgs = [sim.config(g, **(QUEUES if queues else {})) for _, g in work]
    sim.lib.sim_hold(None, 1)
    for (c, _), (p, _o) in zip(work, outs):
        sim.lib.sim_fill(None, p, c.n, 7)
    t = threading.Timer(0.2, sim.lib.sim_hold, (None, 0))
    t.start()
    rc, st = sim.batch([(g, 3, p) for (_, g), (p, _o) in zip(work, outs)], cfgs)
    t.join()
    assert rc == 0 and not any(st)
    for (c, _), (_p, o) in zip(work, outs):
        np.testing.assert_array_equal(o, oracle.dijkstra(c, 3))


def test_deadline_counts_from_the_device_s_start(sim):
    """Earlier work on the stream outlasts the deadline; the solve itself does not."""
    g = sim.graph(ROAD)
    p, out = sim.buffer(ROAD.n)
    stream = sim.lib.sim_stream()
    for call in ("single", "batch"):
        out[:] = 1
        sim.lib.sim_hold(stream, 1)
        sim.lib.sim_fill(stream, p, ROAD.n, 7)
        t = threading.Timer(0.7, sim.lib.sim_hold, (stream, 0))
        t.start()
        cfg = sim.config(g, stream=stream, timeout_ms=300)
        rc = sim.sssp(g, 3, p, cfg) if call == "single" else sim.batch([(g, 3, p)], [cfg])[0]
        t.join()
        assert rc == 0, (call, sim.error())
        np.testing.assert_array_equal(out, oracle.dijkstra(ROAD, 3))


def test_a_solve_that_takes_too_long_ends_at_its_deadline(sim):
    for csr in (ROAD, SKEWED):
        g = sim.graph(csr)
        p, out = sim.buffer(csr.n)
        for call in ("single", "batch"):
            sim.set(steps=10**6, step_ms=20)
            t0 = time.time()
            cfg = sim.config(g, timeout_ms=100)
            rc = sim.sssp(g, 3, p, cfg) if call == "single" else sim.batch([(g, 3, p)], [cfg])[0]
            assert rc == -5 and time.time() - t0 < 2.0, (call, rc)
            sim.set(steps=6, step_ms=0)
            assert sim.sssp(g, 3, p) == 0  # the memory of the late solve is whole
            np.testing.assert_array_equal(out, oracle.dijkstra(csr, 3))


@pytest.mark.parametrize("call", ["single", "batch"])
def test_a_stream_that_never_gets_there_is_not_waited_for(sim, call):
    """As the queue worker's: the call returns some seconds after its deadline
    and what its launches may still touch is not given to another call."""
    g = sim.graph(SKEWED)
    p, out = sim.buffer(SKEWED.n)
    stream = sim.lib.sim_stream()
    sim.lib.sim_hold(stream, 1)
    cfg = sim.config(g, stream=stream, timeout_ms=50)
    t0 = time.time()
    rc = sim.sssp(g, 3, p, cfg) if call == "single" else sim.batch([(g, 3, p)], [cfg])[0]
    assert rc == -5 and 3.0 < time.time() - t0 < 12.0
    q, other = sim.buffer(SKEWED.n)
    for _ in range(3):
        assert sim.sssp(g, 4, q) == 0 and sim.batch([(g, 4, q)])[0] == 0
    sim.lib.sim_hold(stream, 0)  # the late launches run now
    sim.lib.sim_pump()
    np.testing.assert_array_equal(other, oracle.dijkstra(SKEWED, 4))


def test_a_solve_does_not_wait_for_what_others_put_on_its_stream(sim):
    """Another thread goes on putting work on the same stream."""
    g = sim.graph(SKEWED)
    p, out = sim.buffer(SKEWED.n)
    q, _ = sim.buffer(SKEWED.n)
    stream = sim.lib.sim_stream()
    stop = threading.Event()

    def keep_busy():
        while not stop.is_set():
            sim.lib.sim_wait(stream, 2.0)  # two milliseconds of work, always two of them ahead
            time.sleep(0.0015)

    t = threading.Thread(target=keep_busy)
    t.start()
    end = threading.Timer(4.0, stop.set)
    end.start()
    time.sleep(0.05)
    t0 = time.time()
    rc = sim.sssp(g, 3, p, sim.config(g, stream=stream))
    took = time.time() - t0
    stop.set()
    t.join()
    end.cancel()
    assert rc == 0 and took < 2.0, took
    np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 3))


def test_one_deadline_for_both_solvers(sim):
    """A solve that runs out of steps leaves the queue worker what is left of its time."""
    p, out = sim.buffer(SKEWED.n)
    sim.set(steps=10**6, step_ms=1, worker_ms=400)
    for timeout, want in ((600, -5), (4000, 0)):
        g = sim.graph(SKEWED)
        assert sim.sssp(g, 3, p, sim.config(g, timeout_ms=timeout)) == want
        g = sim.graph(SKEWED)
        assert sim.batch([(g, 3, p)], [sim.config(g, timeout_ms=timeout)])[0] == want
    np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 3))


def test_one_deadline_for_all_groups_of_a_batch(sim):
    g = sim.graph(MESH)
    bufs = [sim.buffer(MESH.n) for _ in range(40)]
    sim.set(step_ms=100)  # 0.6 s a group
    rc, st = sim.batch([(g, i, b[0]) for i, b in enumerate(bufs)], [sim.config(g, timeout_ms=900)] * 40)
    assert rc == -5 and st == [0] * 32 + [-5] * 8
    for i in range(32):
        np.testing.assert_array_equal(bufs[i][1], oracle.dijkstra(MESH, i))


def test_no_room_for_a_bulk_solve(sim):
    """Its lists do not fit, the queues do: the queue worker solves, alone and
    in a batch beside a solve that has room."""
    csr = gg.rmat(16, 2, seed=4)
    big, small = sim.graph(csr), sim.graph(SKEWED)
    (p, out), (q, other) = sim.buffer(csr.n), sim.buffer(SKEWED.n)
    assert sim.sssp(small, 3, q) == 0
    sim.set(largest=8 << 20, reset=1)
    assert sim.sssp(big, 3, p) == 0, sim.error()
    np.testing.assert_array_equal(out, oracle.dijkstra(csr, 3))
    assert sim.count("worker") == 1
    for order in ([(small, 3, q), (big, 4, p)], [(big, 4, p), (small, 3, q)]):
        rc, st = sim.batch(order)
        assert rc == 0 and not any(st), sim.error()
        np.testing.assert_array_equal(out, oracle.dijkstra(csr, 4))
        np.testing.assert_array_equal(other, oracle.dijkstra(SKEWED, 3))


class Server:
    def __init__(self, sim, graphs):
        self.sim, self.h = sim, ctypes.c_void_p()
        arr = (ctypes.c_void_p * len(graphs))(*[g.value for g in graphs])
        assert sim.lib.mlmq_server_create(arr, len(graphs), 1 << 28, 8, None, ctypes.byref(self.h)) == 0, sim.error()

    def submit(self, k, src, p):
        t = ctypes.c_uint64()
        assert self.sim.lib.mlmq_server_submit(self.h, k, src, p, ctypes.byref(t)) == 0
        return t.value

    def wait(self, t):
        return self.sim.lib.mlmq_server_wait(self.h, t, 20000)

    def close(self):
        self.sim.lib.mlmq_server_destroy(self.h)


def _until(cond, limit=5.0):
    t0 = time.time()
    while not cond() and time.time() - t0 < limit:
        time.sleep(0.002)
    assert cond()


def test_solves_beside_a_busy_server(sim):
    """A resident kernel leaves no room for a bulk solve's workgroups: solves
    take the queue worker until it has left."""
    served, other = sim.graph(ROAD), sim.graph(SKEWED)
    (p, _), (q, out) = sim.buffer(ROAD.n), sim.buffer(SKEWED.n)
    srv = Server(sim, [served])
    try:
        sim.set(served_ms=1500, reset=1)
        ticket = srv.submit(0, 3, p)
        _until(lambda: sim.count("resident") == 1)
        t0 = time.time()
        assert sim.sssp(other, 5, q) == 0 and sim.batch([(other, 5, q)])[0] == 0
        assert time.time() - t0 < 1.0 and sim.count("worker") == 2 and sim.count("step") == 0
        np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 5))
        assert srv.wait(ticket) == 0
        _until(lambda: sim.count("resident") == 0)

        def bulk_again():
            sim.set(reset=1)
            return sim.sssp(other, 5, q) == 0 and sim.count("step") > 0
        _until(bulk_again)
    finally:
        srv.close()
    sim.set(reset=1)
    assert sim.sssp(other, 5, q) == 0 and sim.count("step") > 0


def test_a_server_kernel_waits_for_bulk_solves_under_way(sim):
    served, other = sim.graph(ROAD), sim.graph(SKEWED)
    (p, _), (q, out) = sim.buffer(ROAD.n), sim.buffer(SKEWED.n)
    srv = Server(sim, [served])
    try:
        sim.set(steps=40, step_ms=5, reset=1)
        got = []
        t = threading.Thread(target=lambda: got.append(sim.sssp(other, 5, q)))
        t.start()
        _until(lambda: sim.count("step") > 3)
        assert srv.wait(srv.submit(0, 3, p)) == 0
        t.join()
        assert got == [0] and sim.count("launches before it") == sim.count("step") >= 40
        np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 5))
    finally:
        srv.close()


def test_a_graph_is_made_beside_a_busy_server(sim):
    """Nothing that its creation does waits for the device to be idle (freeing
    device memory does), and no memory beyond the graph's own stays with it."""
    served = sim.graph(ROAD)
    p, _ = sim.buffer(ROAD.n)
    srv = Server(sim, [served])
    try:
        sim.set(served_ms=1500, reset=1)
        ticket = srv.submit(0, 3, p)
        _until(lambda: sim.count("resident") == 1)
        t0 = time.time()
        for csr in (ROAD, MESH, SKEWED):
            used = sim.count("used")
            g = sim.graph(csr)
            # rows, then tiles (records of 16 bytes, ids, offsets, the few edges past the fourth and over a border) or
            # rows out and in
            assert sim.count("used") - used < 8 * csr.m + 4 * csr.n + 16 * csr.m + 32 * csr.n + (1 << 20)
        assert time.time() - t0 < 1.0 and sim.count("hipFree") == 0
        assert srv.wait(ticket) == 0
    finally:
        srv.close()
    assert g


def _with_hubs(side, hubs, degree):
    """A mesh some of whose vertices have edges to many others nearby."""
    ids = np.arange(side * side).reshape(side, side)
    u = [ids[:, :-1].ravel(), ids[:-1].ravel()]
    v = [ids[:, 1:].ravel(), ids[1:].ravel()]
    rng = np.random.default_rng(1)
    for h in rng.integers(0, side * side, hubs):
        u.append(np.full(degree, h))
        v.append((h + rng.integers(-3 * side, 3 * side, degree)) % (side * side))
    u, v = np.concatenate(u), np.concatenate(v)
    return gg.from_edges(side * side, np.concatenate([u, v]), np.concatenate([v, u]), rng.integers(1, 256, 2 * len(u)))


def test_radius_estimate(sim):
    """Within a factor of two of half the diameter of meshes, small on graphs
    that spread exponentially, whatever the order of their vertices."""
    def radius(csr):
        off, col = csr.off32(), np.ascontiguousarray(csr.col, dtype=np.int32)
        return sim.lib.sim_radius(csr.n, ctypes.c_void_p(off.ctypes.data), ctypes.c_void_p(col.ctypes.data))

    def shuffled(csr):
        p = np.random.default_rng(2).permutation(csr.n)
        return gg.from_edges(csr.n, p[np.repeat(np.arange(csr.n), csr.degrees())], p[csr.col], csr.w)

    for side in (40, 130, 300):
        for csr in (gg.grid(side, side, 0.0, seed=1), gg.grid(side, side, 0.2, seed=1)):
            for g in (csr, shuffled(csr)):
                assert side / 2 <= radius(g) <= 4 * side
    path = gg.from_edges(5000, np.arange(4999), np.arange(1, 5000), np.ones(4999))  # one way: seen from its vertices
    assert 2500 <= radius(path) <= 10000
    assert radius(gg.rmat(14, 16, seed=1)) <= 8
    assert radius(gg.uniform(50000, 200000, seed=1)) <= 24
    assert radius(gg.from_edges(3000, [0], [1], [1])) == 0
    assert radius(gg.from_edges(1, [], [], [])) == 0


def test_deep_graphs_do_not_begin_with_steps(sim):
    """A mesh that one vertex's degree keeps out of tiles is too deep for steps."""
    csr = _with_hubs(260, 1, 40)
    g = sim.graph(csr)
    p, out = sim.buffer(csr.n)
    for bfs in (False, True):
        sim.set(reset=1)
        assert sim.sssp(g, 5, p, bfs=bfs) == 0
        assert sim.count("step") == 0 and sim.count("worker") == 1


def test_a_failed_bulk_solve_is_not_tried_again_at_once(sim):
    g = sim.graph(SKEWED)
    p, out = sim.buffer(SKEWED.n)
    sim.set(steps=10**6)

    def tries(calls, **kw):
        n = 0
        for _ in range(calls):
            sim.set(reset=1)
            assert sim.sssp(g, 5, p, **kw) == 0
            n += sim.count("step") > 0
        return n
    assert tries(8) == 1 and tries(64) == 1 and tries(64) == 1
    np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 5))
    assert tries(1, bfs=True) == 1  # levels have a count of their own
    sim.set(steps=6)
    assert tries(1) == 1 and tries(5) == 5  # it succeeds: every call again
    sim.set(steps=10**6)
    assert tries(8) == 1  # and the count starts over


def _cut(sim, csr, sbits=10, xcap=1024, most=17408, threads=16):
    off, col = csr.off32(), np.ascontiguousarray(csr.col, dtype=np.int32)
    ids, verts, info = np.zeros(csr.n, np.uint32), np.zeros(csr.n, np.uint32), np.zeros(3, np.uint64)
    p = lambda x: ctypes.c_void_p(x.ctypes.data)  # noqa: E731
    t0 = time.time()
    sim.lib.sim_cut(csr.n, p(off), p(col), sbits, xcap, most, threads, p(ids), p(verts), p(info))
    return ids, verts[:int(info[0])], info, time.time() - t0


def _reordered(csr, seed=2):
    p = np.random.default_rng(seed).permutation(csr.n)
    return gg.from_edges(csr.n, p[np.repeat(np.arange(csr.n), csr.degrees())], p[csr.col], csr.w)


@pytest.mark.parametrize("name", ["road", "shuffled road", "mesh", "small", "loops", "hub", "pieces"])
def test_tiles_hold_every_vertex_once(sim, name):
    rng = np.random.default_rng(3)
    csr = {"road": lambda: gg.grid(600, 700, 0.2, seed=1), "shuffled road": lambda: _reordered(gg.grid(500, 500, 0.05, seed=1)),
           "mesh": lambda: gg.grid(40, 5000, 0.0, seed=1), "small": lambda: gg.grid(64, 65, 0.0, seed=1),
           "loops": lambda: gg.from_edges(9000, *(lambda a: (np.concatenate([a, a, a[:-1]]),
                                                             np.concatenate([a, a, a[1:]]), np.ones(3 * len(a) - 1)))(np.arange(9000))),
           "hub": lambda: _with_hubs(120, 3, 700),
           "pieces": lambda: gg.from_edges(200000, *(lambda a: (a[a % 7 != 6], a[a % 7 != 6] + 1, np.ones((a % 7 != 6).sum())))(
               np.arange(199999)))}[name]()
    ids, verts, info, _ = _cut(sim, csr)
    assert len(verts)
    # ids are places of tiles: each once, the first of its tile's
    tile, place = ids >> 10, ids & 1023
    np.testing.assert_array_equal(np.bincount(tile, minlength=len(verts)), verts)
    assert len(np.unique(ids)) == csr.n and (place < verts[tile]).all()
    # what the lists are allocated for
    row = np.repeat(np.arange(csr.n), csr.degrees())
    inside = (tile[row] == tile[csr.col])
    assert info[1] == (~inside).sum() and 4 * info[1] <= csr.m
    loc = np.bincount(row[inside & (row != csr.col)], minlength=csr.n)
    over = np.maximum(loc - 4, 0)
    assert info[2] == over.sum() and np.bincount(tile, weights=over).max() <= 1024
    # tiles are nearly full; the counts do not depend on the threads
    assert len(verts) <= (1.35 if name in ("hub", "pieces") else 1.05) * csr.n / 1024 + 2
    for threads in (1, 3):
        assert (_cut(sim, csr, threads=threads)[2] == info).all()


def test_graphs_that_do_not_fall_into_tiles(sim):
    assert len(_cut(sim, gg.uniform(300000, 600000, 255, seed=1))[1]) == 0  # too many edges would be cut
    assert len(_cut(sim, gg.grid(300, 300, 0.0, seed=1), most=50)[1]) == 0  # too many tiles
    star = gg.from_edges(3000, np.zeros(2999, int), np.arange(1, 3000), np.ones(2999))
    assert len(_cut(sim, star)[1]) == 0  # a row that fits no tile
    one = gg.grid(64, 64, 0.0, seed=1)
    assert _cut(sim, one, sbits=12, xcap=4096)[1].tolist() == [4096]


@pytest.mark.parametrize("queues_faster", [False, True])
def test_autotune_times_queues_and_keeps_the_faster_solver(sim, queues_faster):
    """Every candidate is timed on its queues, whatever the budget; default
    solves go on in bulk unless the queues were faster."""
    for csr, kernel in ((ROAD, "tile"), (SKEWED, "step")):
        for budget in (1, 300):
            g = sim.graph(csr)
            p, out = sim.buffer(csr.n)
            before = sim.config(g).as_dict()
            sim.set(worker_ms=1 if queues_faster else 10, step_ms=2 if queues_faster else 0, reset=1)
            assert sim.lib.mlmq_autotune(g, budget, None) == 0
            timed = sim.count("worker")
            assert timed >= 3 and timed % 3 == 0
            if budget == 300:  # the selector's own pick among them
                assert timed >= 6
            # six launches at least for each of two solves from three sources
            assert sim.count(kernel) >= 36
            for cfg in (None, sim.config(g)):
                sim.set(reset=1)
                assert sim.sssp(g, 5, p, cfg) == 0 and sim.batch([(g, 5, p)], [cfg] if cfg else None)[0] == 0
                assert (sim.count(kernel) > 0, sim.count("worker") > 0) == (not queues_faster, queues_faster)
                np.testing.assert_array_equal(out, oracle.dijkstra(csr, 5))
            # what is no longer the default is a request for queues
            old = sim.config(g)
            for k, v in before.items():
                setattr(old, k, v)
            if old.as_dict() != sim.config(g).as_dict():
                sim.set(reset=1)
                assert sim.sssp(g, 5, p, old) == 0 and sim.count("worker") == 1


def test_the_corpus_is_timed_on_queues(sim):
    """Every template as collect.py asks for it, the graph's default among them."""
    sys.path.insert(0, os.path.join(ROOT, "paper_2602_10080_amd", "selector"))
    import collect
    for csr in (ROAD, SKEWED):
        g = sim.graph(csr)
        p, _ = sim.buffer(csr.n)
        cfgs = [sim.config(g)]
        for t in range(-1, sim.lib.mlmq_candidate_count()):
            c = sim.config(g)
            assert sim.lib.mlmq_candidate_config(g, t, ctypes.byref(c)) == 0
            cfgs.append(c)
        for c in cfgs:
            sim.set(reset=1)
            assert sim.sssp(g, 3, p, collect.on_queues(c)) == 0, sim.error()
            assert sim.count("worker") == 1


def test_a_batch_makes_room_for_a_server_between_its_groups(sim):
    """The group under way ends as it is; what has not begun takes the queue
    worker, and the server's kernel does not wait for the whole batch."""
    served, mesh = sim.graph(ROAD), sim.graph(MESH)
    p, _ = sim.buffer(ROAD.n)
    bufs = [sim.buffer(MESH.n) for _ in range(70)]
    srv = Server(sim, [served])
    try:
        sim.set(steps=20, step_ms=10, reset=1)  # 0.2 s a group of 32
        res = []
        t = threading.Thread(target=lambda: res.append(sim.batch([(mesh, i, b[0]) for i, b in enumerate(bufs)])))
        t.start()
        _until(lambda: sim.count("tile") > 3)
        assert srv.wait(srv.submit(0, 3, p)) == 0
        t.join()
        assert res[0][0] == 0 and not any(res[0][1]) and sim.count("worker") == 1
        assert 20 <= sim.count("launches before it") == sim.count("tile") < 40  # one group's
        for i, (_p, o) in enumerate(bufs):
            np.testing.assert_array_equal(o, oracle.dijkstra(MESH, i))
    finally:
        srv.close()


def test_autotune_beside_a_server(sim):
    """No bulk solve can be timed there: default solves keep it."""
    served, g = sim.graph(ROAD), sim.graph(SKEWED)
    (p, _), (q, out) = sim.buffer(ROAD.n), sim.buffer(SKEWED.n)
    srv = Server(sim, [served])
    try:
        sim.set(served_ms=2500, worker_ms=1, worker_more=0.5)  # later runs are slower than the candidates' first
        ticket = srv.submit(0, 3, p)
        _until(lambda: sim.count("resident") == 1)
        assert sim.lib.mlmq_autotune(g, 20, None) == 0
        assert srv.wait(ticket) == 0
    finally:
        srv.close()
    sim.set(reset=1)
    assert sim.sssp(g, 5, q) == 0 and sim.count("step") > 0
    np.testing.assert_array_equal(out, oracle.dijkstra(SKEWED, 5))
