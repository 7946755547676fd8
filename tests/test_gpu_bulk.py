"""Solves and levels in the library's own configuration (stepping and tiled
solves) at the sizes and forms where their paths change, against the oracle.
Distances are whole numbers: every comparison is exact."""
import threading
import time

import numpy as np
import pytest

import graphgen as gg
import oracle
import paper_2602_10080_amd as mlmq

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def directed(n, pairs, wmax, seed, zero_weights=False):
    """Random directed graph whose last vertex has no edges at all."""
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n - 1, pairs), rng.integers(0, n - 1, pairs)
    w = rng.integers(0 if zero_weights else 1, wmax + 1, pairs).astype(np.uint32)
    return gg.from_edges(n, u, v, w)


def expect(csr, src):
    return oracle.dijkstra(csr, src)


def host(t):
    return t if isinstance(t, np.ndarray) else t.cpu().numpy().view(np.uint32)


FORMS = [
    ("one tile", lambda: gg.grid(24, 37, 0.0, seed=1)),
    ("tile edge", lambda: gg.grid(64, 64, 0.0, seed=2)),          # 4096 vertices: the most of one tile
    ("just above one tile", lambda: gg.grid(17, 241, 0.0, seed=3)),  # 4097
    ("many tiles, ragged", lambda: gg.grid(211, 307, 0.05, seed=4)),
    ("skewed", lambda: gg.rmat(12, 16, seed=5)),
    ("directed", lambda: directed(10007, 80000, 255, 6)),
    ("zero weights", lambda: directed(10007, 80000, 3, 7, True)),
    ("wide weights", lambda: directed(10007, 80000, 1 << 17, 8)),
    ("sparse, mostly unreached", lambda: directed(10007, 9000, 255, 9)),
]


@pytest.mark.parametrize("name,make", FORMS, ids=[f[0] for f in FORMS])
def test_default_solves_equal_the_oracle(name, make):
    csr = make()
    g = mlmq.Graph.from_csr(csr)
    out = mlmq.new_dist(csr.n)
    for src in (0, csr.n // 2, csr.n - 1):  # the directed graphs' last vertex is isolated
        want = expect(csr, src)
        np.testing.assert_array_equal(host(mlmq.sssp(g, src, out=out)), want, err_msg=f"{name} from {src}")
        np.testing.assert_array_equal(mlmq.sssp(g, src, out=np.empty(csr.n, np.uint32)), want)
        np.testing.assert_array_equal(host(mlmq.bfs(g, src, out=out)), oracle.bfs(csr, src))


def test_queues_asked_for_give_the_same_distances():
    for csr in (gg.grid(96, 80, 0.05, seed=1), gg.rmat(13, 8, seed=1)):
        g = mlmq.Graph.from_csr(csr)
        a = host(mlmq.sssp(g, 3)).copy()
        cfg = mlmq.default_config(l0_rows=1, l1_type=2, l2_type=1, bmax=32, bnum=4, delta2_log2=7, delta1=128,
                                  l1_cap=256, th_hub=0)
        np.testing.assert_array_equal(host(mlmq.sssp(g, 3, config=cfg)), a)


def test_a_graph_too_deep_for_steps():
    """A long path with a hub at its end: neither tiles (the hub's degree) nor
    the step limit take it, so the queue worker does."""
    n, arms = 6000, 200
    u = np.concatenate([np.arange(n - 1), np.full(arms, n - 1)])
    v = np.concatenate([np.arange(1, n), n + np.arange(arms)])
    total = n + arms
    csr = gg.from_edges(total, u, v, np.full(len(u), 255, np.uint32))
    g = mlmq.Graph.from_csr(csr)
    np.testing.assert_array_equal(host(mlmq.sssp(g, 0)), expect(csr, 0))


def test_batches_of_more_queries_than_a_group_and_from_two_threads():
    graphs = [gg.rmat(10, 8, seed=1), gg.grid(40, 40, 0.05, seed=2), gg.grid(90, 90, 0.05, seed=3)]
    handles = [mlmq.Graph.from_csr(c) for c in graphs]
    queries = [(k, (17 * i) % graphs[k].n) for i in range(35) for k in range(3)]
    want = {q: expect(graphs[q[0]], q[1]) for q in set(queries)}
    failed = []

    def work():
        try:
            outs, status = mlmq.sssp_batch([handles[k] for k, _ in queries], [s for _, s in queries])
            assert not any(status)
            for q, o in zip(queries, outs):
                np.testing.assert_array_equal(host(o), want[q])
        except BaseException as e:  # noqa: BLE001 (handed to the main thread)
            failed.append(e)

    threads = [threading.Thread(target=work) for _ in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_stretches_without_labels():
    """Weights far above the width of a distance step: most scans find nothing
    in it and go on to the smallest label. Shared launches of many rows have
    workgroups that start when others of the same step have ended."""
    csr = gg.rmat(16, 16, seed=9)
    rng = np.random.default_rng(9)
    w = np.where(rng.random(csr.m) < 0.97, csr.w % 4 + 1, csr.w * 1000).astype(np.uint32)
    csr = gg.Csr(csr.n, csr.off, csr.col, w)
    g = mlmq.Graph.from_csr(csr)
    sources = [int(s) for s in gg.sample_sources(csr, 32, seed=1)]
    want = [expect(csr, s) for s in sources]
    for _ in range(4):
        outs, status = mlmq.sssp_batch([g] * len(sources), sources)
        assert not any(status)
        for o, d in zip(outs, want):
            np.testing.assert_array_equal(host(o), d)
    for s, d in zip(sources[:4], want):
        np.testing.assert_array_equal(host(mlmq.sssp(g, s)), d)


@pytest.mark.parametrize("queues", [False, True])
def test_a_batch_starts_after_work_on_the_default_stream(queues):
    """Fills of the output buffers wait behind a long kernel when the batch is
    called; the solves come after them."""
    graphs = [gg.rmat(12, 16, seed=5), gg.grid(90, 90, 0.05, seed=3), gg.grid(30, 30, 0.0, seed=2)]
    handles = [mlmq.Graph.from_csr(c) for c in graphs]
    outs = [mlmq.new_dist(c.n) for c in graphs]
    cfg = mlmq.default_config(l0_rows=1, l1_type=2, l2_type=1, bmax=32, bnum=4, delta2_log2=7, delta1=128, l1_cap=256,
                              th_hub=0) if queues else None
    for _ in range(2):
        torch.cuda._sleep(100_000_000)
        for o in outs:
            o.fill_(7)
        _, status = mlmq.sssp_batch(handles, [3] * 3, outs=outs, configs=[cfg] * 3)
        assert not any(status)
        for c, o in zip(graphs, outs):
            np.testing.assert_array_equal(host(o), expect(c, 3))


def test_solves_and_batches_beside_a_busy_server():
    """A server that always has queries keeps its kernel on the device; default
    solves go on beside it and finish long before it would leave."""
    served = gg.rmat(16, 16, seed=4)
    h = mlmq.Graph.from_csr(served)
    graphs = [gg.rmat(12, 16, seed=5), gg.grid(90, 90, 0.05, seed=3), gg.grid(30, 30, 0.0, seed=2)]
    handles = [mlmq.Graph.from_csr(c) for c in graphs]
    want = [expect(c, 3) for c in graphs]
    outs = [mlmq.new_dist(served.n) for _ in range(8)]
    srv = mlmq.Server([h], 1 << 30, max_slots=8)
    stop, served_n = threading.Event(), []

    def load():
        while not stop.is_set():
            for t in [srv.submit(0, 17 * k, outs[k]) for k in range(8)]:
                assert srv.wait(t) == 0
                served_n.append(t)

    t = threading.Thread(target=load)
    t.start()
    try:
        end = time.time() + 20
        while not served_n and time.time() < end:
            time.sleep(0.01)
        for _ in range(3):
            for c, g, w in zip(graphs, handles, want):
                t0 = time.time()
                np.testing.assert_array_equal(host(mlmq.sssp(g, 3)), w)
                assert time.time() - t0 < 1.0
            t0 = time.time()
            res, status = mlmq.sssp_batch(handles, [3] * 3)
            assert time.time() - t0 < 1.0 and not any(status)
            for o, w in zip(res, want):
                np.testing.assert_array_equal(host(o), w)
    finally:
        stop.set()
        t.join()
        srv.close()
    assert served_n
    np.testing.assert_array_equal(host(outs[0]), expect(served, 0))


def test_a_shallow_graph_with_a_long_tail():
    """Steps run out on the tail: the queue worker solves, and later calls and
    batches, with and without another try, give the same."""
    core, tail = gg.rmat(12, 16, seed=5), 3000
    hub = gg.max_degree_vertex(core)
    row = np.repeat(np.arange(core.n), core.degrees())
    t = core.n + np.arange(tail)
    u, v = np.concatenate([[hub], t[:-1]]), t
    w = np.full(tail, 9)
    csr = gg.from_edges(core.n + tail, np.concatenate([row, u, v]), np.concatenate([core.col, v, u]),
                        np.concatenate([core.w, w, w]))
    g = mlmq.Graph.from_csr(csr)
    want, levels = expect(csr, 3), oracle.bfs(csr, 3)
    for _ in range(10):
        np.testing.assert_array_equal(host(mlmq.sssp(g, 3)), want)
        np.testing.assert_array_equal(host(mlmq.bfs(g, 3)), levels)
    outs, status = mlmq.sssp_batch([g] * 3, [3] * 3)
    assert not any(status)
    for o in outs:
        np.testing.assert_array_equal(host(o), want)


def test_a_path_of_many_more_hops_than_rounds():
    """100,000 hops: the tiled solve gets to the end by itself (a solve by
    queues reports the time of its waves)."""
    n = 100_000
    rng = np.random.default_rng(2)
    u, w = np.arange(n - 1), rng.integers(1, 256, n - 1)
    csr = gg.from_edges(n, np.concatenate([u, u + 1]), np.concatenate([u + 1, u]), np.concatenate([w, w]))
    g = mlmq.Graph.from_csr(csr)
    out, st = mlmq.sssp(g, 0, stats=True)
    np.testing.assert_array_equal(host(out), np.concatenate([[0], np.cumsum(w)]).astype(np.uint32))
    assert st["wave_ms"] == 0


def test_batches_of_bucket_queues():
    """Queries on bucket rings whose waves are any of the launch's: each query
    has waves that look for work at once, whatever workgroups they are. More
    queries than run at a time, beside one that takes many waves."""
    graphs = [gg.grid(256, 256, 0.05, seed=9)] + [gg.grid(40 + i, 50, 0.05, seed=i) for i in range(30)] + \
             [gg.rmat(10, 8, seed=i) for i in range(6)]
    handles = [mlmq.Graph.from_csr(c) for c in graphs]
    cfg = mlmq.default_config(l0_rows=1, l1_type=2, l2_type=1, bmax=32, bnum=4, delta2_log2=7, delta1=128, l1_cap=256,
                              th_hub=0)
    for _ in range(2):  # the second launch replays the first one's graph
        outs, status, stats = mlmq.sssp_batch(handles, [5] * len(handles), configs=[cfg] * len(handles), stats=True)
        assert not any(status)
        for c, o, st in zip(graphs, outs, stats):
            np.testing.assert_array_equal(host(o), expect(c, 5))
            assert st["l2_writes"] > 0 and st["wave_ms"] > 0


def on_queues(cfg):
    """cfg with a knob changed that its queues do not read: never the default."""
    return cfg.copy(bmax=cfg.bmax // 2) if cfg.l2_type == 2 else cfg.copy(pnum=3)


def overflowing(form, real):
    """A graph in the form of one bulk solve whose largest distance fits, or
    does not, below 2^32 - 1, beside sums that do not (Section 2.1)."""
    if form == "tiles":  # a path of heavy edges over several tiles
        n, w = 6000, (1 << 20) - 1
        u = np.arange(n - 1)
        fits = (2**32 - 2) // w  # hops
        wt = np.full(n - 1, w, np.uint64)
        if not real:
            wt[fits:] = 1  # ends a little below the limit
        return gg.from_edges(n, np.concatenate([u, u[:10]]), np.concatenate([u + 1, u[:10]]),
                             np.concatenate([wt, wt[:10]])), n - 1
    rng = np.random.default_rng(11)
    n = 9000
    u, v = rng.integers(0, n, 40000), rng.integers(0, n, 40000)
    w = rng.integers(1, 1000, 40000)
    # a way round by two edges whose sum is too large, and one vertex far out
    tail = [2**31, 2**31 if real else 2**31 - 10**6]
    # (the last vertex has no edges)
    return gg.from_edges(n + 4, np.concatenate([u, [0, n, n + 1, n]]), np.concatenate([v, [n, n + 1, 1, n + 2]]),
                         np.concatenate([w, [tail[0], tail[1], 2**32 - 1, 2**32 - 5]]) if real else
                         np.concatenate([w, [tail[0], tail[1], 2**32 - 1, 7]])), n + 1


@pytest.mark.parametrize("form", ["tiles", "steps"])
@pytest.mark.parametrize("real", [False, True])
def test_distances_near_the_largest_one(form, real):
    csr, far = overflowing(form, real)
    g = mlmq.Graph.from_csr(csr)
    out, buf = mlmq.new_dist(csr.n), np.empty(csr.n, np.uint32)
    if real:
        for call in (lambda: mlmq.sssp(g, 0, out=out), lambda: mlmq.sssp(g, 0, out=buf)):
            with pytest.raises(mlmq.MlmqError) as e:
                call()
            assert e.value.code == -3
        _, status = mlmq.sssp_batch([g, g], [0, csr.n - 1], outs=[out, mlmq.new_dist(csr.n)])
        assert status == [-3, 0]
        return
    want = expect(csr, 0)
    assert want[far] != 0xFFFFFFFF and int(want[far]) + int(csr.w.max()) >= 2**32 - 1
    out, st = mlmq.sssp(g, 0, out=out, stats=True)
    assert st["wave_ms"] == 0  # no queues
    np.testing.assert_array_equal(host(out), want)
    np.testing.assert_array_equal(mlmq.sssp(g, 0, out=buf), want)
    outs, status = mlmq.sssp_batch([g, g], [0, csr.n - 1])
    assert status == [0, 0]
    np.testing.assert_array_equal(host(outs[0]), want)
    np.testing.assert_array_equal(host(outs[1]), expect(csr, csr.n - 1))


def test_a_batch_of_bulk_solves_with_counters():
    graphs = [gg.rmat(12, 16, seed=5), gg.grid(90, 90, 0.05, seed=3), gg.grid(30, 30, 0.0, seed=2)]
    handles = [mlmq.Graph.from_csr(c) for c in graphs]
    outs, status, stats = mlmq.sssp_batch(handles * 2, [3] * 6, stats=True)
    assert not any(status)
    for c, o, st in zip(graphs * 2, outs, stats):
        want = expect(c, 3)
        np.testing.assert_array_equal(host(o), want)
        reached = int((want != 0xFFFFFFFF).sum())
        assert st["expansions"] > 0 and st["edges"] > 0 and st["pushes"] >= reached // 2
        assert st["wave_ms"] == st["l2_writes"] == st["l1_writes"] == 0


def test_queue_batches_of_changing_layout():
    """The captured launch of a batch on queues: the same number of queries with
    queue memory laid out differently, and the same again."""
    a, b = gg.grid(256, 256, 0.05, seed=41), gg.rmat(12, 8, seed=3)
    ga, gb = mlmq.Graph.from_csr(a), mlmq.Graph.from_csr(b)
    cfgs = [on_queues(ga.config()), on_queues(gb.config())]
    for rep, mix in enumerate(([0, 0, 1], [0, 1, 1], [1, 1, 0], [0, 0, 1], [0, 0, 1])):
        srcs = [(rep * 977 + 13 * i) % (a, b)[k].n for i, k in enumerate(mix)]
        outs, status, stats = mlmq.sssp_batch([(ga, gb)[k] for k in mix], srcs, configs=[cfgs[k] for k in mix], stats=True)
        assert not any(status)
        for k, s, o, st in zip(mix, srcs, outs, stats):
            np.testing.assert_array_equal(host(o), expect((a, b)[k], s), err_msg=str((rep, k, s)))
            assert st["wave_ms"] > 0


def test_queue_solves_on_a_degree_ordered_copy():
    csr = gg.rmat(14, 16, seed=21)
    g = mlmq.Graph.from_csr(csr, degree_order=True)
    cfg = on_queues(g.config())
    for s in [gg.max_degree_vertex(csr)] + [int(x) for x in gg.sample_sources(csr, 2, seed=4)]:
        want = expect(csr, s)
        out, st = mlmq.sssp(g, s, config=cfg, stats=True)
        np.testing.assert_array_equal(host(out), want)
        assert st["wave_ms"] > 0
        np.testing.assert_array_equal(mlmq.sssp(g, s, out=np.empty(csr.n, np.uint32), config=cfg), want)
        np.testing.assert_array_equal(host(mlmq.bfs(g, s, config=cfg.copy(delta1=1, delta2_log2=0))), oracle.bfs(csr, s))
