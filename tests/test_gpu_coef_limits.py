"""GPU parity of the coefficient form where a size or a launch reaches a limit:
look-ups far past a block of edges, launches of more work items than one
dimension of a grid takes, outputs cut into parts, and batches cut into rounds."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2010_08423_amd import inputs
from parity_util import host_threads, say

pytestmark = pytest.mark.gpu

R = None


def setup_module(module):
    global R
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2010_08423_amd as lib

    R = lib
    R.library()


def hub_graph(arrivals, leave, feeders=2000):
    """`arrivals` edges into vertex 0, in order of time from 1 on, `feeders` per
    time; edges from vertex 0 to 40 others at each of the times `leave` (as
    shares of the last arrival's time), and one edge on from each of those."""
    i = np.arange(arrivals)
    last = int(i[-1] // feeders + 1)
    times = np.maximum(1, (np.asarray(leave) * last).astype(np.int64))
    out = 1 + feeders + np.arange(40)
    src = [1 + i % feeders, np.zeros(40 * len(times)), np.tile(out, len(times))]
    dst = [np.zeros(arrivals), np.tile(out, len(times)), np.tile(out, len(times)) + 40]
    t = [1 + i // feeders, np.repeat(times, 40), np.repeat(times, 40) + 1]
    g = inputs.TemporalGraph(1 + feeders + 80, *(np.concatenate(x).astype(np.uint32) for x in (src, dst, t)),
                             name=f"hub{arrivals}")
    return g, last


# The search for the next marked window end goes on past 64 blocks of 1024
# edges in steps of 1024 blocks: one step from some 10^5 arrivals on, a second one
# from 1.12*10^6; with one edge per thread and, from 1.4*10^6 edges on, four.
@pytest.mark.parametrize("arrivals", [100_000, 400_000, 700_000, 1_300_000, 1_500_000])
def test_next_window_end_far_past_a_block(arrivals):
    for leave in ((1.0,), (0.3, 0.97)):
        g, last = hub_graph(arrivals, leave)
        gd = R.Graph.from_inputs(g)
        for k in (3, 4):
            for delta in (2, last // 2, last):
                say("[coef] hub", arrivals, "leave", leave, "k", k, "delta", delta)
                want = oracle.sieve(g.n, g.src, g.dst, g.t, k, delta, 9, threads=host_threads())
                assert R.run(gd, k, delta, 9).fingerprint == want
                assert R.run(gd, k, delta, 9, tuning=R.Tuning(edges_per_tile=16)).fingerprint == want


def star_graph(n, m, into, out, tau, seed):
    """m edges: the share `into` end in vertex 0, the share `out` start there, the rest are random."""
    r = np.random.default_rng(seed)
    a, b = int(m * into), int(m * out)
    src = np.concatenate([r.integers(1, n, a), np.zeros(b), r.integers(1, n, m - a - b)])
    dst = np.concatenate([np.zeros(a), r.integers(1, n, m - a)])
    g = inputs.TemporalGraph(n, src.astype(np.uint32), dst.astype(np.uint32), r.integers(1, tau + 1, m).astype(np.uint32),
                             name=f"star{m}")
    return inputs.add_colours(g, 4, seed=seed)


# One vertex whose arrivals span more runs of a scan than are summed one by one:
# rows of 3 to 126 coefficients (runs sharing a wave from 262144 entries on, and
# runs over two blocks of coefficients), single iterations, and, in the batch,
# long runs.
@pytest.mark.parametrize("m,k", [(30_000, 3), (150_000, 5), (400_000, 4), (60_000, 9)])
def test_carries_over_many_runs(m, k):
    g = star_graph(3000, m, 0.85, 0.08, 2000, seed=k)
    gd = R.Graph.from_inputs(g)
    full, queries, want = 1 << k, [], []
    for delta, motif in ((40, None), (1500, None), (1500, np.array([1, 1, 1, k - 3], np.uint8))):
        say("[coef] star m", m, "k", k, "delta", delta, "motif", motif is not None)
        e = R.run(gd, k, delta, 5, motif=motif, per_iteration=True, tuning=R.Tuning(edges_per_tile=16))
        if k <= 5:
            kw = dict(colour=g.colour, n_colours=4, motif=motif) if motif is not None else {}
            assert e.fingerprint == oracle.sieve(g.n, g.src, g.dst, g.t, k, delta, 5, threads=host_threads(), **kw)
        assert R.run(gd, k, delta, 5, motif=motif).fingerprint == e.fingerprint
        for lo, hi in ((0, full), (1, 3), (full // 3, full - 1)):
            r = R.run(gd, k, delta, 5, motif=motif, it_begin=lo, it_end=hi, per_iteration=True)
            assert np.array_equal(r.per_iteration, e.per_iteration[lo:hi])
        queries.append(inputs.Query(k=k, delta=delta, seed=5, motif=motif))
        want.append(e.fingerprint)
    for q, F in zip(queries, want):
        assert R.run_batch([gd], [q])[0][0].fingerprint == F
    assert [r.fingerprint for r in R.run_batch([gd] * 3, queries)[0]] == want


# Single iterations on many vertices: a table of every vertex's z^L would take
# 8 n 2^k bytes (45 GB) and a launch of more than 2^32 work items.
@pytest.mark.parametrize("n,k", [(1_400_000, 12), (70_000_000, 6)])
def test_iterations_on_many_vertices(n, k):
    m, r = 30_000, np.random.default_rng(k)
    at = np.sort(r.choice(n, size=600, replace=False))  # the few vertices with edges, over the whole range
    g = inputs.TemporalGraph(n, at[r.integers(0, 600, m)].astype(np.uint32), at[r.integers(0, 600, m)].astype(np.uint32),
                             r.integers(1, 400, m).astype(np.uint32), name="spread")
    gd = R.Graph.from_inputs(g)
    say("[coef] iterations n", n, "k", k)
    got = R.run(gd, k, 4, 3, per_iteration=True)
    small = inputs.TemporalGraph(600, np.searchsorted(at, g.src).astype(np.uint32), np.searchsorted(at, g.dst).astype(np.uint32),
                                 g.t, name="packed")
    sd = R.Graph.from_inputs(small)  # the same graph on 600 vertices: other values, the same iterations that vanish
    assert np.array_equal(got.per_iteration != 0, R.run(sd, k, 4, 3, per_iteration=True).per_iteration != 0)
    assert got.fingerprint == R.run(gd, k, 4, 3).fingerprint == int(np.bitwise_xor.reduce(got.per_iteration))
    part = R.run(gd, k, 4, 3, it_begin=8, it_end=24, per_iteration=True, tuning=R.Tuning(edges_per_tile=16))
    assert np.array_equal(part.per_iteration, got.per_iteration[8:24])


def test_literal_level_of_many_slots():
    """A level of 67.2*10^6 slots, a wave each: over 2^32 work items in one launch.
    On a ring whose vertices pass everything on at once, every slot is in the sets."""
    n, times = 4_200_000, 16
    v = np.tile(np.arange(n, dtype=np.uint32), times)
    t = np.repeat(np.arange(1, times + 1, dtype=np.uint32), n)
    gd = R.Graph(n, v, (v + 1) % np.uint32(n), t)
    del v, t
    say("[coef] literal ring")
    got = R.run_literal(gd, 3, 0, 5)
    parts = [R.run_literal(gd, 3, 0, 5, it_begin=a, it_end=b).zeta for a, b in ((0, 5), (5, 8))]  # evaluation form
    assert np.array_equal(got.zeta, parts[0] ^ parts[1]) and (got.reach == 1).all()


# Slots of very uneven length: a hub's with up to 128 edges next to single ones,
# blocks of 1024 edges that hold a few slots, a part of one, or a thousand.
@pytest.mark.parametrize("k,delta", [(3, 4), (5, 60), (7, 4), (8, 20)])
def test_literal_uneven_slots(k, delta):
    r = np.random.default_rng(k)
    n, hubs = 1200, 9000
    src = np.concatenate([r.integers(0, n, 3 * hubs), r.integers(0, n, 4000), np.zeros(600), np.full(500, n - 1)])
    dst = np.concatenate([np.zeros(hubs), np.full(hubs, 600), np.full(hubs, n - 1), r.integers(0, n, 5100)])
    t = np.concatenate([1 + np.arange(3 * hubs) % hubs // 100, r.integers(1, 300, 5100)])
    g = inputs.TemporalGraph(n, *(x.astype(np.uint32) for x in (src, dst, t)), name="uneven")
    inputs.add_colours(g, 4, seed=k)
    gd = R.Graph.from_inputs(g)
    for motif in (None, np.array([1, 1, 0, k - 2], np.uint8)):
        kw = dict(colour=g.colour, n_colours=4, motif=motif) if motif is not None else {}
        say("[coef] literal uneven slots k", k, "delta", delta)
        z, reach = oracle.fine_literal(g.n, g.src, g.dst, g.t, k, delta, 17, threads=host_threads(), **kw)
        got = R.run_literal(gd, k, delta, 17, motif=motif)
        assert np.array_equal(got.zeta, z) and np.array_equal(got.reach, reach)


# Per-slot outputs around the slot length from which a wave goes on where the
# slot's thread stops (16 edges, then 64 at a time), and, from 262144 edges on,
# written in eight parts of the edges with slots across their ends.
@pytest.mark.parametrize("lengths", [(1, 15, 16, 17, 18, 79, 80, 81, 144, 145, 300), (900,) * 310, (70_000,) * 4])
def test_slots_of_every_length(lengths):
    r = np.random.default_rng(len(lengths))
    n = max(lengths) + 2
    src = [np.sort(r.choice(n - 1, size=x, replace=False)) for x in lengths]
    into = np.repeat(np.arange(len(lengths)) % 7, lengths)  # seven vertices, a slot per time
    t = np.repeat(10 + np.arange(len(lengths)) // 7, lengths)
    src = np.concatenate([*src, r.integers(0, n, 500)])
    dst = np.concatenate([np.where(src[:len(into)] == into, n - 1, into), r.integers(0, n, 500)])
    g = inputs.TemporalGraph(n, src.astype(np.uint32), dst.astype(np.uint32),
                             np.concatenate([t, r.integers(1, 12, 500)]).astype(np.uint32), name="lengths")
    gd = R.Graph.from_inputs(g)
    for k in (2, 3, 4):
        say("[coef] slots of up to", max(lengths), "edges, m", len(g.src), "k", k)
        z, reach, F = oracle.fine_grained(g.n, g.src, g.dst, g.t, k, 6, 5, threads=host_threads())
        for it_end in (0, 1 << k):  # (the second run reuses the output buffer)
            got = R.run_fine(gd, k, 6, 5, it_end=it_end)
            assert got.fingerprint == F and np.array_equal(got.reach, reach) and np.array_equal(got.zeta, z)
        only = R.run_fine(gd, k, 6, 5, slots=False)
        assert only.zeta is None and np.array_equal(only.reach, reach)


def test_outputs_of_both_readings_share_a_buffer():
    g = inputs.chung_lu_graph(30_000, 300_000, 2.4, 800, seed=9)
    gd = R.Graph.from_inputs(g)
    fine = oracle.fine_grained(g.n, g.src, g.dst, g.t, 4, 6, 5, threads=host_threads())
    lit = oracle.fine_literal(g.n, g.src, g.dst, g.t, 4, 6, 5, threads=host_threads())
    for _ in range(2):
        for want, got in ((fine, R.run_fine(gd, 4, 6, 5)), (lit, R.run_literal(gd, 4, 6, 5))):
            assert np.array_equal(got.zeta, want[0]) and np.array_equal(got.reach, want[1])


def serve(srv, gid, queries):
    tickets = [srv.submit(gid, q) for q in queries]
    return [srv.poll(t, wait_ms=100_000).fingerprint for t in tickets]


def test_server_stays_in_its_budget():
    """Groups of whole queries (coefficient form, rows in several rounds), of
    parts of ranges (evaluation form) and of both, one after another: what the
    server takes of the device's memory stays within the budget."""
    import threading

    import torch

    g = inputs.uniform_graph(10_000, 100_000, 200, seed=3)
    gd = R.Graph.from_inputs(g)
    whole = [inputs.Query(k=8, delta=60, seed=i) for i in range(18)]
    parts = [inputs.Query(k=8, delta=60, seed=i, it_begin=0, it_end=200) for i in range(18)]
    want = {id(q): R.run(gd, q.k, q.delta, q.seed, it_begin=q.it_begin, it_end=q.it_end).fingerprint for q in whole + parts}
    budget, slack = 2 << 30, 64 << 20
    free0 = torch.cuda.mem_get_info()[0]
    least, stop = [free0], threading.Event()

    def watch():
        while not stop.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])
            stop.wait(0.0005)

    th = threading.Thread(target=watch)
    th.start()
    try:
        srv = R.Server(hbm_budget=budget, streams=1)
        gid = srv.add_graph(gd)
        mixed = [q for pair in zip(whole[:9], parts[:9]) for q in pair]
        for queries in (whole, parts, mixed, whole, parts):
            say("[server] budget: group of", len(queries), "first range", queries[0].it_end, queries[1].it_end)
            assert serve(srv, gid, queries) == [want[id(q)] for q in queries]
        assert srv.stats()["held_bytes"] <= budget
        srv.close()
    finally:
        stop.set()
        th.join()
    say("[server] budget", budget, "taken", free0 - least[0])
    assert free0 - least[0] <= budget + slack


def test_batch_leaves_queries_with_too_large_rows():
    """A small budget: the rows of k = 12 exceed a group's share and the queries run
    in the evaluation form, next to others that fit it a few at a time."""
    g = inputs.uniform_graph(600, 12_000, 40, seed=4)
    gd = R.Graph.from_inputs(g)
    queries = [inputs.Query(k=k, delta=30, seed=10 * k + i) for i in range(3) for k in (12, 5, 9, 7)]
    want = [R.run(gd, q.k, q.delta, q.seed).fingerprint for q in queries]
    need = max(R.footprint(gd, q.k, q.delta) for q in queries)
    for budget in (need + (32 << 20), 4 * need, 4 << 30):
        srv = R.Server(hbm_budget=budget, streams=1)
        gid = srv.add_graph(gd)
        say("[server] rows beyond the share, budget", budget)
        assert serve(srv, gid, queries) == want
        srv.close()


def test_tuned_shapes_give_the_same_results():
    """The launch shapes that the tuner picks belong to the evaluation form, which
    default calls leave to larger k: given as knobs, they run."""
    g = inputs.add_colours(inputs.chung_lu_graph(800, 9000, 2.3, 60, seed=8), 4, seed=8)
    gd = R.Graph.from_inputs(g)
    queries = [inputs.Query(k=k, delta=4, seed=k, motif=None if k % 2 else np.array([1, 1, 2, k - 4], np.uint8)) for k in range(5, 9)]
    want = [oracle.sieve(g.n, g.src, g.dst, g.t, q.k, q.delta, q.seed, threads=host_threads(),
                         **(dict(colour=g.colour, n_colours=4, motif=q.motif) if q.motif is not None else {})) for q in queries]
    for tuned in (R.autotune(gd, queries), R.autotune_batch(gd, queries)):
        assert tuned.edges_per_tile in (8, 16) and tuned.waves_per_block in (1, 2, 4)
        for q, F in zip(queries, want):
            r = R.run(gd, q.k, q.delta, q.seed, motif=q.motif, tuning=tuned, per_iteration=True)
            assert r.fingerprint == F == int(np.bitwise_xor.reduce(r.per_iteration))
        assert [r.fingerprint for r in R.run_batch([gd] * 4, queries, tuning=tuned)[0]] == want
        half = [inputs.Query(k=q.k, delta=q.delta, seed=q.seed, motif=q.motif, it_begin=0, it_end=1 << q.k - 1) for q in queries]
        rest = [inputs.Query(k=q.k, delta=q.delta, seed=q.seed, motif=q.motif, it_begin=1 << q.k - 1, it_end=1 << q.k) for q in queries]
        # (parts of the range run in the evaluation form with the graph's tuned batch shape)
        parts = [r.fingerprint for r in R.run_batch([gd] * 8, half + rest)[0]]
        assert [a ^ b for a, b in zip(parts[:4], parts[4:])] == want


def test_batch_that_runs_out_of_memory_says_so():
    """Queries of the evaluation form whose tables exceed the device's memory, next to
    an invalid one: the call's error and theirs, not a result of zero."""
    gd = R.Graph.from_inputs(inputs.uniform_graph(100_000, 1_000_000, 1000, seed=4))
    queries = [inputs.Query(k=5, delta=3, seed=1), inputs.Query(k=1, delta=3, seed=2)]
    queries += [inputs.Query(k=16, delta=3, seed=i) for i in range(200)]  # 2.2 GB of tables each
    res, st = R.run_batch([gd] * len(queries), queries)
    assert st == R.RS_ENOMEM and res[1].status == R.RS_EINVAL
    assert all(r.status == R.RS_ENOMEM for r in res[2:])
    assert res[0].status == R.RS_OK and res[0].fingerprint == R.run(gd, 5, 3, 1).fingerprint
    # the workspace is as good as before
    res, st = R.run_batch([gd] * 2, [queries[0], inputs.Query(k=5, delta=3, seed=1, it_begin=0, it_end=32)])
    assert st == R.RS_OK and res[0].fingerprint == res[1].fingerprint != 0


def test_batch_of_more_queries_than_a_grid_takes():
    gd = R.Graph.from_inputs(inputs.uniform_graph(30, 200, 20, seed=4))
    some = [inputs.Query(k=3 + i % 3, delta=1 + i % 5, seed=i) for i in range(40)]
    want = [R.run(gd, q.k, q.delta, q.seed).fingerprint for q in some]
    n = 66_000
    res, st = R.run_batch([gd] * n, [some[i % 40] for i in range(n)])
    assert st == R.RS_OK and [r.fingerprint for r in res] == [want[i % 40] for i in range(n)]


def test_literal_with_little_memory_left():
    """Slots of 100 edges: the coefficient form's tables (16 bytes per edge and level)
    take more than the evaluation form, which runs where only that fits."""
    import torch

    n, dsts, times, per = 3001, 400, 100, 100
    s = np.arange(dsts * times)
    src = ((s[:, None] * 37 + np.arange(per) * 29) % n).astype(np.uint32).ravel()
    dst = np.repeat(s % dsts, per).astype(np.uint32)
    t = np.repeat(1 + s // dsts, per).astype(np.uint32)
    args = (12, 1, 5)
    want = R.run_literal(R.Graph(n, src, dst, t), *args)
    gd = R.Graph(n, src, dst, t)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    leave = 1000 << 20
    hold = []
    try:
        while torch.cuda.mem_get_info()[0] > leave + (8 << 20):
            hold.append(torch.empty(torch.cuda.mem_get_info()[0] - leave, dtype=torch.uint8, device="cuda"))
        say("[coef] literal, free", torch.cuda.mem_get_info()[0])
        for _ in range(2):
            got = R.run_literal(gd, *args)
            assert np.array_equal(got.zeta, want.zeta) and np.array_equal(got.reach, want.reach)
    finally:
        del hold
        torch.cuda.empty_cache()
    assert R.run_literal(gd, *args).fingerprint == want.fingerprint


# Backward passes with one and with four edges per thread; at 2.6*10^6 edges the
# rows are sized from the set sizes, and long runs leave their carries to a launch
# of their own.
@pytest.mark.parametrize("m,k,delta", [(1_396_736, 4, 60), (1_400_001, 5, 60), (2_600_000, 8, 60)])
def test_large_graphs(m, k, delta):
    g = inputs.add_colours(inputs.chung_lu_graph(m // 10, m, 2.5, 1000, seed=k), 4, seed=k)
    gd = R.Graph.from_inputs(g)
    for motif in (None, np.array([1, 1, 1, k - 3], np.uint8)):
        say("[coef] large m", m, "k", k, "motif", motif is not None)
        e = R.run(gd, k, delta, 3, motif=motif, per_iteration=True, tuning=R.Tuning(edges_per_tile=16))
        assert R.run(gd, k, delta, 3, motif=motif).fingerprint == e.fingerprint
        for lo, hi in ((0, 1 << k), (3, 9)):
            r = R.run(gd, k, delta, 3, motif=motif, it_begin=lo, it_end=hi, per_iteration=True)
            assert np.array_equal(r.per_iteration, e.per_iteration[lo:hi])


# Graphs whose slots are all of one length, on either side of the lengths from which
# the literal reading stays in the evaluation form.
@pytest.mark.parametrize("k,per,slots", [(6, 10, 200), (6, 11, 200), (7, 10, 200), (7, 11, 200), (10, 9, 200),
                                         (10, 10, 200), (3, 128, 1119), (3, 128, 1120), (3, 129, 1200)])
def test_literal_long_slots(k, per, slots):
    n = 73 if per < 70 else 293  # (so that walks of k vertices exist)
    s = np.arange(slots)
    src = (s[:, None] * 7 + 1 + np.arange(per)) % n
    dst = np.broadcast_to((s[:, None] * 7) % n, src.shape)  # (never among its sources)
    t = np.broadcast_to(1 + s[:, None] // 5, src.shape)
    src, dst, t = (x.ravel().astype(np.uint32) for x in (src, dst, t))
    gd = R.Graph(n, src, dst, t)
    for delta in (2, 12):
        z, reach = oracle.fine_literal(n, src, dst, t, k, delta, 7, threads=host_threads())
        got = R.run_literal(gd, k, delta, 7)
        assert np.array_equal(got.zeta, z) and np.array_equal(got.reach, reach) and got.yes


# A captured batch holds pointers to its graphs' arrays: a graph that takes a destroyed
# one's handle and sizes, but not its memory, is not run with them.
def test_batch_after_graph_is_replaced():
    hip = ctypes.CDLL("libamdhip64.so")
    n, k = 500, 6
    g = inputs.uniform_graph(n, 20000, 60, seed=1)
    held = []
    for i in range(4):
        name = np.random.default_rng(i).permutation(n).astype(np.uint32)  # (so all graphs have as many edges)
        src, dst = name[g.src], name[g.dst]
        z, reach, F = oracle.fine_grained(n, src, dst, g.t, k, 4, 9 + i, threads=host_threads())
        gd = R.Graph(n, src, dst, g.t)
        for _ in range(2):
            parts = [inputs.Query(k=k, delta=4, seed=9 + i, it_begin=a, it_end=b) for a, b in ((0, 20), (20, 64))]
            r, s = R.run_batch([gd] * 2, parts)
            assert s == 0 and r[0].fingerprint ^ r[1].fingerprint == F
        size = 4 * gd.info()["m"]
        gd.close()
        for _ in range(8):
            p = ctypes.c_void_p()
            assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(size)) == 0
            held.append(p)
    for p in held:
        assert hip.hipFree(p) == 0
