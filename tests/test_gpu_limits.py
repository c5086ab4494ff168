"""Calls at the edges of what the library's rules of size and launch choose between, against the CPU
oracle or the call they are a variant of, bit for bit."""
import sys

import numpy as np
import pytest

from paper_1507_03074_amd import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def B():
    import torch
    from paper_1507_03074_amd import binding
    from paper_1507_03074_amd import build as hbuild
    hbuild.ensure_built()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    return binding


def hits(seed, n):
    ev = synth.make_hits(np.random.default_rng([seed, n]), *synth.hits_split(n))
    return tuple(np.asarray(a[:n], np.float32) for a in (ev.x, ev.y, ev.z))


def noalloc_equals_fill_peaks(B, spec, ev, capacity=1 << 20):
    """The no-alloc call's matrix, count and first `capacity` peaks equal ht_fill_peaks'."""
    import torch
    x, y, z = B.hits_to_device(*ev)
    ref, acc = B.new_acc(spec), B.new_acc(spec)
    out, nf = B.new_peaks(capacity)
    B.ht_fill_peaks(spec, x, y, z, ref, out, capacity, nf)
    c, v, n = B.peaks_to_host(out, nf, capacity, allow_truncation=True)
    acc.fill_(7)
    out.fill_(-1)
    B.ht_fill_peaks_noalloc(spec, x, y, z, acc, out, capacity, nf)
    c2, v2, n2 = B.peaks_to_host(out, nf, capacity, allow_truncation=True)
    assert torch.equal(acc, ref) and n2 == n and np.array_equal(c2, c) and np.array_equal(v2, v)
    return n


@pytest.mark.parametrize("threshold", [1, 2, 3, 4])
def test_noalloc_takes_crowded_events_at_low_thresholds(B, threshold):
    """Events from the reported dense_hits on are accepted whatever the threshold."""
    spec = synth.GridSpec(4, 16, 1024, 1024, threshold=threshold)
    for n in (16384, 24576, 39321):
        say("no-alloc, threshold", threshold, "hits", n)
        assert noalloc_equals_fill_peaks(B, spec, hits(1, n)) > 1000


def test_noalloc_layouts(B):
    """Direct lists at 39 000 hits, the counting sort past the array, slices of a matrix whose
    survivors' scratch passes it by far, and the stencil in their place."""
    say("direct lists")
    spec = synth.GridSpec(4, 16, 1024, 1024)
    assert B.ht_debug_launch_plan(spec, [39000], "noalloc")["direct"] == 1
    noalloc_equals_fill_peaks(B, spec, hits(2, 39000))
    assert B.ht_debug_launch_plan(spec, [64000], "noalloc")["direct"] == 0
    noalloc_equals_fill_peaks(B, spec, hits(2, 64000))
    say("slices")
    spec = synth.GridSpec(2, 32, 4096, 2048, threshold=9)
    B.ht_set_tuning(spec, cand_cap=2)
    try:
        assert B.ht_debug_launch_plan(spec, [2500], "noalloc")["sliced"] == 1
        for k in range(2):
            assert noalloc_equals_fill_peaks(B, spec, hits(3, 2500)) > 50
    finally:
        B.ht_set_tuning(spec)
    say("stencil in place of slices")
    spec = synth.GridSpec(4, 16, 2048, 2048, threshold=9)
    assert B.ht_debug_launch_plan(spec, [40000], "noalloc")["n_stencil"] == 1
    assert B.ht_debug_launch_plan(spec, [40000])["n_stencil"] == 0
    assert noalloc_equals_fill_peaks(B, spec, hits(4, 40000)) > 1000


def oracle_run(spec, ev):
    from oracle import oracle
    g = oracle.OracleGrid(*spec.as_tuple())
    M, _ = oracle.fill(g, *ev)
    return (M, *oracle.peaks(g, M))


@pytest.mark.parametrize("graph", ["0", "1"])
def test_batches_around_the_stencil_threshold(B, monkeypatch, graph):
    """The default launches of batches whose largest event lies below and at twice the reported
    dense_hits (8192 on 4x16x256x256), one graph bucket of workgroups; replayed."""
    spec = synth.GridSpec(4, 16, 256, 256, threshold=8)
    monkeypatch.setenv("HT_BATCH_GRAPH", graph)
    batches = ([6585] * 3 + [300], [4500, 4200, 300], [8191, 5000, 300], [8192, 5000, 4095, 300])
    want = {}
    for _ in range(2):
        for sizes in batches:
            say("graph", graph, "sizes", sizes)
            evs = [hits(10 + i, n) for i, n in enumerate(sizes)]
            res = B.fill_peaks_batch(spec, evs)
            for i, n in enumerate(sizes):
                if (i, n) not in want:
                    want[i, n] = oracle_run(spec, evs[i])
                M, c, v, k = want[i, n]
                assert np.array_equal(B.as_u32(res.acc[i]), M), (sizes, i)
                got = res.peaks[i]
                assert got[2] == k and np.array_equal(got[0], c) and np.array_equal(got[1], v), (sizes, i)


def test_request_loop_with_few_crowded_events(B):
    """A loop made for crowded events: batches without one, with one, and single events."""
    import time
    spec = synth.GridSpec(4, 16, 256, 256, threshold=8)
    sizes = [5000] * 3 + [9000, 5000, 300, 4096] + [4100]
    evs = [hits(20 + i, n) for i, n in enumerate(sizes)]
    with B.Server(spec, 2 << 30, peak_capacity=1 << 16, max_hits=9000, max_batch=4, n_streams=2, queue_depth=16) as srv:
        for group in (range(0, 3), range(3, 7), range(7, 8)):
            say("served", [sizes[i] for i in group])
            tickets = [srv.submit(*evs[i]) for i in group]
            for i, t in zip(group, tickets):
                deadline = time.time() + 60
                while (r := srv.poll(t)) is None:
                    assert time.time() < deadline
                    time.sleep(1e-4)
                M, c, v, k = oracle_run(spec, evs[i])
                assert r[2] == k and np.array_equal(r[0], c) and np.array_equal(r[1], v), i


@pytest.mark.parametrize("grid,threshold,sizes", [((2, 4, 40, 2500), 4, (1300, 1400, 2700, 8192, 8193)),
                                                  ((1, 3, 50, 333), 9, (512, 513, 1500)),
                                                  ((1, 3, 33, 14000), 3, (600, 2048, 2049))],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_moderately_long_slab_lists(B, grid, threshold, sizes):
    """Slab lists of one to six times the short-list fill's 512 records in registers, and more: either
    fill, single events and batches."""
    spec = synth.GridSpec(*grid, threshold=threshold)
    evs = [hits(30, n) for n in sizes]
    want = [oracle_run(spec, ev) for ev in evs]
    for n, ev, (M, c, v, k) in zip(sizes, evs, want):
        say(grid, "hits", n, "long", B.ht_debug_launch_plan(spec, [n])["long_lists"])
        acc, gc, gv, gk = B.fill_peaks(spec, *B.hits_to_device(*ev))
        assert np.array_equal(B.as_u32(acc), M) and gk == k and np.array_equal(gc, c) and np.array_equal(gv, v), n
    res = B.fill_peaks_batch(spec, evs)
    for i, (M, c, v, k) in enumerate(want):
        assert np.array_equal(B.as_u32(res.acc[i]), M), i
        assert res.peaks[i][2] == k and np.array_equal(res.peaks[i][0], c) and np.array_equal(res.peaks[i][1], v), i


@pytest.mark.parametrize("shape,threshold,sizes", [((1, 3, 16, 16), 2, (0, 1, 40, 400)), ((1, 3, 64, 256), 2, (300, 700)),
                                                   ((2, 3, 300, 33), 3, (200, 2000)), ((4, 16, 64, 64), 2, (30, 33, 900)),
                                                   ((1, 4, 20, 1), 1, (1, 3, 4, 60)), ((2, 3, 64, 64), 32, (255, 1024, 1025))])
def test_survivor_lists_of_every_size(B, monkeypatch, shape, threshold, sizes):
    """Lists as short as their event: one that holds every survivor of few cells, eight that overflow,
    and events of either kind in one batch and one request loop."""
    import time
    spec = synth.GridSpec(*shape, threshold=threshold)
    evs = []
    for n in sizes:
        ev = synth.make_hits(np.random.default_rng([40, n]), n // 14, n - 12 * (n // 14))
        x, y, z = (np.asarray(a[:n], np.float32).copy() for a in (ev.x, ev.y, ev.z))
        if n > 20:  # many hits alike: large counts
            x[n // 2:], y[n // 2:], z[n // 2:] = x[0], y[0], z[0]
        evs.append((x, y, z))
    want = [oracle_run(spec, ev) for ev in evs]

    def same(i, got, tag):
        M, c, v, k = want[i]
        assert got[2] == k and np.array_equal(got[0], c) and np.array_equal(got[1], v), (tag, sizes[i])
    B.ht_set_tuning(spec, dense_hits=-1)
    try:
        for i, ev in enumerate(evs):
            say(shape, "hits", sizes[i], B.ht_debug_launch_plan(spec, [sizes[i]]))
            acc, *got = B.fill_peaks(spec, *B.hits_to_device(*ev))
            assert np.array_equal(B.as_u32(acc), want[i][0]), sizes[i]
            same(i, got, "event")
            noalloc_equals_fill_peaks(B, spec, ev)
            same(i, B.peaks(spec, acc), "matrix")
        for k in range(4):
            monkeypatch.setenv("HT_BATCH_GRAPH", str(k % 2))
            for pick in ([i for i in range(len(evs))], [0, 0, 1]):
                res = B.fill_peaks_batch(spec, [evs[i] for i in pick])
                for j, i in enumerate(pick):
                    assert np.array_equal(B.as_u32(res.acc[j]), want[i][0])
                    same(i, res.peaks[j], "batch")
        with B.Server(spec, 64 << 20, peak_capacity=1 << 14, max_hits=max(sizes), max_batch=3, n_streams=2, queue_depth=16) as srv:
            for k in range(3):
                tickets = [(i, srv.submit(*evs[i])) for i in range(len(evs))]
                for i, t in tickets:
                    deadline = time.time() + 60
                    while (r := srv.poll(t)) is None:
                        assert time.time() < deadline
                        time.sleep(1e-4)
                    same(i, r, "served")
    finally:
        B.ht_set_tuning(spec)


def fused_equals_oracle(B, spec, ev, want=None):
    M, c, v, k = want or oracle_run(spec, ev)
    acc, gc, gv, gk = B.fill_peaks(spec, *B.hits_to_device(*ev))
    assert np.array_equal(B.as_u32(acc), M) and gk == k and np.array_equal(gc, c) and np.array_equal(gv, v)
    return M, k


def test_default_search_around_the_stencil_threshold(B):
    """The largest event that the paper grid searches from its survivors by default and the smallest
    that takes the stencil (40960 hits: 2.5 times the reported dense_hits)."""
    spec = synth.GridSpec(4, 16, 1024, 1024, threshold=9)
    x, y, z = hits(50, 40960)
    for n, stencil in ((40959, 0), (40960, 1)):
        assert B.ht_debug_launch_plan(spec, [n])["n_stencil"] == stencil
        say("paper grid, hits", n, "stencil", stencil)
        assert fused_equals_oracle(B, spec, (x[:n], y[:n], z[:n]))[1] > 100000


def test_fused_call_overflows_its_survivor_lists(B):
    """More survivors than the lists hold: those of every job of 4 rows and 256 columns, counted here,
    against a quarter of the votes' bound. The search falls back to the masks."""
    from oracle import oracle
    spec = synth.GridSpec(2, 3, 16, 1024, threshold=1, a_min=-20000.0, a_max=20000.0, b_min=-20000.0, b_max=20000.0)
    n = 300
    ev = synth.uniform_hits(np.random.default_rng(n), n, 1000.0, 2500.0)
    plan = B.ht_debug_launch_plan(spec, [n])
    assert plan["rows"] == 4 and plan["n_lists"] == 1 and not plan["few"] and not plan["long_lists"]
    M, _ = fused_equals_oracle(B, spec, ev)
    job = oracle.OracleGrid(*synth.GridSpec(1, 1, 4, 256, threshold=1, phi_sectors=True).as_tuple())
    blocks = M.reshape(6, 4, 4, 4, 256).swapaxes(2, 3).reshape(-1, 1, 1, 4, 256)
    survivors = sum(oracle.peaks(job, np.ascontiguousarray(b))[2] for b in blocks)
    say("survivors", survivors)
    assert survivors > n * 4 * spec.n_a // 4 > spec.n_cells // 32
    res = B.fill_peaks_batch(spec, [ev, ev])
    for got in res.peaks:
        assert got[2] == oracle_run(spec, ev)[3]


def test_fused_call_overflows_its_groups_segments(B):
    """One sector of one theta cell, where a peak is a maximum of its own plane: more peaks in a group
    of jobs than its segment holds (one per 64 cells), from survivor lists and from masks."""
    spec = synth.GridSpec(1, 1, 128, 256, threshold=2, phi_sectors=True)
    B.ht_set_tuning(spec, dense_hits=-1)
    try:
        for n, lists in ((170, 1), (700, 0)):
            ev = synth.uniform_hits(np.random.default_rng(n), n, 1000.0, 2500.0)
            assert B.ht_debug_launch_plan(spec, [n])["n_lists"] == lists
            _, k = fused_equals_oracle(B, spec, ev)
            say("hits", n, "peaks", k)
            assert k > 2 * spec.n_cells // 64
    finally:
        B.ht_set_tuning(spec)
