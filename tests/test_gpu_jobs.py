"""The survivor search (the fill's and the scan's jobs, the peak test from lists and from masks, the
ordered writer) where it can go wrong: rows of every width around the job sizes, tiles of every
height, lists and group segments that overflow, counts up to 2^32 - 1, and the no-alloc call's
slice-by-slice search. Against the CPU oracle, bit for bit."""
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


def oracle_peaks(spec, M):
    from oracle import oracle
    return oracle.peaks(oracle.OracleGrid(*spec.as_tuple()), M)


def same_peaks(spec, got, M, tag):
    oc, ov, on = oracle_peaks(spec, M)
    c, v, n = got
    assert n == on, (tag, n, on)
    assert np.array_equal(c, oc) and np.array_equal(v, ov), tag


# widths around a unit (4), half a wave of units (128), a wave of units (256), and ragged ones
@pytest.mark.parametrize("n_b", [1, 2, 3, 5, 16, 31, 64, 100, 127, 128, 129, 255, 257, 512, 1030])
@pytest.mark.parametrize("n_hits", [30, 900])  # one record per lane at most, and longer lists
def test_every_job_shape_bit_exact(B, n_b, n_hits):
    import torch
    from oracle import oracle
    rng = np.random.default_rng([n_b, n_hits])
    ev = synth.make_hits(rng, n_hits // 15, n_hits - 12 * (n_hits // 15))
    spec = synth.GridSpec(2, 3, 70, n_b, threshold=2)
    M, _ = oracle.fill(oracle.OracleGrid(*spec.as_tuple()), ev.x, ev.y, ev.z)
    x, y, z = B.hits_to_device(ev.x, ev.y, ev.z)
    for rows in (1, 2, 4, 8, 16, 32, 64):
        if 4 * rows * n_b > 56 * 1024:
            continue
        say("n_b", n_b, "hits", n_hits, "rows", rows)
        B.ht_set_tuning(spec, rows=rows, dense_hits=-1)
        try:
            acc, c, v, n = B.fill_peaks(spec, x, y, z)
            torch.cuda.synchronize()
        finally:
            B.ht_set_tuning(spec)
        assert np.array_equal(B.as_u32(acc), M), rows
        same_peaks(spec, (c, v, n), M, "rows %d" % rows)
    c, v, n = B.peaks(spec, torch.from_numpy(M.view(np.int32).copy()).cuda())
    same_peaks(spec, (c, v, n), M, "peaks of a matrix")


@pytest.mark.parametrize("shape", [(1, 3, 64, 256), (2, 3, 512, 1024), (1, 3, 40, 33), (1, 3, 3, 17000)])
def test_crowded_matrices_overflow_lists_and_segments(B, shape):
    """A peak on every other row and column of one slab: more than any group's segment holds, and on
    the larger grids more survivors than the lists hold."""
    import torch
    rng = np.random.default_rng(shape)
    M = np.zeros(shape, np.uint32)
    M[0, 0, ::2, ::2] = rng.integers(1, 4, M[0, 0, ::2, ::2].shape)
    M[0, 1] = rng.integers(0, 2, M[0, 1].shape)
    M[0, 0, 0, 0] = 0xffffffff
    M[0, 0, 0, 1] = 0xffffffff  # a tie at the largest count: the lower cell wins
    for T in (1, 2, 0xffffffff):
        say("crowded matrix", shape, T)
        spec = synth.GridSpec(*shape, threshold=T)
        got = B.peaks(spec, torch.from_numpy(M.view(np.int32).copy()).cuda())
        same_peaks(spec, got, M, (shape, T))
        n = got[2]
        if n > 3:  # truncated inside a group
            c, v, m = B.peaks(spec, torch.from_numpy(M.view(np.int32).copy()).cuda(), capacity=n // 2,
                              allow_truncation=True)
            assert m == n and np.array_equal(c, got[0][:n // 2]) and np.array_equal(v, got[1][:n // 2])


def test_noalloc_searches_in_slices(B):
    """A grid whose masks pass the fixed scratch, admitted because its candidate list is set small:
    the same matrix and peaks as ht_fill_peaks, twice in a row."""
    import torch
    spec = synth.GridSpec(4, 16, 2048, 2048, threshold=9)
    ev = synth.make_event(1, 3)
    x, y, z = B.hits_to_device(ev.x, ev.y, ev.z)
    B.ht_set_tuning(spec, cand_cap=2)
    try:
        ref = B.new_acc(spec)
        ref, c, v, n = B.fill_peaks(spec, x, y, z, acc=ref)
        assert n > 100
        acc = B.new_acc(spec)
        for k in range(2):
            say("sliced no-alloc search", k)
            out, nf = B.new_peaks(1 << 16)
            acc.fill_(7)
            B.ht_fill_peaks_noalloc(spec, x, y, z, acc, out, 1 << 16, nf)
            c2, v2, n2 = B.peaks_to_host(out, nf, 1 << 16)
            assert n2 == n and np.array_equal(c2, c) and np.array_equal(v2, v)
            assert torch.equal(acc, ref)
    finally:
        B.ht_set_tuning(spec)


@pytest.mark.parametrize("ranges", [(-2000.0, 2000.0), (-1e18, 1e18), (-3e38, 3e38), (0.0, 1.5e-45), (-1e-30, 3e-30)])
@pytest.mark.parametrize("rows", [2, 8])
def test_long_lists_with_extreme_hits_bit_exact(B, ranges, rows):
    """Votes that overflow, vanish or would be NaN (1/(2y) infinite, A x infinite, an infinite bin
    scale) through the long-list fill, and on grids that it leaves to the other one."""
    import torch
    from oracle import oracle
    lo, hi = ranges
    spec = synth.GridSpec(1, 3, 21, 64, a_min=lo, a_max=hi, b_min=lo, b_max=hi, threshold=2)
    rng = np.random.default_rng(7)
    n = 3000  # three slabs: more than the 512 records each that make a long list
    scale = rng.choice([1.0, 1e3, 1e-3, 1e18, 1e-18, 1e-25, 3e-39, 1e-42], (2, n))
    x, y = (rng.uniform(-1, 1, (2, n)) * scale).astype(np.float32)
    x[::17] = 0.0
    z = rng.uniform(-2000, 2000, n).astype(np.float32)
    say("ranges", ranges, "rows", rows)
    M, _ = oracle.fill(oracle.OracleGrid(*spec.as_tuple()), x, y, z)
    B.ht_set_tuning(spec, rows=rows, dense_hits=-1)
    try:
        acc, c, v, k = B.fill_peaks(spec, *B.hits_to_device(x, y, z))
        torch.cuda.synchronize()
    finally:
        B.ht_set_tuning(spec)
    assert np.array_equal(B.as_u32(acc), M)
    same_peaks(spec, (c, v, k), M, ranges)


@pytest.mark.parametrize("n_b", [33, 66, 131, 333, 1030])
def test_long_lists_with_ragged_rows(B, n_b):
    """Votes outside the row of the long-list fill are counted in words past it: with rows that are
    not whole units of four columns, none of these is a cell of the survivor search."""
    import torch
    from oracle import oracle
    rng = np.random.default_rng(n_b)
    spec = synth.GridSpec(1, 3, 21, n_b, b_min=-300.0, b_max=300.0, threshold=4)  # many votes outside
    for n in (520, 1500, 4000):
        say("n_b", n_b, "hits", n)
        ev = synth.make_hits(rng, n // 14, n - 12 * (n // 14))
        M, _ = oracle.fill(oracle.OracleGrid(*spec.as_tuple()), ev.x, ev.y, ev.z)
        x, y, z = B.hits_to_device(ev.x, ev.y, ev.z)
        for rows in (1, 4, 8):
            B.ht_set_tuning(spec, rows=rows, dense_hits=-1)
            try:
                acc, c, v, found = B.fill_peaks(spec, x, y, z)
                torch.cuda.synchronize()
            finally:
                B.ht_set_tuning(spec)
            assert np.array_equal(B.as_u32(acc), M), rows
            same_peaks(spec, (c, v, found), M, "rows %d" % rows)


# (cells per axis, threshold) on either side of the two-launch rule's bounds: hits up to 1024, and
# hits * cells per hit * n_a / threshold up to 8192; rows of a unit and less, and past a wave's units
@pytest.mark.parametrize("n_a,n_b,threshold", [(64, 64, 32), (64, 64, 31), (64, 1, 40), (63, 2, 40), (33, 3, 17),
                                               (20, 5, 10), (64, 33, 33), (40, 300, 20), (5, 1030, 3), (4, 16, 1)])
@pytest.mark.parametrize("sectors", [False, True])
def test_tiny_events_in_two_launches(B, monkeypatch, n_a, n_b, threshold, sectors):
    import torch
    from oracle import oracle
    rng = np.random.default_rng([n_a, n_b, threshold, sectors])
    spec = synth.GridSpec(2, 3, n_a, n_b, threshold=threshold, phi_sectors=sectors)
    og = oracle.OracleGrid(*spec.as_tuple())
    evs, want = [], []
    for n in (0, 1, 63, 257, 512, 1023, 1024, 1025):
        say("hits", n)
        ev = synth.make_hits(rng, n // 14, n - 12 * (n // 14))
        x, y, z = (np.array(a[:n], dtype=np.float32) for a in (ev.x, ev.y, ev.z))
        if n > 60:  # many alike (their cells hold large counts), refused ones and extremes among the others
            x[n // 3:], y[n // 3:], z[n // 3:] = x[0], y[0], z[0]
            x[1], y[2], z[3], y[4], y[5] = np.nan, 0.0, np.inf, 1e-40, -1e-30
        M, _ = oracle.fill(og, x, y, z)
        evs.append((x, y, z))
        want.append(M)
        dev = B.hits_to_device(x, y, z)
        acc, c, v, found = B.fill_peaks(spec, *dev)
        torch.cuda.synchronize()
        assert np.array_equal(B.as_u32(acc), M), n
        same_peaks(spec, (c, v, found), M, "hits %d" % n)
        if found > 1:  # a short list: its first peaks and the full count
            acc, c2, v2, found2 = B.fill_peaks(spec, *dev, capacity=found - 1, allow_truncation=True)
            assert found2 == found and np.array_equal(c2, c[:-1]) and np.array_equal(v2, v[:-1]), n
    for evs, want in ((evs[:-1], want[:-1]), (evs, want)):
        for k in range(6):  # by turns launched and as a captured graph, replayed
            monkeypatch.setenv("HT_BATCH_GRAPH", str(k % 2))
            res = B.fill_peaks_batch(spec, evs)
            for i, M in enumerate(want):
                assert np.array_equal(B.as_u32(res.acc[i]), M), (k, i)
                same_peaks(spec, res.peaks[i], M, "event %d" % i)


@pytest.mark.parametrize("shape", [(3, 11, 96, 260), (1, 3, 7, 2000), (8, 32, 40, 64), (2, 3, 300, 33), (5, 1, 64, 1030)])
def test_mask_groups_are_all_searched(B, shape):
    """Every group of the mask search is taken by exactly one workgroup, whatever the number of
    slabs and groups, in single events and batches."""
    import torch
    from oracle import oracle
    rng = np.random.default_rng(shape)
    spec = synth.GridSpec(*shape, threshold=3, phi_sectors=shape[1] < 3)
    og = oracle.OracleGrid(*spec.as_tuple())
    evs, want = [], []
    for n in (20000, 21000, 700):
        ev = synth.make_hits(rng, n // 14, n - 12 * (n // 14))
        evs.append((ev.x, ev.y, ev.z))
        want.append(oracle.fill(og, *evs[-1])[0])
    B.ht_set_tuning(spec, rows=4, dense_hits=-1)
    try:
        for events in (evs, evs * 4):
            say(shape, "events", len(events))
            res = B.fill_peaks_batch(spec, events)
            for i in range(len(events)):
                assert np.array_equal(B.as_u32(res.acc[i]), want[i % 3]), i
                same_peaks(spec, res.peaks[i], want[i % 3], "event %d" % i)
        for h, M in zip(evs, want):
            acc, c, v, n = B.fill_peaks(spec, *B.hits_to_device(*h))
            same_peaks(spec, (c, v, n), M, "one event")
    finally:
        B.ht_set_tuning(spec)


def test_short_lists_with_masks_only(B):
    """Batches whose survivors are many in a job and in all are searched from masks, though the fill
    is the short-list one; with events of few hits, and each event alone, from the lists."""
    from oracle import oracle
    rng = np.random.default_rng(17)
    spec = synth.GridSpec(4, 16, 256, 256, threshold=8)
    og = oracle.OracleGrid(*spec.as_tuple())
    evs = []
    for n in (6585, 300, 5000):
        ev = synth.make_hits(rng, n // 14, n - 12 * (n // 14))
        evs.append((ev.x, ev.y, ev.z))
    want = [oracle.fill(og, *h)[0] for h in evs]
    B.ht_set_tuning(spec, dense_hits=-1)
    try:
        for pick in ([0, 1, 2], [1, 2]):
            say("events", pick)
            res = B.fill_peaks_batch(spec, [evs[i] for i in pick])
            for k, i in enumerate(pick):
                assert np.array_equal(B.as_u32(res.acc[k]), want[i]), i
                same_peaks(spec, res.peaks[k], want[i], "event %d" % i)
        for h, M in zip(evs, want):
            say("one event of", len(h[0]))
            acc, c, v, n = B.fill_peaks(spec, *B.hits_to_device(*h))
            assert np.array_equal(B.as_u32(acc), M)
            same_peaks(spec, (c, v, n), M, "one event")
    finally:
        B.ht_set_tuning(spec)


@pytest.mark.parametrize("n_hits", [9000, 30000])  # survivors from lists, from masks
def test_counts_per_block_of_groups(B, n_hits):
    """Past 8192 groups of jobs the ordered write takes its offsets from counts per 64 groups."""
    import torch
    from oracle import oracle
    rng = np.random.default_rng(n_hits)
    spec = synth.GridSpec(8, 32, 2100, 258, threshold=8)
    ev = synth.make_hits(rng, n_hits // 14, n_hits - 12 * (n_hits // 14))
    M, _ = oracle.fill(oracle.OracleGrid(*spec.as_tuple()), ev.x, ev.y, ev.z)
    x, y, z = B.hits_to_device(ev.x, ev.y, ev.z)
    for k in range(2):
        say("hits", n_hits, "call", k)
        acc, c, v, n = B.fill_peaks(spec, x, y, z)
        same_peaks(spec, (c, v, n), M, "fill_peaks")
        same_peaks(spec, B.peaks(spec, acc), M, "peaks of the matrix")


def test_large_batches_of_narrow_rows_and_mixed_searches(B):
    """Many tiles of long lists on rows of 256 columns take 16 KiB tiles; a batch with a crowded event
    searches those of its events with the stencil that reach the reported threshold (2048 hits)."""
    from oracle import oracle
    rng = np.random.default_rng(23)
    spec = synth.GridSpec(4, 8, 256, 256)
    og = oracle.OracleGrid(*spec.as_tuple())
    evs = []
    for n in (8000, 5000, 3000, 300):
        ev = synth.make_hits(rng, n // 14, n - 12 * (n // 14))
        evs.append((ev.x, ev.y, ev.z))
    want = [oracle.fill(og, *h)[0] for h in evs]
    for pick in ([0, 1, 2, 3] * 4, [2, 3] * 8, [0, 3]):
        say("events", len(pick))
        res = B.fill_peaks_batch(spec, [evs[i] for i in pick])
        for k, i in enumerate(pick):
            assert np.array_equal(B.as_u32(res.acc[k]), want[i]), (k, i)
            same_peaks(spec, res.peaks[k], want[i], "event %d" % i)
