"""What the calls would launch (ht_debug_launch_plan, decided on the host with the calls' own code):
the no-alloc call's limit, launch shapes that are read and set back, and batches whose launches are
chosen by their own events. No GPU needed."""
import pytest

from paper_1507_03074_amd import binding as B
from paper_1507_03074_amd import synth


@pytest.fixture(scope="module")
def lib():
    from paper_1507_03074_amd import build as hbuild
    hbuild.ensure_built()  # a missing or stale library is rebuilt, never tested
    return B.lib()


def al(v):
    return -(-v // 256) * 256


def noalloc_limit(spec, n):
    """Bytes that the documented size rule of ht_fill_peaks_noalloc counts for an event of n hits:
    slab lists (direct where that keeps within the limit), 16 bytes per tile, and the stencil's peak
    words from the reported dense_hits on, else nine bytes per candidate."""
    tl, tu = B.ht_tiling(spec), B.ht_get_tuning(spec)
    slabs, tiles = spec.n_theta * spec.n_phi, tl["n_tiles"]
    fixed = al(4 * (slabs + 1)) + 4 * al(4 * tiles) + al(4 * -(-tiles // tu.group_tiles))
    if tl["lds_fill"] and 0 < tu.dense_hits <= n:
        chunks = -(-spec.n_b // 62)
        rows = -(-spec.n_a // max(1, 512 // chunks))
        rows = max(12, -(-rows // 12) * 12)
        fixed += al(8 * slabs * -(-spec.n_a // rows) * rows * chunks)
    else:
        bound = n * (2 if spec.phi_sectors else 4) * spec.n_a // spec.threshold
        pool = max(tiles * tl["cand_cap"], min(spec.n_cells, bound // 4))
        fixed += al(8 * pool) + al(pool)
    direct = fixed + al(16 * slabs * max(n, 1))
    packed = fixed + 3 * al(16 * n) + al(64 * n + 16)
    return direct if tl["lds_fill"] and 16 * slabs * max(n, 1) <= 1 << 29 and direct <= ROOM else packed


ROOM = (64 << 20) - 295424
GRIDS = [(4, 16, 1024, 1024), (4, 16, 2048, 512), (2, 8, 1024, 1024), (4, 16, 512, 512), (4, 16, 64, 64),
         (1, 3, 16, 16), (3, 7, 501, 333), (4, 16, 2048, 2048), (8, 32, 256, 256), (2, 3, 40, 20000), (1, 3, 2000, 5000)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("sectors", [False, True])
def test_noalloc_accepts_what_its_limit_holds(lib, grid, sectors):
    """Accepted exactly where the documented arithmetic fits, crowded events of low thresholds among
    them, with a layout that fits the array."""
    taken = refused = 0
    for T in (1, 2, 3, 4, 5, 9, 30):
        spec = synth.GridSpec(*grid, threshold=T, phi_sectors=sectors)
        d = B.ht_get_tuning(spec).dense_hits
        sizes = {0, 1, 250, 5000, 16384, 24576, 31129, 39000, 39321, 60000, 400000, 590000, 600000}
        sizes |= {d - 1, d, 2 * d, 2 * d + 1, 5 * d // 2} if d > 0 else set()
        for n in sorted(sizes):
            try:
                plan = B.ht_debug_launch_plan(spec, [n], "noalloc")
            except B.HTError as ex:
                assert ex.code == B.HT_EINVAL and "bytes of scratch" in str(ex)
                plan = None
            assert (plan is not None) == (noalloc_limit(spec, n) <= ROOM), (T, n)
            taken, refused = taken + (plan is not None), refused + (plan is None)
            if plan:
                assert plan["scratch_bytes"] <= ROOM
    assert taken and (refused or grid == (8, 32, 256, 256) or spec.n_cells < 1 << 27)


def test_noalloc_takes_direct_lists_where_they_fit(lib):
    """The slab lists are direct while they and the search's own scratch fit, not what the size rule
    counts beside them."""
    for T in (1, 9):
        spec = synth.GridSpec(4, 16, 1024, 1024, threshold=T)
        for n, direct in ((5000, 1), (16384, 1), (33500, 1), (39000, 1), (64000, 0)):
            assert B.ht_debug_launch_plan(spec, [n], "noalloc")["direct"] == direct, (T, n)


def test_noalloc_slices_only_what_does_not_fit(lib):
    """Slices where the survivors' scratch passes the array, here by two thirds; never for an event
    that the size rule takes for a crowded one, which has the stencil."""
    spec = synth.GridSpec(2, 32, 4096, 2048, threshold=9)
    B.ht_set_tuning(spec, cand_cap=2)
    try:
        assert B.ht_debug_launch_plan(spec, [2500], "noalloc")["sliced"] == 1
        assert B.ht_debug_launch_plan(spec, [2500])["scratch_bytes"] > 5 * ROOM // 3
    finally:
        B.ht_set_tuning(spec)
    spec = synth.GridSpec(4, 16, 2048, 2048, threshold=1)
    assert B.ht_get_tuning(spec).dense_hits == 32768
    plan = B.ht_debug_launch_plan(spec, [40000], "noalloc")
    assert plan["sliced"] == 0 and plan["n_stencil"] == 1


def plans(spec):
    sizes = (0, 250, 1000, 3000, 5000, 12000, 22000, 41000)
    one = [B.ht_debug_launch_plan(spec, [n]) for n in sizes]
    return one + [B.ht_debug_launch_plan(spec, b, "batch") for b in ([250] * 100, [5000, 8000] * 50, list(sizes))]


@pytest.mark.parametrize("grid", [(4, 16, 1024, 1024), (4, 16, 256, 256), (3, 7, 501, 333), (8, 32, 512, 512), (4, 16, 64, 64)],
                         ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("fields", [{}, {"rows": 4}, {"nt_store": 1}, {"dense_hits": -1}, {"dense_hits": 900}, {"nt_store": 2, "rows": 2},
                                    {"tiles_per_block": 4, "group_tiles": 64}], ids=str)
def test_setting_the_reported_shape_changes_no_launch(lib, grid, fields):
    """ht_get_tuning, then ht_set_tuning of what it returned: the same launches for every event size,
    whether fields were set before or not."""
    spec = synth.GridSpec(*grid, threshold=9)
    try:
        B.ht_set_tuning(spec, **fields)
        before, shape = plans(spec), B.ht_get_tuning(spec)
        B.ht_set_tuning(spec, shape)
        assert plans(spec) == before
        assert B.ht_get_tuning(spec).as_dict() == shape.as_dict()
        B.ht_set_tuning(spec)
        unset = plans(spec)
        B.ht_set_tuning(spec, B.ht_get_tuning(spec))
        assert plans(spec) == unset
    finally:
        B.ht_set_tuning(spec)


def test_batches_are_searched_by_their_own_largest_event(lib):
    """The stencil's threshold, long or short lists and the tile height of a batch go by its largest
    event, not by a rounded number of hits; with one event from the stencil's threshold on (2.5 times
    the reported 16384, twice the reported 4096), all from the reported one on take it."""
    paper, small = synth.GridSpec(4, 16, 1024, 1024, threshold=9), synth.GridSpec(4, 16, 256, 256, threshold=8)

    def plan(spec, sizes, call="batch"):
        return B.ht_debug_launch_plan(spec, sizes, call)
    assert plan(paper, [33000, 30000, 20000, 5000])["n_stencil"] == 0
    assert plan(paper, [40959, 30000, 20000, 5000])["n_stencil"] == 0
    assert plan(paper, [40960, 30000, 16384, 16383])["n_stencil"] == 3
    assert plan(small, [4500, 4200, 4100, 300])["n_stencil"] == 0
    p = plan(small, [6585] * 7)
    assert p["n_stencil"] == 0 and p["n_lists"] == 0 and not p["long_lists"]  # masks of the short-list fill
    assert plan(small, [8191] * 7)["n_stencil"] == 0 and plan(small, [8192] + [4096] * 6)["n_stencil"] == 7
    for n in (8193, 9000, 10922):
        p = plan(paper, [n] * 8)
        assert not p["long_lists"] and p["rows"] == plan(paper, [n])["rows"] == 4, n
    assert plan(paper, [10923] * 8)["long_lists"]
    for spec, sizes in ((paper, [9000] * 8), (small, [3000] * 20), (paper, [42000, 20000])):
        assert plan(spec, sizes) == plan(spec, sizes[::-1])
    # a request loop's batches, whatever the largest event that it may get
    for max_hits, want in ((40000, 0), (41000, 0), (60000, 0)):
        assert plan(paper, [max_hits] + [20000] * 8, "serve")["n_stencil"] == want, max_hits
    assert plan(paper, [60000] + [20000] * 7 + [45000], "serve")["n_stencil"] == 8
    assert plan(paper, [60000, 20000], "serve")["n_stencil"] == 0


def test_low_thresholds_are_left_to_the_stencil_earlier(lib):
    """The hits from which the stencil takes an event, by threshold: the reported number up to four
    votes, 2 or 2.5 times it from seven or nine on; one vote per cell also keeps survivors off the
    lists."""
    for grid, d, steps in (((4, 16, 1024, 1024), 16384, {1: 1, 3: 1, 4: 1, 5: 4 / 3, 7: 2, 8: 7 / 3, 9: 2.5, 100: 2.5}),
                           ((4, 16, 256, 256), 4096, {1: 1, 4: 1, 5: 1, 6: 1.5, 7: 2, 8: 2, 100: 2}),
                           ((1, 3, 256, 256), 192, {1: 1, 5: 1, 8: 2})):
        for T, f in steps.items():
            spec = synth.GridSpec(*grid, threshold=T)
            assert B.ht_get_tuning(spec).dense_hits == d
            n = int(d * f)
            assert B.ht_debug_launch_plan(spec, [n - 1])["n_stencil"] == 0, (grid, T)
            assert B.ht_debug_launch_plan(spec, [n])["n_stencil"] == 1, (grid, T)
            B.ht_set_tuning(spec, dense_hits=d + 5)
            try:
                assert [B.ht_debug_launch_plan(spec, [k])["n_stencil"] for k in (d + 4, d + 5)] == [0, 1]
            finally:
                B.ht_set_tuning(spec)
    spec = synth.GridSpec(4, 16, 256, 256, threshold=1)
    assert [B.ht_debug_launch_plan(spec, [n])["n_lists"] for n in (8, 29, 30, 250)] == [1, 1, 0, 0]
    assert B.ht_debug_launch_plan(spec, [8] * 4, "batch")["n_lists"] == 0
    assert B.ht_debug_launch_plan(synth.GridSpec(4, 16, 256, 256, threshold=2), [250])["n_lists"] == 1


def test_one_workgroup_searches_few_cells_only(lib):
    """The one-workgroup search takes events that leave at most 8192 cells at the threshold, 4096 at
    two votes and 256 at one."""
    for (grid, T), sizes in ((((4, 16, 64, 64), 1), {1: 1, 2: 0, 32: 0}), (((4, 16, 64, 64), 2), {32: 1, 33: 0, 64: 0}),
                             (((4, 16, 64, 64), 3), {96: 1, 97: 0}), (((4, 16, 64, 64), 8), {250: 1, 256: 1, 257: 0}),
                             (((4, 16, 1024, 1024), 1), {1: 0, 2: 0}), (((2, 4, 16, 14336), 1), {4: 1, 5: 0, 128: 0})):
        for n, few in sizes.items():
            spec = synth.GridSpec(*grid, threshold=T)
            for plan in (B.ht_debug_launch_plan(spec, [n]), B.ht_debug_launch_plan(spec, [n] * 3, "batch")):
                assert plan["few"] == few and plan["tiny"] <= few, (grid, T, n)


def test_long_slab_lists_with_few_survivors_keep_the_survivor_lists(lib):
    """Events of a few slabs, of more than 512 records each, but with few survivors: the short-list fill
    and the search from lists, as for shorter ones; the long-list fill where survivors are many, at low
    thresholds sooner, and past six times that length."""
    for grid, T, sectors, sizes in (((2, 4, 256, 9000), 9, False, {1300: 0, 1392: 0, 2700: 0, 7200: 0, 8192: 0, 8193: 1}),
                                    ((2, 4, 256, 9000), 3, False, {1392: 0, 2048: 0, 3413: 1}),
                                    ((1, 3, 2000, 5000), 9, False, {522: 0, 2048: 0, 3000: 1}),
                                    ((4, 4, 1024, 1024), 9, True, {2785: 0, 3276: 0, 4000: 1, 5000: 1}),
                                    ((4, 16, 1024, 1024), 9, False, {10922: 0, 10923: 1, 14142: 1}),
                                    ((2, 4, 256, 9000), 1, False, {1300: 0, 1392: 1})):
        for n, long_l in sizes.items():
            spec = synth.GridSpec(*grid, threshold=T, phi_sectors=sectors)
            plan = B.ht_debug_launch_plan(spec, [n])
            assert plan["long_lists"] == long_l and plan["n_lists"] == (0 if long_l or T == 1 else 1), (grid, T, n)


def test_small_events_take_little_scratch(lib):
    """The survivor lists are as long as the event may need: the scratch of small events is mostly
    their slab lists, and large batches of them keep direct lists."""
    G = synth.GridSpec
    for grid, T, n, most in (((1, 3, 16, 16), 3, 40, 5 << 10), ((1, 3, 16, 16), 2, 400, 24 << 10), ((4, 16, 64, 64), 8, 250, 420 << 10),
                             ((4, 16, 64, 64), 8, 1000, 1200 << 10), ((4, 16, 1024, 1024), 9, 5000, 24 << 20)):
        spec = G(*grid, threshold=T)
        for call, sizes in (("event", [n]), ("batch", [n] * 50), ("serve", [n] * 9)):
            events = len(sizes) - (call == "serve")
            assert B.ht_debug_launch_plan(spec, sizes, call)["scratch_bytes"] <= events * (most + (12 << 10)), (grid, call)
    plan = B.ht_debug_launch_plan(G(1, 3, 16, 16, threshold=3), [40] * 65535, "batch")
    assert plan["direct"] and plan["scratch_bytes"] < 1 << 29
    assert B.ht_debug_launch_plan(G(4, 16, 64, 64, threshold=8), [250] * 20000, "batch")["direct"]


def test_launch_plan_validated_on_host(lib):
    spec = synth.WORKLOADS[0].grid
    for bad in ([], [-1], [5, 5], [1 << 29]):
        with pytest.raises(B.HTError) as ex:
            B.ht_debug_launch_plan(spec, bad)
        assert ex.value.code == B.HT_EINVAL
    with pytest.raises(B.HTError):
        B.ht_debug_launch_plan(synth.GridSpec(1, 3, 16385, 64), [5], "noalloc")
    assert B.ht_debug_launch_plan(synth.GridSpec(1, 3, 16385, 64), [5])["scratch_bytes"] > 0
