"""The library's host code (plans, buffers, fallbacks) over a device that
computes nothing: what each call asks the kernels for, and what it does when
memory ends.  Runs without a GPU."""
import numpy as np
import pytest

import hostapi
import hostcheck
import oracle as O
import workloads as W

ENOMEM, ECAPACITY, EINVAL = -2, -5, -1
ROT = W.random_rotations(1, seed=3)[0]


@pytest.fixture(scope="module")
def tess():
    import paper_1208_3206_amd as t
    return t


@pytest.fixture
def dev(tess):
    return hostapi.Device(tess)


# The slope bound of the crease form, the mean pixel value times 64 / width
# (times the mean density for rho^2): the one the host twin runs, whose error
# the oracle tests hold
@pytest.mark.parametrize("size", [(64, 64), (300, 77), (1024, 2048)])
@pytest.mark.parametrize("quantity", ["density", "density2", "unit"])
def test_steep_bound_is_the_host_twins(dev, size, quantity):
    lat = dev.build((32, 32, 32), total_mass=3.0)
    for view in (W.z_view(*size), W.rotated_view(ROT, *size)):
        view = dict(view, quantity=quantity)
        assert dev.project(lat, view) == 0, dev.error()
        div = size[0] / 64.0
        du, dv = view["extent"][0] / size[0], view["extent"][1] / size[1]
        if quantity == "unit":
            assert dev.log.bmax_per_q == pytest.approx(1.0 / (du * dv * size[0] * size[1]) / div, rel=1e-12)
        else:
            # all the mass in view, per pixel and pixel area; the mean density is 3
            mean = 3.0 / (du * dv) / (size[0] * size[1]) * (3.0 if quantity == "density2" else 1.0)
            assert dev.log.crease_bmax == pytest.approx(mean / div, rel=1e-12)


# Which images take the edge form by themselves: at the lines of the rule,
# periodic images and windows, lattices with and without periods; what is
# forced stays forced
FORMS = [
    # dims, periodic, view, quantity, edges
    ((64, 64, 64), True, W.z_view(95), "density", 0), ((64, 64, 64), True, W.z_view(97), "density", 1),
    ((64, 64, 64), True, W.z_view(97), "density2", 1), ((64, 64, 64), True, W.z_view(97), "unit", 1),
    ((101, 101, 102), True, W.z_view(80), "density", 0), ((102, 102, 102), True, W.z_view(80), "density", 1),
    ((128, 128, 128), True, W.z_view(100), "unit", 0), ((128, 128, 128), True, W.z_view(100), "density2", 0),
    ((64, 64, 64), True, W.rotated_view(ROT, 512), "density", 0),
    ((128, 128, 128), True, W.rotated_view(ROT, 160), "density", 0),
    ((32, 32, 32), True, W.rotated_view(ROT, 400, side=2.0), "density", 1),
    ((48, 48, 48), True, W.rotated_view(ROT, 300, side=2.0), "density2", 0),
    ((33, 33, 33), False, W.rotated_view(ROT, 383, side=2.0), "density", 0),
    ((33, 33, 33), False, W.rotated_view(ROT, 400, side=2.0), "density", 1),
]


@pytest.mark.parametrize("dims,periodic,view,quantity,edges", FORMS)
def test_automatic_form(dev, dims, periodic, view, quantity, edges):
    lat = dev.build(dims, periodic=periodic)
    view = dict(view, quantity=quantity)
    assert dev.project(lat, view) == 0 and dev.log.edges == edges
    assert dev.batch([lat], [view]) == 0 and dev.log.edges == edges
    bound = dev.log.crease_bmax
    for form, want in (("edges", 1), ("per_tetrahedron", 0)):
        assert dev.project(lat, view, form=form) == 0 and dev.log.edges == want
    # coarse images of large lattices: the tighter bound, where it is not forced
    coarse = edges and view["wrap"] and view["width"] < 1.5 * dims[0]
    assert dev.log.crease_bmax / bound == pytest.approx(32.0 if coarse else 1.0)


# ... whose FP64 sums are then no further from the exact image than the
# per-tetrahedron form's at its own bound: rms within a twentieth (the rms of
# ten lattices lies within 4 %), the largest error alike
@pytest.mark.parametrize("n,size,growth", [(64, (50, 50), 8.0), (64, (20, 20), 4.0), (80, (30, 110), 6.0)])
def test_coarse_images_are_as_exact_by_edges(n, size, growth):
    xyz = W.zeldovich(n, n // 4, growth, seed=3)
    view = W.z_view(*size)
    ref, _ = O.project_region(*xyz, (n, n, n), view)
    err = [hostcheck.pipeline(*xyz, (n, n, n), view, tile_rows=32, crease_div=size[0] / k, edges=e)[0] - ref
           for e, k in ((False, 64.0), (True, 2.0))]
    rms = [np.sqrt((e ** 2).mean()) for e in err]
    assert rms[1] <= 1.05 * rms[0]
    assert np.abs(err[1]).max() <= 1.05 * np.abs(err[0]).max()


# A caller's tile rows go with tiles up to 512 wide, on periodic images too:
# an image of the largest side in rows one high stays within the tile limit,
# and a tile too large for the LDS stays refused
def test_given_tile_rows_keep_wide_tiles(dev):
    lat = dev.build((8, 8, 8))
    for call in (dev.project, lambda lat, v, **t: dev.batch([lat], [v], **t), dev.noalloc):
        assert call(lat, W.z_view(512, 8200), tile_rows=1) == 0, dev.error()
        assert (dev.log.Th, dev.log.Tw) == (1, 512)
        assert call(lat, W.z_view(200), tile_rows=100) == EINVAL
    assert dev.project(lat, W.z_view(512, 16384), tile_rows=1) == 0, dev.error()
    assert dev.project(lat, W.z_view(512)) == 0 and (dev.log.Th, dev.log.Tw) == (32, 128)


# Payloads for own records at a shape's first call: one tetrahedron in 64 (and
# 65,536) where the edge form always was the automatic one, all for the coarse
# images; then from the count
@pytest.mark.parametrize("n,width,first", [(64, 97, 64), (128, 512, 64), (64, 380, 64), (32, 256, 64), (102, 80, 1)])
def test_first_guess_of_own_records(dev, n, width, first):
    lat, ntets = dev.build((n, n, n)), 6 * n ** 3
    guess = ntets if first == 1 else min(ntets, ntets // 64 + 65536)
    dev.counts(own=1000)
    for tune, want in ((dict(own_capacity=5000, form="edges"), 5000), ({}, guess), ({}, 1000 + 125 + 4096)):
        # (a stream has what its own calls have counted)
        assert dev.project(lat, W.z_view(width), stats=True, stream=2 if tune else 1, **tune) == 0, dev.error()
        assert dev.log.edges == 1 and dev.log.stored == want


# a workspace limit that held a periodic image of 4 pixels per cell with that
# guess (128^3 -> 512^2 in tiles of 32 x 512: 2,066,967,552 bytes)
def test_limit_of_a_periodic_image_at_four_pixels_per_cell(dev):
    lat = dev.build((128, 128, 128))
    assert dev.project(lat, W.z_view(512), tile_rows=32, chunk=12768, workspace_limit=2066967552) == 0, dev.error()


# Under a workspace limit a call takes the plan that needs least memory: limits
# (bytes) that hold these images, single and twice in a batch of 10^5 pairs a
# list, to the byte
SLAB = dict(W.z_view(200), slab=(-0.1, 0.2))
PERSP = W.perspective_view(np.eye(3), (0.5, 0.5, 0.05), 200, 200, extent=(2.0, 2.0))
LIMITS = [
    ((64, 64, 64), W.z_view(200), 270644072, 510970692), ((32, 32, 32), W.z_view(512), 47279532, 123605352),
    ((64, 64, 64), W.z_view(512), 272719732, 513637352), ((50, 50, 50), SLAB, 135431360, 135453876),
    ((50, 50, 50), dict(W.z_view(200), method="centroids"), 135431360, 135453876),
    ((50, 50, 50), PERSP, 135431360, 135453876), ((128, 128, 128), W.z_view(200), 2064376260, 3927094244),
    ((128, 128, 128), W.z_view(100), 2131035504, 2131118480),
    ((128, 128, 128), W.rotated_view(ROT, 512), 2133885664, 2138531980),
    ((97, 120, 75), W.z_view(1000, 707), 877422196, 1691801120), ((8, 8, 8), W.z_view(512, 16384), 81146456, 1987038632),
]


@pytest.mark.parametrize("dims,view,single,batch", LIMITS)
def test_workspace_limits_that_hold_a_call(tess, dims, view, single, batch):
    dev = hostapi.Device(tess)
    lat = dev.build(dims)
    base = dev.held()
    assert dev.project(lat, view, workspace_limit=single - (1 << 20)) == ENOMEM
    assert dev.held() == base  # (refused before anything is allocated)
    assert dev.project(lat, view, workspace_limit=single) == 0, dev.error()
    assert dev.held() <= base + single
    dev = hostapi.Device(tess)
    dev.counts(100000, 5000)
    lat = dev.build(dims)
    assert dev.batch([lat], [view] * 2, workspace_limit=batch) == 0, dev.error()


# ... and so do calls with a capacity of their own, whose pairs are counted in
# that plan's tiles and form
@pytest.mark.parametrize("tune", [dict(pair_capacity=10 ** 6), dict(own_capacity=10 ** 5)])
def test_given_capacities_keep_tiles_and_forms(dev, tune):
    lat = dev.build((128, 128, 128))
    assert dev.project(lat, W.z_view(100), **tune) == 0 and dev.log.edges == 0
    assert dev.project(lat, W.z_view(512), **tune) == 0 and (dev.log.Th, dev.log.Tw) == (32, 512)
    assert dev.project(lat, W.z_view(100)) == 0 and dev.log.edges == 1
    assert dev.project(lat, W.z_view(512)) == 0 and (dev.log.Th, dev.log.Tw) == (32, 128)


# When memory ends, a call that fits in its smaller plan is drawn by that, with
# nothing kept of the attempt: the budget here is what the smaller plan takes
def budget_of(tess, dims, call):
    """Bytes that a device holds after `call` of the smaller plan (the calls under a limit take it)."""
    dev = hostapi.Device(tess)
    dev.counts(1000, 500)
    lat = dev.build(dims)
    for _ in range(2):
        assert call(dev, lat, workspace_limit=1 << 50) == 0, dev.error()
    return dev.held()


SLABS = [dict(W.z_view(400), slab=(a, a + 0.02)) for a in np.linspace(-0.5, 0.48, 50)]


def test_slab_stack_without_memory_is_drawn_slab_by_slab(tess):
    def call(dev, lat, **tune):
        return dev.batch([lat], SLABS, **tune)
    budget = budget_of(tess, (48, 48, 48), call)
    dev = hostapi.Device(tess)
    dev.counts(1000, 500)
    lat = dev.build((48, 48, 48))
    assert call(dev, lat) == 0 and dev.log.stack_setups > 0 and dev.held() > budget
    dev = hostapi.Device(tess)
    dev.counts(1000, 500)
    lat = dev.build((48, 48, 48))
    dev.budget(budget + 4096)
    for k in range(3):
        dev.reset()
        assert call(dev, lat) == 0, dev.error()
        assert dev.lib.fake_last_error() == 0 and dev.held() <= budget + 4096
        # (later calls replay the graph)
        assert dev.log.stack_setups == 0 and dev.log.graph_launches == 1
        assert k == 0 or dev.log.mallocs == dev.log.frees == dev.log.failed_mallocs == 0


def test_coarse_image_without_memory_is_drawn_per_tetrahedron(tess):
    def call(dev, lat, **tune):
        return dev.project(lat, W.z_view(100), **tune)
    dims = (128, 128, 128)
    budget = budget_of(tess, dims, call)
    dev = hostapi.Device(tess)
    dev.counts(1000, 500)
    lat = dev.build(dims)
    dev.budget(budget + 4096)
    for k in range(3):
        dev.reset()
        dev.capturing(k == 2)
        assert call(dev, lat) == 0, dev.error()
        assert dev.log.edges == 0 and dev.lib.fake_last_error() == 0 and dev.held() <= budget + 4096
        assert k == 0 or dev.log.mallocs == dev.log.frees == dev.log.failed_mallocs == dev.log.illegal == 0


# ... a batch too, whichever of its views is the coarse one, and the views that
# are finer keep the edge form
@pytest.mark.parametrize("order", [(0, 1), (1, 0), (2, 1), (1,)])
def test_coarse_batch_without_memory(tess, order):
    dims, box = (128, 128, 128), (1.0, 1.0, 4.0)
    eye = np.eye(3)
    # 2.5 and 1.2 pixels per cell of the periodic images, a window
    kinds = [dict(W.z_view(200), center=(0.5, 0.5, 2.0)),
             dict(W.z_view(200), rot=eye[[2, 0, 1]].ravel().tolist(), center=(0.5, 0.5, 2.0), extent=(4.0, 1.0)),
             W.rotated_view(ROT, 200)]
    views = [kinds[k] for k in order]

    def run(budget=None, **tune):
        dev = hostapi.Device(tess)
        dev.counts(1000, 500)
        lat = dev.build(dims, box=box)
        if budget:
            dev.budget(budget)
        for _ in range(2):
            assert dev.batch([lat], views, **tune) == 0, dev.error()
        return dev
    lean, free = run(workspace_limit=1 << 50), run()
    assert free.log.edge_setups > lean.log.edge_setups
    tight = run(budget=lean.held() + 4096)
    assert tight.lib.fake_last_error() == 0 and tight.held() <= lean.held() + 4096
    if 0 not in order:
        assert free.held() > lean.held() and tight.log.failed_mallocs > 0
        assert tight.log.edges == 0


# A call refused for want of memory leaves nothing for the next one to report
def test_refused_call_does_not_fail_the_next(dev):
    lat = dev.build((64, 64, 64))
    dev.budget(dev.held() + (1 << 20))
    for call in (lambda: dev.project(lat, W.z_view(512)), lambda: dev.batch([lat], [W.z_view(512)])):
        assert call() == ENOMEM
        assert dev.lib.fake_last_error() == 0
    dev.budget()
    assert dev.project(lat, W.z_view(512)) == 0, dev.error()


# A limit holds after calls without one too, whose plan may have taken more:
# what it made larger is given back (but not under capture)
@pytest.mark.parametrize("dims,view,single,batch", LIMITS)
def test_workspace_limit_after_a_call_without(tess, dims, view, single, batch):
    dev = hostapi.Device(tess)
    lat = dev.build(dims)
    base = dev.held()
    assert dev.project(lat, view) == 0
    over = dev.held() > base + single + 4096
    dev.capturing(1)
    assert dev.project(lat, view, workspace_limit=single + 4096) == (ENOMEM if over else 0)
    assert dev.log.illegal == 0
    dev.capturing(0)
    for _ in range(2):
        assert dev.project(lat, view, workspace_limit=single + 4096) == 0, dev.error()
    assert dev.held() <= base + single + 4096


# The allocation-free projection refuses what does not fit its scratch in the
# automatic form, and keeps wide tiles, of fewer pairs, where these take all
# the room that is left
@pytest.mark.parametrize("n,width,rc,tile", [
    (32, 256, 0, (32, 128)), (40, 320, 0, (32, 128)), (43, 344, 0, (32, 344)), (44, 352, 0, (32, 352)),
    (50, 200, ECAPACITY, None), (48, 400, ECAPACITY, None), (50, 64, 0, (32, 64)), (52, 60, 0, (64, 60))])
def test_allocation_free_plans(dev, n, width, rc, tile):
    lat = dev.build((n, n, n))
    assert dev.noalloc(lat, W.z_view(width)) == rc
    if tile:
        assert (dev.log.Th, dev.log.Tw) == tile
        assert dev.log.edges == (1 if width >= 1.5 * n else 0)


# Plans read from a tune cache file: room for own records as the call asks, or
# the first guess for any of the batch's views
def test_cached_plan_has_room_for_own_records(tess, tmp_path, monkeypatch):
    monkeypatch.setenv("TESS_TUNE_CACHE", str(tmp_path / "tune.json"))
    n, ntets = 128, 6 * 128 ** 3
    window, coarse, fine = W.rotated_view(ROT, 100), W.z_view(100), dict(W.z_view(100), quantity="unit")
    cases = [((64,) * 3, [W.z_view(128)] * 2, {}, 6 * 64 ** 3 // 64 + 65536),
             ((64,) * 3, [W.z_view(128)] * 2, dict(own_capacity=7000), 7000),
             ((n,) * 3, [window, coarse], {}, ntets), ((n,) * 3, [coarse, fine], {}, ntets)]
    for first in (True, False):  # tuned and saved, then read by another process
        for dims, views, tune, room in cases:
            dev = hostapi.Device(tess)
            dev.counts(1000, 500)
            lat = dev.build(dims)
            assert dev.batch([lat], views, **tune) == 0, dev.error()
            if not first:
                assert dev.log.rasters == len(views)  # (no tuning)
                assert dev.log.edge_setups == len([v for v in views if v is not window and v is not fine])
                assert dev.log.own_room == room


# A batch's graphs, with and without the fragment count, are both kept: calls
# that ask for statistics now and then capture neither again
def test_batches_with_and_without_stats_keep_their_graphs(dev):
    lat = dev.build((32, 32, 32))
    views = [W.z_view(128)] * 3
    for k in range(6):
        assert dev.batch([lat], views, stats=k % 2 == 1) == 0, dev.error()
        if k == 2:  # (the first counts settle the capacities)
            dev.reset()
    assert dev.log.graphs == 0 and dev.log.graph_launches == 3
    assert dev.batch([lat], views[:2]) == 0 and dev.log.graphs == 1


# Work items of a window: 512 entries at least, then about 200 items of up to
# 1,024, then what fills the chip
@pytest.mark.parametrize("pairs,chunk", [(1000, 512), (102000, 512), (160000, 800), (220000, 1024), (500000, 1024),
                                         (2400000, 4096), (40000000, 9765)])
def test_work_items_of_windows(dev, pairs, chunk):
    lat = dev.build((32, 32, 32))
    dev.counts(pairs)
    for _ in range(2):  # one tile; the second call knows its pairs
        assert dev.project(lat, W.rotated_view(ROT, 100, 64), stats=True) == 0
    assert dev.log.Th == 64 and dev.log.chunk == chunk
