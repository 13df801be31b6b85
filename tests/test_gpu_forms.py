"""The form and the work items chosen for an image, against the general
per-tetrahedron form, over sizes where either could go wrong."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tess():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1208_3206_amd as t
    return t


def lattice(tess, n, growth, **kw):
    import torch
    if growth == 0.0:
        xyz = W.undisplaced(n)
    else:
        xyz = W.zeldovich(n, min(4, (n - 1) // 2), growth, seed=17)
    return tess.build(*[torch.from_numpy(a).cuda() for a in xyz], (n, n, n), **kw)


def same(a, b):
    # FP64 sums of the same terms in another order (4e-11 of the maximum
    # between the forms), rounded once to FP32
    a, b = a.double(), b.double()
    return bool(((a - b).abs() <= 1.2e-7 * b.abs() + 1e-10 * b.max()).all())


# periodic images from a pixel for many cells to many pixels a cell: one
# pixel, a row, tetrahedra wider than the image, most of them steep (own
# records), undisplaced walls; one tile and several
@pytest.mark.parametrize("n,size,growth,quantity", [
    (8, (1, 1), 3.0, "density"), (9, (17, 1), 2.0, "density"), (24, (7, 5), 8.0, "density"),
    (33, (16, 16), 0.5, "density"), (40, (61, 33), 0.2, "unit"), (64, (100, 75), 6.0, "density2"),
    (12, (40, 24), 0.0, "density"), (48, (600, 70), 1.0, "density"), (100, (150, 150), 0.3, "density")])
def test_periodic_image_equals_the_per_tetrahedron_form(tess, n, size, growth, quantity):
    lat = lattice(tess, n, growth)
    view = dict(W.z_view(*size), quantity=quantity)
    for _ in range(2):  # first guesses of the capacities, then learned ones
        auto, st = tess.project(lat, view, stats=True)
        ref, sr = tess.project(lat, view, tune=tess.make_tune(form="per_tetrahedron"), stats=True)
        assert same(auto, ref)
        assert same(tess.project(lat, view), ref)
        for k in ("tets", "zero_volume", "inverted", "fp64_dets"):
            assert st[k] == sr[k], k
        assert abs(st["fragments"] - sr["fragments"]) <= 1e-6 * sr["fragments"] + 8


# entries per work item: fewer than a lane each, one wavefront's, not a
# multiple of anything, more than every list
@pytest.mark.parametrize("form", ["edges", "per_tetrahedron"])
@pytest.mark.parametrize("chunk", [64, 1000, 7177, 10 ** 6])
def test_work_item_sizes(tess, form, chunk):
    lat = lattice(tess, 40, 3.0)
    view = W.z_view(333, 150)
    ref = tess.project(lat, view, tune=tess.make_tune(form=form))
    img, st = tess.project(lat, view, tune=tess.make_tune(form=form, chunk=chunk), stats=True)
    assert same(img, ref) and st["overflow"] == 0


def test_noalloc_keeps_its_largest_lattice(tess):
    # 50^3 does not fit the allocation-free scratch in the edge form
    import torch
    lat = lattice(tess, 50, 1.0)
    view = W.z_view(64)
    out = torch.empty((64, 64), device="cuda")
    tess.project_noalloc(lat, view, out)
    assert same(out, tess.project(lat, view, tune=tess.make_tune(form="per_tetrahedron")))


# An image's scratch is cleared in one launch, ranges of very different
# lengths together: an image drawn after a larger one, periodic and a window
# of it, is the per-tetrahedron form's, with its counts
@pytest.mark.parametrize("quantity", ["density", "unit"])
@pytest.mark.parametrize("n,size", [(2, (1, 1)), (5, (33, 17)), (16, (64, 200))])
def test_nothing_is_left_of_the_image_before(tess, n, size, quantity):
    big, lat = lattice(tess, 32, 4.0), lattice(tess, n, 0.0 if n == 2 else 1.0)
    view = dict(W.z_view(*size), quantity=quantity)
    large = dict(W.z_view(256, 256), quantity=quantity)
    for tune in (tess.make_tune(form="edges"), tess.make_tune(form="per_tetrahedron")):
        tess.project(big, large, tune=tune)
        img, st = tess.project(lat, view, tune=tune, stats=True)
        tess.project(big, large)
        ref, sr = tess.project(lat, view, tune=tune, stats=True)
        assert same(img, ref)
        assert (st["tets"], st["zero_volume"]) == (sr["tets"], sr["zero_volume"])
        assert st["tets"] + st["zero_volume"] <= 6 * n ** 3 and st["fragments"] > 0


# The lists' prefix sum over (tiles x segments) counts: within one block of
# 4096, over a few, over more blocks than a block has threads (4.2 million)
@pytest.mark.parametrize("n,size,tiles", [
    (8, (64, 64), (32, 32)), (24, (250, 130), (8, 16)), (64, (1000, 900), (4, 16))])
def test_prefix_sum_sizes(tess, n, size, tiles):
    lat = lattice(tess, n, 1.0)
    view = W.z_view(*size)
    kw = dict(form="per_tetrahedron")
    ref, sr = tess.project(lat, view, tune=tess.make_tune(**kw), stats=True)
    kw.update(tile_rows=tiles[0], tile_cols=tiles[1])
    tess.project(lat, view, tune=tess.make_tune(**kw), stats=True)  # (a first guess of the pairs may overflow)
    img, st = tess.project(lat, view, tune=tess.make_tune(**kw), stats=True)
    assert same(img, ref)
    # (a pixel that a footprint's edge touches may fall either way at another tile's seam)
    assert abs(st["fragments"] - sr["fragments"]) <= 1e-6 * sr["fragments"] + 8
    assert st["overflow"] == 0


# Most tetrahedra of a strongly displaced window keep their own records (more
# than the first guess): a batch of a new shape has counted them before it
# draws.
def test_first_batch_of_a_window_has_room_for_its_own_records(tess):
    import torch
    lat = tess.build(*[torch.from_numpy(a).cuda() for a in W.zeldovich(64, 16, 8.0)], (64, 64, 64))
    views = [W.rotated_view(r, 203) for r in W.random_rotations(2, 1)]
    img, st = tess.project_batch([lat], views, stats=True)
    assert st["overflow"] == 0
    for i, v in enumerate(views):
        assert same(img[0, i], tess.project(lat, v, tune=tess.make_tune(form="per_tetrahedron")))


# A workspace limit that the per-tetrahedron form meets is met by the
# automatic form of a coarse image too, single and in a batch
@pytest.mark.parametrize("batch", [False, True])
def test_coarse_windows_fit_the_limits_of_the_per_tetrahedron_form(tess, batch):
    import torch
    lat = lattice(tess, 24, 2.0)
    view = W.rotated_view(W.random_rotations(1, 1)[0], 64)
    ref = tess.project(lat, view, tune=tess.make_tune(form="per_tetrahedron"))

    def drawn(form, limit):
        with torch.cuda.stream(torch.cuda.Stream()):  # (a workspace of its own)
            tune = tess.make_tune(form=form, workspace_limit=limit)
            try:
                img = tess.project_batch([lat], [view], tune=tune)[0, 0] if batch else tess.project(lat, view, tune=tune)
            except tess.TessError as e:
                assert e.status == -2
                return False
            torch.cuda.current_stream().synchronize()
            assert same(img, ref)
            return True

    seen = set()
    for limit in [int(2 ** (20 + k / 2)) for k in range(0, 16, 1)]:
        tet, auto = drawn("per_tetrahedron", limit), drawn("auto", limit)
        assert auto or not tet, limit
        seen.add(tet)
    assert seen == {False, True}
