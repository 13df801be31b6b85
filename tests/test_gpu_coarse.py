"""Coarse periodic images of large lattices (the edge form with a bound of its
own on steep footprints), and the workspace given back to a call's limit, against
the per-tetrahedron form."""
import pytest

import workloads as W
from test_gpu_forms import lattice, same, tess  # noqa: F401

pytestmark = pytest.mark.gpu


# a pixel for many cells to 1.5 pixels a cell, one row, undisplaced walls, most
# of the tetrahedra steep and few; the first call has room for all own records,
# the second for as many as were counted
@pytest.mark.parametrize("size,growth", [((150, 150), 0.3), ((40, 25), 5.0), ((97, 1), 2.0), ((1, 1), 3.0), ((128, 64), 0.0)])
def test_coarse_image_equals_the_per_tetrahedron_form(tess, size, growth):  # noqa: F811
    lat = lattice(tess, 102, growth)
    view = W.z_view(*size)
    ref, sr = tess.project(lat, view, tune=tess.make_tune(form="per_tetrahedron"), stats=True)
    for k in range(2):
        img, st = tess.project(lat, view, stats=True)
        assert st["own_records"] > 0 and st["overflow"] == 0, k
        assert same(img, ref)
        assert same(tess.project(lat, view), ref)
        assert same(tess.project_batch([lat], [view, view])[0, 1], ref)
        for key in ("tets", "zero_volume", "inverted", "fp64_dets"):
            assert st[key] == sr[key], key
        assert abs(st["fragments"] - sr["fragments"]) <= 1e-6 * sr["fragments"] + 8


# A call under a limit gives back what calls without it made larger; batches
# captured before it draw the same after it, with and without statistics
def test_workspace_given_back_between_batches(tess):  # noqa: F811
    import torch
    lat = lattice(tess, 48, 2.0)
    views = [W.z_view(300, 200)] * 3
    ref = tess.project(lat, views[0], tune=tess.make_tune(form="per_tetrahedron"))
    with torch.cuda.stream(torch.cuda.Stream()):  # (a workspace of its own)
        out = torch.empty((1, 3, 200, 300), device="cuda")
        small = W.z_view(16)
        few = tess.project(lat, small)
        for _ in range(3):
            for stats in (False, True):
                out.zero_()
                tess.project_batch([lat], views, out=out, stats=stats)
                torch.cuda.current_stream().synchronize()
                for k in range(3):
                    assert same(out[0, k], ref)
            # (fits in an empty workspace, not beside the batch's edge buffers)
            img = tess.project(lat, small, tune=tess.make_tune(workspace_limit=150 << 20))
            torch.cuda.current_stream().synchronize()
            assert same(img, few)
