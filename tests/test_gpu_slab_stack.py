"""Stacks of depth slabs drawn at once, against the same views one by one."""
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


def lattices(tess, n, growths):
    import torch
    return [tess.build(*[torch.from_numpy(a).cuda() for a in W.zeldovich(n, 4, g, seed=3)], (n, n, n)) for g in growths]


def cuts(*edges):
    return list(zip(edges[:-1], edges[1:]))


Z = W.z_view
ROT = W.rotated_view(W.random_rotations(1, seed=3)[0], 75, 41, side=1.7)
# slabs side by side, with gaps, overlapping, equal, and in an order that is no
# stack; images of one tile and of several, ragged; cells 150 pixels wide
CASES = {
    "side_by_side": (12, Z(64), cuts(-1.5, *np.linspace(-0.5, 0.5, 9), 1.5)),
    "gaps_ragged": (13, Z(97, 70), [(-0.6, -0.3), (-0.1, 0.0), (0.05, 0.06), (0.4, 2.0)]),
    "overlapping": (12, Z(64), [(-0.7, 0.1), (-0.7, 0.1), (-0.2, 0.3), (0.0, 0.3)]),
    "not_sorted": (12, Z(64), [(0.1, 0.4), (-0.7, 0.1)]),
    "rotated": (12, ROT, cuts(-0.9, -0.2, 0.1, 0.35, 0.9)),
    "unit_wide": (12, dict(Z(1100, 90), quantity="unit"), cuts(-1.5, -0.1, 0.2, 1.5)),
    "large_cells": (9, Z(1400, 1300), cuts(-1.5, 0.0, 1.5)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_stack_equals_single_slabs(tess, case):
    n, view, slabs = CASES[case]
    lats = lattices(tess, n, (2.0, 5.0))
    views = [dict(view, slab=(float(a), float(b))) for a, b in slabs]
    for _ in range(2):  # the call that counts its pairs, and one that knows them
        imgs, st = tess.project_batch(lats, views, stats=True)
        frags = tets = 0
        for i, lat in enumerate(lats):
            for k, v in enumerate(views):
                one, so = tess.project(lat, v, stats=True)
                a, b = imgs[i, k].double(), one.double()
                # the same FP64 terms in another order, rounded once to FP32
                assert bool(((a - b).abs() <= 1.2e-7 * b.abs() + 1e-12 * b.max()).all()), (i, k)
                frags += so["fragments"]
                tets += so["tets"]
        assert st["tets"] == tets
        assert abs(st["fragments"] - frags) <= 1e-6 * frags + 8 and st["overflow"] == 0


def test_stack_beyond_its_learned_capacity(tess):
    # a shape whose pairs were learned on an undisplaced lattice, then a
    # strongly displaced one: drawn by the overflow raster, then by the lists
    n, view = 24, Z(48)
    views = [dict(view, slab=(float(a), float(b))) for a, b in cuts(-1.5, *np.linspace(-0.5, 0.5, 25), 1.5)]
    calm, wild = lattices(tess, n, (0.0, 12.0))
    tess.project_batch([calm], views, stats=True)
    first, st = tess.project_batch([wild], views, stats=True)
    assert st["overflow"] == len(views)
    again, st2 = tess.project_batch([wild], views, stats=True)
    assert st2["overflow"] == 0 and st2["bin_pairs"] == st["bin_pairs"]
    a, b = first.double(), again.double()
    assert bool(((a - b).abs() <= 1.2e-7 * b.abs() + 1e-12 * b.max()).all())
