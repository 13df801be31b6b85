"""Depth slabs of undisplaced lattices seen along their axes: every face
parallel to the view is a wall, pixel centres lie on walls, and a pixel belongs
to one side of each."""
import itertools

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tess():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1208_3206_amd as t
    return t


def flat(dims, box, reverse):
    k, j, i = np.meshgrid(*[np.arange(n) for n in dims[::-1]], indexing="ij")
    q = [(v.ravel() / n * L).astype(np.float32) for v, n, L in zip((i, j, k), dims, box)]
    return [a[::-1].copy() for a in q] if reverse else q


# lattices whose spacings round, in both orders of their tracers, along every
# signed axis; a pixel on the wrong side of a wall is off by a whole chord, the
# rest by the FP32 rounding.  (A wall's two tetrahedra place it in their own
# cubes' frames; where those round apart, as in 20 planes over a box of 7.5, a
# pixel on it may still fall to both or neither.)
@pytest.mark.parametrize("dims,box,center,size,quantity", [
    ((5, 2, 31), (1.0, 1.0, 1.0), (0.0, 0.1, 0.5), (513, 31), "unit"),
    ((2, 31, 3), (1.0, 1.0, 1.0), (0.0, 1.3, 0.5), (31, 513), "density2"),
    ((8, 5, 2), (1.0, 1.0, 1.0), (0.1, 0.0, 0.0), (513, 31), "density"),
    ((10, 7, 12), (1.0, 1.0, 1.0), (0.5, 0.5, 0.5), (100, 60), "density"),
    ((9, 11, 13), (2.0, 1.0, 3.0), (1.0, 0.5, 1.5), (99, 65), "density")])
def test_walls_of_undisplaced_lattices(tess, dims, box, center, size, quantity):
    import torch
    deep = max(box)
    cuts = [-0.61 * deep, -0.27 * deep, -0.083 * deep, 0.24 * deep, 0.66 * deep]
    for reverse in (False, True):
        xyz = flat(dims, box, reverse)
        lat = tess.build(*[torch.from_numpy(a).cuda() for a in xyz], dims, box=box)
        for perm in itertools.permutations(range(3)):
            for signs in itertools.product((1, -1), repeat=2):
                rot = np.eye(3)[list(perm)] * np.array([signs[0], signs[1], 1])[:, None]
                view = dict(rot=rot.ravel().tolist(), center=center, extent=[box[perm[0]], box[perm[1]]], wrap=1,
                            width=size[0], height=size[1], quantity=quantity)
                views = [dict(view, slab=s) for s in zip(cuts[:-1], cuts[1:])]
                imgs = tess.project_batch([lat], views)[0].double().cpu().numpy()
                for k, v in enumerate(views):
                    ref, _ = O.project_region(*xyz, dims, v, box=box)
                    one = tess.project(lat, v).double().cpu().numpy()
                    for got in (imgs[k], one):
                        off = np.abs(got - ref) > 2e-7 * ref + 1e-9 * ref.max()
                        assert not off.any(), (reverse, perm, signs, k, int(off.sum()))
