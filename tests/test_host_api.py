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
