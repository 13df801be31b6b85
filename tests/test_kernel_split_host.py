"""The per-tetrahedron code in the kernels' own split of it, on the CPU: the
edge form's setup in two passes against one, and depth slabs deposited as
values by a wavefront's lanes, alone and as a stack, against the oracle."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle as O
import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_1208_3206_amd", "csrc")
SRC, LIB = os.path.join(HERE, "hostcheck", "kernels.cpp"), os.path.join(HERE, "hostcheck", "libkernels.so")
P = ctypes.POINTER


@pytest.fixture(scope="module")
def lib():
    newest = max(os.path.getmtime(p) for p in (SRC, os.path.join(CSRC, "tess_tet.h"), os.path.join(CSRC, "tess_internal.h")))
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        tmp = LIB + ".tmp%x" % os.getpid()
        subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-arch=gfx950", "-O2", "-std=c++17", "-fPIC", "-shared",
                        "-I", CSRC, "-I", os.path.join(ROOT, "include"), SRC, "-o", tmp], check=True, capture_output=True)
        os.replace(tmp, LIB)
    L = ctypes.CDLL(LIB)
    L.hk_slabs.restype = ctypes.c_longlong
    return L


def scene_args(xyz, dims, view, periodic=True):
    xyz = [np.ascontiguousarray(a, dtype=np.float32) for a in xyz]
    keep = [(ctypes.c_int32 * 3)(*dims), (ctypes.c_double * 9)(*[float(v) for v in view["rot"]]),
            (ctypes.c_double * 2)(*[float(v) for v in view["extent"]]), xyz]
    q = {"unit": 0, "density": 1, "density2": 2}[view.get("quantity", "density")]
    args = [a.ctypes.data_as(P(ctypes.c_float)) for a in xyz] + [
        keep[0], int(periodic), keep[1], keep[2], int(view["width"]), int(view["height"]), int(view.get("wrap", 0)), q]
    return args, keep


ROT = W.random_rotations(1, seed=3)[0]
SETUPS = {
    "wrap": (16, 4.0, W.z_view(128), 64.0, True), "steep": (16, 4.0, W.z_view(128), 4.0, True),
    "rotated": (16, 4.0, W.rotated_view(ROT, 120, 110), 64.0, True), "coarse": (24, 5.0, W.z_view(20), 2.0, True),
    "density2": (16, 4.0, dict(W.z_view(128), quantity="density2"), 64.0, True),
    "undisplaced": (16, 0.0, W.z_view(96), 64.0, True), "open": (12, 3.0, W.rotated_view(ROT, 90), 64.0, False),
    "wide": (4, 6.0, W.z_view(23, 19), 64.0, True), "pixel": (8, 3.0, W.z_view(1), 64.0, True),
}


# Bit for bit: the same expressions on the same numbers
@pytest.mark.parametrize("case", sorted(SETUPS))
def test_two_pass_setup_equals_one_pass(lib, case):
    n, growth, view, bound, periodic = SETUPS[case]
    xyz = W.zeldovich(n, max(1, n // 4), growth, seed=7) if growth else W.undisplaced(n)
    args, keep = scene_args(xyz, (n, n, n), view, periodic)
    out = (ctypes.c_longlong * 6)()
    lib.hk_setup(*args, ctypes.c_double(bound), out)
    assert list(out[:4]) == [0, 0, 0, 0], "words that differ: slope changes, silhouettes, own records, counters"
    assert out[4] > 0 and out[4] >= out[5]
    if case in ("steep", "coarse"):
        assert out[5] > 0.05 * 6 * n ** 3


SLABS = [(-1.5, -0.31), (-0.31, -0.1), (-0.1, 0.02), (0.02, 0.021), (0.021, 0.4), (0.4, 1.5)]


# held to the bar of the row-sum form's slab tests
@pytest.mark.parametrize("stack", [0, 1])
@pytest.mark.parametrize("kind,lanes,tile", [("z", 1, (8, 40)), ("z", 64, (32, 96)), ("rotated", 64, (16, 17)),
                                             ("undisplaced", 64, (8, 64)), ("large", 64, (64, 256))])
def test_slabs_as_values_match_oracle(lib, kind, lanes, tile, stack):
    n = 4 if kind == "large" else 12
    xyz = W.undisplaced(n) if kind == "undisplaced" else W.zeldovich(n, max(1, n // 3), 5.0, seed=5)
    view = {"z": W.z_view(96, 72), "rotated": W.rotated_view(ROT, 80, 64), "undisplaced": W.z_view(64, 48),
            "large": W.z_view(256, 200)}[kind]
    args, keep = scene_args(xyz, (n, n, n), view)
    out = np.zeros((len(SLABS), view["height"], view["width"]))
    t = np.array(SLABS, dtype=np.float64)
    frags = lib.hk_slabs(*args, t.ctypes.data_as(P(ctypes.c_double)), len(SLABS), stack, *tile, lanes,
                         out.ctypes.data_as(P(ctypes.c_double)))
    want = 0
    for k, slab in enumerate(SLABS):
        ref, st = O.project_region(*xyz, (n, n, n), dict(view, slab=slab))
        want += st["fragments"]
        assert np.abs(out[k] - ref).max() <= 1e-8 * np.abs(ref).max(), k
    if kind != "undisplaced":  # (there pixel centres lie on the slabs' faces and edges)
        assert abs(frags - want) <= 1e-6 * want + 4
