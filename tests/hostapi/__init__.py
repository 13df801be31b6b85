"""Builds and loads the library's host code over a device that computes
nothing (fake_hip.cpp), for tests of allocation, fallbacks and plans without a
GPU.  Every device() is a fresh copy of the library with its own state."""
import ctypes
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_1208_3206_amd", "csrc")
LIB = os.path.join(HERE, "libhostapi.so")
SRC = [os.path.join(CSRC, "tess_api.cpp"), os.path.join(HERE, "fake_hip.cpp")]
DEPS = SRC + [os.path.join(CSRC, "tess_internal.h"), os.path.join(CSRC, "tess_host.h"),
              os.path.join(ROOT, "include", "tess.h")]


def build():
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(p) for p in DEPS):
        tmp = LIB + ".tmp%x" % os.getpid()
        subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                        "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", *SRC, "-o", tmp],
                       check=True, capture_output=True)
        os.replace(tmp, LIB)
    return LIB


class Log(ctypes.Structure):
    _fields_ = ([(k, ctypes.c_longlong) for k in
                 ("setups", "edge_setups", "stack_setups", "rasters", "direct_rasters", "counting_rasters", "mallocs",
                  "frees", "failed_mallocs", "graphs", "graph_launches", "illegal")]
                + [(k, ctypes.c_int32) for k in ("edges", "Th", "Tw", "chunk", "block", "nstack")]
                + [("ntet", ctypes.c_int64), ("stored", ctypes.c_int64), ("crease_bmax", ctypes.c_double),
                   ("bmax_per_q", ctypes.c_double), ("cap", ctypes.c_ulonglong), ("max_items", ctypes.c_ulonglong), ("own_room", ctypes.c_int64)])


class Device:
    """The library over an idle device; calls return the status."""

    def __init__(self, tess):
        self.t = tess
        # (a file of its own: the loader would hand out one loaded copy)
        fd, path = tempfile.mkstemp(suffix=".so")
        os.close(fd)
        shutil.copyfile(build(), path)
        self.lib = ctypes.CDLL(path)
        os.unlink(path)
        L, vp = self.lib, ctypes.c_void_p
        L.tess_last_error.restype = ctypes.c_char_p
        L.fake_held.restype = ctypes.c_size_t
        L.fake_budget.argtypes = [ctypes.c_size_t]
        L.fake_counts.argtypes = [ctypes.c_ulonglong, ctypes.c_ulonglong]
        L.tess_free.argtypes = [vp]
        self.log = Log.in_dll(L, "fake_log")

    def build(self, dims, **kw):
        d = self.t.build_desc(dims, **kw)
        h, p = ctypes.c_void_p(), ctypes.c_void_p(1 << 40)
        assert self.lib.tess_build(ctypes.byref(d), p, p, p, None, None, ctypes.byref(h)) == 0, self.error()
        return h

    def error(self):
        return self.lib.tess_last_error().decode()

    def reset(self):
        self.lib.fake_reset()

    def counts(self, pairs_per_list=1, own=0):
        self.lib.fake_counts(pairs_per_list, own)

    def budget(self, nbytes=(1 << 64) - 1):
        self.lib.fake_budget(nbytes)

    def held(self):
        return self.lib.fake_held()

    def capturing(self, on):
        self.lib.fake_capturing(int(on))

    def project(self, lat, view, stats=False, stream=1, **tune):
        v, t, st = self.t.make_view(view), self.t.make_tune(**tune), self.t.TessStats()
        rc = self.lib.tess_project(lat, ctypes.byref(v), ctypes.byref(t), ctypes.c_void_p(1 << 41),
                                   ctypes.byref(st) if stats else None, ctypes.c_void_p(stream))
        self.stats = st
        return rc

    def noalloc(self, lat, view, **tune):
        v, t = self.t.make_view(view), self.t.make_tune(**tune)
        return self.lib.tess_project_noalloc(lat, ctypes.byref(v), ctypes.byref(t), ctypes.c_void_p(1 << 41), None)

    def batch(self, lats, views, stats=False, stream=1, **tune):
        L = (ctypes.c_void_p * len(lats))(*lats)
        V = (self.t.TessView * len(views))(*[self.t.make_view(v) for v in views])
        t, st = self.t.make_tune(**tune), self.t.TessStats()
        rc = self.lib.tess_project_batch(L, len(lats), V, len(views), ctypes.byref(t), ctypes.c_void_p(1 << 41),
                                         ctypes.byref(st) if stats else None, ctypes.c_void_p(stream))
        self.stats = st
        return rc
