"""The library's host code built against tests/fake_hip.cpp (no device code, no GPU)."""
import contextlib
import ctypes as C
import os
import re
import subprocess

import numpy as np

from paper_2603_15780_amd import build as B
from paper_2603_15780_amd import sg

HERE = os.path.dirname(os.path.abspath(__file__))
LAUNCH = C.CFUNCTYPE(C.c_int, C.c_char_p, C.c_int, C.POINTER(C.c_void_p))


def build(out_dir) -> str:
    inc = ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC]
    objs, bins = [], set()
    for s in B.SOURCES:
        o = os.path.join(out_dir, s + ".o")
        host = ["--offload-arch=gfx950", "--offload-host-only"] if s.endswith(".hip") else []
        subprocess.run([B.HIPCC, *host, "-O1", "-std=c++17", "-fPIC", "-ffp-contract=on", *inc, "-c",
                        os.path.join(B.CSRC, s), "-o", o], check=True, capture_output=True)
        objs.append(o)
        bins |= set(re.findall(r"__hip_fatbin_\w+", subprocess.run(["nm", "-u", o], check=True, capture_output=True,
                                                                 text=True).stdout))
    lib = os.path.join(out_dir, "libsg_host.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"),
                    *objs, *[f"-Wl,--defsym={b}=fake_fatbin" for b in bins], "-Wl,-Bsymbolic", "-o", lib], check=True)
    return lib


def arr(*shape, dtype=np.float32):
    return np.zeros(shape, dtype)


def ptr(a):
    return a.ctypes.data if a is not None else None


class Lib:
    """The C functions with numpy arrays in the place of device memory."""

    def __init__(self, path):
        self.L = C.CDLL(path)
        for name in dir(sg.lib()):   # (the signatures that the binding has declared)
            f = getattr(sg.lib(), name)
            if name.startswith("sg_") and f.argtypes is not None:
                getattr(self.L, name).argtypes, getattr(self.L, name).restype = f.argtypes, f.restype
        self.L.sg_last_error.restype = C.c_char_p
        self.L.fake_malloc_limit.argtypes = [C.c_size_t]

    @contextlib.contextmanager
    def on_launch(self, fn):
        """fn(kernel name, device, args) -> HIP error or None, at each launch."""
        cb = LAUNCH(lambda name, dev, args: fn(re.sub(r"^_ZN2sg12_GLOBAL__N_1\d+(k_[a-z0-9_]+?)(I|E).*", r"\1",
                                                      name.decode()), dev, args) or 0)
        self.L.fake_on_launch(cb)
        try:
            yield
        finally:
            self.L.fake_on_launch(LAUNCH())

    def mesh(self, X, F):
        X, F = np.ascontiguousarray(X, np.float32), np.ascontiguousarray(F, np.int32)
        h = C.c_void_p()
        rc = self.L.sg_mesh_create(ptr(X), len(X), ptr(F), len(F), None, None, 1, C.byref(h))
        assert rc == 0, self.L.sg_last_error()
        return h

    def exp(self, h, n, **kw):
        o = sg.opts(**kw)
        f, b, v = arr(n, dtype=np.int32), arr(n, 3), arr(n, 3)
        out = [arr(n, dtype=np.int32), arr(n, 3), arr(n, 3), arr(n, 3)]
        return self.L.sg_exp(h, n, ptr(f), ptr(b), ptr(v), *[ptr(x) for x in out], None, None, None, C.byref(o), None)

    def backward(self, h, mode, n, saved=True, grad_X=None, **kw):
        o = sg.opts(**kw)
        f, b, v, g = arr(n, dtype=np.int32), arr(n, 3), arr(n, 3), arr(n, 3)
        fo, bo, vo, st = (arr(n, dtype=np.int32), arr(n, 3), arr(n, 3), arr(n, dtype=np.int32)) if saved else [None] * 4
        gv, gb = arr(n, 3), arr(n, 3)
        return self.L.sg_exp_backward(h, mode, n, ptr(f), ptr(b), ptr(v), ptr(fo), ptr(bo), ptr(vo), ptr(st), ptr(g),
                                      ptr(gv), ptr(gb), ptr(grad_X), C.byref(o), None)

    def pi_exp(self, h, n, step=0.01, search=sg.PI_GRID):
        f, b, v = arr(n, dtype=np.int32), arr(n, 3), arr(n, 3)
        out = [arr(n, dtype=np.int32), arr(n, 3), arr(n, 3), arr(n, 3)]
        po = sg.pi_opts(step, None, search)
        return self.L.sg_pi_exp(h, n, ptr(f), ptr(b), ptr(v), 0, None, *[ptr(x) for x in out], None, None, None, C.byref(po),
                                None)

    def pi_backward(self, h, n, step=0.01):
        f, b, v, g, gv, gb = arr(n, dtype=np.int32), *[arr(n, 3) for _ in range(5)]
        po = sg.pi_opts(step)
        return self.L.sg_pi_backward(h, sg.BWD_GFD, n, ptr(f), ptr(b), ptr(v), None, None, ptr(g), ptr(gv), ptr(gb),
                                     C.byref(po), None, None)
