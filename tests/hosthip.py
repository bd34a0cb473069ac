"""The library's host runtime over host_hip.cpp: models and engines on CPU tensors whose
launches are recorded and can be made to fail, for the routes and the error paths of calls."""
import ctypes as C
import gc
import os
import subprocess
from collections import Counter

import numpy as np
import torch

HERE = os.path.dirname(os.path.abspath(__file__))


def build(out_dir):
    from paper_2104_02646_amd import build as b, gsim as gs
    lib = os.path.join(out_dir, "libgsim_host.so")
    absent = os.path.join(out_dir, "absent.cpp")  # entry points of the kernel sources
    with open(absent, "w") as f:
        for name in gs.ABI_SYMBOLS:
            if name.split("_")[1] in ("controller", "rigid", "raster"):
                f.write('extern "C" int %s() { return %d; }\n' % (name, gs.GSIM_E_UNSUPPORTED))
    src = [os.path.join(b.CSRC, s) for s in b.HOST_SOURCES] + [os.path.join(HERE, "host_hip.cpp"), absent]
    subprocess.check_call([b.CLANGXX, "-x", "c++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + b.INCLUDE, "-I" + b.CSRC, *src, "-o",
                           lib])
    return lib


class Stream:
    """Anything with an address: the recorded calls only pass it on."""

    def __init__(self):
        self.buf = C.create_string_buffer(8)
        self.cuda_stream = C.addressof(self.buf)


class HostHip:
    def __init__(self, lib):
        self.lib = C.CDLL(lib)
        self.lib.host_hip_calls.restype = C.c_char_p
        self.lib.host_hip_fail.argtypes = [C.c_char_p, C.c_int]
        self.stream = Stream()

    def reset(self):
        self.lib.host_hip_reset()

    def fail(self, name, nth=1):
        self.lib.host_hip_fail(name.encode(), nth)

    def names(self):
        return self.lib.host_hip_calls().decode().split()

    def count(self):
        return Counter(self.names())

    def model(self, bodies, dtype=torch.float32, **kw):
        """(model, parameters, x0, v0)"""
        from paper_2104_02646_amd import gsim as gs
        m = gs.Model(bodies, dtype, device="cpu", stream=self.stream, **kw)
        x, v = (gs.soa(np.concatenate([getattr(b, k) for b in bodies]), dtype, "cpu") for k in ("x0", "v0"))
        return m, m.params_from_bodies(), x, v


def use(lib, monkeypatch):
    """The binding over `lib` until the patches are undone."""
    from paper_2104_02646_amd import gsim as gs, serve
    gc.collect()
    monkeypatch.setattr(gs, "LIB_PATH", lib)
    monkeypatch.setattr(gs, "_lib", None)
    monkeypatch.setattr(serve, "_ready", False)
    h = HostHip(lib)
    default = gs._stream
    monkeypatch.setattr(gs, "_stream", lambda s=None: default(h.stream if s is None else s))
    gs.load()
    h.reset()
    return h
