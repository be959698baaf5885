"""The library linked with tests/hip_stub.c in the place of the HIP runtime, for tests of its host side on the CPU.

`stubbed(monkeypatch)` gives the binding with that library loaded and the library itself, whose stub_* functions count
launches and allocations and make launches fail; `context` makes a context in host memory."""
import ctypes as C
import glob
import os
import subprocess
import tempfile

import numpy as np
import pytest

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
_path = None


def _build():
    global _path
    if _path is None:
        from paper_1711_10984_amd import build as B
        clang = os.path.join(ROCM, "lib", "llvm", "bin", "clang")
        if not os.path.exists(clang):
            pytest.skip("ROCm compilers not available")
        objs = sorted(glob.glob(os.path.join(B.HERE, "_build", "lbm_*.o")))
        if len(objs) < len(B.SRC):
            B.build()
            objs = sorted(glob.glob(os.path.join(B.HERE, "_build", "lbm_*.o")))
        out = os.path.join(tempfile.mkdtemp(prefix="lbm_stub_"), "liblbm_stub.so")
        src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub.c")
        # symbolic: the library's calls go to the stub, also where the process holds a HIP runtime
        subprocess.run([clang, "-O1", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-o", out, src] + objs +
                       ["-lstdc++", "-lpthread", "-lm"], check=True, capture_output=True, text=True)
        _path = out
    return _path


def stubbed(monkeypatch):
    from paper_1711_10984_amd import lbm
    lib = lbm.load_library(_build())
    lib.stub_launched.argtypes, lib.stub_launched.restype = [C.c_char_p], C.c_long
    lib.stub_fail.argtypes = [C.c_long, C.c_long]
    lib.stub_last_grid.restype = C.c_uint
    lib.stub_host_allocs.restype = lib.stub_host_live.restype = C.c_long
    lib.stub_reset()
    monkeypatch.setattr(lbm, "_lib", lib)
    return lbm, lib


class Context:
    """A context over host memory; `close` destroys it."""

    def __init__(self, lbm, shapes, drops, precision=0, stream=1, **params):
        self.lbm, self.shapes, self.ndrop = lbm, shapes, [len(d) for d in drops]
        cfgs = [lbm.make_config(dict(nx=nx, ny=ny, **params), precision) for nx, ny in shapes]
        nbytes = lbm.lbm_workspace_bytes(cfgs, self.ndrop)
        self.memory = np.zeros(nbytes + 256, np.uint8)
        at = -(-self.memory.ctypes.data // 256) * 256
        n = sum(nx * ny for nx, ny in shapes)
        table = [lbm.make_droplet(d) for ds in drops for d in ds]
        self.h = lbm.lbm_init_batch(cfgs, at, nbytes, stream, np.zeros(n), np.zeros(n), None, self.ndrop, table)

    def centres(self, inst=0):
        return [(d.x, d.y) for d in self.lbm.lbm_droplets(self.h, inst, self.ndrop[inst])]

    def close(self):
        self.lbm.lbm_destroy(self.h)
