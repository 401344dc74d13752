"""The host runtime built against hip_stub.cpp, for CPU tests of what it launches.

No GPU is involved: a launch records the states it would read and write, a
read-out returns the number of steps done to the state, and launches that touch
one state in no order, or hold two step chunks of one instance, count as faults.
"""
import ctypes
import os
import subprocess

from paper_0907_1720_amd import build as B
from paper_0907_1720_amd import lbm

HERE = os.path.dirname(os.path.abspath(__file__))
REG, SLABS, TILES, LDS, LDS_SLABS, LDS_TILES, STREAM, READ, INIT = range(9)


def compile_to(path):
    src = [os.path.join(B.CSRC, f) for f in ("runtime.cpp", "coeffs.cpp")] + [os.path.join(HERE, "hip_stub.cpp")]
    cmd = ([B.CLANG] + B.HOST_FLAGS + [f"-I{B.INCLUDE}", f"-I{B.CSRC}", "-shared", "-Wl,-Bsymbolic,-z,defs", "-o", path]
           + src)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]


class HostRuntime:
    """Puts the library built at `path` in the place of the HIP one until close()."""

    def __init__(self, path):
        self._saved = (lbm.LIB_PATH, lbm._lib)
        lbm.LIB_PATH, lbm._lib = path, None
        self.lib = lbm.library()
        self.lib.stub_limit.argtypes = [ctypes.c_size_t]
        self.lib.stub_slab_wait.restype = ctypes.c_longlong
        for name in ("stub_foreign", "stub_device"):
            getattr(self.lib, name).argtypes = [ctypes.c_size_t]
            getattr(self.lib, name).restype = ctypes.c_void_p

    def close(self):
        lbm.LIB_PATH, lbm._lib = self._saved

    def reset(self):
        self.lib.stub_reset()

    def limit(self, more=None):
        """Bytes of device memory that may be allocated from now on (None: any)."""
        self.lib.stub_limit(ctypes.c_size_t(-1).value if more is None else more)

    def faults(self):
        text = ctypes.create_string_buffer(256)
        n = self.lib.stub_faults(text, 256)
        return n, text.value.decode()

    def launches(self, *kinds):
        """(kind, stream, workgroups, steps, tag, blocks, nodes per lane, jobs) of the launches
        since reset(); for whole instances, the percentage of a CU's waves filled instead of a tag, and
        bytes of LDS instead of blocks."""
        out = []
        for k in range(self.lib.stub_launches()):
            r = (ctypes.c_int64 * 8)()
            self.lib.stub_launch(k, r)
            if not kinds or r[0] in kinds:
                out.append(tuple(r))
        return out
