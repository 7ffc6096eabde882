"""The library's host code on a host double of the HIP runtime (tests/host_double.c): which kernels
a call launches, with which arguments, and what it returns when a launch fails.  No GPU is used and
no kernel runs.

Run as a child process, so that the double never meets the runtime that torch loads:
`double(code, tmp_path)` returns what the code, which starts with `from host_double import *`, prints
with `emit`.
"""
import ctypes as C
import json
import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LAUNCH = C.CFUNCTYPE(C.c_int, C.c_char_p, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32, C.POINTER(C.c_void_p))
CALL = C.CFUNCTYPE(None, C.c_char_p, C.c_void_p, C.c_void_p, C.c_size_t)


def double(code, tmp_path):
    so = str(tmp_path / "libhost_double.so")
    subprocess.run([shutil.which("gcc") or "cc", "-O1", "-std=c99", "-Wall", "-fPIC", "-shared", "-o", so,
                    os.path.join(HERE, "host_double.c")], check=True)
    r = subprocess.run([sys.executable, "-c", "import sys; sys.path[:0] = [%r, %r]\nfrom host_double import *\n%s"
                        % (HERE, ROOT, code)], env=dict(os.environ, HOST_DOUBLE=so), capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, (r.stdout[-2000:], r.stderr[-4000:])
    return json.loads(r.stdout.strip().splitlines()[-1])


def emit(v):
    print(json.dumps(v), flush=True)


class Runtime:
    """The double, the library bound to it, and the record of launches and calls."""

    def __init__(self):
        self.launches = []  # (kernel, grid, threads, template arguments)
        self.calls = []     # (name, dst, src, bytes)
        self.fail = lambda kernel: False
        self.on_launch = lambda kernel, args: None
        self.dev = C.CDLL(os.environ["HOST_DOUBLE"], mode=C.RTLD_GLOBAL)
        self._cbs = LAUNCH(self._launch), CALL(self._call)
        self.dev.double_callbacks(*self._cbs)
        from paper_2304_04214_amd import _abi
        self.A, self.L = _abi, _abi.lib()

    def _launch(self, name, gx, gy, gz, threads, args):
        kernel = re.search(r"(?<=\d)([a-z][a-z0-9_]*_kernel)", name.decode())
        kernel = kernel.group(1) if kernel else name.decode()
        targs = re.search("_kernelI((?:L[bi][0-9]+E)+)E", name.decode())
        targs = [int(v) for v in re.findall("L[bi]([0-9]+)E", targs.group(1))] if targs else []
        self.launches.append((kernel, (gx, gy, gz), threads, targs))
        self.on_launch(kernel, args)
        return 1 if self.fail(kernel) else 0

    def _call(self, name, dst, src, n):
        self.calls.append((name.decode(), dst, src, n))

    def channel(self, nx, ny, nz, *, storage=0, ywall=2, xbc=0, wall_model=0, wall_avg=0, modes=16, fluct=True):
        """A handle on state buffers that nothing dereferences, with bound inlet inputs if xbc = 1."""
        A, c = self.A, self.A.Config()
        c.nx, c.ny, c.nz, c.storage, c.ywall, c.xbc = nx, ny, nz, storage, ywall, xbc
        c.wall_model, c.wall_avg, c.newton_iters = wall_model, wall_avg, 4
        c.tau0, c.cs_smag, c.kappa, c.b_reich, c.y_wall, c.u_conv = 0.6, 0.1, 0.41, 7.8, 0.5, 0.1
        h, p = C.c_void_p(), self.plane
        st = self.L.lbm_create(C.byref(c), p(0), p(1), p(2), p(3), None, C.byref(h))
        assert st == A.LBM_OK, st
        if xbc:
            s = A.Stg()
            s.n_modes, s.n_bins = modes, 1
            for k, f in enumerate(("q", "sigma", "kmag", "d", "phi", "omega", "u_rans", "R", "amp_bin", "bin_of_y",
                                   "u_in", "fluct")):
                setattr(s, f, p(100 + k).value)
            if not fluct:
                s.fluct = None
            self.u_in, self.fluct, self.stg = p(110).value, p(111).value, s
            assert self.L.stg_inlet_fill(h, C.byref(s), 0.0) == A.LBM_OK
        self.launches.clear()
        self.calls.clear()
        return h

    @staticmethod
    def plane(k):
        """Address of the k-th of far-apart buffers."""
        return C.c_void_p((k + 1) << 32)

    @classmethod
    def array(cls, ks):
        return (C.c_void_p * max(len(ks), 1))(*[cls.plane(k) for k in ks])
