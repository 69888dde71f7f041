"""The library over a stand-in HIP runtime that records launches and runs
nothing (hip_standin.c), for checks of its host side without a GPU. The stand-in
must be loaded ahead of the library and of any real HIP runtime, so ``run`` gives
each check a process of its own."""
import ctypes
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
WORKSPACE = 1 << 44  # an address that nothing reads or writes


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _Entry(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", _Dim3), ("block", _Dim3), ("arg", ctypes.c_void_p * 2)]


def run(tmp_path, code: str) -> str:
    """Runs `code` in a process where ``standin.load()`` works; returns what it printed."""
    so = os.path.join(str(tmp_path), "libhip_standin.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    os.path.join(HERE, "hip_standin.c"), "-o", so], check=True)
    env = dict(os.environ, HIP_STANDIN=so, PYTHONPATH=os.pathsep.join([HERE, ROOT]))
    r = subprocess.run([sys.executable, "-c", "import standin\n" + code], env=env, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    return r.stdout


class Recorder:
    def __init__(self):
        self.hip = ctypes.CDLL(os.environ["HIP_STANDIN"], mode=ctypes.RTLD_GLOBAL)
        from paper_1901_02716_amd import _lib

        self.lib, self.m = _lib.load(), _lib
        self._count = ctypes.c_int.in_dll(self.hip, "standin_count")
        self._log = ctypes.cast(ctypes.addressof(ctypes.c_char.in_dll(self.hip, "standin_log")),
                                ctypes.POINTER(_Entry))
        self.fail_event = ctypes.c_int.in_dll(self.hip, "standin_fail_event")
        self.ms = ctypes.c_float.in_dll(self.hip, "standin_ms")

    def launches(self, call, *args):
        """What `call` enqueued: (kernel name, grid, block, first two arguments) each."""
        self._count.value = 0
        rc = call(*args)
        return rc, [(e.name.decode(), (e.grid.x, e.grid.y), (e.block.x, e.block.y), tuple(e.arg))
                    for e in self._log[: self._count.value]]

    def config(self, q, n, precision, seed=0):
        c = self.m.Config(lattice=q, precision=precision, dx=0.1, nu=0.05, rho_ref=1.0, seed=seed)
        for i, v in enumerate(tuple(n) + (1,) * (3 - len(n))):
            c.n[i] = v
        return c

    def handle(self, q, n, precision, walls=""):
        c = self.config(q, n, precision)
        c.workspace, c.workspace_bytes = WORKSPACE, self.lib.maclab_workspace_bytes(ctypes.byref(c))
        h = ctypes.c_void_p()
        assert self.lib.maclab_init(ctypes.byref(c), ctypes.byref(h)) == 0
        self.walls(h, walls)
        return h

    def walls(self, h, axes):
        u = (ctypes.c_double * 3)()
        for ax in axes:
            for side in (0, 1):
                assert self.lib.maclab_set_bc(h, 2 * "xyz".index(ax) + side, self.m.FIXED, 1.0, u) == 0

    def batch(self, sizes, precision):
        cfgs = (self.m.Config * len(sizes))(*[self.config(9, n, precision) for n in sizes])
        b = ctypes.c_void_p()
        need = self.lib.maclab_batch_workspace_bytes(cfgs, len(sizes))
        assert self.lib.maclab_batch_init(cfgs, len(sizes), WORKSPACE, need, ctypes.byref(b)) == 0
        return b

    def buffer(self, h):
        """Address of the buffer that holds the state now."""
        rc, log = self.launches(self.lib.maclab_save_state, h, ctypes.c_void_p(WORKSPACE - 4096))
        assert rc == 0 and len(log) == 1 and log[0][0] == "copy"
        return log[0][3][0]


def load() -> Recorder:
    return Recorder()
