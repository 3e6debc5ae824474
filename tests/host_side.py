"""Runs host code of the library on the CPU: a child process loads fake_hip.c
(kernels do nothing) in the place of the HIP runtime, then libtau1.so."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2312_14742_amd import tau1
lib = tau1._lib()
i32 = ctypes.c_int
def get(name):
    return i32.in_dll(fake, "fake_" + name).value
def put(name, v):
    i32.in_dll(fake, "fake_" + name).value = v
class Ctx:
    def __init__(self, samples, lattice=19, precision="f32", g=(1e-6, 0, 0), graph_chunk=0,
                 kernel=-1, tile=-1, tune_cache=None):
        samples = [tau1.Sample(s) for s in samples]
        d, keep = tau1._desc(samples, lattice, precision, g, graph_chunk, kernel, tile, (0, 0),
                             tune_cache)
        n = ctypes.c_size_t(0)
        assert lib.tau1_workspace_size(ctypes.byref(d), ctypes.byref(n)) == 0
        self.mem = np.zeros(n.value // 8 + 64)
        d.workspace = (self.mem.ctypes.data + 255) // 256 * 256
        d.workspace_bytes = n.value
        self.p = ctypes.c_void_p(None)
        self.shape = samples[0].solid.shape
        st = lib.tau1_create(ctypes.byref(d), ctypes.byref(self.p))
        assert st == 0, st
    def step(self, n):
        assert lib.tau1_step(self.p, n) == 0
    def read(self):
        d, u = np.zeros(self.shape), np.zeros((3,) + self.shape)
        return lib.tau1_moments_drho(self.p, 0, d.ctypes.data, u.ctypes.data), d, u
    def permeability(self):
        k, m = ctypes.c_double(0), ctypes.c_double(0)
        return lib.tau1_permeability(self.p, 0, 0, ctypes.byref(k), ctypes.byref(m))
    def info(self):
        inf = tau1.tau1_info()
        assert lib.tau1_get_info(self.p, ctypes.byref(inf)) == 0
        return inf
    def close(self):
        lib.tau1_destroy(self.p)
def fluid(nx, ny, nz):
    return np.zeros((nz, ny, nx), np.uint8)
"""


def run_host(tmp_path, body, *args):
    """Runs `body` after PRELUDE (sys.argv[3:] = args); its assertions are the test."""
    shim = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-pthread", "-o", shim,
                    os.path.join(HERE, "fake_hip.c")], check=True)
    code = PRELUDE + textwrap.dedent(body)
    res = subprocess.run([sys.executable, "-c", code, shim, ROOT, *map(str, args)],
                         capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr
