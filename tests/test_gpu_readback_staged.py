"""Readback where no pinned host memory is to be had: the fields and the
permeability come through the workspace's staging area, with the same bits.  A
child process puts a hipHostMalloc that always fails before the HIP runtime's."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = "int hipHostMalloc(void **p, unsigned long n, unsigned f) { *p = 0; ++refused; return 2; }"
CODE = """
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL) if sys.argv[1] else None
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import hashlib
import numpy as np
from paper_2312_14742_amd import tau1
from test_gpu_readback import state
h = hashlib.sha256()
for dims in [(3, 2, 1), (64, 64, 65), (160, 128, 130)]:
    solid, drho, u = state(*dims, seed=7 + sum(dims))
    with tau1.Sim([tau1.Sample(solid, drho, u)], precision="f64", g=(1e-5, 0, 0)) as sim:
        for steps in (0, 3):
            sim.step(steps)
            for a in (*sim.moments(0), *sim.rho_u(0), np.array(sim.permeability(0))):
                h.update(a.tobytes())
    with tau1.Sim([tau1.Sample(solid, drho, u)], precision="f64") as sim:
        d, v = sim.moments(0)
        assert np.array_equal(d, drho) and np.array_equal(v, u), dims
if shim is not None:
    assert ctypes.c_int.in_dll(shim, "refused").value > 0
print("hash", h.hexdigest(), flush=True)
"""


def run(shim):
    res = subprocess.run([sys.executable, "-c", CODE, shim, ROOT], capture_output=True,
                         text=True, timeout=100)
    assert res.returncode == 0, res.stdout + res.stderr
    return [ln for ln in res.stdout.splitlines() if ln.startswith("hash")]


def test_staged_readback_has_the_same_bits(tmp_path):
    shim = str(tmp_path / "no_pinned.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-x", "c", "-", "-o", shim],
                   input="int refused;\n" + SHIM, text=True, check=True)
    print("[case] readback without pinned memory", flush=True)
    assert run(shim) == run("")


def test_last_context_goes_without_waiting_for_other_streams():
    """Giving the pinned blocks back waits for the whole device: tau1_destroy
    must not, nor may it hold up the contexts that follow."""
    import torch
    from paper_2312_14742_amd import tau1
    from test_gpu_readback import state
    solid, drho, u = state(64, 64, 40, seed=5)
    a = torch.randn(8192, 8192, device="cuda:0")
    side = torch.cuda.Stream()
    torch.matmul(a, a)
    torch.cuda.synchronize()
    print("[case] destroy beside a busy stream", flush=True)
    sim = tau1.Sim([tau1.Sample(solid, drho, u)], precision="f64")
    sim.moments(0)
    done = torch.cuda.Event()
    with torch.cuda.stream(side):
        for _ in range(40):
            b = torch.matmul(a, a)
        done.record(side)
    sim.close()
    assert not done.query()
    with tau1.Sim([tau1.Sample(solid, drho, u)], precision="f64") as nxt:
        d, v = nxt.moments(0)
        assert np.array_equal(d, drho) and np.array_equal(v, u)
    torch.cuda.synchronize()
    del b
