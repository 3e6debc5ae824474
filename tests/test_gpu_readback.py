"""Readback through pinned slots of 2^18 nodes: one slot, a last slot of few
nodes, more slots than are in flight (copied by worker threads), either array
alone, and several contexts and threads at a time."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2312_14742_amd import tau1

pytestmark = pytest.mark.gpu


def state(nx, ny, nz, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    solid = (rng.random((nz, ny, nx)) < 0.3).astype(np.uint8)
    fl = solid == 0
    return solid, rng.uniform(-1e-3, 1e-3, solid.shape) * fl, \
        rng.uniform(-0.05, 0.05, (3,) + solid.shape) * fl


@pytest.mark.parametrize("dims", [(3, 2, 1), (64, 64, 64), (64, 64, 65), (128, 128, 66),
                                  (150, 131, 97)])
def test_initial_state_comes_back(dims):
    """FP64, g = 0: the uploaded fields come back as they are."""
    solid, drho, u = state(*dims, seed=sum(dims))
    print(f"[case] readback {dims}", flush=True)
    with tau1.Sim([tau1.Sample(solid, drho, u)], precision="f64") as sim:
        for _ in range(2):
            d, v = sim.moments(0)
            assert np.array_equal(d, drho) and np.array_equal(v, u)
        rho, v = sim.rho_u(0)
        assert np.array_equal(rho, 1.0 + drho) and np.array_equal(v, u)
        # either array alone
        lib = tau1._lib()
        only_d, only_u = np.empty_like(drho), np.empty_like(u)
        assert lib.tau1_moments_drho(sim._c(), 0, only_d.ctypes.data, None) == 0
        assert lib.tau1_moments_drho(sim._c(), 0, None, only_u.ctypes.data) == 0
        assert lib.tau1_moments_drho(sim._c(), 0, None, None) == 0
        assert np.array_equal(only_d, drho) and np.array_equal(only_u, u)
        m = ctypes.c_double(0.0)
        assert lib.tau1_permeability(sim._c(), 0, 0, None, ctypes.byref(m)) == 0
        assert abs(m.value - (solid == 0).sum() - drho.sum()) <= 1e-9


def test_threads_read_at_once():
    samples = [state(96, 80, 50 + 10 * i, seed=i) for i in range(4)]
    sims = [tau1.Sim([tau1.Sample(*s)], precision="f64") for s in samples]
    bad = []

    def read(i):
        for _ in range(5):
            d, v = sims[i].moments(0)
            if not (np.array_equal(d, samples[i][1]) and np.array_equal(v, samples[i][2])):
                bad.append(i)

    print("[case] readback from four threads", flush=True)
    ts = [threading.Thread(target=read, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for s in sims:
        s.close()
    assert not bad
