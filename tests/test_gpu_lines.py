"""The row kernel (kernel 0: one node per lane, windows of at most 62 nodes,
rows of 64 nodes without neighbour lanes) at the edges of its windows and
z-segments, against the FP64 oracle."""
import numpy as np
import pytest

from paper_2312_14742_amd import inputs

from gpu_helpers import (UNIT_ROUNDOFF, assert_f64_parity, reduced_errors, run_gpu, run_oracle)

pytestmark = pytest.mark.gpu

G = (1e-5, -2e-5, 3e-6)
# one window with and without room, exactly 64 nodes, two and three windows,
# a last window of few nodes; one plane, and segments of several planes
DIMS = [(2, 3, 1), (31, 2, 2), (61, 4, 3), (62, 3, 5), (63, 5, 4), (64, 3, 4), (65, 4, 3),
        (124, 3, 3), (125, 2, 4), (187, 5, 2), (62, 90, 180), (64, 100, 170)]


@pytest.mark.parametrize("q", [15, 19, 27])
@pytest.mark.parametrize("dims", DIMS)
def test_window_edges_f64(q, dims):
    nx, ny, nz = dims
    solid, drho, u = inputs.random_state(nx, ny, nz, seed=nx + 7 * ny + 31 * nz)
    print(f"[case] rows f64 q={q} dims={dims}", flush=True)
    sim, out = run_gpu([(solid, drho, u)], q, "f64", G, 4, kernel=0)
    assert_f64_parity(out[0], run_oracle(q, solid, drho, u, G, 4), solid)
    sim.close()


@pytest.mark.parametrize("prec", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("dims", [(63, 5, 4), (64, 3, 4), (125, 2, 4), (62, 90, 180)])
def test_window_edges_reduced(prec, dims):
    """Bounds of one storage rounding per step (the other kernels' bounds)."""
    nx, ny, nz = dims
    solid, drho, u = inputs.random_state(nx, ny, nz, seed=3 + nx)
    print(f"[case] rows {prec} dims={dims}", flush=True)
    sim, out = run_gpu([(solid, drho, u)], 19, prec, G, 4, kernel=0)
    err = reduced_errors(out[0], run_oracle(19, solid, drho, u, G, 4), solid)
    eps = UNIT_ROUNDOFF[prec]
    assert err["u_rel_l2"] <= 8.0 * eps, err
    assert err["drho_abs"] <= (2.0 * eps + 16.0 * 2.0 ** -24) * np.abs(u).max(), err
    sim.close()
