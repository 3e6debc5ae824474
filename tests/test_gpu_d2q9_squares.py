"""D2Q9 launches of several steps on overlapping squares of 32 nodes: lattices
smaller than a square's halo, just beside a square's edge, and large enough for
each number of steps per launch; step counts that leave a shorter last launch."""
import numpy as np
import pytest

import oracle

from test_gpu_d2q9 import gpu_run, oracle_run, random_state

pytestmark = pytest.mark.gpu

LID = dict(wall_u=(0.1, 0.02, 0.0), g=(1e-4, -2e-5))
PRESSURE = dict(x_boundary=1, rho_in=1.01, rho_out=0.99)


@pytest.mark.parametrize("steps", [1, 7, 23])
@pytest.mark.parametrize("nx,ny,kind", [
    (2, 3, "lid"), (12, 12, "lid"), (13, 25, "lid"), (65, 33, "lid"), (300, 290, "lid"),
    (3, 13, "pressure"), (24, 12, "pressure"), (37, 40, "pressure"), (620, 90, "pressure")])
def test_squares_match_oracle(nx, ny, kind, steps):
    st = random_state(nx, ny, seed=nx + ny, wall_frac=0.1, lid=kind == "lid",
                      pressure=kind == "pressure")
    bc = LID if kind == "lid" else PRESSURE
    print(f"[case] d2q9 squares {nx}x{ny} {kind} steps={steps}", flush=True)
    sim, d, u = gpu_run(st, steps, graph_chunk=10, **dict(bc))
    ref = oracle_run(st, steps, **dict(bc))
    fl = st.types == 0
    assert np.abs(d - ref.drho)[fl].max(initial=0.0) <= 1e-12
    assert np.abs(u - ref.u).max() <= 1e-12 * max(np.abs(ref.u).max(), 1e-300)
    assert np.all(d[~fl] == 0) and np.all(u[:, ~fl] == 0)
    assert sim.info()["steps_done"] == steps
    sim.close()
