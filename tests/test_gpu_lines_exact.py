"""Kernel 0's arithmetic.  FP64, the reference of the other modes, is the plain
evaluation of the update, bit for bit; no rounding of FP32 leans to one side.
Sizes at the edges of the row kernel's windows and z-segments, and rows of a few
nodes."""
import numpy as np
import pytest

import oracle
from paper_2312_14742_amd import inputs

import plain_step
from gpu_helpers import run_gpu

pytestmark = pytest.mark.gpu

G = (1e-5, -2e-5, 3e-6)
DIMS = [(1, 5, 3), (3, 4, 1), (8, 6, 5), (17, 16, 9), (62, 3, 5), (63, 2, 4), (64, 3, 4),
        (125, 4, 3), (187, 3, 2)]


def same(got, ref):
    return np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("q", [15, 19, 27])
def test_fp64_bits_of_the_plain_step(q):
    for dims in DIMS:
        solid, drho, u = inputs.random_state(*dims, seed=sum(dims))
        d, v = plain_step.start(solid, drho, u, G)
        print(f"[case] exact q={q} {dims}", flush=True)
        sim, out = run_gpu([(solid, drho, u)], q, "f64", G, 0, kernel=0)
        for n in (1, 6):
            sim.step(n)
            for _ in range(n):
                d, v = plain_step.step(q, solid, d, v, G)
            assert same(sim.moments(0), plain_step.fields(solid, d, v, G)), (dims, n)
        sim.close()


@pytest.mark.parametrize("q", [15, 19, 27])
@pytest.mark.parametrize("dims", [(48, 40, 36), (150, 40, 33), (64, 50, 45)])
def test_fp64_bits_of_the_oracle(q, dims):
    """g = 0: the state is the oracle's (v = u), and so are its bits."""
    s = inputs.random_state(*dims, seed=q)
    print(f"[case] exact f64 oracle q={q} {dims}", flush=True)
    sim, out = run_gpu([s], q, "f64", (0.0, 0.0, 0.0), 20, kernel=0)
    ref = oracle.run(q, oracle.State(*s), (0.0, 0.0, 0.0), 20)
    assert same(out[0], (ref.drho, ref.u))
    sim.close()


@pytest.mark.parametrize("q", [15, 19, 27])
@pytest.mark.parametrize("dims", [(150, 50, 40), (2, 400, 380)])
def test_fp32_step_has_no_bias(q, dims):
    """The regression of one step's error on the exact value.  The weights' unit
    (1/72, 1/36, 1/216) is 7.45e-9 too large as a float: used as it is, density or
    velocity has that slope in every step.  Roundings to nearest of a random state
    scatter by about 2^-24 of the summed terms, a few times the value: over 3e5
    nodes the slope of that scatter is below 1e-9, well within the bound of half the
    unit's."""
    solid, drho, u = inputs.random_state(*dims, seed=q)
    g = (0.0, 0.0, 0.0)
    print(f"[case] fp32 bias q={q} {dims}", flush=True)
    sim, out = run_gpu([(solid, drho, u)], q, "f32", g, 0, kernel=0)
    ref = oracle.run(q, oracle.State(solid, *out[0]), g, 1)   # from the state as stored
    sim.step(1)
    got = sim.moments(0)
    sim.close()
    for name, a, b in (("drho", got[0], ref.drho), ("u", got[1], ref.u)):
        slope = np.sum((a - b) * b) / np.sum(b * b)
        print(f"[err] fp32 bias q={q} {dims} {name}: {slope:.2e}", flush=True)
        assert abs(slope) <= 0.5 * 7.45e-9, (name, slope)
