"""Kernel 0 is the plain evaluation of the update, bit for bit, in every
precision: FP64 mode is the reference of the others, and no operation of the
FP32 modes is less than correctly rounded.  Sizes at the edges of the row
kernel's windows and z-segments, and rows of a few nodes."""
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


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("q", [15, 19, 27])
def test_bits_of_the_plain_step(q, prec):
    for dims in DIMS:
        solid, drho, u = inputs.random_state(*dims, seed=sum(dims))
        d, v = plain_step.start(solid, drho, u, G, prec)
        print(f"[case] exact q={q} {prec} {dims}", flush=True)
        sim, out = run_gpu([(solid, drho, u)], q, prec, G, 0, kernel=0)
        for n in (1, 6):
            sim.step(n)
            for _ in range(n):
                d, v = plain_step.step(q, solid, d, v, G, prec)
            assert same(sim.moments(0), plain_step.fields(solid, d, v, G)), (dims, n)
        sim.close()


def test_bits_after_many_steps():
    """A rounding that leans to one side in every step would collect here."""
    solid, drho, u = inputs.random_state(37, 11, 9, seed=4)
    d, v = plain_step.start(solid, drho, u, G, "f32")
    print("[case] exact f32, 500 steps", flush=True)
    sim, _ = run_gpu([(solid, drho, u)], 19, "f32", G, 500, kernel=0)
    for _ in range(500):
        d, v = plain_step.step(19, solid, d, v, G, "f32")
    assert same(sim.moments(0), plain_step.fields(solid, d, v, G))
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
