"""Kernel 0 on rows of a few nodes (one node per thread): in FP64 the bits of the
plain step, and in every precision those of the row kernel, whichever of the two
a context's samples lead to."""
import numpy as np
import pytest

from paper_2312_14742_amd import inputs, tau1

import plain_step
from gpu_helpers import run_gpu

pytestmark = pytest.mark.gpu

G = (1e-5, -2e-5, 3e-6)


@pytest.mark.parametrize("q", [15, 19, 27])
def test_fp64_bits_of_the_plain_step(q):
    for dims in [(1, 300, 20), (2, 1, 4000), (3, 100, 41), (8, 97, 90)]:
        solid, drho, u = inputs.random_state(*dims, seed=sum(dims))
        d, v = plain_step.start(solid, drho, u, G)
        print(f"[case] nodes q={q} {dims}", flush=True)
        sim, _ = run_gpu([(solid, drho, u)], q, "f64", G, 3, kernel=0)
        for _ in range(3):
            d, v = plain_step.step(q, solid, d, v, G)
        ref = plain_step.fields(solid, d, v, G)
        got = sim.moments(0)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]), dims
        sim.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("q", [15, 19, 27])
@pytest.mark.parametrize("shapes", [
    [(1, 300, 40), (70, 9, 8), (64, 5, 6), (2, 3, 1)],      # one node per thread
    [(8, 97, 90), (1, 300, 20), (3, 100, 41), (150, 60, 60)]])  # row windows
def test_batch_has_the_bits_of_each_sample_alone(shapes, q, prec):
    samples = [inputs.random_state(*s, seed=sum(s)) for s in shapes]
    print(f"[case] nodes batch q={q} {shapes} {prec}", flush=True)
    sim, outs = run_gpu(samples, q, prec, G, 5, kernel=0)
    for s, (d, u) in zip(samples, outs):
        with tau1.Sim([tau1.Sample(*s)], lattice=q, precision=prec, g=G, kernel=0) as alone:
            alone.step(5)
            a = alone.moments(0)
            assert np.array_equal(a[0], d) and np.array_equal(a[1], u)
    sim.close()
