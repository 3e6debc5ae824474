"""The numpy step of the exactness tests against the oracle, on the CPU."""
import numpy as np
import pytest

import oracle
from paper_2312_14742_amd import inputs

import plain_step


@pytest.mark.parametrize("q", [15, 19, 27])
def test_step_is_the_oracles(q):
    """g = 0, where the library's state is the oracle's (v = u): bit for bit."""
    solid, drho, u = inputs.random_state(13, 9, 7, seed=q)
    g = (0.0, 0.0, 0.0)
    d, v = plain_step.start(solid, drho, u, g)
    for _ in range(10):
        d, v = plain_step.step(q, solid, d, v, g)
    ref = oracle.run(q, oracle.State(solid, drho, u), g, 10)
    assert np.array_equal(d, ref.drho) and np.array_equal(v, ref.u)
