"""D2Q9 under a caller's stream capture, repeated calls that end beside a graph's
length, and batches: several steps per launch must not show."""
import numpy as np
import pytest

import oracle
from paper_2312_14742_amd import tau1

from test_gpu_d2q9 import oracle_run, random_state

pytestmark = pytest.mark.gpu

LID = dict(wall_u=(0.1, 0.02, 0.0), g=(1e-4, -2e-5))


def make(sts, **kw):
    samples = [tau1.Sample(st.types[None], st.drho[None],
                           np.stack([st.u[0][None], st.u[1][None], 0 * st.u[0][None]]))
               for st in sts]
    return tau1.Sim(samples, lattice=9, precision="f64", g=(*LID["g"], 0.0),
                    wall_u=LID["wall_u"], **kw)


def check(sim, i, st, steps):
    d, u = sim.moments(i)
    ref = oracle_run(st, steps, **dict(LID))
    fl = st.types == 0
    assert np.abs(d[0] - ref.drho)[fl].max(initial=0.0) <= 1e-12
    assert np.abs(u[:2, 0] - ref.u).max() <= 1e-12 * max(np.abs(ref.u).max(), 1e-300)


@pytest.mark.parametrize("steps", [2, 4, 10, 20])
def test_captured_steps_replay(steps):
    """An even number of steps, captured once, advances the state at each replay."""
    import torch
    st = random_state(61, 47, seed=steps, wall_frac=0.1, lid=True, pressure=False)
    print(f"[case] d2q9 captured steps={steps}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim = make([st])
        sim.step(steps)
        sim.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(steps)
        for n in range(1, 4):
            graph.replay()
            torch.cuda.synchronize()
            check(sim, 0, st, steps * (1 + n))
        sim.close()


def test_repeated_calls_beside_the_graph_length():
    st = random_state(70, 41, seed=3, wall_frac=0.1, lid=True, pressure=False)
    print("[case] d2q9 repeated calls", flush=True)
    sim = make([st], graph_chunk=20)
    done = 0
    for k in (20, 27, 30, 21, 1, 46, 30, 30, 13):
        sim.step(k)
        done += k
        check(sim, 0, st, done)
    sim.close()


def test_batch_of_different_sizes():
    sts = [random_state(nx, ny, seed=nx, wall_frac=0.1, lid=True, pressure=False)
           for nx, ny in ((3, 5), (64, 31), (130, 90), (12, 200), (33, 33))]
    print("[case] d2q9 batch", flush=True)
    sim = make(sts, graph_chunk=10)
    sim.step(27)
    for i, st in enumerate(sts):
        check(sim, i, st, 27)
    sim.close()
