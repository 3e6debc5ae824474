"""The automatic choice of z-segments: as short as one plane on small lattices.
It gives the bits of a fixed tile, and a batch whose lane layouts mix the chunk
tile with short segments fits its work list."""
import numpy as np
import pytest

from paper_2312_14742_amd import inputs, tau1

from gpu_helpers import run_gpu

pytestmark = pytest.mark.gpu

G = (1e-5, -2e-5, 3e-6)


@pytest.mark.parametrize("dims", [(16, 5, 1), (48, 9, 37), (80, 4, 3), (32, 70, 2), (64, 6, 1),
                                  (128, 33, 17), (512, 3, 2), (96, 130, 65)])
@pytest.mark.parametrize("layout", [-1, 0])
def test_automatic_segments_same_bits(dims, layout):
    nx, ny, nz = dims
    solid, drho, u = inputs.random_state(nx, ny, nz, seed=11 + nx + nz)
    print(f"[case] automatic segments {dims} layout={layout}", flush=True)
    auto, oa = run_gpu([(solid, drho, u)], 19, "f32", G, 5, kernel=1, layout=layout)
    tile = 14 if auto.info()["layout"] else 2
    fixed, of = run_gpu([(solid, drho, u)], 19, "f32", G, 5, kernel=1, layout=layout, tile=tile)
    assert oa[0][0].tobytes() == of[0][0].tobytes()
    assert oa[0][1].tobytes() == of[0][1].tobytes()
    auto.close()
    fixed.close()


def test_autotune_mixes_chunk_tile_and_segments():
    """A sample with half of its chunks stored has far more 64-chunk items than
    16-plane row items; beside a sample without chunk records, whose layout
    runs a z-march in the chunk tile's trial, both lists fit."""
    rng = np.random.Generator(np.random.PCG64(3))
    a = (rng.random((32, 8, 64)) < 0.55).astype(np.uint8)
    b = np.zeros((20, 8, 128), np.uint8)
    print("[case] autotune, chunk tile beside short segments", flush=True)
    with tau1.Sim([tau1.Sample(a), tau1.Sample(b)], lattice=19, precision="f32", g=G) as sim, \
            tau1.Sim([tau1.Sample(a), tau1.Sample(b)], lattice=19, precision="f32", g=G,
                     tile=14) as ref:
        sim.autotune(2)
        sim.step(4)
        ref.step(4)
        for i in range(2):
            x, y = sim.moments(i), ref.moments(i)
            assert x[0].tobytes() == y[0].tobytes() and x[1].tobytes() == y[1].tobytes()
