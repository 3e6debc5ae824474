"""Shared-row z-march launches of more than 2048 blocks of four rows, far more than
are resident at a time.  (Where a workgroup takes two blocks, the second one's
first rows go to the LDS slots that the waves still read at the end of the
first: an item that ends at an odd plane and one that starts at an even plane
use the same slot.)  The bits have to be those of a few long segments."""
import numpy as np
import pytest

from paper_2312_14742_amd import inputs, tau1

pytestmark = pytest.mark.gpu

G = (1e-5, -2e-5, 3e-6)
GRID = 2048


def blocks(sim):
    return sim.info()["work_items"] // 4


def same(a, b, n):
    for i in range(n):
        x, y = a.moments(i), b.moments(i)
        assert x[0].tobytes() == y[0].tobytes() and x[1].tobytes() == y[1].tobytes(), i


@pytest.mark.parametrize("q,prec", [(19, "f32"), (15, "f32"), (27, "f16")])
@pytest.mark.parametrize("dims,tile,one", [
    ((64, 3600, 33), 12, 15),       # packed, segments of 16, the last one of one plane
    ((64, 3600, 33), 4, 7),         # dense
    ((128, 376, 81), -1, 15),       # automatic segments
    ((96, 1100, 127), -1, 15)])
def test_several_items_per_workgroup(q, prec, dims, tile, one):
    nx, ny, nz = dims
    s = inputs.random_state(nx, ny, nz, seed=50 + nx + nz)
    print(f"[case] item passes q={q} {prec} {dims} tile={tile}", flush=True)
    with tau1.Sim([tau1.Sample(*s)], lattice=q, precision=prec, g=G, kernel=1, tile=tile) as many, \
            tau1.Sim([tau1.Sample(*s)], lattice=q, precision=prec, g=G, kernel=1, tile=one) as ref:
        assert blocks(ref) <= GRID
        if tile >= 0:
            assert blocks(many) > GRID
        for _ in range(3):
            many.step(4)
            ref.step(4)
            same(many, ref, 1)


@pytest.mark.parametrize("tile,one", [(12, 15), (4, 7), (-1, 15)])
def test_several_items_per_workgroup_one_launch(tile, one):
    """A batch of several row lengths in one launch: a workgroup may take items
    of rows of different lengths, whose slots lie at different places."""
    shapes = [(64, 1200, 17), (320, 400, 17), (96, 1100, 33), (256, 300, 33), (160, 900, 19)]
    samples = [inputs.random_state(*d, seed=70 + d[0]) for d in shapes]
    print(f"[case] item passes, one launch, tile={tile}", flush=True)
    mk = [tau1.Sample(*s) for s in samples]
    with tau1.Sim(mk, lattice=19, precision="f32", g=G, kernel=1, tile=tile,
                  batch_graph=3) as many, \
            tau1.Sim(mk, lattice=19, precision="f32", g=G, kernel=1, tile=one,
                     batch_graph=1) as ref:
        assert many.info()["launches_per_step"] == 1
        if tile >= 0:
            assert blocks(many) > GRID
        for _ in range(3):
            many.step(4)
            ref.step(4)
            same(many, ref, len(shapes))
