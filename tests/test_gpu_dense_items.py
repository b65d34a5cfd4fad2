"""Material that is dense at rest (40 particles to a cell) filling its blocks only
in part: a small context adds up the same work items as one large enough not to
cut any, so node sums agree bit for bit (the blocks share no node, one item each,
and the integer sums of an item have no order)."""
import numpy as np
import pytest

from gpu_util import announce
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu

RES = 32


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


def _scene(seed, n, lo, hi, per_cell):
    rng = np.random.default_rng(seed)
    x = ((rng.uniform(lo, hi, size=(n, 3)) + 8 * rng.choice([0, 2], size=(n, 1)) + 0.5) / RES).astype(np.float32)
    return scenes.Scene("dense", x, rng.normal(size=(n, 3)).astype(np.float32), RES, 1.0 / RES, 1e-4, (0.0, -9.8, 0.0), 3,
                        scenes.FLUID, 1e4, 0.3, 1000.0, 0.0, 0, (1.0 / RES) ** 3 / per_cell, [], np.zeros((1, 0, 7)),
                        np.zeros((1, 0, 6)))


@pytest.mark.parametrize("block", [4, 8])
def test_part_filled_dense_blocks(mpm, block):
    # two cubes of 4^3 cells (block edge 8) or 2^3 cells (4), an eighth of their blocks
    announce("dense items", block)
    edge = block // 2
    sc = _scene(1, 2 * 40 * edge ** 3, 8.01, 8.0 + edge - 0.01, 40.0)
    filler = _scene(2, 2 * 8192 * 128 + 1024, 8.01, 15.99, 40.0)      # over 256 CUs x 8,192 particles
    grids = []
    for made in ([sc], [sc, filler]):
        sim = mpm.Sim(made)
        sim.set_option(mpm.OPT_BLOCK, block)
        sim.set_option(mpm.OPT_CHUNK, 8192)
        sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
        sim.set_state(*(np.concatenate(a) for a in zip(*[(m.x, m.v, np.zeros((m.n, 3, 3), np.float32),
                                                           np.tile(np.eye(3, dtype=np.float32), (m.n, 1, 1))) for m in made])))
        sim.step(1)
        grids.append(sim.get_grid(0))
        sim.close()
    for a, b in zip(*grids):
        np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
