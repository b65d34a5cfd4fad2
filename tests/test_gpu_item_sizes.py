"""Work items cut to the number of CUs: contexts with fewer particles than
CUs x chunk (256 CUs: items of 64 up to 16,384 particles, then 128, ...) and
the first sizes above, against the oracle: the grid mass and momentum of the
second substep's P2G from the state after the first (mass 1e-6, momentum 1e-5,
FP32 sums of a node's contributions in fixed point), separate and fused
launches."""
import numpy as np
import pytest

from gpu_util import announce, momentum_floor, rel_l2
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


@pytest.mark.parametrize("n,block,fuse", [(1, 4, 1), (65, 8, 0), (16384, 8, 1), (16385, 4, 0), (16385, 8, 1),
                                          (40001, 4, 1)])
def test_item_sizes(mpm, orc, n, block, fuse):
    announce("item sizes", "n", n, "B", block, "fuse", fuse)
    sc = scenes.small_scene(91, n=n, res=32, model=scenes.HENCKY_VM, dt=1e-4)
    sim = mpm.Sim([sc])
    sim.set_option(mpm.OPT_BLOCK, block)
    sim.set_option(mpm.OPT_FUSE, fuse)
    sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
    sim.step(1)
    x, v, C, F = sim.get_state(0)
    o = orc.Oracle(sc, x=x, v=v, C=C, F=F)
    om, op = o.p2g()
    assert sim.sync() == mpm.OK
    sim2 = mpm.Sim([sc])
    sim2.set_option(mpm.OPT_BLOCK, block)
    sim2.set_option(mpm.OPT_FUSE, fuse)
    sim2.set_option(mpm.OPT_CAPTURE_GRID, 1)
    sim2.step(2)                       # substep 1's P2G is fused into substep 0's G2P
    gm, gp = sim2.get_grid(0)
    assert rel_l2(gm, om) <= 1e-6
    assert rel_l2(gp, op, momentum_floor(sc, om.sum())) <= 1e-5
    sim.close()
    sim2.close()


def test_dense_blocks_keep_their_items(mpm):
    """40 particles to a cell in a small context: the blocks are not cut, so the
    launch configuration with the same chunk gives the same sums, bit for bit
    (one item per block: no order of float additions enters between blocks that
    share no node)."""
    rng = np.random.default_rng(3)
    n = 2 * 2560
    lo = np.repeat([4.5, 16.5], n // 2)[:, None] + rng.uniform(0.01, 3.99, size=(n, 3))
    sc = scenes.small_scene(92, n=n, res=32, model=scenes.FLUID, colliders=False, dt=1e-4)
    sc.x = (lo * sc.dx).astype(np.float32)
    sc.v = rng.normal(size=(n, 3)).astype(np.float32)
    grids = []
    for copies in (1, 230):                # 5,120 particles, and enough scenes for chunks of 8,192 uncut
        announce("dense blocks, scenes", copies)
        sim = mpm.Sim([sc] + [scenes.small_scene(93, n=9200, res=32, model=scenes.FLUID, colliders=False)] * (copies - 1))
        sim.set_option(mpm.OPT_CHUNK, 8192)
        sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
        sim.step(1)
        grids.append(sim.get_grid(0))
        sim.close()
    assert np.array_equal(grids[0][0], grids[1][0]) and np.array_equal(grids[0][1], grids[1][1])
