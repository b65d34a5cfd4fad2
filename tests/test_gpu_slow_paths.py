"""Particles outside their work item's tile, few and many to a wave (the
wave-wide and the lane-by-lane slow paths of P2G, G2P and the fused launch):
the material drifts without a re-sort, then the grid momentum of the next
substep's P2G is compared with the oracle's P2G of the same state,
|p_gpu - p_orc|_2 / max(|p_orc|_2, sum m |g| dt) <= 1e-5, mass to 1e-6, and one
more substep's positions to 1e-5 dx and velocities to 1e-5 (FP32 sums of 27 terms)."""
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


@pytest.mark.parametrize("block", [4, 8])
@pytest.mark.parametrize("fuse", [0, 1])
@pytest.mark.parametrize("cells", [0.05, 0.6, 2.5])     # drift since the re-sort
def test_drifted_particles(mpm, orc, cells, fuse, block):
    announce("slow paths", "drift", cells, "fuse", fuse, "B", block)
    sc = scenes.small_scene(77, n=6000, res=32, model=scenes.HENCKY_VM, colliders=False, dt=1e-4)
    sub = 12
    speed = cells * sc.dx / (sub * sc.dt)
    sc.v = (0.02 * sc.v + speed * np.array([0.57, 0.57, -0.57], np.float32)).astype(np.float32)
    sim = mpm.Sim([sc])
    sim.set_option(mpm.OPT_BLOCK, block)
    sim.set_option(mpm.OPT_FUSE, fuse)
    sim.set_option(mpm.OPT_SORT_EVERY, 1000)
    sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
    sim.step(sub)
    x, v, C, F = sim.get_state(0)
    assert sim.sync() == mpm.OK
    o = orc.Oracle(sc, x=x, v=v, C=C, F=F)
    om, op = o.p2g()
    sim.step(1)
    gm, gp = sim.get_grid(0)
    assert rel_l2(gm, om) <= 1e-6
    assert rel_l2(gp, op, momentum_floor(sc, om.sum())) <= 1e-5
    o = orc.Oracle(sc, x=x, v=v, C=C, F=F)
    o.step(1)
    x1, v1, _, _ = sim.get_state(0)
    assert np.abs(x1 - o.x).max() <= 1e-5 * sc.dx + 1e-7
    assert rel_l2(v1, o.v) <= 1e-5
    sim.close()
