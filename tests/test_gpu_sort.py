"""The counting sort's order, straight from the creation order: a permutation
of each scene's own particles, in non-decreasing Morton order of their grid
blocks; sizes around a wave, a workgroup and its last partial one, on both
sides of the size from which a thread takes eight particles."""
import numpy as np
import pytest

from gpu_util import announce
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


def _morton(b):
    key = np.zeros(len(b), np.int64)
    for bit in range(8):
        for d in range(3):
            key |= ((b[:, d] >> bit) & 1) << (3 * bit + d)
    return key


@pytest.mark.parametrize("counts", [(1,), (63, 65, 1), (255, 257, 2049), (40001, 2047), (524287,), (524288,),
                                    (300007, 250001, 100)])
@pytest.mark.parametrize("same", [0, 1])       # 1: every particle of a scene in one block
def test_sort_order(mpm, counts, same):
    announce("sort order", counts, same)
    batch = [scenes.small_scene(s, n=n, res=32, model=scenes.NEO_HOOKEAN, colliders=False) for s, n in enumerate(counts)]
    rng = np.random.default_rng(9)
    for sc in batch:
        u = rng.uniform(12.6, 16.4, (sc.n, 3)) if same else rng.uniform(3.6, 28.4, (sc.n, 3))
        sc.x = (u * sc.dx).astype(np.float32)
    sim = mpm.Sim(batch)
    order, lo = sim.order(), 0
    for sc in batch:
        pid = order[lo:lo + sc.n] - lo
        assert np.array_equal(np.sort(pid), np.arange(sc.n))
        base = np.floor(sc.x * np.float32(1.0 / sc.dx) - np.float32(0.5)).astype(np.int64) // 4
        assert np.all(np.diff(_morton(base)[pid]) >= 0)
        lo += sc.n
    sim.close()


@pytest.mark.parametrize("n_scenes", [1, 2, 3, 4, 5])      # 512 bins each: up to 2,048 planned by one workgroup
def test_plan_covers_every_scene(mpm, orc, n_scenes):
    """The work lists of scenes planned together: every scene's grid mass after
    a substep is the oracle's (a block or item left out, or counted twice, is a
    particle's mass off; FP32 sums, 1e-6)."""
    announce("plan", n_scenes)
    batch = [scenes.small_scene(s, n=700 + 431 * s, res=32, model=scenes.NEO_HOOKEAN, colliders=False)
             for s in range(n_scenes)]
    sim = mpm.Sim(batch)
    sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
    sim.step(1)
    for s, sc in enumerate(batch):
        gm, _ = sim.get_grid(s)
        om, _ = orc.Oracle(sc).p2g()
        assert np.linalg.norm(gm - om) <= 1e-6 * np.linalg.norm(om)
    assert sim.sync() >= 0
    sim.close()
