"""A state handed in and given out keeps its bits whichever kernels convert it:
all scenes at once (sorted as they are read) or scene by scene (converted, sorted
later), read back before or after the sort.  The particles fill blocks that share
no grid nodes, one work item each, so nothing depends on an order of additions:
C as read back, the node sums of the P2G and the network's input are compared bit
for bit.  The strains reach over the range of the Hencky series, particles past
it and within it side by side."""
import numpy as np
import pytest

from gpu_util import announce
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu

RES, PER_BLOCK = 32, 64   # 64: the smallest work item, so no block is cut in two


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


def _scene(seed, model, per_block=PER_BLOCK):
    rng = np.random.default_rng(seed)
    blocks = np.array([(i, j, k) for i in (1, 4) for j in (1, 4) for k in (1, 4)])
    x = (blocks[:, None, :] * 4 + 0.5 + rng.uniform(0.01, 3.99, size=(8, per_block, 3))) / RES
    n = 8 * per_block
    order = rng.permutation(n)                       # creation order: the blocks' particles mixed
    x = x.reshape(n, 3)[order].astype(np.float32)
    F = np.eye(3) + rng.choice([0.01, 0.06, 0.15], n)[:, None, None] * rng.normal(size=(n, 3, 3))
    sc = scenes.Scene("bits", x, rng.normal(size=(n, 3)).astype(np.float32), RES, 1.0 / RES, 5e-5, (0.0, -9.8, 0.0), 3,
                      model, 1e4, 0.3, 1000.0, 0.0, 0, (1.0 / RES) ** 3 / 8, [], np.zeros((1, 0, 7)), np.zeros((1, 0, 6)))
    return sc, (x, sc.v, (2 * rng.normal(size=(n, 3, 3))).astype(np.float32), F.astype(np.float32))


def _features(sim):
    import torch
    feat = torch.zeros((len(sim.scenes), RES, RES, RES, 8), device="cuda")
    grid0 = torch.zeros((len(sim.scenes), RES, RES, RES, 4), device="cuda")
    torch.cuda.synchronize()
    sim.sur_features(feat, grid0)
    assert sim.sync() == 0
    return feat.cpu().numpy(), grid0.cpu().numpy()


@pytest.mark.parametrize("model", [scenes.NEO_HOOKEAN, scenes.HENCKY_VM, scenes.FLUID])
def test_state_bits_do_not_follow_the_route(mpm, model):
    announce("state bits", model)
    made = [_scene(s, model) for s in (1, 2)]
    whole = tuple(np.concatenate([st[k] for _, st in made]) for k in range(4))
    got = []
    for per_scene in (False, True, False):
        sim = mpm.Sim([sc for sc, _ in made])
        if per_scene:
            for s, (_, st) in enumerate(made):
                sim.set_state(*st, scene=s)
        else:
            sim.set_state(*whole)
        before = sim.get_state(-1)[2]
        feat, grid0 = _features(sim)                 # sorts the particles that are not yet
        got.append((before, sim.get_state(-1)[2], feat, grid0))
        sim.close()
    for other in got[1:]:
        for name, a, b in zip(("C", "C after the sort", "features", "node sums"), got[0], other):
            np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32), err_msg=name)
    np.testing.assert_array_equal(got[0][0], got[0][1])


@pytest.mark.parametrize("chunk", [128, 2048])
def test_surrogate_input_does_not_follow_the_batch(mpm, chunk):
    """A small context cuts its blocks to the number of CUs, a large one does not: the
    network's input of a scene is the same in both, and from call to call, as long as
    its blocks fit the chunk."""
    announce("surrogate input", chunk)
    small = [_scene(3, scenes.HENCKY_VM, per_block=120)]
    filler = _scene(4, scenes.HENCKY_VM, per_block=4 * chunk * 256 // 8 // 3)
    got = []
    for made in (small, small + [filler], small):
        sim = mpm.Sim([sc for sc, _ in made])
        sim.set_option(mpm.OPT_CHUNK, chunk)
        sim.set_state(*(np.concatenate([st[k] for _, st in made]) for k in range(4)))
        for _ in range(2):
            feat, grid0 = _features(sim)
            got.append((feat[0], grid0[0]))
        sim.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))
