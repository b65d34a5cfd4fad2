"""Particles past the grid's edge (their base cell is clamped, the run goes on
with a warning): the weights stay the quadratics of the offset, which sum to 1
for any offset, so mass and momentum are kept.  Few and many of them to a wave
(the wave-wide and the lane-by-lane slow paths), P2G, G2P and the fused launch,
against the same substeps in FP64.

Bars: node sums 1e-5 (FP32, 27 terms, sum |w| at most 3 an axis, sums of nodes
at worst 5 times smaller than their terms), velocities 1e-4 (their quotients)."""
import numpy as np
import pytest

from gpu_util import announce, rel_l2
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu

RES, DT, RHO = 16, 1e-4, 1000.0
DX = 1.0 / RES


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


def _weights(x):
    xi = x / DX
    base = np.clip(np.floor(xi - 0.5).astype(int), 0, RES - 3)
    f = xi - base
    return base, f, np.stack([0.5 * (1.5 - f) ** 2, 0.75 - (f - 1) ** 2, 0.5 * (f - 0.5) ** 2], 2)


def _stencil(x):
    base, f, w = _weights(x)
    for o in np.ndindex(3, 3, 3):
        i = base + o
        yield (i[:, 0], i[:, 1], i[:, 2]), w[:, 0, o[0]] * w[:, 1, o[1]] * w[:, 2, o[2]], (np.array(o) - f) * DX


def _p2g(x, v, C, mass):
    gm, gp = np.zeros((RES,) * 3), np.zeros((RES,) * 3 + (3,))
    for i, w, d in _stencil(x):
        np.add.at(gm, i, w * mass)
        np.add.at(gp, i, (w * mass)[:, None] * (v + np.einsum("pij,pj->pi", C, d)))
    return gm, gp


def _g2p(x, gm, gp):
    """No gravity, no stress: node velocity, walls of 3 nodes, back to the particles."""
    vg = np.where(gm[..., None] > 0, gp / np.where(gm == 0, 1, gm)[..., None], 0.0)
    for a in range(3):
        lo, hi = [slice(None)] * 3, [slice(None)] * 3
        lo[a], hi[a] = slice(0, 3), slice(RES - 3, RES)
        vg[tuple(lo) + (a,)] = np.maximum(vg[tuple(lo) + (a,)], 0)
        vg[tuple(hi) + (a,)] = np.minimum(vg[tuple(hi) + (a,)], 0)
    v, C = np.zeros_like(x), np.zeros(x.shape + (3,))
    for i, w, d in _stencil(x):
        v += w[:, None] * vg[i]
        C += 4 / DX ** 2 * w[:, None, None] * vg[i][:, :, None] * d[:, None, :]
    return x + DT * v, v, C


@pytest.mark.parametrize("block", [4, 8])
@pytest.mark.parametrize("inside", [40, 3])              # inside particles to one outside
@pytest.mark.parametrize("axis,high", [(0, False), (2, True)])
def test_particles_past_the_edge(mpm, axis, high, inside, block):
    announce("past the edge", axis, high, inside, block)
    rng = np.random.default_rng(7)
    n_out = 4 * 4 * 12 if inside == 3 else 4 * 4 * 2
    n = n_out * (inside + 1)
    x = np.empty((n, 3))
    out = np.arange(n) % (inside + 1) == 0
    edge = np.where(out, rng.uniform(-0.3, -0.02, n), rng.uniform(0.5, 1.5, n))
    x[:, axis] = (RES - 1 - edge if high else edge) * DX
    for a in range(3):
        if a != axis:
            x[:, a] = rng.uniform(6.0, 10.0, n) * DX
    x = x.astype(np.float32)
    v = rng.normal(size=(n, 3)).astype(np.float32)
    C = (2 * rng.normal(size=(n, 3, 3))).astype(np.float32)
    vol = DX ** 3 / 8
    sc = scenes.Scene("edge", x, v, RES, DX, DT, (0.0, 0.0, 0.0), 3, scenes.NEO_HOOKEAN, 1e-3, 0.3, RHO, 0.0, 0, vol, [],
                      np.zeros((1, 0, 7)), np.zeros((1, 0, 6)))
    ref = x.astype(np.float64), v.astype(np.float64), C.astype(np.float64)
    grids, states = [], []
    for _ in range(3):
        grids.append(_p2g(*ref, RHO * vol))
        ref = _g2p(ref[0], *grids[-1])
        states.append(ref)
    np.testing.assert_allclose(grids[0][0].sum(), n * RHO * vol, rtol=1e-9)
    for fuse in (0, 1):
        for steps in (1, 3):                             # in one call: the last P2G of three is a fused launch
            sim = mpm.Sim([sc])
            sim.set_option(mpm.OPT_BLOCK, block)
            sim.set_option(mpm.OPT_FUSE, fuse)
            sim.set_option(mpm.OPT_CAPTURE_GRID, 1)
            sim.set_state(x, v, C, np.tile(np.eye(3, dtype=np.float32), (n, 1, 1)))
            sim.step(steps)
            assert sim.sync() == 1                       # MPM_WARN_CLAMPED
            gm, gp = sim.get_grid(0)
            x1, v1, _, _ = sim.get_state(0)
            sim.close()
            what = (fuse, steps)
            assert rel_l2(gm.reshape((RES,) * 3), grids[steps - 1][0]) <= 1e-5, what
            assert rel_l2(gp.reshape((RES,) * 3 + (3,)), grids[steps - 1][1]) <= 1e-5, what
            assert rel_l2(v1, states[steps - 1][1]) <= 1e-4, what
            assert np.abs(x1 - states[steps - 1][0]).max() <= 1e-5 * DX + 1e-7, what
