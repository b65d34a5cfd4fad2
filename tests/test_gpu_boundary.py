"""State in and out through device arrays (taken by the boundary kernels
themselves) against the same calls with host arrays (through the context's own
buffer), bit for bit: sizes around a workgroup, one scene of several, arrays
that start off a 16-byte boundary, and arrays that overlap (which take the
buffer, so the later array wins where two share memory)."""
import numpy as np
import pytest

from gpu_util import announce, random_state
from paper_2302_04659_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    from paper_2302_04659_amd import mpm as m
    return m


def _sim(mpm, counts):
    return mpm.Sim([scenes.small_scene(s, n=n, res=16, model=m, colliders=False)
                    for s, (n, m) in enumerate(zip(counts, (scenes.HENCKY_VM, scenes.NEO_HOOKEAN, scenes.FLUID)))])


def _state(sim, scene, seed):
    rng = np.random.default_rng(seed)
    scs = sim.scenes if scene < 0 else [sim.scenes[scene]]
    cf = [random_state(sc, seed) for sc in scs]
    x = np.concatenate([sc.x for sc in scs])
    return (x, rng.normal(size=x.shape).astype(np.float32), np.concatenate([c for c, _ in cf]),
            np.concatenate([f for _, f in cf]))


@pytest.mark.parametrize("counts,scene,off", [((1,), -1, 0), ((255, 1, 257), -1, 1), ((300, 513, 64), 1, 3),
                                              ((256, 1024, 5), -1, 0)])
def test_device_arrays_match_host_arrays(mpm, counts, scene, off):
    import torch
    announce("boundary", counts, scene, off)
    sim, ref = _sim(mpm, counts), _sim(mpm, counts)
    st = _state(sim, scene, 5)
    ref.set_state(*st, scene=scene)
    buf = torch.zeros(sum(a.size for a in st) + 8, device="cuda")
    dev, pos = [], off
    for a in st:
        dev.append(buf[pos:pos + a.size].view(a.shape))
        dev[-1].copy_(torch.from_numpy(a))
        pos += a.size
    torch.cuda.synchronize()
    sim.set_state_device(*dev, scene=scene)
    for step in (0, 1):
        if step:
            ref.set_state(*_state(ref, -1, 6))
            sim.set_state(*_state(sim, -1, 6))
        want = ref.get_state(scene)
        buf.zero_()
        torch.cuda.synchronize()
        sim.get_state_device(*dev, scene=scene)
        assert sim.sync() >= 0
        for w, d in zip(want, dev):
            assert np.array_equal(w.reshape(-1), d.cpu().numpy().reshape(-1))
        assert float(buf[:off].abs().sum()) == 0.0 and float(buf[pos:].abs().sum()) == 0.0
    sim.close()
    ref.close()


def test_overlapping_arrays_take_the_buffer(mpm):
    import torch
    sim = _sim(mpm, (700,))
    want = sim.get_state(0)
    F = torch.zeros(700 * 9, device="cuda")
    C = torch.zeros(700 * 9, device="cuda")
    v = torch.zeros(700 * 3, device="cuda")
    torch.cuda.synchronize()
    sim.get_state_device(F[:2100], v, C, F)      # x inside F: F is written last
    sim.sync()
    assert np.array_equal(F.cpu().numpy(), want[3].reshape(-1))
    sim.close()
