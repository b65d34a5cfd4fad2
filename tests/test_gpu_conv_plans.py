"""The 3^3 and upsampling convolutions on tiles of several positions: 4, 6 and 8
rows to a wave, positions and channels over several waves, boxes that no tile
divides, channel slices that are no 16-byte pieces, a halo of more than 64 KB of
LDS.  The shapes are asked of the planner first (a change of it that moves a
case to another kind of tile fails here, not silently).

Against FP64 on BF16-rounded inputs: FP32 outputs within 1e-5 * sum |terms|,
BF16 outputs within one BF16 rounding more, channels outside the slice untouched."""
import numpy as np
import pytest

from gpu_util import announce
from nn_plans import Plans

pytestmark = pytest.mark.gpu

CASES = [
    # kind, n, input spatial, cx, x_off, cin, cy, y_off, cout, rows, waves along positions, LDS past 64 KB
    ("c3", 8, (33, 17, 39), 36, 4, 32, 16, 0, 16, 6, 3, False),
    ("c3", 7, (28, 22, 29), 40, 8, 32, 23, 3, 20, 6, 4, False),
    ("c3", 8, (34, 13, 40), 32, 0, 32, 32, 0, 32, 8, 2, False),
    ("c3", 5, (38, 10, 35), 32, 0, 32, 64, 0, 64, 4, 2, False),
    ("c3", 8, (13, 22, 35), 64, 0, 64, 128, 0, 128, 6, 4, False),
    ("c3", 8, (39, 24, 38), 128, 0, 128, 24, 4, 20, 6, 6, True),
    ("up", 8, (13, 12, 17), 44, 12, 32, 20, 0, 20, 4, 3, False),
    ("up", 7, (13, 9, 17), 32, 0, 32, 64, 0, 64, 6, 2, False),
    ("up", 5, (16, 7, 13), 96, 0, 96, 130, 2, 128, 8, 3, False),
]


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return Plans(str(tmp_path_factory.mktemp("nn_plan")))


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{'x'.join(map(str, c[2]))}-{c[5]}to{c[8]}" for c in CASES])
def test_planned_tiles(plans, case):
    import torch
    from paper_2302_04659_amd import unet
    kind, n, sp, cx, x_off, cin, cy, y_off, cout, rows, waves, big = case
    announce("nn conv plans", *case)
    p = plans.conv(unet.KIND[kind], n, *sp, cin, cout)
    osp = tuple(2 * a for a in sp) if kind == "up" else sp
    assert (p["FR"], p["PW"], p["lds"] > 65536) == (rows, waves, big) and p["TZ"] > 1 and p["TX"] > 1
    g = torch.Generator(device="cpu").manual_seed(300 + CASES.index(case))
    bf = lambda t: t.to(torch.bfloat16).double()
    X = bf(torch.randn((n,) + sp + (cx,), generator=g)).cuda()
    W = bf(torch.randn((27, cin, cout), generator=g) / np.sqrt(27 * cin)).cuda()
    b = (0.1 * torch.randn(cout, generator=g)).cuda()

    def reference(x, w, bias):
        if kind == "up":
            x = x.repeat_interleave(2, 1).repeat_interleave(2, 2).repeat_interleave(2, 3)
        pad = torch.zeros((n, osp[0] + 2, osp[1] + 2, osp[2] + 2, cin), dtype=torch.float64, device="cuda")
        pad[:, 1:-1, 1:-1, 1:-1] = x
        y = bias.double().expand(n * osp[0] * osp[1] * osp[2], cout).clone()
        for t in range(27):
            a, c, e = t // 9, t // 3 % 3, t % 3
            y += pad[:, a:a + osp[0], c:c + osp[1], e:e + osp[2]].reshape(-1, cin) @ w[t]
        return y.reshape((n,) + osp + (cout,))

    xs = X[..., x_off:x_off + cin]
    ref, bound = reference(xs, W, b), reference(xs.abs(), W.abs(), b.abs())
    L, s = unet.nn_lib(), torch.cuda.current_stream().cuda_stream
    x_d, w_d = X.to(torch.bfloat16).contiguous(), W.float().contiguous()
    fw = torch.zeros(27 * cin * ((cout + 15) // 16 * 16), dtype=torch.int16, device="cuda")
    assert L.mpm_nn_pack(w_d.data_ptr(), unet.KIND[kind], cin, cout, 0, fw.data_ptr(), s) == 0
    y = torch.full((n,) + osp + (cy,), 1.0, dtype=torch.bfloat16, device="cuda")
    y32 = torch.full(ref.shape, float("nan"), device="cuda")
    assert L.mpm_nn_conv(unet.KIND[kind], x_d.data_ptr(), n, *sp, cx, x_off, cin, fw.data_ptr(), b.data_ptr(), 0,
                         y.data_ptr(), cy, y_off, cout, y32.data_ptr(), cout, s) == 0
    assert bool(((y32.double() - ref).abs() <= 1e-5 * bound + 1e-30).all())
    got = y[..., y_off:y_off + cout].double()
    assert bool(((got - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * bound + 1e-30).all())
    rest = torch.cat([y[..., :y_off], y[..., y_off + cout:]], dim=-1)
    assert bool((rest == 1.0).all())
