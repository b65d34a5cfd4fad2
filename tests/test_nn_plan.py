"""Invariants of the convolutions' tile plans that the kernels rely on (waves within
the launch bounds, halo extents, LDS, exact reciprocals, covered outputs), over
random boxes and channel counts of every kind."""
import random

import numpy as np
import pytest

from nn_plans import Plans

LDS_OF_A_CU = 160 * 1024


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return Plans(str(tmp_path_factory.mktemp("nn_plan")))


def _shape(r, kind):
    n = r.choice([1, 1, 2, 3, 8, 64])
    d, h, w = (r.choice([r.randint(1, 12), r.randint(1, 64), r.randint(1, 300)]) for _ in range(3))
    if kind == 2:
        d, h, w = 2 * d, 2 * h, 2 * w
    return n, d, h, w


def _out(kind, d, h, w):
    return (2 * d, 2 * h, 2 * w) if kind == 1 else ((d // 2, h // 2, w // 2) if kind == 2 else (d, h, w))


def _exact(magic, d, most):
    v = np.arange(most, dtype=np.uint64)
    return d == 1 or np.array_equal((v * np.uint64(magic)) >> np.uint64(32), v // np.uint64(d))


@pytest.mark.parametrize("seed", range(4))
def test_convolution_plans(plans, seed):
    r = random.Random(seed)
    for _ in range(150):
        kind, cin, cout = r.choice([(0, 8, r.choice([16, 32])), (0, 32 * r.randint(1, 4), r.choice([4, 16, 20, 32, 64, 128])),
                                    (1, 32 * r.randint(1, 4), r.choice([16, 32, 64, 128]))])
        n, d, h, w = _shape(r, kind)
        p, (od, oh, ow) = plans.conv(kind, n, d, h, w, cin, cout), _out(kind, d, h, w)
        what = (kind, n, d, h, w, cin, cout, p)
        TZ, TX, FR = p["TZ"], p["TX"], p["FR"]
        assert p["tiles_x"] * TX >= ow and p["tiles_y"] * FR >= oh and p["tiles_z"] * TZ >= od, what
        # halo rows and columns that the taps of a tile starting at o0 reach (upsampling: coarse rows)
        for o0 in (0, TX, 3 * TX):
            need = TX + 2 if kind == 0 else ((o0 + TX) >> 1) - ((o0 - 1) >> 1) + 1
            assert p["HX"] >= need, what
        for o0 in (0, TZ, 3 * TZ):
            need = TZ + 2 if kind == 0 else ((o0 + TZ) >> 1) - ((o0 - 1) >> 1) + 1
            assert p["HZ"] >= need, what
        if cin == 8:
            assert TZ * TX <= 64 and p["HY"] == FR + 2 and p["lds"] >= 16 * p["HZ"] * p["HY"] * p["HX"], what
        else:
            assert FR % 2 == 0 and p["HY"] >= (FR + 2 if kind == 0 else (FR + 2 >> 1) + 1), what
            assert p["lds"] >= 64 * p["HZ"] * p["HY"] * p["HX"], what
            assert TZ * TX <= 16 * p["PW"] and p["PW"] * p["CW"] <= (8 if p["NF"] == 2 and FR == 8 else 16), what
            assert 16 * p["NF"] * p["CW"] * p["nco"] >= cout, what
            assert _exact(p["mHY"], p["HY"], p["HZ"] * p["HY"]), what
        assert p["lds"] <= LDS_OF_A_CU, what
        assert _exact(p["mTX"], TX, 16 * max(p["PW"], 4)) and _exact(p["mHX"], p["HX"], p["HZ"] * p["HY"] * p["HX"]), what


@pytest.mark.parametrize("seed", range(4))
def test_weight_gradient_plans(plans, seed):
    r = random.Random(10 + seed)
    for _ in range(150):
        kind = r.randint(0, 3)
        cin, cout = 16 * r.randint(1, 8), r.choice([4, 16, 20, 32, 48, 64, 100, 128])
        n, d, h, w = _shape(r, kind)
        od, oh, ow = _out(kind, d, h, w)
        chunk = r.choice([16, 256, 8192, 1 << 30])
        p = plans.wgrad(kind, n, d, h, w, cin, cout, chunk)
        what = (kind, n, d, h, w, cin, cout, chunk, p)
        NT, S = {0: (3, 1), 1: (3, 1), 2: (2, 2), 3: (1, 1)}[kind]
        NF, RY = 2 if cout > 16 else 1, S * 3 + NT
        npos, nvox = 32 * p["ns"], n * od * oh * ow
        ntiles = n * p["tiles_x"] * p["tiles_y"] * p["tiles_z"]
        assert p["TZ"] * p["TX"] <= npos and p["ncf"] * p["nch"] * p["nkh"] == 4, what
        assert p["tiles_x"] * p["TX"] >= ow and p["tiles_y"] * 4 >= oh and p["tiles_z"] * p["TZ"] >= od, what
        assert p["HX"] >= S * (p["TX"] - 1) + NT and p["HX"] % 2 == 0, what
        assert 16 * p["ncf"] * p["ncb"] >= cin and 16 * NF * p["nch"] * p["ncg"] >= cout and p["nvar"] == NT * p["ncb"] * p["ncg"], what
        # every tile in one group, every group with a tile, partial sums within the caller's buffer
        assert p["groups"] * p["tpg"] >= ntiles > (p["groups"] - 1) * p["tpg"], what
        assert p["groups"] <= -(-nvox // chunk), what
        xrow, grow = 32 * p["ncf"], 32 * NF * p["nch"]
        assert p["g_off"] >= 4 * npos and p["x_off"] - p["g_off"] >= 4 * npos * grow, what
        nx = p["TZ"] * RY * p["HX"]
        assert p["lds"] - p["x_off"] >= nx * xrow and p["lds"] <= LDS_OF_A_CU, what
        assert (p["TZ"] - 1) * RY * p["HX"] * xrow < 1 << 20 and S * p["TX"] < 1 << 16, what   # a position's table entry
        if p["nkh"] > 1:
            assert p["lds"] >= p["ncf"] * p["nch"] * NT * NT * NF * 1024, what
        assert _exact(p["mTX"], p["TX"], npos) and _exact(p["mHX"], p["HX"], nx) and _exact(p["mNP"], npos, 4 * npos), what
