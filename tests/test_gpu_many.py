"""Parameter updates of many tensors in one call: Adam against its formula in
64 bits (a handful of FP32 roundings of the step, lr wide at most: 1e-5 lr, and
one of the parameter), with sizes around the 1,024 elements of a workgroup,
tensors off a 16-byte boundary and more of them than one launch takes; packed
fragments of padded rows against those of a contiguous copy, bit for bit."""
import ctypes as ct

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need the MI355X"
    return torch


@pytest.mark.parametrize("count", [1, 5, 48, 49, 97])
def test_adam_many(torch, count):
    from paper_2302_04659_amd.unet import nn_lib
    L, rng = nn_lib(), np.random.default_rng(count)
    sizes = [(1, 3, 1023, 1024, 1025, 4096, 5001)[i % 7] for i in range(count)]
    offs = [i % 4 if i % 3 == 0 else 0 for i in range(count)]
    host = [[(rng.normal(size=n) * s).astype(np.float32) for s in (1.0, 0.1, 0.01)]
            + [(1e-4 * rng.random(n)).astype(np.float32)] for n in sizes]
    dev = [[torch.zeros(n + 8, device="cuda")[o:o + n] for _ in range(4)] for n, o in zip(sizes, offs)]
    for hs, ds in zip(host, dev):
        for h, d in zip(hs, ds):
            d.copy_(torch.from_numpy(h))
    lr, b1, b2, eps, t = 1e-3, 0.9, 0.999, 1e-8, 3
    ptrs = ct.c_void_p * count
    arrs = [ptrs(*[d[i].data_ptr() for d in dev]) for i in range(4)]
    n = (ct.c_longlong * count)(*sizes)
    s = torch.cuda.current_stream().cuda_stream
    assert L.mpm_nn_adam_many(count, *arrs, n, lr, b1, b2, eps, t, s) == 0
    assert L.mpm_nn_adam_many(0, *arrs, n, lr, b1, b2, eps, t, s) == -1
    n[count - 1] = 0
    assert L.mpm_nn_adam_many(count, *arrs, n, lr, b1, b2, eps, t, s) == -1     # nothing queued
    torch.cuda.synchronize()
    f = np.float64
    b1, b2 = f(np.float32(b1)), f(np.float32(b2))
    for (p, g, m, v), ds in zip(host, dev):
        p, g, m, v = (a.astype(f) for a in (p, g, m, v))
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        step = lr * (m / (1 - b1 ** t)) / (np.sqrt(v / (1 - b2 ** t)) + eps)
        got = ds[0].cpu().numpy().astype(f)
        # 1 - beta in FP32 carries 2^-24 / (1 - beta): 6e-7 and 6e-5 of it
        assert np.all(np.abs(got - (p - step)) <= 2.0 ** -23 * np.abs(p) + 1e-4 * np.abs(step) + 1e-5 * lr)


@pytest.mark.parametrize("kind,taps,ci,co,transpose", [(0, 27, 64, 32, 0), (0, 27, 16, 48, 1), (0, 27, 8, 32, 0),
                                                       (1, 27, 16, 20, 0), (2, 8, 32, 64, 0), (3, 1, 48, 4, 1)])
def test_pack_many_padded_rows(torch, kind, taps, ci, co, transpose):
    from paper_2302_04659_amd.unet import nn_lib
    L = nn_lib()
    w = torch.randn(taps, ci + 8, co, device="cuda")
    flat = w[:, :ci, :].contiguous()
    size = taps * ((ci + 15) // 16 * 16) * ((co + 15) // 16 * 16)
    one, many = (torch.zeros(size, dtype=torch.int16, device="cuda") for _ in range(2))
    s = torch.cuda.current_stream().cuda_stream
    assert L.mpm_nn_pack(flat.data_ptr(), kind, ci, co, transpose, one.data_ptr(), s) == 0
    i, p = ct.c_int * 1, ct.c_void_p * 1
    assert L.mpm_nn_pack_many(1, p(w.data_ptr()), i(kind), i(ci + 8), i(ci), i(co), i(transpose),
                              p(many.data_ptr()), s) == 0
    assert L.mpm_nn_pack_many(1, p(w.data_ptr()), i(kind), i(ci - 1), i(ci), i(co), i(transpose),
                              p(many.data_ptr()), s) == -1
    torch.cuda.synchronize()
    assert torch.equal(one, many)
    if kind == 0 and ci == 64:          # the order itself: element ((t KC2 + c) NF + n) 64 8 + lane 8 + e
        t, c, n, lane, e = 5, 1, 1, 37, 3
        at = (((t * 2 + c) * 2 + n) * 64 + lane) * 8 + e
        ref = flat[t, 32 * c + 8 * (lane // 16) + e, 16 * n + lane % 16].to(torch.bfloat16)
        assert int(one[at]) == int(ref.view(torch.int16))
