"""The forms of the Hencky series at the limits of their ranges, host build of
mpm_math.hpp against 64 bits: hencky_invariant_strain (rollouts; |b - I|_F up to
0.6, more terms past 0.35), hencky_series_strain (up to 0.35) and the form of the
kernels that take states in and give them out.

Bar on the log strain: 5e-6 |e| (a chain of about 40 roundings) plus 1e-6 (the
roundings of F F^T, entries of size 1)."""
import ctypes as ct
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_04659_amd", "csrc")
SOURCE = """
#include "%s/mpm_math.hpp"
extern "C" void strain(int form, const float *F, int n, int plastic, float yield_eps, float *e, int *ok)
{
    mpm::Material m{1, plastic, 1.0f, 1.0f, yield_eps};
    for (int p = 0; p < n; p++) {
        float G[9];
        for (int k = 0; k < 9; k++) G[k] = F[9 * p + k] - (k %% 4 == 0 ? 1.0f : 0.0f);
        ok[p] = form == 0 ? mpm::hencky_invariant_strain(G, m, e + 6 * p)
                          : (form == 1 ? mpm::hencky_series_strain(G, m, e + 6 * p) : mpm::state_hencky_series(G, e + 6 * p));
    }
}
""" % CSRC
LIMIT = (0.6, 0.35, 0.35)


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    d = tmp_path_factory.mktemp("strain")
    src, lib = str(d / "strain.cpp"), str(d / "strain.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", lib, src],
                   check=True, capture_output=True)
    fn = ct.CDLL(lib).strain
    fn.argtypes = [ct.c_int, ct.c_void_p, ct.c_int, ct.c_int, ct.c_float, ct.c_void_p, ct.c_void_p]
    return fn


def _states(rng, n, near):
    """F with |F F^T - I|_F spread over 0 .. 0.8, some of it close to the limits `near`."""
    out = np.empty((n, 3, 3), np.float32)
    for p in range(n):
        target = rng.choice(near) * (1 + rng.uniform(-0.02, 0.02)) if rng.random() < 0.4 else rng.uniform(0.0, 0.8)
        d = rng.normal(size=3)
        if rng.random() < 0.2:
            d = np.array([-1.0, 0.0, 0.0])                 # all of it in one compressed direction
        d *= target / np.linalg.norm(d)
        Q, R = (np.linalg.qr(rng.normal(size=(3, 3)))[0] for _ in range(2))
        Q, R = Q * np.linalg.det(Q), R * np.linalg.det(R)
        out[p] = Q @ np.diag(np.sqrt(np.maximum(1 + d, 0.05))) @ Q.T @ (R if rng.random() < 0.5 else np.eye(3))
    return out


# the third form has no yield test
@pytest.mark.parametrize("form,yield_eps", [(0, None), (0, 0.05), (0, 0.2), (1, None), (1, 0.05), (1, 0.2), (2, None)])
def test_series_at_their_limits(forms, form, yield_eps):
    F = _states(np.random.default_rng(5), 3000, (0.35, 0.6))
    n = len(F)
    e, ok = np.zeros((n, 6), np.float32), np.zeros(n, np.int32)
    forms(form, F.ctypes.data, n, yield_eps is not None, yield_eps or 0.0, e.ctypes.data, ok.ctypes.data)
    F64 = F.astype(np.float64)
    b = F64 @ F64.transpose(0, 2, 1)
    nb = np.linalg.norm((b - np.eye(3)).reshape(n, 9), axis=1)
    lam, V = np.linalg.eigh(b)
    ref = (V * (0.5 * np.log(lam))[:, None, :]) @ V.transpose(0, 2, 1)
    dev = ref - np.trace(ref, axis1=1, axis2=2)[:, None, None] / 3 * np.eye(3)
    nd = np.linalg.norm(dev.reshape(n, 9), axis=1)
    det = np.linalg.det(F64)
    limit, tol = LIMIT[form], 1e-5
    takes, refuses = (nb < limit - tol) & (det > 0.5 + tol), (nb > limit + tol) | (det < 0.5 - tol)
    if yield_eps is not None:
        takes &= nd < yield_eps - tol
        refuses |= nd > yield_eps + tol
    assert takes.sum() > 200 and refuses.sum() > 200
    assert ok[takes].all() and not ok[refuses].any()
    idx = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
    got = np.stack([e[:, idx.index((min(i, j), max(i, j)))] for i in range(3) for j in range(3)], axis=1)
    err = np.linalg.norm(got - ref.reshape(n, 9), axis=1)[ok == 1]
    assert (err <= 5e-6 * np.linalg.norm(ref.reshape(n, 9), axis=1)[ok == 1] + 1e-6).all(), err.max()
