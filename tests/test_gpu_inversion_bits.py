"""The register-resident inversion up to 128 electrons is, bit for bit, the
rank-1 Gauss-Jordan elimination with a fused multiply-add per entry and step,
pivots by the largest |entry| (the smallest row on ties): the panels and the
FP64 matrix instructions change no rounding."""
import ctypes as ct
import ctypes.util

import numpy as np
import pytest

from tests.gpu_common import make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu

_libm = ct.CDLL(ctypes.util.find_library("m"))
_libm.fma.restype = ct.c_double
_libm.fma.argtypes = [ct.c_double] * 3


def _eliminate(D):
    """D[i][e] -> its inverse [e][i] and the pivots in step order."""
    fma, n = _libm.fma, D.shape[0]
    M = [list(map(float, r)) for r in D]
    used, perm, piv = [False] * n, [], []
    for k in range(n):
        p = max((i for i in range(n) if not used[i]), key=lambda i: (abs(M[i][k]), -i))
        pv, row = M[p][k], M[p]
        inv = 1.0 / pv
        for i in range(n):
            if i == p:
                continue
            r = M[i]
            f = -(r[k] * inv)
            M[i] = [fma(f, pv + 1.0 if c == k else row[c], r[c]) for c in range(n)]
        used[p] = True
        perm.append(p)
        piv.append(pv)
    X = np.empty((n, n))
    for k in range(n):
        rs = 1.0 / piv[k]
        for e in range(n):
            x = M[perm[k]][e] + (1.0 - piv[k] if e == k else 0.0)
            X[k, perm[e]] = x * rs
    return X, np.array(piv)


@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 15, 16, 17, 33, 63, 65, 80])
def test_rank_one_steps_bit_for_bit(n):
    print(f"[case] inversion bits n={n}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=n // 3 + 2, n_up=n, n_dn=1, seed=n + 40)
    R = walkers_near(sysm, 2, seed=n)
    out = run_gpu_forward(make_gpu_system(sysm, A_up, A_dn), R, "fp64")
    for w in range(2):
        X, piv = _eliminate(out["C_up"][w, 0].T)
        np.testing.assert_array_equal(out["Dinv_up"][w], X)
        # the logs' own rounding and the order of their sum
        assert abs(out["logdet"][w, 0] - np.log(np.abs(piv)).sum()) <= 1e-13 * (n + np.abs(np.log(np.abs(piv))).sum())
