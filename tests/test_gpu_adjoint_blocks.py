"""FP32 dA by electron where the 32-MO blocks of a workgroup's 224 are partly
used (1, 2, 3, 4, 5 and 7 blocks, and a second workgroup), against the oracle
adjoint from the same inverse, within the bound of
tests/test_gpu_adjoint.py."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import U32, dA_tol, max_survivors
from tests.systems import random_tiny, walkers_near
from tests.test_gpu_adjoint import _abs_bounds, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn,W", [(32, 31, 33), (33, 2, 3), (65, 64, 2), (129, 97, 2), (193, 128, 2), (225, 10, 2)])
def test_mo_blocks(n_up, n_dn, W):
    print(f"[case] fp32 dA blocks n={n_up}/{n_dn} W={W}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 8 + 2, n_up=n_up, n_dn=n_dn, seed=n_up)
    R = walkers_near(sysm, W, seed=n_dn)
    g, _, dAu, dAd, out = _run(sysm, A_up, A_dn, R, "fp32")
    tol = (64 + 64 + 2 * max_survivors(sysm, R[:1])) * U32
    _, rdAu, rdAd = oracle.backward(sysm, A_up, A_dn, R, out["Dinv_up"], out["Dinv_dn"], g)
    bA, _ = _abs_bounds(sysm, A_up, A_dn, R, out, g)
    for got, want, b, n in ((dAu, rdAu, bA[0], n_up), (dAd, rdAd, bA[1], n_dn)):
        assert np.all(np.abs(got - want) <= max(tol, dA_tol("fp32", W, n)) * b + 1e-300)
