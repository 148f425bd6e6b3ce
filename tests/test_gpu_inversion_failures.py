"""A pivot that fails in any panel of the register-resident inversion: every
wave of the workgroup leaves at that panel, the matrix is reported singular
with a NaN inverse, and the matrices around it are bit for bit what they are
without it."""
import numpy as np
import pytest

from tests.gpu_common import make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 40, 96, 129, 200, 224])
def test_zero_column_at_every_step(n):
    """Walker 2 k has electron k out of reach of every AO: column k of D is
    zero, the pivot of step k fails.  The walkers between are ordinary."""
    print(f"[case] failing pivot at every step n={n}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=n // 3 + 2, n_up=n, n_dn=1, seed=n)
    R = walkers_near(sysm, 2 * n, seed=n + 1)
    S = make_gpu_system(sysm, A_up, A_dn)
    ok = run_gpu_forward(S, R, "fp64")
    assert np.all(ok["sign"] != 0)
    far = R.copy()
    for k in range(n):
        far[2 * k, k] = [400.0, -300.0, 250.0]
    out = run_gpu_forward(S, far, "fp64")
    bad, good = slice(0, None, 2), slice(1, None, 2)
    assert np.all(out["status"][bad] & 1) and not np.any(out["status"][good] & 5)
    assert np.all(np.isneginf(out["logdet"][bad, 0])) and np.all(out["sign"][bad, 0] == 0)
    assert np.all(np.isnan(out["Dinv_up"][bad]))
    for k in ("logdet", "sign", "Dinv_up", "drift", "lap"):
        np.testing.assert_array_equal(out[k][good], ok[k][good], err_msg=k)
    np.testing.assert_array_equal(out["logdet"][bad, 1], ok["logdet"][bad, 1])


@pytest.mark.parametrize("n", [5, 16, 21, 100, 129, 160, 201, 224])
def test_subnormal_pivot(n):
    """One orbital scaled by 2^-1040: the last pivot is a subnormal number
    whose reciprocal overflows.  log|det| and sign are those of the unscaled
    matrix but for the factor; the walker is not singular, but its inverse and
    with it the drift are not finite (status 4).

    Bound: each of the row's entries and updates (the products' chain over the
    AOs, n elimination steps) rounds to a multiple of 2^-1074, 2^-35 of the
    unscaled row's units each: |d log|det|| <= (AOs + n + 2) 2^-35 sum_e
    |D^-1[e][row]|, twice for the second order, and the unscaled 1e-10."""
    print(f"[case] subnormal pivot n={n}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=n // 3 + 2, n_up=n, n_dn=1, seed=n)
    R = walkers_near(sysm, 6, seed=n + 1)
    S = make_gpu_system(sysm, A_up, A_dn)
    ok = run_gpu_forward(S, R, "fp64")
    for row in (0, n - 1):
        A = A_up.copy()
        A[row] *= 2.0 ** -1040
        S.set_mo(0, A)
        g = run_gpu_forward(S, R, "fp64")
        assert not np.any(g["status"] & 1) and np.all(g["status"] & 4)
        np.testing.assert_array_equal(g["sign"], ok["sign"])
        bound = 2 * (sysm.n_basis + n + 2) * 2.0 ** -35 * np.abs(ok["Dinv_up"][:, :, row]).sum(1) + 1e-10 * (1 + 1040)
        assert np.all(np.abs(g["logdet"][:, 0] - (ok["logdet"][:, 0] - 1040 * np.log(2.0))) <= bound)
