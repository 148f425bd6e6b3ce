"""The register-resident inversion at the edges of its 16-column panels and
tiles against the oracle (the bounds of tests/gpu_common.py), and what it
reports for matrices whose pivots are not ordinary numbers."""
import numpy as np
import pytest

from tests.gpu_common import compare_forward, make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn", [(2, 1), (15, 14), (16, 16), (17, 16), (31, 18), (48, 47), (81, 80), (96, 95),
                                       (113, 112), (145, 144), (160, 159), (177, 176), (193, 192), (209, 208)])
def test_panel_and_tile_edges(n_up, n_dn):
    """One electron fewer, exactly and one more than whole panels, in every
    register shape."""
    print(f"[case] inversion edges n_up={n_up} n_dn={n_dn}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=max(2, (n_up + n_dn) // 6 + 1), n_up=n_up, n_dn=n_dn, seed=n_up * 5 + n_dn)
    R = walkers_near(sysm, 3, seed=n_up)
    S = make_gpu_system(sysm, A_up, A_dn)
    for mode in ("fp64", "fp32"):
        compare_forward(sysm, A_up, A_dn, R, run_gpu_forward(S, R, mode), mode)


@pytest.mark.parametrize("n", [20, 100, 200])
def test_pivots_that_are_no_ordinary_numbers(n):
    """An infinite entry is the largest of its column: a non-finite pivot
    (log|det| NaN, sign 0).  NaN is never a pivot: a row of them is left over
    at the end, as is a row of zeros (log|det| -inf, sign 0).  A row scaled
    by 2^-1000 is a pivot like any other."""
    print(f"[case] special pivots n={n}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=n // 3 + 2, n_up=n, n_dn=1, seed=n)
    R = walkers_near(sysm, 2, seed=n + 1)
    S = make_gpu_system(sysm, A_up, A_dn)
    ok = run_gpu_forward(S, R, "fp64")
    for row in (0, 17, n - 1):
        for value, status in ((np.inf, 4), (np.nan, 1), (0.0, 1)):
            A = A_up.copy()
            A[row] = np.where(A[row] == 0, 1.0, A[row]) * value if np.isinf(value) else value
            S.set_mo(0, A)
            g = run_gpu_forward(S, R, "fp64")
            # infinite coefficients of both signs meet in one sum: NaN
            if np.isinf(value) and np.isnan(g["C_up"][:, 0, :, row]).all():
                status = 1
            assert np.all(g["sign"][:, 0] == 0) and np.all(g["status"] & status), (row, value)
            ld = g["logdet"][:, 0]
            assert np.all(np.isneginf(ld)) if status == 1 else np.all(np.isnan(ld)), (row, value, ld)
            assert np.all(np.isnan(g["Dinv_up"]))
            np.testing.assert_array_equal(g["logdet"][:, 1], ok["logdet"][:, 1])
        A = A_up.copy()
        A[row] *= 2.0 ** -1000
        S.set_mo(0, A)
        g = run_gpu_forward(S, R, "fp64")
        # exactly scaled by a power of two: the same but for that factor
        np.testing.assert_array_equal(g["sign"], ok["sign"])
        np.testing.assert_allclose(g["logdet"][:, 0], ok["logdet"][:, 0] - 1000 * np.log(2.0), rtol=1e-12)
