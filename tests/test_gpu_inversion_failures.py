"""A pivot that fails in any panel of the register-resident inversion: every
wave of the workgroup leaves at that panel, the matrix is reported singular
with a NaN inverse, and the matrices around it are bit for bit what they are
without it."""
import dataclasses

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


@pytest.mark.parametrize("n", [5, 40, 129, 224])
def test_infinite_pivot_at_every_step(n):
    """An entry that overflows (no NaN beside it): walker 2 k has electron k
    alone on an atom of its own, whose AO (3.4 at the nucleus) takes part only
    in the last orbital, with a coefficient of 1.7e308.  That orbital is scaled
    by 2^-400 elsewhere, so that no earlier step takes its row (which would
    spread infinities of both signs).  Column k of D holds the entry, +inf,
    and zeros: the pivot of step k is infinite, log|det| NaN, sign 0 and the
    status non-finite, not singular."""
    print(f"[case] infinite pivot at every step n={n}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=n // 3 + 2, n_up=n, n_dn=1, seed=n)
    sysm = dataclasses.replace(
        sysm, atom_xyz=np.concatenate([sysm.atom_xyz, [[90.0, 0.0, 0.0]]]), atom_heavy=np.append(sysm.atom_heavy, True),
        shell_atom=np.append(sysm.shell_atom, np.int32(sysm.n_atoms)), shell_l=np.append(sysm.shell_l, np.int32(0)),
        shell_nprim=np.append(sysm.shell_nprim, np.int32(1)), prim_exp=np.append(sysm.prim_exp, 8.0),
        prim_coef=np.append(sysm.prim_coef, 1.0))
    A_up = np.concatenate([A_up, np.zeros((n, 1))], axis=1)
    A_dn = np.concatenate([A_dn, np.zeros((1, 1))], axis=1)
    A_up[n - 1] *= 2.0 ** -400
    near = dataclasses.replace(sysm, atom_xyz=sysm.atom_xyz[:-1])
    R = walkers_near(near, 2 * n, seed=n + 1)
    ok = run_gpu_forward(make_gpu_system(sysm, A_up, A_dn), R, "fp64")
    A_up[n - 1, -1] = 1.7e308
    for k in range(n):
        R[2 * k, k] = [90.0, 0.0, 0.0]
    out = run_gpu_forward(make_gpu_system(sysm, A_up, A_dn), R, "fp64")
    bad, good = slice(0, None, 2), slice(1, None, 2)
    for k in range(n):
        column = np.zeros(n)
        column[n - 1] = np.inf
        np.testing.assert_array_equal(out["C_up"][2 * k, 0, k], column)
    assert not np.any(np.isnan(out["C_up"][:, 0]))
    assert np.all(out["status"][bad] & 4) and not np.any(out["status"][bad] & 1)
    assert np.all(np.isnan(out["logdet"][bad, 0])) and np.all(out["sign"][bad, 0] == 0)
    assert np.all(np.isnan(out["Dinv_up"][bad]))
    for k in ("logdet", "sign", "Dinv_up", "drift", "lap"):
        np.testing.assert_array_equal(out[k][good], ok[k][good], err_msg=k)
