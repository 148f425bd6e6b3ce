"""Both spins of a call in one launch per phase: each spin's FP64 outputs are
bit for bit those of the spin by itself, also where the two spins' inversions
share a register shape and where they cannot (a tiny matrix beside a large
one, exact beside rounded pivot comparison, register-resident beside blocked)."""
import copy

import numpy as np
import pytest

from tests.gpu_common import make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn", [(100, 7), (100, 8), (113, 5), (96, 20), (129, 128), (224, 40), (230, 30), (240, 226)])
def test_each_spin_as_by_itself(n_up, n_dn):
    print(f"[case] spins together n_up={n_up} n_dn={n_dn}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 6 + 1, n_up=n_up, n_dn=n_dn, seed=n_up + 7 * n_dn)
    R = walkers_near(sysm, 3, seed=n_up)
    both = run_gpu_forward(make_gpu_system(sysm, A_up, A_dn), R, "fp64")
    none = np.zeros((0, A_up.shape[1]))
    for s, key in enumerate(("up", "dn")):
        one = copy.copy(sysm)
        one.n_up, one.n_dn = (n_dn if s else n_up), 0  # either spin as the up spin
        el = slice(n_up, n_up + n_dn) if s else slice(0, n_up)
        S = make_gpu_system(one, A_dn if s else A_up, none)
        alone = run_gpu_forward(S, np.ascontiguousarray(R[:, el]), "fp64")
        for k in ("C", "Dinv"):
            np.testing.assert_array_equal(both[f"{k}_{key}"], alone[f"{k}_up"])
        for k in ("logdet", "sign"):
            np.testing.assert_array_equal(both[k][:, s], alone[k][:, 0])
        for k in ("drift", "lap"):
            np.testing.assert_array_equal(both[k][:, el], alone[k])


@pytest.mark.parametrize("n_up,n_dn,n_det,W", [(12, 5, 40, 3), (33, 8, 7, 2), (9, 0, 3, 2), (130, 120, 3, 2), (230, 12, 2, 2)])
def test_each_determinant_as_a_forward(n_up, n_dn, n_det, W):
    """Determinants inverted in groups: each one's log|det| and sign bit for
    bit those of a forward with its orbitals alone."""
    import torch
    print(f"[case] determinants n_up={n_up} n_dn={n_dn} n_det={n_det}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 6 + 2, n_up=n_up, n_dn=n_dn, seed=n_up)
    rng = np.random.default_rng(n_up)
    R = walkers_near(sysm, W, seed=n_up + 1)
    orb = [np.concatenate([A, rng.normal(size=(4, A.shape[1])) / np.sqrt(A.shape[1])]) if len(A) else A for A in (A_up, A_dn)]
    occ = np.array([np.concatenate([rng.permutation(len(o))[:n] for o, n in zip(orb, (n_up, n_dn))])
                    for _ in range(n_det)], np.int32)
    S = make_gpu_system(sysm, A_up, A_dn)
    for s in range(2):
        if len(orb[s]):
            S.set_orbitals(s, orb[s])
    out = S.multidet_forward(torch.from_numpy(R).cuda(), occ, rng.normal(size=n_det), "fp64")
    T = make_gpu_system(sysm, A_up, A_dn)
    for K in range(n_det):
        T.set_mo(0, orb[0][occ[K, :n_up]])
        if n_dn:
            T.set_mo(1, orb[1][occ[K, n_up:]])
        one = run_gpu_forward(T, R, "fp64")
        np.testing.assert_array_equal(out["det_logdet"][K].cpu().numpy(), one["logdet"])
        np.testing.assert_array_equal(out["det_sign"][K].cpu().numpy(), one["sign"])


@pytest.mark.parametrize("W", [1985, 1986, 2100])
def test_walker_order_changes_nothing(W):
    """FP64: C and what follows from it, for the first walkers of a call whose
    tiles take the walkers in an order of their own (from 65536 electrons on)
    or not, are bit for bit those of a call of these walkers alone (one tile,
    no order): the products are one chain over the slots, to which slots that
    survive for other walkers add zeros."""
    print(f"[case] walker order W={W}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=6, n_up=17, n_dn=16, seed=W)
    R = walkers_near(sysm, W, seed=5)
    S = make_gpu_system(sysm, A_up, A_dn)
    all_, few = run_gpu_forward(S, R, "fp64"), run_gpu_forward(S, np.ascontiguousarray(R[:20]), "fp64")
    for k in ("C_up", "C_dn", "Dinv_up", "Dinv_dn", "logdet", "sign", "drift", "lap", "status"):
        np.testing.assert_array_equal(all_[k][:20], few[k])
