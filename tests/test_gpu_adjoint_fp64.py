"""FP64 dA by electron at the edges of its tiles (16 MOs in groups of 80,
224 MOs a workgroup, 64 slots a chunk, 32 walkers a batch), against the oracle
adjoint from the same inverse.

Bound: |dA - ref| <= 1e-10 sum |G| |chi|, the configurations' bound of
tests/test_gpu_adjoint.py (a sum of W terms in FP64 is within W 2^-53 of it,
the AO values within some 2^-48)."""
import numpy as np
import pytest

import oracle
from tests.systems import random_tiny, walkers_near
from tests.test_gpu_adjoint import _abs_bounds
from tests.gpu_common import make_gpu_system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn,W", [(3, 1, 1), (16, 15, 32), (17, 0, 33), (80, 20, 5), (81, 80, 2), (161, 17, 2), (230, 5, 2)])
def test_tile_edges_and_singular_walkers(n_up, n_dn, W):
    import torch
    print(f"[case] fp64 dA n={n_up}/{n_dn} W={W}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=max(2, (n_up + n_dn) // 8 + 2), n_up=n_up, n_dn=n_dn, seed=n_up + W)
    R = walkers_near(sysm, W, seed=n_up)
    g = np.random.default_rng(W).normal(size=(W, 2))
    if W > 1:  # one singular walker, with g = 0 and its inverse NaN
        R[W - 1, 1] = R[W - 1, 0]
        g[W - 1] = 0.0
    S = make_gpu_system(sysm, A_up, A_dn)
    Rt = torch.from_numpy(R).cuda()
    out = S.forward(Rt, "fp64")
    if W > 1:  # (two electrons at one place need not cancel exactly)
        out["Dinv_up"][W - 1] = float("nan")
    _, dAu, dAd = S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], torch.from_numpy(g).cuda(), "fp64")
    ref = {k: np.nan_to_num(out[k].cpu().numpy()) for k in ("Dinv_up", "Dinv_dn")}
    _, rdAu, rdAd = oracle.backward(sysm, A_up, A_dn, R, ref["Dinv_up"], ref["Dinv_dn"], g)
    bA, _ = _abs_bounds(sysm, A_up, A_dn, R, ref, g)
    for got, want, b in ((dAu, rdAu, bA[0]), (dAd, rdAd, bA[1])):
        if b.size:
            assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-10 * b + 1e-300)
