"""FP64 dA of small calls (up to 32 electrons of a spin, one walker group of up
to 128 walkers or a plan's adj_group): the same bits on every call, and within
the bound of tests/test_gpu_adjoint_fp64.py of the oracle adjoint."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import make_gpu_system
from tests.systems import random_tiny, walkers_near
from tests.test_gpu_adjoint import _abs_bounds

pytestmark = pytest.mark.gpu


def _case(n_up, n_dn, W):
    import torch
    sysm, A_up, A_dn = random_tiny(n_atoms=max(2, (n_up + n_dn) // 8 + 2), n_up=n_up, n_dn=n_dn, seed=n_up + W)
    R = walkers_near(sysm, W, seed=n_up)
    g = np.random.default_rng(W).normal(size=(W, 2))
    S = make_gpu_system(sysm, A_up, A_dn)
    return sysm, A_up, A_dn, R, g, S, torch.from_numpy(R).cuda(), torch.from_numpy(g).cuda()


def _check(sysm, A_up, A_dn, R, g, out, dA):
    ref = {k: out[k].cpu().numpy() for k in ("Dinv_up", "Dinv_dn")}
    _, rdAu, rdAd = oracle.backward(sysm, A_up, A_dn, R, ref["Dinv_up"], ref["Dinv_dn"], g)
    bA, _ = _abs_bounds(sysm, A_up, A_dn, R, ref, g)
    for got, want, b in ((dA[0], rdAu, bA[0]), (dA[1], rdAd, bA[1])):
        assert np.all(np.abs(got - want) <= 1e-10 * b + 1e-300)


# (33, 32): the spin of 33 has atomics, the other one not
@pytest.mark.parametrize("n_up,n_dn,W,same", [(32, 31, 128, (0, 1)), (22, 22, 64, (0, 1)), (33, 32, 40, (1,)), (3, 0, 1, (0,))])
def test_backward_repeats(n_up, n_dn, W, same):
    print(f"[case] fp64 dA repeats n={n_up}/{n_dn} W={W}", flush=True)
    sysm, A_up, A_dn, R, g, S, Rt, gt = _case(n_up, n_dn, W)
    out = S.forward(Rt, "fp64")
    runs = [[x.cpu().numpy() for x in S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], gt, "fp64")[1:]] for _ in range(12)]
    _check(sysm, A_up, A_dn, R, g, out, runs[0])
    for r in runs[1:]:
        for s in same:
            np.testing.assert_array_equal(r[s], runs[0][s])
    # dA += adds the same sum once more
    import torch
    dA = tuple(torch.from_numpy(x.copy()).cuda() for x in runs[0])
    twice = S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], gt, "fp64", dA=dA, accumulate=True)[1:]
    for s in same:
        np.testing.assert_array_equal(twice[s].cpu().numpy(), 2.0 * runs[0][s])


@pytest.mark.parametrize("batched", [0, 1])
@pytest.mark.parametrize("W,group", [(100, 0), (300, 512)])
def test_plan_repeats(W, group, batched):
    import torch
    from paper_1209_6630_amd.api import Plan
    print(f"[case] fp64 dA repeats in a plan W={W} adj_group={group} batched={batched}", flush=True)
    sysm, A_up, A_dn, R, g, S, Rt, gt = _case(24, 17, W)
    P = Plan([S], [W], "fp64", graph=True)
    P.tuning = dict(adj_group=group, batched=batched)
    out = S.alloc_outputs(W, "fp64")
    dR = torch.empty_like(Rt)
    dA = tuple(torch.empty((n, S.n_basis), dtype=torch.float64, device="cuda") for n in (24, 17))
    P.bind(0, Rt, out, g=gt, dR=dR, dA=dA)
    runs = []
    for _ in range(8):
        P.launch()
        torch.cuda.synchronize()
        runs.append([x.cpu().numpy() for x in dA])
    _check(sysm, A_up, A_dn, R, g, out, runs[0])
    for r in runs[1:]:
        for s in range(2):
            np.testing.assert_array_equal(r[s], runs[0][s])


@pytest.mark.parametrize("accumulate", [False, True])
def test_both_spins_add_to_one_dA(accumulate):
    """One dA for both spins (the same coefficients): the spins' sums are
    added to it, or it is their sum."""
    import torch
    print(f"[case] fp64 one dA for both spins accumulate={accumulate}", flush=True)
    sysm, A_up, A_dn, R, g, S, Rt, gt = _case(12, 12, 30)
    out = S.forward(Rt, "fp64")
    _, up, dn = S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], gt, "fp64")
    one = torch.full((12, S.n_basis), 3.0 if accumulate else 7.0, dtype=torch.float64, device="cuda")
    S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], gt, "fp64", dA=(one, one), accumulate=accumulate)
    want = up + dn + (3.0 if accumulate else 0.0)
    # two additions, in either order
    bound = 4 * 2.0 ** -53 * (up.abs() + dn.abs() + 3.0)
    assert bool(((one - want).abs() <= bound).all())
