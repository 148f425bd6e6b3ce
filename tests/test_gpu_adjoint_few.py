"""FP64 adjoint on the two sides of the line between dA by 32-electron range
(few walkers) and by electron, one spin on each side among them, within the
bound of tests/test_gpu_adjoint_fp64.py of the oracle adjoint; and the few
walkers' time, which by electron is that of a whole batch of 32."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import make_gpu_system
from tests.systems import random_tiny, walkers_near
from tests.test_gpu_adjoint import _abs_bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_drift", [False, True])
@pytest.mark.parametrize("n_up,n_dn,W", [(97, 96, 1), (128, 127, 3), (128, 98, 3), (129, 31, 2), (161, 60, 5), (161, 160, 6), (230, 226, 10)])
def test_both_sides(n_up, n_dn, W, use_drift):
    import torch
    print(f"[case] fp64 dA few walkers n={n_up}/{n_dn} W={W} drift={use_drift}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 8 + 2, n_up=n_up, n_dn=n_dn, seed=n_up + W)
    R = walkers_near(sysm, W, seed=n_up)
    g = np.random.default_rng(W).normal(size=(W, 2))
    S = make_gpu_system(sysm, A_up, A_dn)
    Rt = torch.from_numpy(R).cuda()
    out = S.forward(Rt, "fp64")
    dR, dAu, dAd = S.backward(Rt, out["Dinv_up"], out["Dinv_dn"], torch.from_numpy(g).cuda(), "fp64",
                              drift=out["drift"] if use_drift else None)
    ref = {k: out[k].cpu().numpy() for k in ("Dinv_up", "Dinv_dn")}
    rdR, rdAu, rdAd = oracle.backward(sysm, A_up, A_dn, R, ref["Dinv_up"], ref["Dinv_dn"], g)
    bA, bR = _abs_bounds(sysm, A_up, A_dn, R, ref, g)
    for got, want, b in ((dAu, rdAu, bA[0]), (dAd, rdAd, bA[1]), (dR, rdR, bR)):
        assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-10 * b + 1e-300)


def test_one_walker_of_many_electrons_is_quick():
    """One walker's adjoint of 866 electrons a spin (by range 0.9 ms, by
    electron 8.8) takes at most a third of that of 64 walkers (by
    electron in either case, about 12 ms)."""
    import torch
    print("[case] fp64 dA of one walker, 866 electrons a spin", flush=True)
    import qsl_synth as q
    sysm, A_up, A_dn, R = q.make_config("1731e", W=64)
    S = make_gpu_system(sysm, A_up, A_dn)

    def time(W):
        Rt = torch.from_numpy(np.ascontiguousarray(R[:W])).cuda()
        Di = [torch.zeros((W, n, n), dtype=torch.float64, device="cuda") for n in (sysm.n_up, sysm.n_dn)]
        g = torch.ones((W, 2), dtype=torch.float64, device="cuda")
        dr = torch.zeros_like(Rt)
        dA = tuple(torch.empty((n, S.n_basis), dtype=torch.float64, device="cuda") for n in (sysm.n_up, sysm.n_dn))
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        best = float("inf")
        for _ in range(5):
            e[0].record()
            S.backward(Rt, *Di, g, "fp64", dA=dA, drift=dr)
            e[1].record()
            e[1].synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        return best

    assert time(1) * 3 <= time(64)


def _plan(S, Rt, gt, group, dR, dA):
    from paper_1209_6630_amd.api import Plan
    W = Rt.shape[0]
    P = Plan([S], [W], "fp64", graph=False)
    P.tuning = dict(batched=1, adj_group=group)
    out = S.alloc_outputs(W, "fp64")
    P.bind(0, Rt, out, g=gt, dR=dR, dA=dA)
    P.launch()
    return P, out


@pytest.mark.parametrize("n_up,n_dn,W,group", [(40, 39, 47, 1), (40, 30, 90, 8), (40, 17, 90, 40), (129, 20, 13, 5)])
def test_small_groups_of_a_plan(n_up, n_dn, W, group):
    import torch
    print(f"[case] fp64 dA small groups n={n_up}/{n_dn} W={W} group={group}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 8 + 2, n_up=n_up, n_dn=n_dn, seed=n_up + W)
    R = walkers_near(sysm, W, seed=n_up)
    g = np.random.default_rng(W).normal(size=(W, 2))
    S = make_gpu_system(sysm, A_up, A_dn)
    Rt, gt = torch.from_numpy(R).cuda(), torch.from_numpy(g).cuda()
    dR = torch.empty_like(Rt)
    dA = tuple(torch.empty((n, S.n_basis), dtype=torch.float64, device="cuda") for n in (n_up, n_dn))
    P, out = _plan(S, Rt, gt, group, dR, dA)
    ref = {k: out[k].cpu().numpy() for k in ("Dinv_up", "Dinv_dn")}
    rdR, rdAu, rdAd = oracle.backward(sysm, A_up, A_dn, R, ref["Dinv_up"], ref["Dinv_dn"], g)
    bA, bR = _abs_bounds(sysm, A_up, A_dn, R, ref, g)
    for got, want, b in ((dA[0], rdAu, bA[0]), (dA[1], rdAd, bA[1]), (dR, rdR, bR)):
        assert np.all(np.abs(got.cpu().numpy() - want) <= 1e-10 * b + 1e-300)


def test_groups_of_one_walker_are_no_batches_of_32():
    """dA of 512 walkers of 79 electrons a spin in groups of one: by range 3.3
    times the time of groups of 32, by electron 29 times; at most 8 allowed."""
    import torch
    from paper_1209_6630_amd import _lib
    import qsl_synth as q
    print("[case] fp64 dA in groups of one walker", flush=True)
    sysm, A_up, A_dn, R = q.make_config("158e", W=512)
    S = make_gpu_system(sysm, A_up, A_dn)
    Rt = torch.from_numpy(R).cuda()
    gt = torch.ones((512, 2), dtype=torch.float64, device="cuda")
    dR = torch.empty_like(Rt)
    dA = tuple(torch.empty((n, S.n_basis), dtype=torch.float64, device="cuda") for n in (sysm.n_up, sysm.n_dn))

    def ms(group):
        P, _ = _plan(S, Rt, gt, group, dR, dA)
        torch.cuda.synchronize()
        _lib.profile_enable(True)
        try:
            _lib.profile_read()
            for _ in range(5):
                P.launch()
            return _lib.profile_read()["adjoint_dA"][1] / 5
        finally:
            _lib.profile_enable(False)

    assert ms(1) <= 8 * ms(32)
