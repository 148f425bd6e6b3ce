"""Determinants in several uneven groups (a launch holds at most 65536
matrices): each one's log|det| and sign bit for bit those of a forward with its
orbitals alone, and the combination of the forwards' drift and Laplacian.

Bound of the combination: w_K = c_K Det_K / Psi from logs and exponentials of
numbers below 2^7 in size is within 1e-13 (1 + sum |w|) of itself (the sum's
cancellation), each term's product and the sum of n_det terms within 1e-15."""
import numpy as np
import pytest

from tests.gpu_common import make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


# 10000 walkers: groups of 3 and 2 of five determinants; 6000: of 4 and 3 of
# seven, without spin-down electrons; 17000: one at a time
@pytest.mark.parametrize("n_up,n_dn,W,n_det", [(3, 2, 10000, 5), (4, 0, 6000, 7), (2, 2, 17000, 3)])
def test_groups(n_up, n_dn, W, n_det):
    import torch
    print(f"[case] determinant groups n={n_up}/{n_dn} W={W} n_det={n_det}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=3, n_up=n_up, n_dn=n_dn, seed=n_det)
    rng = np.random.default_rng(W)
    R = walkers_near(sysm, W, seed=n_up + 1)
    nb = A_up.shape[1]
    orb = [np.concatenate([A, rng.normal(size=(3, nb)) / np.sqrt(nb)]) if len(A) else A for A in (A_up, A_dn)]
    occ = np.array([np.concatenate([rng.permutation(len(o))[:n] for o, n in zip(orb, (n_up, n_dn))])
                    for _ in range(n_det)], np.int32)
    coef = rng.normal(size=n_det)
    S = make_gpu_system(sysm, A_up, A_dn)
    for s in range(2):
        if len(orb[s]):
            S.set_orbitals(s, orb[s])
    got = S.multidet_forward(torch.from_numpy(R).cuda(), occ, coef, "fp64")
    got = {k: v.cpu().numpy() for k, v in got.items() if not k.startswith("_")}
    T = make_gpu_system(sysm, A_up, A_dn)
    one = []
    for K in range(n_det):
        T.set_mo(0, orb[0][occ[K, :n_up]])
        if n_dn:
            T.set_mo(1, orb[1][occ[K, n_up:]])
        one.append(run_gpu_forward(T, R, "fp64"))
        np.testing.assert_array_equal(got["det_logdet"][K], one[K]["logdet"])
        np.testing.assert_array_equal(got["det_sign"][K], one[K]["sign"])
    L = np.array([f["logdet"].sum(1) for f in one]) + np.log(np.abs(coef))[:, None]
    sg = np.array([f["sign"].astype(float).prod(1) for f in one]) * np.sign(coef)[:, None]
    m = L.max(0)
    t = sg * np.exp(L - m)
    psi = t.sum(0)
    np.testing.assert_array_equal(got["sign"], np.sign(psi))
    w = t / psi
    amp = np.abs(w).sum(0)
    np.testing.assert_allclose(got["logpsi"], m + np.log(np.abs(psi)), rtol=0, atol=1e-12 * amp.max())
    for k in ("drift", "lap"):
        x = np.array([f[k].reshape(W, -1) for f in one])
        want = (w[:, :, None] * x).sum(0)
        bound = 2e-13 * (1 + amp)[:, None] * (np.abs(w)[:, :, None] * np.abs(x)).sum(0) + 1e-300
        assert np.all(np.abs(got[k].reshape(W, -1) - want) <= bound), k


@pytest.mark.parametrize("W_ws,nd_ws,W,n_det", [(17000, 2, 16384, 2), (33000, 4, 9000, 3)])
def test_workspace_of_a_larger_call(W_ws, nd_ws, W, n_det):
    """A workspace sized for more walkers (whose groups are smaller, so that
    it may hold less) serves fewer, with the same outputs; one byte less than
    a single determinant at a time needs is refused."""
    import ctypes as ct
    import torch
    from paper_1209_6630_amd._lib import MultidetArgs, lib
    print(f"[case] determinants' workspace {W_ws}x{nd_ws} for {W}x{n_det}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=5, n_up=10, n_dn=9, seed=4)
    S = make_gpu_system(sysm, A_up, A_dn)
    R = torch.from_numpy(walkers_near(sysm, W, seed=2)).cuda()
    occ = np.array([np.concatenate([np.roll(np.arange(10), K), np.arange(9)]) for K in range(n_det)], np.int32)
    coef = np.linspace(1.0, 2.0, n_det)
    want = S.multidet_forward(R, occ, coef, "fp64")
    n = ct.c_size_t()
    assert lib().qsl_multidet_workspace_size(S._h, W_ws, 0, nd_ws, ct.byref(n)) == 0
    got = {k: torch.zeros_like(v) for k, v in want.items() if not k.startswith("_")}
    ws = torch.empty(n.value, dtype=torch.uint8, device="cuda")

    def call(ws_bytes):
        a = MultidetArgs(W, R.data_ptr(), 0, n_det, occ.ctypes.data_as(ct.POINTER(ct.c_int32)),
                         coef.ctypes.data_as(ct.POINTER(ct.c_double)), got["logpsi"].data_ptr(), got["sign"].data_ptr(),
                         got["drift"].data_ptr(), got["lap"].data_ptr(), got["status"].data_ptr(),
                         got["det_logdet"].data_ptr(), got["det_sign"].data_ptr(), ws.data_ptr(), ws_bytes)
        return lib().qsl_multidet_forward(S._h, ct.byref(a), ct.c_void_p(torch.cuda.current_stream().cuda_stream))

    assert call(ws.numel()) == 0
    torch.cuda.synchronize()
    for k, v in got.items():
        np.testing.assert_array_equal(v.cpu().numpy(), want[k].cpu().numpy(), err_msg=k)
    assert lib().qsl_multidet_workspace_size(S._h, W, 0, 1, ct.byref(n)) == 0
    assert call(n.value - 1) == 4
