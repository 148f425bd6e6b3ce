"""FP64 products on an orbital set of more than 2^31 coefficients (33000 AO
slots x 65536 orbitals; 86 GB of the library's copies): offsets of the last
atom's rows pass 2^31.  Three one-orbital determinants of one electron at that
atom against the oracle's AO values (1e-12 of the absolute sum, the bound of
tests/gpu_common.py)."""
import ctypes as ct

import numpy as np
import pytest

import oracle
from tests.systems import make_tiny

pytestmark = pytest.mark.gpu


def test_rows_past_2_31():
    import torch
    from paper_1209_6630_amd._lib import check, lib
    from paper_1209_6630_amd.api import System
    free, _ = torch.cuda.mem_get_info()
    if free < 150 << 30:
        pytest.skip("needs 150 GiB of device memory")
    print("[case] fp64 products, 33000 slots x 65536 orbitals", flush=True)
    n_atoms, n_orb = 4125, 65536
    xyz = np.zeros((n_atoms, 3))
    xyz[:, 0] = 25.0 * np.arange(n_atoms)
    shells = [(a, 0, [0.3 + 0.2 * k], [1.0]) for a in range(n_atoms) for k in range(8)]
    sysm = make_tiny(shells, xyz, 1, 0)
    S = System.from_synth(sysm)
    A = torch.zeros((n_orb, S.n_basis), dtype=torch.float64, device="cuda")
    tail = np.random.default_rng(0).normal(size=(n_orb, 16))
    A[:, -16:] = torch.from_numpy(tail).cuda()
    check(lib().qsl_set_orbitals(S._h, 0, ct.c_void_p(A.data_ptr()), n_orb, S.n_basis, 1,
                                 ct.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    del A
    orbitals = [0, 40001, n_orb - 1]
    R = np.array([[[25.0 * (n_atoms - 1) + 0.4, -0.3, 0.2]]])
    out = S.multidet_forward(torch.from_numpy(R).cuda(), np.array(orbitals, np.int32)[:, None], np.ones(3), "fp64")
    torch.cuda.synchronize()
    idx, B, _ = oracle.ao_eval(sysm, R[0, 0])
    assert idx.min() >= S.n_basis - 16
    for K, o in enumerate(orbitals):
        a = tail[o, idx - (S.n_basis - 16)]
        c, scale = a @ B[0], np.abs(a) @ np.abs(B[0])
        got = float(out["det_logdet"][K, 0, 0])
        assert abs(got - np.log(abs(c))) <= 2e-12 * scale / abs(c) + 1e-15
        assert int(out["det_sign"][K, 0, 0]) == np.sign(c)
    S.close()
    torch.cuda.empty_cache()
