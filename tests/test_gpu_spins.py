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
