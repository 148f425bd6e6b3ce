"""One C and one D^-1 buffer for both spins, for callers that need neither: the
spins run one after the other and log|det|, sign, drift and Laplacian are bit
for bit those of a call with buffers of their own; the shared buffers end with
the second spin's values."""
import numpy as np
import pytest

from tests.gpu_common import make_gpu_system
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_up,n_dn,W,mode", [(20, 20, 40, "fp64"), (33, 9, 65, "fp32"), (130, 129, 3, "bf16x3"), (230, 20, 2, "fp64")])
@pytest.mark.parametrize("share", ["C", "Dinv", "both", "cross"])
def test_shared_between_spins(n_up, n_dn, W, mode, share):
    import torch
    print(f"[case] shared outputs n={n_up}/{n_dn} W={W} {mode} {share}", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=(n_up + n_dn) // 6 + 2, n_up=n_up, n_dn=n_dn, seed=n_up)
    R = torch.from_numpy(walkers_near(sysm, W, seed=n_dn)).cuda()
    S = make_gpu_system(sysm, A_up, A_dn)
    want = S.forward(R, mode)
    out = S.alloc_outputs(W, mode)
    if share in ("C", "both"):
        out["C_dn"] = out["C_up"].view(-1)[:out["C_dn"].numel()].view_as(out["C_dn"])
    if share in ("Dinv", "both"):
        out["Dinv_dn"] = out["Dinv_up"].view(-1)[:out["Dinv_dn"].numel()].view_as(out["Dinv_dn"])
    if share == "cross":  # the second spin's C over the first one's inverse
        buf = torch.empty(max(out["Dinv_up"].numel(), out["C_dn"].numel()), dtype=torch.float64, device="cuda")
        out["Dinv_up"] = buf[:out["Dinv_up"].numel()].view_as(out["Dinv_up"])
        out["C_dn"] = buf.view(out["C_dn"].dtype)[:out["C_dn"].numel()].view_as(out["C_dn"])
    S.forward(R, mode, out=out)
    torch.cuda.synchronize()
    for k in ("logdet", "sign", "drift", "lap", "status", "C_dn", "Dinv_dn"):
        np.testing.assert_array_equal(out[k].cpu().numpy(), want[k].cpu().numpy(), err_msg=k)
