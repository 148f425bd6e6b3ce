"""The FP64 products at the edges of their MO blocks (16), workgroup shapes (128
and 256 MOs) and walker tiles (32), against the oracle (bounds of
tests/gpu_common.py); and the uneven batch, whose small systems run in the
largest one's shape, bit for bit as alone."""
import numpy as np
import pytest

from tests.gpu_common import compare_forward, make_gpu_system, run_gpu_forward
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


def _system(n_up, n_dn, W):
    sysm, A_up, A_dn = random_tiny(n_atoms=max(2, (n_up + n_dn) // 6 + 1), n_up=n_up, n_dn=n_dn, seed=n_up + 3 * n_dn)
    return sysm, A_up, A_dn, walkers_near(sysm, W, seed=n_up)


@pytest.mark.parametrize("n_up,n_dn,W", [(1, 1, 33), (16, 15, 32), (17, 16, 31), (64, 63, 2), (128, 127, 1),
                                         (129, 128, 2), (241, 240, 1), (257, 256, 1)])
def test_block_and_tile_edges(n_up, n_dn, W):
    print(f"[case] fp64 products n_up={n_up} n_dn={n_dn} W={W}", flush=True)
    sysm, A_up, A_dn, R = _system(n_up, n_dn, W)
    S = make_gpu_system(sysm, A_up, A_dn)
    compare_forward(sysm, A_up, A_dn, R, run_gpu_forward(S, R, "fp64"), "fp64")


@pytest.mark.parametrize("persistent", [0, 1])
def test_mixed_shapes_in_one_launch(persistent):
    print(f"[case] fp64 mixed shapes persistent={persistent}", flush=True)
    import torch
    from paper_1209_6630_amd.api import Plan
    items = [_system(150, 130, 5), _system(20, 19, 40), _system(3, 0, 7)]
    systems = [make_gpu_system(m, a, b) for m, a, b, _ in items]
    alone = [run_gpu_forward(S, it[3], "fp64") for S, it in zip(systems, items)]
    P = Plan(systems, [it[3].shape[0] for it in items], "fp64", graph=False)
    P.tuning = dict(persistent=persistent)
    outs = []
    for i, (S, it) in enumerate(zip(systems, items)):
        R = torch.from_numpy(np.ascontiguousarray(it[3])).cuda()
        outs.append(S.alloc_outputs(R.shape[0], "fp64"))
        P.bind(i, R, outs[-1])
    P.launch()
    torch.cuda.synchronize()
    for ref, out in zip(alone, outs):
        for k, v in ref.items():
            np.testing.assert_array_equal(out[k].cpu().numpy(), v, err_msg=k)
