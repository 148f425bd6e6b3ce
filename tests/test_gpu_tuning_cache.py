"""A tuning cache written for other kernels is not applied: its values mean
other shapes and forms there."""
import json

import numpy as np
import pytest

from tests.gpu_common import make_gpu_system
from tests.systems import random_tiny, walkers_near

pytestmark = pytest.mark.gpu


def test_entry_of_other_kernels_is_tuned_again(tmp_path):
    import torch
    from paper_1209_6630_amd.api import Plan
    print("[case] tuning cache of other kernels", flush=True)
    sysm, A_up, A_dn = random_tiny(n_atoms=4, n_up=9, n_dn=8, seed=3)
    S = make_gpu_system(sysm, A_up, A_dn)
    R = torch.from_numpy(walkers_near(sysm, 40, seed=1)).cuda()
    g = torch.ones((40, 2), dtype=torch.float64, device="cuda")
    cache = tmp_path / "tune.json"

    def plan():
        P = Plan([S], [40], "fp64", graph=False)
        dA = tuple(torch.empty((n, S.n_basis), dtype=torch.float64, device="cuda") for n in (9, 8))
        P.bind(0, R, S.alloc_outputs(40, "fp64"), g=g, dR=torch.empty_like(R), dA=dA)
        return P

    plan().autotune(str(cache))
    entry = json.loads(cache.read_text())["qslater_autotune"][0]
    parts = entry["key"].split("|")
    old = "|".join(p for p in parts if not p.startswith("kernels"))
    assert old != entry["key"]
    # 3 walkers a group: no candidate of the tuner
    line = json.dumps(dict(entry, key=old, adj_group=3))
    cache.write_text('{"qslater_autotune": [\n' + line + "\n]}\n")
    P = plan()
    assert P.autotune(str(cache))["adj_group"] != 3
    keys = [e["key"] for e in json.loads(cache.read_text())["qslater_autotune"]]
    assert keys == [old, entry["key"]]
