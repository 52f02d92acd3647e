"""The context-free FP64 sum (work items of 64 i and whole tiles of 64 j): the
oracle's forces to the FP64 bar (1e-12 normwise) at the edges of its tiles and
of its rules (4096 waves, 2^18 partial rows, the large items from 64513 on), with unequal masses."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 64, 65, 129, 1500, 4096, 4097, 16385, 64512, 64513])
@pytest.mark.parametrize("masses", ["equal", "unequal"])
def test_static_fp64(orc, n, masses):
    import torch
    import paper_2506_06269_amd as S
    s = dict(W.nfw_halo(n, seed=n))
    if masses == "unequal":
        s["m"] = s["m"] * np.random.default_rng(n).uniform(0.5, 1.5, n)
    ax, ay, az, pot, an = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0, 0.01, want_norm=True)
    dev = S.state_to_device(s)
    for f in ("ax", "ay", "az", "pot"):
        dev[f].fill_(float("nan"))
    S.sidm_gravity_static(dict(n=n, eps=0.01), dev, S.SIDM_PREC_FP64)
    torch.cuda.synchronize()
    o = S.state_to_host(dev)
    e = np.sqrt((o["ax"] - ax) ** 2 + (o["ay"] - ay) ** 2 + (o["az"] - az) ** 2)
    assert np.all(e <= 1e-12 * an)
    assert np.all(np.abs(o["pot"] - pot) <= 1e-12 * np.abs(pot))
