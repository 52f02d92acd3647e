"""Cycles of block steps whose idle ticks lie between ticks that end a step: the
largest bin in use is neither 0 nor the halo's max_bin (asserted from the
oracle's bins), so that ticks are skipped and run in turn, alone, beside a halo
with fewer ticks, and on a context whose previous cycle had no idle tick; the
FP64 bar of block steps (1e-12 of the largest magnitude)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

XV = ("x", "y", "z", "vx", "vy", "vz")


@pytest.mark.parametrize("sizes", [(3000,), (8200,), (8200, 500)])
@pytest.mark.parametrize("etas", [(0.1, 0.1), (0.2, 0.2), (0.006, 0.2, 0.1)])
def test_skipped_and_run_in_turn(orc, sizes, etas):
    import torch
    import paper_2506_06269_amd as S
    max_bin = 4
    parts, off = [], []
    for q, n in enumerate(sizes):
        s = dict(W.nfw_halo(n, seed=40 + q))
        s["id"] = np.arange(n, dtype=s["id"].dtype)
        s["ax"], s["ay"], s["az"], s["pot"] = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0,
                                                          0.01)
        s["h"] = np.zeros(n)
        off.append(sum(sizes[:q]))
        parts.append(s)
    dev = S.state_to_device({f: np.concatenate([p[f] for p in parts]) for f in parts[0]})
    ctx = S.sidm_create(0, sum(sizes), len(sizes))
    for cyc, eta in enumerate(etas):
        halos = [dict(offset=off[q], n=n, eps=0.01, sigma_m=1.0, dt=1.0 / 16, k=16, seed=5,
                      steps=dict(eta=eta, max_bin=max_bin - 2 * q))
                 for q, n in enumerate(sizes)]
        before = S.state_to_host(dev)
        S.sidm_kdk_step(ctx, halos, dev, cyc, S.SIDM_PREC_FP64)
        torch.cuda.synchronize()
        out = S.state_to_host(dev)
        for q, h in enumerate(halos):
            sl = slice(h["offset"], h["offset"] + h["n"])
            ref = {f: v[sl].copy() for f, v in before.items()}
            p = orc.make_params(G=1.0, eps=0.01, sigma_m=1.0, dt=h["dt"], k=16, seed=5,
                                steps=h["steps"])
            if q == 0:
                deepest = orc.time_bin(p, ref["ax"], ref["ay"], ref["az"]).max()
                assert deepest == max_bin if eta < 0.01 else 0 < deepest < max_bin
            orc.kdk_step(ref, p, cyc)
            for f in XV:
                assert np.max(np.abs(out[f][sl] - ref[f])) <= 1e-12 * np.max(np.abs(ref[f]))
    S.sidm_destroy(ctx)
