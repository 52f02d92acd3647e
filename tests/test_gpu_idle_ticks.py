"""Ticks of a cycle at which no particle's step ends do no cell list and no
forces: cycles on a context that has made no cell list before, with every
tick but the last idle, with some idle, and with none, on both sides of the
size up to which one workgroup sorts a halo, alone and beside a halo with
fewer ticks; the FP64 bar of block steps (1e-12 of the largest magnitude)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

XV = ("x", "y", "z", "vx", "vy", "vz")


@pytest.mark.parametrize("sizes", [(3000,), (8200,), (8200, 500)])
@pytest.mark.parametrize("eta,bins", [(1e3, "one"), (0.025, "some"), (0.006, "deep")])
def test_cycles_with_idle_ticks(orc, sizes, eta, bins):
    import torch
    import paper_2506_06269_amd as S
    parts, halos, off = [], [], 0
    for q, n in enumerate(sizes):
        s = dict(W.nfw_halo(n, seed=40 + q))
        s["id"] = np.arange(n, dtype=s["id"].dtype)
        s["ax"], s["ay"], s["az"], s["pot"] = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0,
                                                          0.01)
        s["h"] = np.zeros(n)
        halos.append(dict(offset=off, n=n, eps=0.01, sigma_m=1.0, dt=1.0 / 16, k=16, seed=5,
                          steps=dict(eta=eta, max_bin=4 - 2 * q)))
        parts.append(s)
        off += n
    state = {f: np.concatenate([p[f] for p in parts]) for f in parts[0]}
    dev = S.state_to_device(state)
    ctx = S.sidm_create(0, off, len(sizes))
    for cyc in range(2):
        before = S.state_to_host(dev)
        S.sidm_kdk_step(ctx, halos, dev, cyc, S.SIDM_PREC_FP64)
        torch.cuda.synchronize()
        out = S.state_to_host(dev)
        for h in halos:
            sl = slice(h["offset"], h["offset"] + h["n"])
            ref = {f: v[sl].copy() for f, v in before.items()}
            p = orc.make_params(G=1.0, eps=0.01, sigma_m=1.0, dt=h["dt"], k=16, seed=5,
                                steps=h["steps"])
            used = orc.time_bin(p, ref["ax"], ref["ay"], ref["az"])
            if bins == "one":
                assert used.max() == 0
            orc.kdk_step(ref, p, cyc)
            for f in XV:
                assert np.max(np.abs(out[f][sl] - ref[f])) <= 1e-12 * np.max(np.abs(ref[f]))
