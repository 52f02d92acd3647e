"""Symmetric FP64 tiles where their work items are longer than the shortest
(2^20 particles, in a large and in the smallest launch shape): sampled particles
to the FP64 bar (1e-12 normwise) against the oracle, with equal and unequal
masses and one that dominates; and the sums over an item's tiles, which lose
no more than a run of 32 tiles' roundings however long the item is."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

N = (1 << 20) + 77


def _forces(s, halo, ireg, nt):
    import torch
    import paper_2506_06269_amd as S
    n = s["x"].size
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    S.sidm_set_launch_shape(ctx, ireg, nt, False)
    S.sidm_gravity(ctx, [halo], dev, S.SIDM_PREC_FP64)
    torch.cuda.synchronize()
    out = S.state_to_host(dev)
    S.sidm_destroy(ctx)
    return [out[f] for f in ("ax", "ay", "az", "pot")]


@pytest.mark.parametrize("ireg,nt", [(8, 256), (2, 128)])
@pytest.mark.parametrize("masses", ["equal", "drawn", "one dominates"])
def test_sampled(orc, ireg, nt, masses):
    s = dict(W.nfw_halo(N, seed=17))
    rng = np.random.default_rng(2)
    if masses == "drawn":
        s["m"] = s["m"] * rng.uniform(0.5, 1.5, N)
    elif masses == "one dominates":
        s["m"] = s["m"].copy()
        s["m"][N // 3] = 10.0 * s["m"].sum()
    q = rng.choice(N, 256, replace=False)
    ax, ay, az, pot, an = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0, 0.01, query=q,
                                      want_norm=True)
    got = [g[q] for g in _forces(s, dict(n=N, eps=0.01), ireg, nt)]
    e = np.sqrt((got[0] - ax) ** 2 + (got[1] - ay) ** 2 + (got[2] - az) ** 2) / an
    ep = np.abs(got[3] - pot) / np.abs(pot)
    print(f"{ireg}x{nt} {masses}: e_a {e.max():.2e} e_phi {ep.max():.2e}", flush=True)
    assert e.max() < 1e-12 and ep.max() < 1e-12


def test_long_items_keep_small_tiles():
    """One heavy particle pulls a small group, first in the sorted order, along
    x; the other 2^20 are far off along x, and a tile of 128 of them pulls with
    0.45 of 2^-53 of the heavy one's force, less than half an ulp of it.  Summed
    plainly over the item's tiles (some 256 in this shape) each of them would be
    lost, 1.3e-14 in all; a run of 32 tiles loses at most 32 x 5.0e-17 = 1.6e-15.
    The bar adds 16 of 2^-53 for the heavy term (its separation, square, reciprocal
    root cubed and products) and for the total's scaling."""
    rng = np.random.default_rng(5)
    n, group, d = N, 128, 0.05
    s = {f: np.zeros(n) for f in ("x", "y", "z", "vx", "vy", "vz")}
    s["id"] = np.arange(n, dtype=np.uint32)
    # the group at the low corner of the box, the heavy one d further along x
    for f in ("x", "y", "z"):
        s[f][:group] = rng.uniform(0.0, 1e-6, group)
        s[f][group:] = (0.0 if f != "x" else 1.0) + rng.uniform(0.0, 1e-4, n - group)
    s["x"][group - 1] = d
    eps = 0.01
    heavy = d / (d * d + eps * eps) ** 1.5
    far = 1.0 / (1.0 + eps * eps) ** 1.5
    light = 0.45 * 2.0 ** -53 * heavy / (128 * far)
    s["m"] = np.full(n, light)
    s["m"][group - 1] = 1.0
    got = _forces(s, dict(n=n, eps=eps), 2, 128)
    L = np.longdouble
    worst = 0.0
    for i in range(0, group - 1, 8):
        dx = s["x"].astype(L) - L(s["x"][i])
        dy = s["y"].astype(L) - L(s["y"][i])
        dz = s["z"].astype(L) - L(s["z"][i])
        r2 = dx * dx + dy * dy + dz * dz + L(np.float64(eps) * np.float64(eps))
        r2[i] = 1
        w = s["m"].astype(L) / (r2 * np.sqrt(r2))
        w[i] = 0
        ref = (w * dx).sum()
        worst = max(worst, float(abs(L(got[0][i]) - ref) / ref))
    print(f"worst {worst:.2e}", flush=True)
    assert worst < (32 * 0.45 + 16) * 2.0 ** -53


@pytest.mark.parametrize("masses", ["equal", "one dominates"])
def test_wide_boxes_by_mass(orc, masses):
    """A box of 2^19 softenings: the totals hold the force at its edge when the
    masses are equal, and do not when one of 41460 holds almost all mass (their
    unit goes with n times the largest mass, the force with the mass): such a
    halo gives the one-sided sums bit for bit."""
    import torch
    import paper_2506_06269_amd as S
    n, eps = 41460, 0.01
    s = dict(W.nfw_halo(n, seed=6))
    s["z"] = s["z"].copy()
    s["z"][123] = 2.0 ** 19 * eps + s["z"].min()
    if masses != "equal":
        s["m"] = np.full(n, 1e-8)
        s["m"][5] = 1.0
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    halo = dict(n=n, eps=eps)
    out = []
    for min_n in (4096, 0):
        S.sidm_set_symmetric(ctx, min_n)
        S.sidm_gravity(ctx, [halo], dev, S.SIDM_PREC_FP64)
        torch.cuda.synchronize()
        h = S.state_to_host(dev)
        out.append([h[f] for f in ("ax", "ay", "az", "pot")])
    S.sidm_destroy(ctx)
    same = all(np.array_equal(a, b) for a, b in zip(*out))
    assert same == (masses != "equal")
    ax, ay, az, pot, an = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0, eps, want_norm=True)
    got = out[0]
    e = np.sqrt((got[0] - ax) ** 2 + (got[1] - ay) ** 2 + (got[2] - az) ** 2) / an
    assert e.max() < 1e-12 and np.max(np.abs(got[3] - pot) / np.abs(pot)) < 1e-12
