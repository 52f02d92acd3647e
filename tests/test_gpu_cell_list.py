"""The cell list at the sizes where its launches change: halos sorted by one
workgroup (up to 8192 particles, in four widths), the general sort with one
key past a whole tile, its three tile sizes, and batches with rank digits and
gaps.  A particle lost, doubled or out of place in the sorted order changes a
neighbour distance, so the kernel sizes must equal the oracle's bit for bit
(the bar of the kNN tests)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

K = 8


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2506_06269_amd as S
    assert torch.cuda.is_available()
    S.lib()
    return S


def _check(S, orc, parts, gap=0):
    import torch
    halos, off, s = [], 0, {}
    for p in parts:
        n = p["x"].size
        halos.append(dict(n=n, offset=off, eps=0.01, k=min(K, n - 1)))
        off += n + gap
    for f in ("x", "y", "z", "vx", "vy", "vz", "m", "id"):
        s[f] = np.zeros(off, dtype=parts[0][f].dtype)
        for h, p in zip(halos, parts):
            s[f][h["offset"]:h["offset"] + h["n"]] = p[f]
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, off, len(halos))
    S.sidm_knn_h(ctx, halos, dev)
    torch.cuda.synchronize()
    got = dev["h"].cpu().numpy()
    for h, p in zip(halos, parts):
        ref = orc.knn_tree(p["x"], p["y"], p["z"], p["id"], h["k"])
        assert np.array_equal(got[h["offset"]:h["offset"] + h["n"]], ref), h
    S.sidm_destroy(ctx)


@pytest.mark.parametrize("n", [2, 63, 1024, 1025, 2049, 4097, 8192, 8193, 65537, 262144, 262145,
                               524289])
def test_one_halo(S, orc, n):
    print(f"cell list n={n}", flush=True)
    _check(S, orc, [W.nfw_halo(n, seed=n)])


def test_ties_in_the_key(S, orc):
    """Many particles with one Morton code (clumps far smaller than a cell):
    the order among them is the caller's."""
    for n in (5000, 20000):
        _check(S, orc, [W.clustered(n, seed=n, n_clumps=3, width=1e-7)])


@pytest.mark.parametrize("sizes", [(8192, 2, 1000, 4097), (8193, 2, 100, 4097), (3000,) * 20 + (9000,)])
@pytest.mark.parametrize("gap", [0, 37])
def test_batches(S, orc, sizes, gap):
    print(f"cell list batch {sizes} gap={gap}", flush=True)
    _check(S, orc, [W.nfw_halo(n, seed=7 + i) for i, n in enumerate(sizes)], gap)
