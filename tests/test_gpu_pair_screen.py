"""The pair pass: its matrix-core screen must let every pair through that the
exact test accepts.  The pairs counted are those of all i < j in double
precision (the same operations, so the numbers are equal): at the edges of the
screen's tiles (32 rows and columns, 64 candidates), with kernel sizes over
five decades (the scale of a batch is that of its widest), far from the
origin, and at lengths that single precision does not hold."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _count(s):
    n = 0
    for i in range(s["x"].size - 1):
        dx, dy, dz = (s[f][i + 1:] - s[f][i] for f in "xyz")
        hs = s["h"][i] + s["h"][i + 1:]
        n += int(np.count_nonzero((dx * dx + dy * dy) + dz * dz < hs * hs))
    return n


@pytest.mark.parametrize("n", [2, 31, 33, 63, 65, 97, 129, 1000, 4097])
@pytest.mark.parametrize("kind", ["knn", "decades", "offset", "tiny", "huge"])
def test_all_pairs_found(orc, n, kind):
    import torch
    import paper_2506_06269_amd as S
    s = dict(W.nfw_halo(n, seed=n))
    if n > 64:
        s["h"] = orc.knn(s["x"], s["y"], s["z"], s["id"], min(16, n - 1))
    else:
        s["h"] = np.full(n, 0.5 * np.abs(s["x"]).mean())
    if kind == "decades":
        s["h"] = s["h"] * 10.0 ** np.random.default_rng(n).uniform(-4.0, 1.0, n)
    scale = {"tiny": 2.0 ** -130, "huge": 2.0 ** 130}.get(kind, 1.0)
    for f in ("x", "y", "z", "h"):
        s[f] = s[f] * scale
    if kind == "offset":
        s["x"] = s["x"] + 1e6
    if scale != 1.0:
        for f in ("vx", "vy", "vz"):
            s[f] = np.zeros(n)   # no candidates of the exact decision
    halo = dict(n=n, eps=0.01, k=16, sigma_m=1e-3, dt=1e-6, seed=3)
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    S.sidm_scatter(ctx, [halo], dev, 1)
    diag = S.diag_buffer(1)
    S.sidm_diagnostics(ctx, [halo], dev, diag)
    torch.cuda.synchronize()
    assert S.read_diag(diag)[0]["n_pairs"] == _count(s)
