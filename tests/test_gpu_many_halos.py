"""Tidal radii of batches against calls with one halo: very many small halos
beside a large one (more workgroups than one grid holds, if every halo had the
large one's number of them), and both sides of the rule that gives each of many
small halos one wave.  The mass sums of a halo are grouped by the call's other
halos: 1e-12, the bar of the tidal tests."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _check(orc, sizes, some):
    import torch
    import paper_2506_06269_amd as S
    total = sum(sizes)
    p = W.place_on_orbit(W.nfw_halo(total, seed=5))
    _, _, _, hp = orc.host_field(p["x"], p["y"], p["z"], orc.make_params(host=W.host_params()))
    p["pot"] = hp - np.random.default_rng(1).uniform(1.0, 2.0, hp.size)
    off = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    halos = [dict(n=int(n), offset=int(o), eps=0.01, host=W.host_params())
             for n, o in zip(sizes, off)]
    dev = S.state_to_device(p)
    ctx = S.sidm_create(0, total, len(halos))
    got = S.sidm_tidal_radius(ctx, halos, dev)
    S.sidm_destroy(ctx)
    torch.cuda.synchronize()
    one = S.sidm_create(0, total, 1)
    for h in some:
        ref = S.sidm_tidal_radius(one, [halos[h]], dev)[0]
        assert got[h]["index"] == ref["index"] and got[h]["status"] == ref["status"], h
        for f in ("r_tidal", "mass", "x", "y", "z"):
            assert got[h][f] == pytest.approx(ref[f], rel=1e-12), (h, f)
    S.sidm_destroy(one)


def test_many_beside_a_large_one(orc):
    small = 33000
    _check(orc, [2] * small + [65536], (0, 1, small // 2, small - 1, small))


@pytest.mark.parametrize("n_halos", [2, 256, 257, 700])
@pytest.mark.parametrize("largest", [3, 64, 65, 4096, 4097])
def test_waves_and_workgroups(orc, n_halos, largest):
    sizes = [2 + (7 * i) % (largest - 1) for i in range(n_halos - 1)] + [largest]
    _check(orc, sizes, (0, 1, n_halos // 2, n_halos - 1))
