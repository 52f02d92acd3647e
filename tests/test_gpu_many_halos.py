"""A call of very many small halos beside a large one (more workgroups than one
grid holds, if every halo had the large one's number of them): the tidal radii
are those of calls with one halo."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_tidal_radius_of_many_halos(orc):
    import torch
    import paper_2506_06269_amd as S
    small, big = 33000, 65536
    p = W.place_on_orbit(W.nfw_halo(2 * small + big, seed=5))
    _, _, _, hp = orc.host_field(p["x"], p["y"], p["z"], orc.make_params(host=W.host_params()))
    p["pot"] = hp - np.random.default_rng(1).uniform(1.0, 2.0, hp.size)
    halos = [dict(n=2, offset=2 * i, eps=0.01, host=W.host_params()) for i in range(small)]
    halos.append(dict(n=big, offset=2 * small, eps=0.01, host=W.host_params()))
    dev = S.state_to_device(p)
    ctx = S.sidm_create(0, 2 * small + big, len(halos))
    got = S.sidm_tidal_radius(ctx, halos, dev)
    S.sidm_destroy(ctx)
    torch.cuda.synchronize()
    one = S.sidm_create(0, 2 * small + big, 1)
    for h in (0, 1, small // 2, small - 1, small):
        ref = S.sidm_tidal_radius(one, [halos[h]], dev)[0]
        assert got[h] == ref, h
    S.sidm_destroy(one)
