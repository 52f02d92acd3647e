"""The tidal radius's bisection (several steps per pass over the particles) where
it can go wrong: halos of one and two workgroups and of more than the passes
have, a batch with unequal masses, no crossing inside the halo, and no finite
potential.  Radius and enclosed mass against the oracle's bisection to 1e-12 (the
bar of the oracle's own tidal test), the mass exactly the sum of the members'
where they are equal."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2506_06269_amd as S
    assert torch.cuda.is_available()
    S.lib()
    return S


def _self_potential(p):
    """Lowest at the halo's first particle."""
    phi = np.zeros(p["x"].size)
    phi[0] = -1.0
    return phi


def _total_potential(orc, halo, p):
    _, _, _, hp = orc.host_field(p["x"], p["y"], p["z"], orc.make_params(host=halo["host"]))
    return hp + 1e3 * _self_potential(p)


def _check(S, orc, parts, halos):
    s = {f: np.concatenate([p[f] for p in parts]) for f in parts[0]}
    s["pot"] = np.concatenate([_total_potential(orc, h, p) for h, p in zip(halos, parts)])
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, s["x"].size, len(halos))
    got = S.sidm_tidal_radius(ctx, halos, dev)
    for g, h, p in zip(got, halos, parts):
        r, mass, _, st = orc.tidal_radius(p["x"], p["y"], p["z"], p["m"], _self_potential(p),
                                          orc.make_params(host=h["host"]))
        print(f"n={h['n']} r_t {g['r_tidal']!r} oracle {r!r} status {g['status']}", flush=True)
        assert g["status"] == st and g["index"] == h["offset"]
        assert g["r_tidal"] == pytest.approx(r, rel=1e-12)
        assert g["mass"] == pytest.approx(mass, rel=1e-12)
    S.sidm_destroy(ctx)


@pytest.mark.parametrize("n", [2, 255, 256, 257, 513, 65536, 65537, 140000])
def test_sizes(S, orc, n):
    p = W.place_on_orbit(W.nfw_halo(n, seed=n))
    _check(S, orc, [p], [dict(n=n, offset=0, eps=0.01, host=W.host_params())])


def test_batch_with_unequal_masses(S, orc):
    parts, halos, off = [], [], 0
    rng = np.random.default_rng(2)
    for i, n in enumerate((300, 70000, 5, 1000)):
        p = W.place_on_orbit(W.nfw_halo(n, seed=40 + i))
        if i % 2:
            p["m"] = p["m"] * rng.uniform(0.5, 1.5, n)
        parts.append(p)
        halos.append(dict(n=n, offset=off, eps=0.01, host=W.host_params()))
        off += n
    _check(S, orc, parts, halos)


def test_no_crossing_and_no_centre(S, orc):
    """A host without mass never wins (status 1, the whole mass); without a
    finite potential there is no centre."""
    n = 3000
    p = W.nfw_halo(n, seed=1)
    h = dict(n=n, offset=0, eps=0.01, host=dict(rho_s=1e-12, r_s=1.0, center=(50.0, 0.0, 0.0)))
    _check(S, orc, [p], [h])
    dev = S.state_to_device(dict(p, pot=np.full(n, np.nan)))
    ctx = S.sidm_create(0, n, 1)
    g = S.sidm_tidal_radius(ctx, [h], dev)[0]
    assert g["index"] == -1 and g["mass"] == 0.0
    S.sidm_destroy(ctx)
