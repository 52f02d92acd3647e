"""Symmetric tiles of the FP64 direct sum (each unordered pair once, totals in
128-bit fixed point): the oracle's forces to the FP64 bar (1e-12 normwise) in
every launch shape on both sides of the smallest halo that takes them, with a
host, unequal, negative and zero masses; the same bits on repeated calls and
when other halos share the call; halos that the fixed-point totals cannot hold
(a value that is not finite, a box far larger than the softening) give the
one-sided sums bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

MIN_N = 40960


@pytest.fixture(scope="module")
def S():
    import torch
    import paper_2506_06269_amd as S
    assert torch.cuda.is_available()
    S.lib()
    return S


def _forces(S, ctx, halos, dev):
    import torch
    for f in ("ax", "ay", "az", "pot"):
        dev[f].fill_(float("nan"))
    S.sidm_gravity(ctx, halos, dev, S.SIDM_PREC_FP64)
    torch.cuda.synchronize()
    out = S.state_to_host(dev)
    return [out[f] for f in ("ax", "ay", "az", "pot")]


def _oracle(orc, s, eps, host=None):
    ax, ay, az, pot, an = orc.gravity(s["x"], s["y"], s["z"], s["m"], 1.0, eps, want_norm=True)
    if host is not None:
        hx, hy, hz, hp = orc.host_field(s["x"], s["y"], s["z"], orc.make_params(host=host))
        ax, ay, az, pot = ax + hx, ay + hy, az + hz, pot + hp
        an = an + np.sqrt(hx ** 2 + hy ** 2 + hz ** 2)
    return ax, ay, az, pot, an


def _check(got, ref, pot_norm=None):
    ax, ay, az, pot, an = ref
    e = np.sqrt((got[0] - ax) ** 2 + (got[1] - ay) ** 2 + (got[2] - az) ** 2) / an
    ep = np.abs(got[3] - pot) / (np.abs(pot) if pot_norm is None else pot_norm)
    print(f"max e_a {e.max():.2e} e_phi {ep.max():.2e}", flush=True)
    assert e.max() < 1e-12 and ep.max() < 1e-12


@pytest.mark.parametrize("n", [MIN_N - 1, MIN_N, MIN_N + 1, 43210])
def test_sizes_and_shapes(S, orc, n):
    s = W.place_on_orbit(W.nfw_halo(n, seed=n))
    halo = dict(n=n, eps=0.01, host=W.host_params())
    ref = _oracle(orc, s, 0.01, W.host_params())
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    for ireg, nt in (S.SHAPES if n == 43210 else [(4, 256)]):
        print(f"n={n} {ireg}x{nt}", flush=True)
        S.sidm_set_launch_shape(ctx, ireg, nt, True)
        got = _forces(S, ctx, [halo], dev)
        _check(got, ref)
        again = _forces(S, ctx, [halo], dev)
        assert all(np.array_equal(a, b) for a, b in zip(got, again))
    S.sidm_destroy(ctx)


@pytest.mark.parametrize("kind", ["drawn", "signs", "some zero", "all zero"])
def test_masses(S, orc, kind):
    n = MIN_N + 77
    s = W.nfw_halo(n, seed=3)
    rng = np.random.default_rng(4)
    s["m"] = {"drawn": lambda: rng.uniform(0.5, 1.5, n) / n,
              "signs": lambda: rng.choice((-3.0, 1.0), n) / n,
              "some zero": lambda: rng.choice((0.0, 1.0), n) / n,
              "all zero": lambda: np.zeros(n)}[kind]()
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    got = _forces(S, ctx, [dict(n=n, eps=0.02)], dev)
    if kind == "all zero":
        assert all(np.all(g == 0.0) for g in got)
        return
    ref = _oracle(orc, s, 0.02)
    # the scales of the sums of magnitudes
    *_, pm, an = orc.gravity(s["x"], s["y"], s["z"], np.abs(s["m"]), 1.0, 0.02, want_norm=True)
    _check(got, ref[:4] + (an,), np.abs(pm))
    S.sidm_destroy(ctx)


def test_batch_equals_single_calls(S, orc):
    """A large halo's bits do not depend on the halos that share its call (one
    with other masses, one below the threshold)."""
    sizes = (MIN_N + 1000, 5000, MIN_N + 300)
    parts = [W.nfw_halo(n, seed=20 + i) for i, n in enumerate(sizes)]
    parts[2]["m"] = np.random.default_rng(1).uniform(0.5, 1.5, sizes[2]) / sizes[2]
    s = {f: np.concatenate([p[f] for p in parts]) for f in parts[0]}
    halos, off = [], 0
    for n in sizes:
        halos.append(dict(n=n, offset=off, eps=0.01))
        off += n
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, off, len(halos))
    got = _forces(S, ctx, halos, dev)
    for h, p in zip(halos, parts):
        part = [g[h["offset"]:h["offset"] + h["n"]] for g in got]
        _check(part, _oracle(orc, p, 0.01))
    one = S.state_to_device(parts[2])
    c1 = S.sidm_create(0, sizes[2], 1)
    alone = _forces(S, c1, [dict(n=sizes[2], eps=0.01)], one)
    o = halos[2]["offset"]
    assert all(np.array_equal(g[o:o + sizes[2]], a) for g, a in zip(got, alone))
    S.sidm_destroy(ctx)
    S.sidm_destroy(c1)


@pytest.mark.parametrize("kind", ["nan position", "infinite mass", "nan mass", "far particle",
                                  "tiny softening"])
def test_left_to_the_one_sided_sums(S, kind):
    """The decision is the device's; the result is that of the one-sided tiles."""
    n, eps = MIN_N + 500, 0.01
    s = W.nfw_halo(n, seed=6)
    if kind == "nan position":
        s["y"][777] = np.nan
    elif kind == "infinite mass":
        s["m"][5] = np.inf
    elif kind == "nan mass":
        s["m"][5] = np.nan
    elif kind == "far particle":
        s["z"][123] = 1e5
    else:
        eps = 1e-6
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    got = _forces(S, ctx, [dict(n=n, eps=eps)], dev)
    S.sidm_set_symmetric(ctx, 0)
    ref = _forces(S, ctx, [dict(n=n, eps=eps)], dev)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b, equal_nan=True)
    if kind == "nan position":
        assert all(np.all(np.isnan(g)) for g in got)
    S.sidm_destroy(ctx)


def test_graph_replays(S):
    """A captured call replayed between eager work gives the eager bits."""
    import torch
    n = MIN_N + 40
    s = W.nfw_halo(n, seed=8)
    dev = S.state_to_device(s)
    ctx = S.sidm_create(0, n, 1)
    halos = [dict(n=n, eps=0.01)]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ref = _forces(S, ctx, halos, dev)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        S.sidm_gravity(ctx, halos, dev, S.SIDM_PREC_FP64)
    for _ in range(3):
        for f in ("ax", "ay", "az", "pot"):
            dev[f].fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        out = S.state_to_host(dev)
        assert all(np.array_equal(out[f], r) for f, r in zip(("ax", "ay", "az", "pot"), ref))
    S.sidm_destroy(ctx)
