"""Kernel sizes where distances are infinite: only real particles are counted
and read, whatever the size of the searched sphere.  A particle at infinity is
infinitely far from finite ones, and its distance to another one there is not a
number: h is infinite where k others are comparable, NaN where they are not;
finite particles that have k finite others keep the oracle's h."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _knn(s, k, h0):
    import torch
    import paper_2506_06269_amd as S
    n = s["x"].size
    dev = S.state_to_device(s)
    dev["h"].copy_(torch.from_numpy(h0))
    ctx = S.sidm_create(0, n, 1)
    S.sidm_knn_h(ctx, [dict(n=n, eps=0.01, k=k)], dev)
    torch.cuda.synchronize()
    h = dev["h"].cpu().numpy()
    S.sidm_destroy(ctx)
    return h


@pytest.mark.parametrize("axis", ["x", "y", "z"])
def test_too_few_comparable_distances(axis):
    """Five particles, two at infinity: for those, three of k = 4 others."""
    s = dict(W.maxwell_box(5, seed=3))
    s[axis] = s[axis].copy()
    s[axis][:2] = np.inf
    h = _knn(s, 4, np.zeros(5))
    assert np.all(np.isnan(h[:2])) and np.all(np.isposinf(h[2:]))


@pytest.mark.parametrize("n", [20, 21, 22, 23, 90])
@pytest.mark.parametrize("h0", [0.0, 1e200])
@pytest.mark.parametrize("axis", ["x", "z"])
def test_sphere_without_bound(orc, n, h0, axis):
    """A previous kernel size whose square overflows, of the particle at infinity."""
    s = dict(W.maxwell_box(n, seed=n))
    s[axis] = s[axis].copy()
    s[axis][0] = np.inf
    hint = np.zeros(n)
    hint[0] = h0
    k = 8
    h = _knn(s, k, hint)
    assert np.isposinf(h[0])
    t = [s[f][1:] for f in ("x", "y", "z")]
    ref, _ = orc.knn(*t, s["id"][1:], k, want_list=True)
    assert np.array_equal(h[1:], ref)
