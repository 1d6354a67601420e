"""Waves on tiles: every orbit is run once and to the same bits whatever the
grid deals to which wave -- whole rounds, the last round's tiles on one block
per CU or on every slot, blocks of every size, and the batched launch's queue.
And the window test on the scaled momenta against the directions' angles."""
import math

import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu

ROUND = 2048 * 64   # orbits of one round with the tangent on 256 CUs; half of one without


@pytest.fixture(scope="module")
def aw():
    need_gpu()
    import paper_1107_4107_amd as m
    return m


@pytest.mark.parametrize("tangent", [True, False])
@pytest.mark.parametrize("n", [1, 65, 4 * 64 + 1, 1024 * 64 + 3, ROUND - 1, ROUND, ROUND + 1, ROUND + 1025 * 64,
                               2 * ROUND + 64 * 5 + 7, 2 * ROUND + 2049 * 64])
def test_every_orbit_once_whatever_the_grid(aw, n, tangent):
    print_case("wave tiles", n, tangent)
    e = aw.Ensemble(eps=1e-2, n_steps=2, ic_kind="box", n_orbits=n, seed_ic=7, tangent=tangent)
    ref = aw.map_ensemble(e, want_state=True)
    others = [aw.map_ensemble(e, want_state=True, tuning=aw.Tuning(block=b)) for b in (64, 256)]
    others.append(aw.map_ensemble(e, want_state=True, tuning=aw.Tuning(orbits_per_lane=2)))
    small = aw.Ensemble(eps=1e-2, n_steps=5, ic_kind="box", n_orbits=77, seed_ic=8, tangent=tangent)
    others.append(aw.map_ensembles([e, small], want_state=True)[0])
    for o in others:
        np.testing.assert_array_equal(np_(o.orbit_out), np_(ref.orbit_out))
        np.testing.assert_array_equal(np_(o.state), np_(ref.state))
        np.testing.assert_array_equal(np_(o.cls), np_(ref.cls))


@pytest.mark.parametrize("window", [(0.55, 1.05, -0.25, 0.25), (-math.pi, math.pi, -1.0, 1.0),
                                    (-math.pi, math.pi, -0.5, 1.0), (-math.pi, math.pi, -1.0, -0.2),
                                    (-3.0, 2.5, -1.0, 0.9), (0.0, math.pi, 0.0, 1.0), (-math.pi / 2, 0.0, 0.3, 0.7)])
def test_window_test_against_the_angles(aw, window):
    """eps = 0 keeps P, so bit 1 of the class is the test of the initial
    direction.  Directions within 1e-12 of an edge may fall either side (the
    test's products carry a few roundings of 1e-16); the axes, whose angles
    are edges of some windows, lie inside a closed window."""
    import torch
    print_case("window test", window)
    rng = np.random.default_rng(9)
    P = np.concatenate([rng.normal(size=(3, 20000)), np.array([[1.0, 0, 0, 1], [0, 1.0, 0, 0], [0, 0, 1.0, 0.0]])], axis=1)
    ic = np.concatenate([rng.uniform(0, 6, P.shape), P])
    e = aw.Ensemble(eps=0.0, n_steps=3, ic_kind="explicit", n_orbits=P.shape[1], tangent=False, window=window,
                    stay_in_window=True)
    r = aw.map_ensemble(e, torch.as_tensor(ic, dtype=torch.float64, device="cuda"))
    left = (np_(r.cls) & 2) != 0
    phi, mu = np.arctan2(P[1], P[0]), P[2] / np.sqrt((P * P).sum(0))
    m = np.minimum.reduce([phi - window[0], window[1] - phi, mu - window[2], window[3] - mu])
    if window[0] == -math.pi and window[1] == math.pi:
        m = np.minimum(mu - window[2], window[3] - mu)
    if window[2] == -1.0 and window[3] == 1.0:
        m = np.minimum(phi - window[0], window[1] - phi) if window[1] - window[0] < 6.28 else np.ones_like(m)
    sure = np.abs(m) > 1e-12
    assert sure.sum() > 19000 or window[3] - window[2] == 2.0
    np.testing.assert_array_equal(left[sure], m[sure] < 0)
