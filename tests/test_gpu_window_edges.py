"""The remained-in-the-window test on the edges of the window.

The initial momentum is tested as it was given: half-plane products against the
edge directions for phi, p_z against mu |P| with |P| rounded once.  At eps = 0
momenta never change, so an orbit is marked as having left exactly if its
initial momentum fails that test, for momenta of small whole numbers on edges
they lie on exactly (mu = 3/5 of (4, 0, 3)) or to rounding (phi = atan2(2, 3))
alike, and however the run is split."""
import math

import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu

PHIS = sorted({math.atan2(j, i) for i in range(-3, 4) for j in range(-3, 4) if i or j})
MUS = [-1.0, -0.8, -0.6, -0.5, 0.0, 0.6, 0.8, 1.0]


def _momenta():
    g = np.arange(-4.0, 5.0)
    p = np.array(np.meshgrid(g, g, g, indexing="ij")).reshape(3, -1)
    return p[:, np.any(p != 0.0, axis=0)]


def _inside(p, win):
    """The test of a momentum as given, in binary64."""
    lo, hi, mlo, mhi = win
    ok = np.ones(p.shape[1], bool)
    if (lo, hi) != (-math.pi, math.pi):
        c0 = math.cos(lo) * p[1] - math.sin(lo) * p[0]
        c1 = p[0] * math.sin(hi) - p[1] * math.cos(hi)
        ok &= (c0 >= 0) & (c1 >= 0) if hi - lo <= math.pi else ~((c0 < 0) & (c1 < 0))
    if (mlo, mhi) != (-1.0, 1.0):
        r = np.sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2])
        ok &= (p[2] >= mlo * r) & (p[2] <= mhi * r)
    return ok


@pytest.mark.parametrize("mus", [(-1.0, 1.0), (-0.8, 0.6), (0.6, 0.8), (-0.6, 1.0), (0.0, 0.8), (-1.0, -0.6)])
def test_momenta_on_the_edges_stay(mus):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("window edges", mus)
    p = _momenta()
    n = p.shape[1]
    ic = torch.as_tensor(np.concatenate([np.full((3, n), 0.25), p]), device="cuda")
    carry = torch.empty((aw.NCARRY, n), dtype=torch.float64, device="cuda")
    out = torch.empty((aw.NOUT, n), dtype=torch.float64, device="cuda")
    cls = torch.empty((n,), dtype=torch.uint8, device="cuda")
    wins = [(a, b) for i, a in enumerate(PHIS) for b in PHIS[i + 1::3]] + [(-math.pi, math.pi)]
    for w in wins:
        win = (*w, *mus)
        e = aw.Ensemble(eps=0.0, n_steps=3, ic_kind="explicit", n_orbits=n, tangent=False, window=win,
                        stay_in_window=True)
        want = ~_inside(p, win)
        left = (np_(aw.map_ensemble(e, ic).cls) >> 1) & 1
        np.testing.assert_array_equal(left.astype(bool), want, err_msg=str(win))
        for a, b in ((0, 1), (1, 3)):
            aw.map_ensemble_steps(e, carry, a, b, ic=ic, orbit_out=out, cls=cls)
        np.testing.assert_array_equal(((np_(cls) >> 1) & 1).astype(bool), want, err_msg=str(win))
