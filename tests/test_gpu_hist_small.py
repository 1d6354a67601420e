"""The one-launch histogram of few items against numpy, on both sides of the
rule that chooses it (65536 items; items x tiles), with odd image sizes whose
last tiles are ragged, every item dropped, no item, crowded tiles, and the
accumulating window density.  Counts and drops are exact; a bin's sum of at
most 65600 values below 1 in another order is within 1e-11."""
import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu


@pytest.mark.parametrize("values", [True, False])
@pytest.mark.parametrize("n,W,H", [(0, 40, 33), (1, 1, 1), (1023, 32, 32), (8191, 33, 65), (8193, 900, 31), (65536, 512, 512),
                                   (65537, 512, 512), (65536, 513, 512), (20000, 1500, 1500), (60000, 7, 3)])
def test_counts_sums_and_drops(n, W, H, values):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("small histogram", n, W, H, values)
    rng = np.random.default_rng(n + W)
    a, b, v = rng.uniform(-0.1, 1.1, n), rng.uniform(-0.1, 1.1, n), rng.uniform(0, 1, n)
    if n > 100:
        a[: n // 3] = 0.31          # a crowded bin row
        a[-1], b[-2], a[-3], b[-4] = np.nan, np.inf, 1.0, 0.0
    dev = lambda x: torch.as_tensor(x, dtype=torch.float64, device="cuda")  # noqa: E731
    counts, sums, dropped = aw.histogram2d(dev(a), dev(b), dev(v) if values else None, (0, 0), (1, 1), W, H)
    with np.errstate(invalid="ignore"):
        fi, fj = np.floor(a * W), np.floor(b * H)
        ok = np.isfinite(a) & np.isfinite(b) & (fi >= 0) & (fi < W) & (fj >= 0) & (fj < H)
    at = fj[ok].astype(np.int64) * W + fi[ok].astype(np.int64)
    np.testing.assert_array_equal(np_(counts).reshape(-1), np.bincount(at, minlength=W * H))
    assert int(np_(dropped)[0]) == n - ok.sum()
    if values:
        np.testing.assert_allclose(np_(sums).reshape(-1), np.bincount(at, weights=v[ok], minlength=W * H), rtol=1e-11,
                                   atol=0)


def test_window_counts_add_up_and_match_the_sorted_path():
    """32000 orbits take the one-launch path, 70000 the sorted one: the first
    32000 orbits' counts must be the same in both, added to what was there."""
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("window counts, small and sorted")
    spec = aw.ImageSpec(kind="hist_vdir", W=96, H=70)
    got = {}
    for n, extra in ((32000, 0), (70000, 1)):
        e = aw.Ensemble(eps=1e-2, n_steps=40, ic_kind="sphere", n_orbits=n, energy=1.0, seed_ic=3, tangent=False)
        carry = torch.empty((aw.NCARRY, n), dtype=torch.float64, device="cuda")
        cnt = torch.full((70, 96), 5, dtype=torch.int32, device="cuda")
        aw.window_density(e, carry, 0, 2, 20, spec, cnt, tuning=aw.Tuning(lanes_per_orbit=1))
        got[n] = np_(cnt).astype(np.int64) - 5
        assert got[n].sum() == 2 * n
    rest = aw.Ensemble(eps=1e-2, n_steps=40, ic_kind="explicit", n_orbits=38000, tangent=False)
    full = aw.Ensemble(eps=1e-2, n_steps=40, ic_kind="sphere", n_orbits=70000, energy=1.0, seed_ic=3, tangent=False)
    ic = aw.generate_ic(full)[0][:, 32000:].contiguous()
    carry = torch.empty((aw.NCARRY, 38000), dtype=torch.float64, device="cuda")
    cnt = torch.zeros((70, 96), dtype=torch.int32, device="cuda")
    aw.window_density(rest, carry, 0, 2, 20, spec, cnt, ic=ic, tuning=aw.Tuning(lanes_per_orbit=1))
    np.testing.assert_array_equal(got[32000] + np_(cnt), got[70000])
