"""The histogram sorted in segments of 4096 items against numpy: items on both
sides of whole segments and of the 1024 segments scanned at a time, images of
1 to 1024 tiles and one tile past that (the sort over the whole range),
uniform, crowded (tiles of several chunks), ordered by tile (a segment's items
in one run) and all dropped.  Counts and drops are exact; a bin's sum of up to
n values below 1 in another order is within n * 2^-52 relative."""
import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu


def data(n, how):
    rng = np.random.default_rng(n)
    a, b = rng.uniform(-0.02, 1.02, n), rng.uniform(-0.02, 1.02, n)
    if how == "crowded":
        a[n // 7:], b[n // 7:] = 0.4 + 1e-3 * a[n // 7:], 0.6 + 1e-3 * b[n // 7:]
    if how == "ordered":
        a, b = np.sort(a), np.sort(b)
    if how == "dropped":
        a += 2.0
    a[0], b[1], a[2], b[3] = np.nan, np.inf, 1.0, 1.0
    return a, b, rng.uniform(0, 1, n)


@pytest.mark.parametrize("values", [True, False])
@pytest.mark.parametrize("n,W,H,how", [
    (65537, 32, 32, "uniform"), (69631, 33, 31, "crowded"), (69632, 512, 512, "ordered"), (69633, 512, 480, "uniform"),
    (100001, 1024, 1024, "uniform"), (100001, 1025, 1024, "uniform"), (200000, 1024, 1024, "ordered"),
    (300000, 250, 333, "crowded"), (300000, 90, 70, "dropped"), (4194304, 512, 512, "uniform"),
    (4194305, 200, 7, "crowded"), (4500003, 700, 600, "ordered")])
def test_counts_sums_and_drops(n, W, H, how, values):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("segments", n, W, H, how, values)
    a, b, v = data(n, how)
    dev = lambda x: torch.as_tensor(x, dtype=torch.float64, device="cuda")  # noqa: E731
    for closed in (False, True):
        counts, sums, dropped = aw.histogram2d(dev(a), dev(b), dev(v) if values else None, (0, 0), (1, 1), W, H,
                                               closed_upper=closed)
        with np.errstate(invalid="ignore"):
            fi, fj = np.floor(a * W), np.floor(b * H)
            if closed:
                fi[a == 1.0], fj[b == 1.0] = W - 1, H - 1
            ok = np.isfinite(a) & np.isfinite(b) & (fi >= 0) & (fi < W) & (fj >= 0) & (fj < H)
        at = fj[ok].astype(np.int64) * W + fi[ok].astype(np.int64)
        np.testing.assert_array_equal(np_(counts).reshape(-1), np.bincount(at, minlength=W * H))
        assert int(np_(dropped)[0]) == n - ok.sum()
        if values:
            np.testing.assert_allclose(np_(sums).reshape(-1), np.bincount(at, weights=v[ok], minlength=W * H),
                                       rtol=n * 2.0**-52, atol=0)
