"""The sine and cosine function of the step loops as the kicks call it: two
angles at a time (two lanes per orbit), three (one lane, with and without the
tangent), against one at a time bit for bit -- whose replay by the table
generator is tested elsewhere -- and against the values in extended precision.

Arguments in nodes (pi/2048): random ones over the torus and up to 1e9, nodes
and midpoints and their neighbours, where the rounding decides the node, tiny
and signed zeros, the range's end at 2^51, and non-finite ones.  The error of a
sine is the rounding of its table entry and of its last sum, of a cosine those
and the first sum's, half an ulp of 1 (2^-54) each; the coefficients' errors
stay below 2e-18."""
import ctypes
import os

import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _device(x, angles, aligned):
    import torch
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_1107_4107_amd", "libaw_probe.so"))
    fn = lib.awp_sincos_nodes
    fn.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
    xd = torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    s, c = torch.full_like(xd, 7.0), torch.full_like(xd, 7.0)
    torch.cuda.synchronize()
    assert fn(xd.data_ptr(), s.data_ptr(), c.data_ptr(), xd.numel(), angles, aligned, None) == 0
    torch.cuda.synchronize()
    return np_(s), np_(c)


def _arguments():
    rng = np.random.default_rng(31)
    k = np.arange(-6000.0, 6000.0)
    mid = k + 0.5
    parts = [rng.uniform(-5e3, 5e3, 100_000), rng.uniform(-1e9, 1e9, 100_000), rng.uniform(-1.0, 1.0, 10_000),
             k, mid, np.nextafter(mid, np.inf), np.nextafter(mid, -np.inf),
             np.array([0.0, -0.0, 5e-324, -5e-324, 1e-300, 4096.0, -4096.0, 2.0 ** 50 + 1.25, -(2.0 ** 50) + 3,
                       2.0 ** 51 - 0.5, np.inf, -np.inf, np.nan, 1.0])]
    return np.concatenate(parts)


@pytest.mark.parametrize("angles,aligned", [(1, 0), (2, 1), (3, 1), (3, 0)])
def test_angles_of_a_kick(angles, aligned):
    need_gpu()
    print_case("node angles", angles, aligned)
    x = _arguments()
    s, c = _device(x, angles, aligned)
    s1, c1 = _device(x, 1, 0)
    np.testing.assert_array_equal(s.view(np.uint64), s1.view(np.uint64))
    np.testing.assert_array_equal(c.view(np.uint64), c1.view(np.uint64))
    fin = np.isfinite(x)
    assert np.all(np.isnan(s[~fin])) and np.all(np.isnan(c[~fin]))
    a = np.fmod(x[fin], 4096.0).astype(np.longdouble) * (np.longdouble("3.14159265358979323846264338327950288") / 2048)
    assert np.max(np.abs(s[fin] - np.sin(a))) <= 2 * 2.0 ** -54 + 2e-18
    assert np.max(np.abs(c[fin] - np.cos(a))) <= 3 * 2.0 ** -54 + 2e-18


@pytest.mark.parametrize("n", [1, 2, 3, 4, 255, 769])
def test_ragged_ends(n):
    need_gpu()
    print_case("node angles, ragged", n)
    x = np.linspace(-5000.0, 5000.0, n)
    s1, c1 = _device(x, 1, 0)
    for angles, aligned in ((2, 1), (3, 1), (3, 0)):
        s, c = _device(x, angles, aligned)
        assert np.array_equal(s, s1) and np.array_equal(c, c1)
