"""The propagation kernels' scaled units: angles in table nodes (pi/2048), the
z components of momentum and tangent times sqrt 2.

The node-unit sine and cosine must reproduce their replay by the table
generator bit for bit; their error is three roundings of at most half an ulp
of 1 (table entry, c1, result), 1.67e-16, plus the reference's own rounding.
A carry written in radians (without the units flag) is taken over: its
conversion perturbs the state by an ulp, which 200 further steps at
eps = 1e-2 amplify by at most exp(2 sqrt(eps) 200 h) = 13, with the
propagation's own rounding well inside 1e-10."""
import ctypes
import importlib.util
import os

import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _probe(x):
    import torch
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_1107_4107_amd", "libaw_probe.so"))
    lib.awp_sincos_node.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p]
    xd = torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")
    s, c = torch.empty_like(xd), torch.empty_like(xd)
    torch.cuda.synchronize()
    assert lib.awp_sincos_node(xd.data_ptr(), s.data_ptr(), c.data_ptr(), xd.numel(), None) == 0
    torch.cuda.synchronize()
    return np_(s), np_(c)


def _gen():
    path = os.path.join(ROOT, "paper_1107_4107_amd", "csrc", "gen_sincos_tab.py")
    spec = importlib.util.spec_from_file_location("gen_sincos_tab", path)
    g = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(g)
    return g


def test_node_sincos_matches_its_model_and_mpmath():
    need_gpu()
    print_case("node sincos")
    import mpmath as mp
    rng = np.random.default_rng(21)
    k = np.arange(-9000, 9000, 3).astype(np.float64)
    x = np.concatenate([rng.uniform(-5e3, 5e3, 4000), rng.uniform(-1e9, 1e9, 1000), k, k + 0.5,
                        np.nextafter(k + 0.5, np.inf), np.nextafter(k + 0.5, -np.inf),
                        [0.0, -0.0, 5e-324, 4096.0, 2.0 ** 50, -(2.0 ** 50) + 3]])
    s, c = _probe(x)
    g = _gen()
    tab = g.constants()[0]
    w, t, _, _, _ = g.node_constants()
    pick = np.concatenate([rng.choice(x.size, 1500, replace=False), np.arange(x.size - 6, x.size)])
    for i in pick:
        ms, mc = g.device_sincos_node(float(x[i]), tab, w, t)
        assert s[i] == ms and c[i] == mc, (x[i], s[i], ms, c[i], mc)
        a = mp.mpf(float(x[i])) * mp.pi / 2048
        assert abs(s[i] - float(mp.sin(a))) <= 2.3e-16 and abs(c[i] - float(mp.cos(a))) <= 2.3e-16
    s, c = _probe(np.array([np.inf, -np.inf, np.nan, 0.0]))
    assert np.all(np.isnan(s[:3])) and np.all(np.isnan(c[:3])) and s[3] == 0.0 and c[3] == 1.0


@pytest.mark.parametrize("tangent,lanes", [(True, 0), (False, 1), (False, 2)])
def test_carry_in_radians_is_taken_over(tangent, lanes):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("carry in radians", tangent, lanes)
    e = aw.Ensemble(eps=1e-2, n_steps=300, nx=21, ny=17, base=(0.1, 0.2, 0.3, 0, 0, 0.7), tangent=tangent)
    N = e.size
    t = aw.Tuning(lanes_per_orbit=lanes)
    ref = aw.map_ensemble(e, want_state=True)
    carry = torch.empty((aw.NCARRY, N), dtype=torch.float64, device="cuda")
    aw.map_ensemble_steps(e, carry, 0, 100, tuning=t)
    assert np.all(np_(carry)[21] == 2.0)
    step = np.pi / 2048
    carry[0:2] *= step
    carry[2] *= 0.5 * step
    for row in (5, 8, 11, 17):
        carry[row] *= np.sqrt(0.5)
    carry[21] = 0.0
    out = torch.empty((aw.NOUT, N), dtype=torch.float64, device="cuda")
    st = torch.empty((12, N), dtype=torch.float64, device="cuda")
    aw.map_ensemble_steps(e, carry, 100, 200, tuning=t)
    assert np.all(np_(carry)[21] == 2.0)
    aw.map_ensemble_steps(e, carry, 200, 300, orbit_out=out, state=st, tuning=t)
    rows = slice(0, 9) if tangent else slice(3, 9)
    np.testing.assert_allclose(np_(out)[rows], np_(ref.orbit_out)[rows], rtol=1e-9, atol=1e-10)
    np.testing.assert_allclose(np_(st), np_(ref.state), rtol=1e-9, atol=1e-10)
