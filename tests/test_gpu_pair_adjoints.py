"""The adjoints with two lanes per orbit against one: indicators and gradients
must be the same bit for bit, at the edges of a wave's 32 pairs and of a block,
for every form, at eps = 0 too, for the stored and the store-free sweep, with
segments kept and recomputed."""
import numpy as np
import pytest

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu


@pytest.mark.parametrize("form,eps", [("s6", 2e-2), ("s6", 0.0), ("y6", 2e-2), ("s4", 1e-2), ("s2", 1e-2), ("stdmap", 2e-2),
                                      ("stdmap", 0.0)])
@pytest.mark.parametrize("n", [1, 31, 33, 130, 1025])
def test_same_bits(n, form, eps):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("pair adjoints", n, form, eps)
    rng = np.random.default_rng(n)
    ic = torch.as_tensor(rng.uniform(0, 6, (6, n)), device="cuda")
    up = torch.as_tensor(rng.normal(size=n), device="cuda")
    one, two = (aw.Tuning(lanes_per_orbit=k) for k in (1, 2))
    for tan, grad, need in ((False, aw.indicator_grad, aw.grad_workspace_bytes),
                            (True, aw.ftle_grad, aw.ftle_grad_workspace_bytes)):
        e = aw.Ensemble(eps=eps, n_steps=45, ic_kind="explicit", n_orbits=n, tangent=tan, map_form=form)
        for rev in (False, True):
            bare = torch.empty(need(e, 12, rev), dtype=torch.uint8, device="cuda")  # nothing kept: recomputed
            for ws in (None, bare):
                a, b = (grad(e, ic, **{"grad_L" if tan else "grad_J": up}, ckpt_every=12, tuning=t, workspace=ws,
                             reversible=rev) for t in (one, two))
                for x, y in zip(a, b):
                    np.testing.assert_array_equal(np_(x), np_(y))
