"""The adjoints keep the step states of as many trailing segments as the
caller's workspace holds and recompute the others: the same states either way,
so the results must be bitwise equal for every workspace size, and nothing may
be written past ws_bytes.  Intervals that do and do not divide the run, a
multiple of 4 and not; sizes from the smallest workspace to one with room for
every segment, with a few bytes to spare."""
import pytest

import numpy as np

from gpu_util import gpu, need_gpu, np_, print_case

pytestmark = gpu


@pytest.mark.parametrize("ftle", [False, True])
@pytest.mark.parametrize("T,ck", [(120, 20), (131, 37), (90, 50), (64, 64), (53, 7)])
def test_results_do_not_depend_on_the_workspace(ftle, T, ck):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("adjoint workspace", ftle, T, ck)
    n, rows = 193, 12 if ftle else 6
    g = torch.Generator(device="cuda").manual_seed(5)
    ic = 6.0 * torch.rand((6, n), dtype=torch.float64, device="cuda", generator=g)
    e = aw.Ensemble(eps=1e-2, n_steps=T, ic_kind="explicit", n_orbits=n, tangent=ftle)
    call, size = ((aw.ftle_grad, aw.ftle_grad_workspace_bytes) if ftle else
                  (aw.indicator_grad, aw.grad_workspace_bytes))
    need = size(e, ck)
    n_seg = -(-T // ck)
    seg = need - (2 * n * (T // 8) if ftle else 0) - 8 * rows * n * (n_seg + 1)
    ref = [np_(t) for t in call(e, ic, ckpt_every=ck)]      # allocates room for every segment
    for extra in sorted({0, seg - 1, seg, 2 * seg + 5, (n_seg - 1) * seg, n_seg * seg + 11}):
        buf = torch.full((need + extra + 4096,), 171, dtype=torch.uint8, device="cuda")
        got = call(e, ic, ckpt_every=ck, workspace=buf[:need + extra])
        for a, b in zip(got, ref):
            np.testing.assert_array_equal(np_(a), b, err_msg=f"{extra} bytes more than needed")
        assert bool((buf[need + extra:] == 171).all()), "written past the workspace"
