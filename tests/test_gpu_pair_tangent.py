"""Two lanes per orbit against one: every output, state, class, image, carry and
window count must be the same bit for bit, at the edges of the 32-orbit tiles,
for every form, with and without the tangent, in one launch and in chunks that
pass a carry from one way to the other."""
import pytest

from gpu_util import gpu, need_gpu, print_case

pytestmark = gpu


def ens(aw, n, form, tan, steps=37):
    return aw.Ensemble(eps=2e-2, n_steps=steps, ic_kind="sphere", n_orbits=n, energy=1.0, seed_ic=5, tangent=tan,
                       map_form=form)


def same(torch, *pairs):
    for a, b in pairs:
        assert torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)) and torch.equal(torch.isnan(a), torch.isnan(b))


@pytest.mark.parametrize("form,tan", [("s6", True), ("s6", False), ("y6", True), ("s4", False), ("s2", True),
                                      ("stdmap", True), ("stdmap", False)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 4099])
def test_outputs_and_chunks(n, form, tan):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("pair lanes", n, form, tan)
    e = ens(aw, n, form, tan)
    one, two = (aw.Tuning(lanes_per_orbit=k, renorm_every=4) for k in (1, 2))
    a, b = (aw.map_ensemble(e, want_state=True, tuning=t) for t in (one, two))
    same(torch, (a.orbit_out, b.orbit_out), (a.state, b.state), (a.cls, b.cls))
    new = lambda rows: torch.zeros((rows, n), dtype=torch.float64, device="cuda")  # noqa: E731
    carries = []
    for ways in ((one, one, one), (two, one, two), (one, two, one), (two, two, two)):
        carry, out, state = new(aw.NCARRY), new(aw.NOUT), new(12)
        seen = []
        for (k0, k1), t in zip(((0, 5), (5, 24), (24, 37)), ways):
            last = dict(orbit_out=out, state=state) if k1 == 37 else {}
            aw.map_ensemble_steps(e, carry, k0, k1, tuning=t, **last)
            seen.append(carry.clone())
        same(torch, (out, a.orbit_out), (state, a.state))
        carries.append(seen[:2])
    for c in carries[1:]:
        same(torch, *zip(c, carries[0]))


@pytest.mark.parametrize("n", [65, 1000])
def test_images_and_windows(n):
    need_gpu()
    import torch
    import paper_1107_4107_amd as aw
    print_case("pair lanes images", n)
    one, two = (aw.Tuning(lanes_per_orbit=k) for k in (1, 2))
    grid = aw.Ensemble(eps=1e-2, n_steps=60, ic_kind="grid2", nx=33, ny=n // 33 + 1, tangent=True)
    for e, spec in ((grid, aw.ImageSpec(kind="ic_grid", field=2, W=33, H=n // 33 + 1)),
                    (ens(aw, n, "s6", True), aw.ImageSpec(kind="hist_vdir", W=40, H=30))):
        a, b = (aw.indicator_image(e, spec, tuning=t) for t in (one, two))
        same(torch, *((x, y) for x, y in zip(a, b) if isinstance(x, torch.Tensor)))
