"""The performance cases of the ensemble mapper: what a user's program calls,
with the sizes of this repository's own workloads and horizons short enough
that two correct binary64 evaluations of the same orbits still agree.

Every call goes through the package's public entry points.  The horizon of a
case is bounded by its eps: at the hyperbolic fixed point X = P = 0 of eq. 2
a deviation grows like exp(2 sqrt(eps) t), and 2 sqrt(eps) T h is kept below
about 12.  The per-step cost does not depend on the horizon, so the cases
stand for the long runs too.

exact() evaluates the same orbits in plain torch (binary64): the map stage by
stage in the printed (x, y, z) frame, gradients by torch's own autograd.
"""
import math

import numpy as np
import torch

import paper_1107_4107_amd as aw

TWO_PI = 2.0 * math.pi
H = aw.H_PAPER


# ---------------------------------------------------------------------------
# The cases.
# ---------------------------------------------------------------------------
def listed():
    return [
        # A few explicit orbits and their final states, as a script that follows
        # single orbits calls it: launch, table fill and latency.
        dict(name="orbits_257", call="map", n=257, steps=200, eps=1e-2, form="s6", tangent=True, state=True),
        # The 64 x 64 indicator image over 1000 steps: fewer waves than the chip has SIMDs.
        dict(name="chi_image_64", call="image", nx=64, ny=64, steps=900, eps=1e-2, form="s6", tangent=True, cls=False),
        # The large slice: the indicator image and the class map.
        dict(name="chi_image_1024", call="image", nx=1024, ny=1024, steps=1000, eps=1e-3, form="s6", tangent=True,
             cls=True),
        # Uniform orbits of the torus and momentum box, momentum drift averaged on a 512 x 512 image.
        dict(name="box_drift_image", call="box", n=1_000_003, steps=400, eps=5e-3, form="s6", tangent=True, W=512,
             H=512),
        # The density of the direction of V on the whole momentum sphere, state
        # only, at the effective perturbation 2 eps/E = 0.005 of the weak regime.
        dict(name="sphere_density", call="sphere", n=2_000_000, steps=200, eps=5e-2, energy=20.0, form="s6",
             stay=False, W=1024, H=512),
        # The zoomed density with the remained-within-the-area test at every step.
        dict(name="zoom_stay", call="sphere", n=500_001, steps=300, eps=5e-2, energy=0.75, form="s6", stay=True,
             W=256, H=256),
        # The injected cloud: direction counts over consecutive windows, state carried, 3.2e4 orbits.
        dict(name="cloud_windows", call="window", n=32_000, windows=3, steps=200, eps=2e-2, energy=15.0, form="s6",
             W=512, H=512),
        # A long run cut into chunks with the state carried in memory, 7-stage composition.
        dict(name="chunked_run", call="steps", n=300_007, chunks=4, steps=100, eps=5e-3, form="y6", tangent=True),
        # An eps sweep over slices of different size and horizon in one persistent launch.
        dict(name="eps_sweep_batch", call="batch", n_ens=16, side=256, steps=900, form="s6", tangent=True),
        # The gradient of the mean momentum drift through autograd: forward, then the checkpointed adjoint.
        dict(name="grad_drift", call="grad_j", n=262_144, steps=400, ckpt=100, eps=1e-2, form="s6", reversible=False),
        # The gradient of the finite-time Lyapunov growth, second-order adjoint.
        dict(name="grad_ftle", call="grad_l", n=32_761, steps=300, ckpt=100, eps=1e-2, form="s6", reversible=False),
        # The histogram reduction on a caller's keys and values.
        dict(name="histogram_3e6", call="hist", n=3_000_001, W=512, H=512, values=True, crowded=False),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _ilog(rng, lo, hi):
    return max(lo, min(hi, int(round(_log(rng, lo, hi)))))


def _horizon(rng, eps, lo=20, hi=1000, work=None):
    """Steps, log-spread, within the horizon eps allows and, for n orbits, within `work` orbit steps."""
    top = min(hi, int(95.0 / math.sqrt(eps)))
    if work is not None:
        top = min(top, int(work))
    return _ilog(rng, min(lo, max(2, top)), max(2, top))


def draw(rng):
    """A case of the same ranges: every call, tiny to large and odd sizes, all map forms and options."""
    call = rng.choice(["map", "map", "image", "image", "box", "sphere", "sphere", "window", "steps", "batch", "grad_j",
                       "grad_l", "hist", "hist"])
    form = rng.choice(["s6", "s6", "s6", "y6", "s4", "s2", "stdmap"])
    eps = _log(rng, 1e-4, 5e-2)
    if call == "map":
        n = _ilog(rng, 1, 300_000)
        return dict(call=call, n=n, steps=_horizon(rng, eps, work=2e8 / n), eps=eps, form=form,
                    tangent=rng.random() < 0.7, state=rng.random() < 0.5)
    if call == "image":
        nx, ny = _ilog(rng, 16, 1024), _ilog(rng, 16, 1024)
        return dict(call=call, nx=nx, ny=ny, steps=_horizon(rng, eps, work=1e9 / (nx * ny)), eps=eps, form=form,
                    tangent=True, cls=rng.random() < 0.5)
    if call == "box":
        n = _ilog(rng, 3_000, 2_000_000)
        return dict(call=call, n=n, steps=_horizon(rng, eps, work=5e8 / n), eps=eps, form=form,
                    tangent=rng.random() < 0.7, W=_ilog(rng, 32, 700), H=_ilog(rng, 32, 700))
    if call == "sphere":
        n = _ilog(rng, 3_000, 3_000_000)
        eps = _log(rng, 1e-2, 1e-1)
        stay = rng.random() < 0.4
        energy = eps * (_log(rng, 12.0, 30.0) if stay else _log(rng, 15.0, 400.0))
        return dict(call=call, n=n, steps=_horizon(rng, eps, hi=300, work=4e8 / n), eps=eps, energy=energy, form=form,
                    stay=stay, W=_ilog(rng, 64, 1024), H=_ilog(rng, 64, 512))
    if call == "window":
        n = _ilog(rng, 1_000, 100_000)
        eps = _log(rng, 1e-2, 5e-2)
        windows = rng.randint(1, 4)
        return dict(call=call, n=n, windows=windows, steps=max(10, int(95.0 / math.sqrt(eps)) // (windows + 1)),
                    eps=eps, energy=rng.uniform(5.0, 30.0), form=form, W=_ilog(rng, 64, 512), H=_ilog(rng, 64, 512))
    if call == "steps":
        n = _ilog(rng, 500, 500_000)
        chunks = rng.randint(2, 5)
        total = _horizon(rng, eps, lo=100, hi=800, work=3e8 / n)
        return dict(call=call, n=n, chunks=chunks, steps=max(1, total // chunks), eps=eps, form=form,
                    tangent=rng.random() < 0.6)
    if call == "batch":
        return dict(call=call, n_ens=rng.randint(2, 24), side=_ilog(rng, 32, 300), steps=_ilog(rng, 50, 900),
                    form=form, tangent=True)
    if call in ("grad_j", "grad_l"):
        eps = _log(rng, 1e-3, 3e-2)
        n = _ilog(rng, 64, 200_000 if call == "grad_j" else 80_000)
        return dict(call=call, n=n, steps=_horizon(rng, eps, lo=40, hi=400, work=1e8 / n), ckpt=rng.choice([20, 50, 100, 1000]),
                    eps=eps, form=form, reversible=rng.random() < 0.4)
    return dict(call="hist", n=_ilog(rng, 1_000, 8_000_000), W=_ilog(rng, 16, 900), H=_ilog(rng, 16, 900),
                values=rng.random() < 0.7, crowded=rng.random() < 0.3)


# ---------------------------------------------------------------------------
# What a user's program holds before the call.
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand(g, n, lo, hi):
    return lo + (hi - lo) * torch.rand((n,), dtype=torch.float64, device="cuda", generator=g)


def _explicit(case, g, tangent, seed):
    """Random orbits of the torus with momenta of the box, [6, N]."""
    n = case["n"]
    ic = torch.stack([_rand(g, n, 0.0, TWO_PI) for _ in range(6)])
    e = aw.Ensemble(eps=case["eps"], n_steps=case["steps"], map_form=case["form"], ic_kind="explicit", n_orbits=n,
                    seed_tangent=seed, tangent=tangent)
    return e, ic


def _slice(eps, nx, ny, steps, form, seed, tangent=True):
    """The (px, py) slice over [0, 2 pi)^2 at an x, y, z and p_z of the seed's own."""
    r = np.random.default_rng(seed)
    base = tuple(float(v) for v in (r.uniform(0, 0.5), r.uniform(0, 0.5), r.uniform(0, 0.5), 0, 0, r.uniform(0, 1)))
    return aw.Ensemble(eps=eps, n_steps=steps, map_form=form, nx=nx, ny=ny, base=base, seed_tangent=seed,
                       tangent=tangent)


def _batch(case, seed):
    """Slices with eps log-spread over 1e-4..1e-2 and sizes and horizons drawn as in the sweep workload."""
    r = np.random.default_rng(case["n_ens"])
    k = case["n_ens"]
    sides = r.choice([max(8, case["side"] // 4), max(8, case["side"] // 2), case["side"]], k)
    steps = r.choice([max(1, case["steps"] // 10), max(1, case["steps"] // 3), case["steps"]], k)
    return [_slice(10.0 ** (-4.0 + 2.0 * i / (k - 1)), int(sides[i]), int(sides[i]), int(steps[i]), case["form"],
                   seed + i, case["tangent"]) for i in range(k)]


def _zoom(stay):
    return (0.55, 1.05, -0.25, 0.25) if stay else (-math.pi, math.pi, -1.0, 1.0)


def prepare(case, seed):
    call = case["call"]
    g = _gen(seed)
    if call == "map":
        e, ic = _explicit(case, g, case["tangent"], seed)
        return dict(call=call, e=e, ic=ic, state=case["state"])
    if call == "image":
        e = _slice(case["eps"], case["nx"], case["ny"], case["steps"], case["form"], seed, case["tangent"])
        return dict(call=call, e=e, spec=aw.ImageSpec(kind="ic_grid", field=aw.OUT_CHI, W=case["nx"], H=case["ny"]),
                    cls=case["cls"])
    if call == "box":
        e = aw.Ensemble(eps=case["eps"], n_steps=case["steps"], map_form=case["form"], ic_kind="box",
                        n_orbits=case["n"], seed_ic=seed, tangent=case["tangent"])
        return dict(call="image", e=e, cls=False,
                    spec=aw.ImageSpec(kind="hist_p0", field=aw.OUT_DP2, W=case["W"], H=case["H"]))
    if call == "sphere":
        w = _zoom(case["stay"])
        e = aw.Ensemble(eps=case["eps"], n_steps=case["steps"], map_form=case["form"], ic_kind="sphere",
                        n_orbits=case["n"], energy=case["energy"], window=w, seed_ic=seed, tangent=False,
                        stay_in_window=case["stay"])
        spec = aw.ImageSpec(kind="hist_vdir", W=case["W"], H=case["H"],
                            lo=(w[0], w[2]) if case["stay"] else None, hi=(w[1], w[3]) if case["stay"] else None)
        return dict(call="image", e=e, spec=spec, cls=case["stay"])
    if call == "window":
        c = math.sqrt(case["energy"])
        e = aw.Ensemble(eps=case["eps"], n_steps=case["windows"] * case["steps"], map_form=case["form"],
                        ic_kind="cloud", n_orbits=case["n"], energy=case["energy"], cloud=(c, c, 0.01, 0.01),
                        seed_ic=seed, tangent=False)
        a = math.pi / 4
        spec = aw.ImageSpec(kind="hist_vdir", W=case["W"], H=case["H"], lo=(a - 0.5, -0.5), hi=(a + 0.5, 0.5))
        return dict(call=call, e=e, spec=spec, windows=case["windows"], steps=case["steps"],
                    carry=torch.empty((aw.NCARRY, case["n"]), dtype=torch.float64, device="cuda"),
                    counts=torch.zeros((case["H"], case["W"]), dtype=torch.int32, device="cuda"))
    if call == "steps":
        n = case["n"]
        e = aw.Ensemble(eps=case["eps"], n_steps=case["chunks"] * case["steps"], map_form=case["form"],
                        ic_kind="box", n_orbits=n, seed_ic=seed, tangent=case["tangent"])
        return dict(call=call, e=e, steps=case["steps"],
                    carry=torch.empty((aw.NCARRY, n), dtype=torch.float64, device="cuda"),
                    out=torch.empty((aw.NOUT, n), dtype=torch.float64, device="cuda"),
                    cls=torch.empty((n,), dtype=torch.uint8, device="cuda"))
    if call == "batch":
        return dict(call=call, ens=_batch(case, seed), spec=aw.ImageSpec(kind="ic_grid", field=aw.OUT_CHI, W=0, H=0))
    if call in ("grad_j", "grad_l"):
        e, ic = _explicit(case, g, call == "grad_l", seed)
        up = _rand(g, case["n"], 0.5, 1.5)
        s = dict(call=call, e=e, up=up, ckpt=case["ckpt"], reversible=case["reversible"], form=case["form"])
        if call == "grad_j":
            s["ic"] = ic.t().contiguous().requires_grad_()
            s["eps"] = torch.tensor(case["eps"], dtype=torch.float64, requires_grad=True)
        else:
            s["ic"] = ic
            s["work"] = torch.empty((aw.ftle_grad_workspace_bytes(e, case["ckpt"], case["reversible"]),),
                                    dtype=torch.uint8, device="cuda")
        return s
    n = case["n"]
    if case["crowded"]:   # a momentum cloud, as the injected cloud's image
        a = 0.5 + 0.02 * torch.randn((n,), dtype=torch.float64, device="cuda", generator=g)
        b = 0.5 + 0.02 * torch.randn((n,), dtype=torch.float64, device="cuda", generator=g)
    else:
        a, b = _rand(g, n, -0.01, 1.01), _rand(g, n, -0.01, 1.01)
    v = _rand(g, n, 0.0, 1.0) if case["values"] else None
    return dict(call="hist", a=a, b=b, v=v, W=case["W"], H=case["H"])


def run(s):
    call = s["call"]
    if call == "map":
        r = aw.map_ensemble(s["e"], s["ic"], want_state=s["state"])
        return dict(out=r.orbit_out, state=r.state, cls=r.cls)
    if call == "image":
        img, cnt, cls = aw.indicator_image(s["e"], s["spec"], want_class=s["cls"])
        return dict(img=img, cnt=cnt, cls=cls)
    if call == "window":
        s["counts"].zero_()
        aw.window_density(s["e"], s["carry"], 0, s["windows"], s["steps"], s["spec"], s["counts"])
        return dict(counts=s["counts"])
    if call == "steps":
        T = s["e"].n_steps
        for k in range(0, T, s["steps"]):
            aw.map_ensemble_steps(s["e"], s["carry"], k, k + s["steps"], orbit_out=s["out"], cls=s["cls"])
        return dict(out=s["out"], cls=s["cls"])
    if call == "batch":
        imgs, cnts, _ = aw.indicator_images(s["ens"], s["spec"])
        return dict(img=imgs, cnt=cnts)
    if call == "grad_j":
        J = aw.IndicatorJ.apply(s["ic"], s["eps"], s["e"].n_steps, H, s["form"], s["ckpt"], s["reversible"])
        gic, geps = torch.autograd.grad(J, (s["ic"], s["eps"]), s["up"])
        return dict(J=J.detach(), gic=gic, geps=geps)
    if call == "grad_l":
        L, gic, geps = aw.ftle_grad(s["e"], s["ic"], grad_L=s["up"], ckpt_every=s["ckpt"], workspace=s["work"],
                                    reversible=s["reversible"])
        return dict(L=L, gic=gic, geps=geps)
    counts, sums, dropped = aw.histogram2d(s["a"], s["b"], s["v"], (0.0, 0.0), (1.0, 1.0), s["W"], s["H"])
    return dict(counts=counts, sums=sums, dropped=dropped)


# ---------------------------------------------------------------------------
# The work a pass cannot do without.
# ---------------------------------------------------------------------------
KICKS = {"s6": 9, "y6": 7, "s4": 3, "s2": 1, "stdmap": 1}


def _step_flops(form, tangent):
    """Floating-point operations of one map step: per kick three sine/cosine
    pairs (21 each), the force (9) and with the tangent the Hessian product
    (22); a drift takes 6 or 12; 10 for the drift indicator."""
    k = KICKS[form]
    return k * (72 + (22 if tangent else 0)) + (k + (form != "stdmap")) * (12 if tangent else 6) + 10


def work(case):
    call = case["call"]
    if call == "hist":
        n, bins = case["n"], case["W"] * case["H"]
        return {"bytes": n * (24 if case["values"] else 16) + bins * (12 if case["values"] else 4), "flops": 6 * n}
    if call == "batch":
        ens = _batch(case, 0)
        return {"bytes": sum(8 * e.nx * e.ny for e in ens),
                "flops": sum(e.nx * e.ny * e.n_steps * _step_flops(case["form"], case["tangent"]) for e in ens)}
    if call == "image":
        n = case["nx"] * case["ny"]
        return {"bytes": n * (9 if case["cls"] else 8), "flops": n * case["steps"] * _step_flops(case["form"], case["tangent"])}
    n = case["n"]
    if call == "map":
        return {"bytes": n * (48 + 73 + (96 if case["state"] else 0)),
                "flops": n * case["steps"] * _step_flops(case["form"], case["tangent"])}
    if call in ("box", "sphere"):
        return {"bytes": 12 * case["W"] * case["H"],
                "flops": n * case["steps"] * _step_flops(case["form"], call == "box" and case["tangent"])}
    if call == "window":
        return {"bytes": 4 * case["W"] * case["H"] + 8 * aw.NCARRY * n,
                "flops": n * case["windows"] * case["steps"] * _step_flops(case["form"], False)}
    if call == "steps":
        return {"bytes": n * (73 + 2 * 8 * aw.NCARRY * (case["chunks"] - 1)),
                "flops": n * case["chunks"] * case["steps"] * _step_flops(case["form"], case["tangent"])}
    # a forward pass for the value, and a reverse pass of about its cost and a half
    fwd = n * case["steps"] * _step_flops(case["form"], call == "grad_l")
    return {"bytes": n * 8 * (6 + 1 + 1 + 7), "flops": int(2.5 * fwd)}


# ---------------------------------------------------------------------------
# exact(): the same values in plain torch, binary64.
# ---------------------------------------------------------------------------
def _signed(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _shr(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _u01(seed, c):
    """SplitMix64 output number c of the stream seeded with `seed`, as a uniform of [0, 1)."""
    z = (c + 1) * _signed(0x9E3779B97F4A7C15) + _signed(seed)
    z = (z ^ _shr(z, 30)) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _signed(0x94D049BB133111EB)
    z = z ^ _shr(z, 31)
    return _shr(z, 11).to(torch.float64) * 2.0 ** -53


def _index(n, step):
    return torch.arange(n, dtype=torch.int64, device="cuda") * step


def _w0(seed, n):
    u = torch.stack([2.0 * _u01(seed, _index(n, 16) + k) - 1.0 for k in range(6)])
    return u / u.square().sum(0).sqrt()


def _hp(X):
    return torch.cos(X[0]) * torch.cos(X[1]) * (1.0 + torch.cos(2.0 * X[2]))


def _start(case, seed, e=None):
    """Initial states [6, N] of a case's ensemble (of one slice e of a batch)."""
    call = case["call"]
    if call in ("image", "batch"):
        i = _index(e.nx * e.ny, 1)
        cols = [torch.full((e.nx * e.ny,), v, dtype=torch.float64, device="cuda") for v in e.base]
        cols[3] = (i % e.nx).to(torch.float64) * (TWO_PI / e.nx)
        cols[4] = (i // e.nx).to(torch.float64) * (TWO_PI / e.ny)
        return torch.stack(cols)
    n = case["n"]
    if call in ("box", "steps"):
        return torch.stack([TWO_PI * _u01(seed, _index(n, 16) + k) for k in range(6)])
    if call == "sphere":
        w = _zoom(case["stay"])
        c = _index(n, 16)
        X = torch.stack([TWO_PI * _u01(seed, c + k) for k in range(3)])
        mu = w[2] + (w[3] - w[2]) * _u01(seed, c + 3)
        phi = w[0] + (w[1] - w[0]) * _u01(seed, c + 4)
        p = torch.sqrt(2.0 * (case["energy"] - case["eps"] * _hp(X)))
        st = torch.sqrt(1.0 - mu * mu)
        return torch.cat([X, torch.stack([p * st * torch.cos(phi), p * st * torch.sin(phi), p * mu])])
    raise ValueError(call)


def _weights(form):
    """Kick weights of a form (fractions of h) and the drifts between them."""
    g1 = 1.0 / (2.0 - 2.0 ** (1.0 / 3.0))
    d1 = 1.0 / (2.0 - 2.0 ** (1.0 / 5.0))
    s4 = [g1, 1.0 - 2.0 * g1, g1]
    if form == "stdmap":
        return [1.0], None
    if form == "s2":
        k = [1.0]
    elif form == "s4":
        k = s4
    elif form == "s6":
        k = [d * g for d in (d1, 1.0 - 2.0 * d1, d1) for g in s4]
    else:   # the real solution of the 7-stage order conditions with the smallest stages
        w = np.array([0.784513610477560, 0.235573213359357, -1.17767998417887])
        for _ in range(4):   # Newton's method on the order conditions
            jac = np.empty((3, 3))
            for q in range(3):
                d = np.zeros(3)
                d[q] = 1e-7
                jac[:, q] = (_order(w + d) - _order(w - d)) / 2e-7
            w = w - np.linalg.solve(jac, _order(w))
        k = [w[0], w[1], w[2], 1.0 - 2.0 * w.sum(), w[2], w[1], w[0]]
    return k, [0.5 * k[0]] + [0.5 * (a + b) for a, b in zip(k[:-1], k[1:])] + [0.5 * k[-1]]


def _order(w):
    """The conditions b = c = d = 0 of a symmetric composition w3 w2 w1 w0 w1 w2 w3 of order 6 (w = w3, w2, w1)."""
    w0 = 1.0 - 2.0 * w.sum()
    a, b, c, d = w0, w0 ** 3, w0 ** 5, 0.0
    for v in (w[2], w[1], w[0]):
        d += (a * v ** 3 - b * v) * (a + v) / 6.0
        a, b, c = a + 2 * v, b + 2 * v ** 3, c + 2 * v ** 5
    return np.array([b, c, d])


def _step(X, P, eps, k, dr, D=None, DP=None):
    """One map step of state (and tangent), in (x, y, z)."""
    def drift(t):
        nonlocal X, D
        X = X + (t * H) * P
        if D is not None:
            D = D + (t * H) * DP

    def kick(t):
        nonlocal P, DP
        S, C = torch.sin(X), torch.cos(X)
        a = 2.0 * t * H * eps
        c2 = C[2] * C[2]
        cs = C[2] * S[2]
        if D is not None:
            xy = C[0] * C[1]
            hxx = a * xy * c2
            hxy = -a * S[0] * S[1] * c2
            hxz = -2.0 * a * S[0] * C[1] * cs
            hyz = -2.0 * a * C[0] * S[1] * cs
            hzz = 2.0 * a * xy * (c2 - S[2] * S[2])
            DP = DP + torch.stack([hxx * D[0] + hxy * D[1] + hxz * D[2], hxy * D[0] + hxx * D[1] + hyz * D[2],
                                   hxz * D[0] + hyz * D[1] + hzz * D[2]])
        P = P + torch.stack([a * S[0] * C[1] * c2, a * C[0] * S[1] * c2, 2.0 * a * C[0] * C[1] * cs])

    if dr is None:
        kick(k[0])
        drift(1.0)
    else:
        for t, w in zip(dr, k):
            drift(t)
            kick(w)
        drift(dr[-1])
    return X, P, D, DP


def _propagate(s0, eps, T, form, tangent_seed=None, window=None):
    """Outputs [9, N] and final state [12 or 6, N] of the orbits, and those that left the window."""
    k, dr = _weights(form)
    X, P = s0[:3], s0[3:]
    n = s0.shape[1]
    D = DP = None
    growth = torch.zeros((n,), dtype=torch.float64, device="cuda")
    if tangent_seed is not None:
        w = _w0(tangent_seed, n)
        D, DP = w[:3], w[3:]
    drift2 = torch.zeros((n,), dtype=torch.float64, device="cuda")
    left = _outside(P, window) if window else torch.zeros((n,), dtype=torch.bool, device="cuda")
    for i in range(T):
        X, P, D, DP = _step(X, P, eps, k, dr, D, DP)
        drift2 = drift2 + (P - s0[3:]).square().sum(0)
        if window:
            left = left | _outside(P, window)
        if D is not None and (i % 50 == 49 or i == T - 1):
            norm = (D.square().sum(0) + DP.square().sum(0)).sqrt()
            growth = growth + norm.log()
            D, DP = D / norm, DP / norm
    th = T * H
    V = (X - s0[:3]) / th
    nan = torch.full((n,), math.nan, dtype=torch.float64, device="cuda")
    L = growth if D is not None else nan
    E = [0.5 * (p * p).sum(0) + eps * _hp(x) for x, p in ((X, P), (s0[:3], s0[3:]))]
    out = torch.stack([L, L / th, L / math.log(1.0 + th), V[0], V[1], V[2], (P - s0[3:]).square().sum(0), drift2 / T,
                       E[0] - E[1]])
    return out, torch.cat([X, P] + ([D, DP] if D is not None else [])), left


def _outside(P, w):
    phi, mu = torch.atan2(P[1], P[0]), P[2] / P.square().sum(0).sqrt()
    return (phi < w[0]) | (phi > w[1]) | (mu < w[2]) | (mu > w[3])


def _hist(a, b, v, lo, hi, W, Hh, closed, keep=None):
    """Counts and sums [H, W] of the keys, bin by floor((key - lo)/(hi - lo) * W)."""
    fi, fj = torch.floor((a - lo[0]) / (hi[0] - lo[0]) * W), torch.floor((b - lo[1]) / (hi[1] - lo[1]) * Hh)
    if closed:
        fi = torch.where((fi == W) & (a == hi[0]), W - 1.0, fi)
        fj = torch.where((fj == Hh) & (b == hi[1]), Hh - 1.0, fj)
    ok = (fi >= 0) & (fi < W) & (fj >= 0) & (fj < Hh)
    if keep is not None:
        ok = ok & keep
    at = (fj * W + fi)[ok].to(torch.int64)
    cnt = torch.bincount(at, minlength=W * Hh).to(torch.float64)
    sums = torch.bincount(at, weights=v[ok], minlength=W * Hh) if v is not None else None
    return cnt.reshape(Hh, W), sums.reshape(Hh, W) if sums is not None else None


def _gradients(ic, eps, T, form, up, w0=None):
    """(indicator, its gradient in ic [6, N], in eps per orbit) by autograd,
    segment by segment; the indicator is J, or L for a tangent start w0."""
    k, dr = _weights(form)
    n, seg = ic.shape[1], max(1, min(20, 300_000 * 20 // ic.shape[1]))
    e = torch.full((n,), float(eps), dtype=torch.float64, device="cuda")
    tan = w0 is not None

    def segment(s, ee, p0, steps):
        X, P = s[:3], s[3:6]
        D, DP = (s[6:9], s[9:12]) if tan else (None, None)
        acc = 0.0
        for _ in range(steps):
            X, P, D, DP = _step(X, P, ee, k, dr, D, DP)
            acc = acc + (P - p0).square().sum(0)
        return torch.cat([X, P, D, DP] if tan else [X, P]), acc

    ends, s, J = [torch.cat([ic, w0]) if tan else ic], None, 0.0
    cuts = list(range(0, T, seg)) + [T]
    with torch.no_grad():
        for a, b in zip(cuts[:-1], cuts[1:]):
            s, acc = segment(ends[-1], e, ic[3:], b - a)
            J = J + acc / T
            ends.append(s)
    bar = torch.zeros_like(s)
    if tan:
        n2 = s[6:].square().sum(0)
        bar[6:] = up * s[6:] / n2
        J = 0.5 * n2.log() - 0.5 * w0.square().sum(0).log()
    ebar, pbar = torch.zeros_like(e), torch.zeros_like(ic[3:])
    for i in range(len(cuts) - 2, -1, -1):
        s = ends[i].detach().requires_grad_()
        ee, p0 = e.clone().requires_grad_(), ic[3:].clone().requires_grad_()
        s1, acc = segment(s, ee, p0, cuts[i + 1] - cuts[i])
        loss = (s1 * bar).sum() + (0.0 if tan else (up * acc / T).sum())
        got = torch.autograd.grad(loss, (s, ee, p0), allow_unused=True)
        bar, ebar = got[0], ebar + got[1]
        if not tan:
            pbar = pbar + got[2]
    gic = bar[:6].clone()
    gic[3:] += pbar
    return J, gic, ebar


def exact(case, seed):
    s, call = prepare(case, seed), case["call"]
    eps, form = case.get("eps"), case.get("form")
    if call == "hist":
        c, v = _hist(s["a"], s["b"], s["v"], (0.0, 0.0), (1.0, 1.0), case["W"], case["H"], False)
        return dict(counts=None, sums=v, dropped=None)
    if call == "window":
        return None
    stages = KICKS[form] * case["steps"]
    if call == "batch":
        if sum(e.n_steps for e in s["ens"]) * KICKS[form] > 90_000:
            return None
        imgs = [_propagate(_start(case, seed, e), e.eps, e.n_steps, form, e.seed_tangent)[0][2].reshape(e.ny, e.nx)
                for e in s["ens"]]
        return dict(img=imgs, cnt=None)
    if call in ("grad_j", "grad_l"):
        if stages > (4000 if call == "grad_j" else 2700):
            return None
        ic = (s["ic"].detach().t() if call == "grad_j" else s["ic"]).contiguous()
        v, gic, ge = _gradients(ic, eps, case["steps"], form, s["up"], _w0(seed, case["n"]) if call == "grad_l" else None)
        if call == "grad_j":
            return dict(J=v, gic=gic.t().contiguous(), geps=ge.sum())
        return dict(L=v, gic=gic, geps=ge)
    if call == "steps":
        stages *= case["chunks"]
    if stages * (2.0 if (case.get("nx", 1) * case.get("ny", 1) > 500_000 or case.get("n", 1) > 500_000) else 1.0) > 20_000:
        return None
    T = s["e"].n_steps
    tan = s["e"].seed_tangent if s["e"].tangent else None
    if call == "map":
        out, st, _ = _propagate(s["ic"], eps, T, form, tan)
        return dict(out=out, state=st if case["state"] and tan is not None else None, cls=None)
    s0 = _start(case, seed, s["e"])
    out, _, left = _propagate(s0, eps, T, form, tan, _zoom(True) if case.get("stay") else None)
    if call == "image":
        return dict(img=out[2].reshape(case["ny"], case["nx"]), cnt=None, cls=None)
    if call == "box":
        c, v = _hist(s0[3], s0[4], out[6], (0.0, 0.0), (TWO_PI, TWO_PI), case["W"], case["H"], False)
        return dict(img=torch.where(c > 0, v / c.clamp(min=1.0), 0.0), cnt=None, cls=None)
    if call == "sphere":
        w = _zoom(case["stay"])
        phi, mu = torch.atan2(out[4], out[3]), out[5] / out[3:6].square().sum(0).sqrt()
        c, _ = _hist(phi, mu, None, (w[0], w[2]), (w[1], w[3]), case["W"], case["H"], True, ~left)
        area = (w[1] - w[0]) / case["W"] * (w[3] - w[2]) / case["H"]
        return dict(img=c / (case["n"] * area), cnt=None, cls=None)
    return dict(out=out, cls=None)
