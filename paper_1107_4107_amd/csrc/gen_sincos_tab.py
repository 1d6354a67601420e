"""Writes aw_sincos_tab.h: constants of the table-driven FP64 sin/cos of the
propagation and adjoint kernels.

The kernels hold their angles in units of the table's nodes, a = 2048 x/pi, so
that the reduction is exact: q = nearest integer to a (by adding 1.5 * 2^52,
whose low mantissa word then holds q in two's complement), r = a - q,
|r| <= 1/2.  With k = q mod 4096 and (S_k, C_k) = (sin, cos)(k pi/2048) read
from a 4096-entry table held in LDS they turn the entry by the angle r pi/2048
with three shears (turn),
    c1 = C - t S,  s = S + w c1,  c = c1 - t s,
with t = tan(r pi/4096) = r (T0 + T1 r^2) and w = sin(r pi/2048) =
r (W0 + W1 r^2): near-minimax fits in r^2 on [0, 1/4] at 60 digits (mpmath
Chebyshev interpolation) whose leading coefficients are pi/4096 and pi/2048.
The table carries the signs of every quadrant, so no parity correction
follows.  Its byte offset 16 k is the low word of the rounding sum shifted left
by 4 and cut to 16 bits.

The whole device sequence is replayed here in double precision with each
fused multiply-add rounded once (exactly, through mpmath), against mpmath's
sin and cos; the errors are written into the header.  The probe library also
runs the rotation behind a reduction in radians -- x = q pi/2048 + r by a
two-part Cody-Waite step (pi/2048 = PI_A/2048 + PI_B/2048, exact scalings of
the two-part pi) -- and from the doubled angle, node 2q and remainder 2r, for
cos z sin z = sin(2z)/2 and cos^2 z = (1 + cos 2z)/2: device_sincos and
device_zterms.

Run:  python gen_sincos_tab.py > aw_sincos_tab.h
"""
import random
import struct
import sys

import mpmath as mp

mp.mp.dps = 60
N_TAB = 4096
MAGIC = 1.5 * 2.0 ** 52


def fma(a, b, c):
    """a * b + c rounded once to double."""
    return float(mp.mpf(a) * mp.mpf(b) + mp.mpf(c))


def lo32(t):
    return struct.unpack("<Q", struct.pack("<d", t))[0] & 0xFFFFFFFF


def turn(tab, k, r, w, t):
    """(sin, cos) of node k turned by r nodes."""
    S, C = tab[2 * k], tab[2 * k + 1]
    u = r * r
    sw = r * fma(w[1], u, w[0])
    tn = r * fma(t[1], u, t[0])
    c1 = fma(-tn, S, C)
    s = fma(sw, c1, S)
    return s, fma(-tn, s, c1)


def radian_reduce(x, inv, pa, pb):
    """(low word of the rounding sum, remainder in radians) of x by pi/2048."""
    m = fma(x, inv, MAGIC)
    q = m - MAGIC
    r = fma(-q, pa, x)
    return lo32(m), fma(-q, pb, r)


def device_sincos(x, tab, w, t, inv, pa, pb):
    lo, r = radian_reduce(x, inv, pa, pb)
    return turn(tab, lo % N_TAB, r * inv, w, t)


def device_zterms(z, tab, w, t, inv, pa, pb):
    """(cos z sin z, cos^2 z) from the table at the doubled angle."""
    lo, r = radian_reduce(z, inv, pa, pb)
    s, c = turn(tab, (2 * lo) % N_TAB, (r + r) * inv, w, t)
    return 0.5 * s, fma(0.5, c, 0.5)


def node_constants():
    """Shear coefficients (W0, W1), (T0, T1) of one node unit with their fit
    errors relative to the angle, and the two-part conversions nodes per radian
    (hi, lo), sqrt 2 (hi, lo) and radians per node."""
    step = mp.pi / 2048

    def cubic(f, lead):
        # f(r) = lead r + r^3 g(r^2): one coefficient for g on u = r^2 in [0, 1/4]
        def g(u):
            if u == 0:
                u = mp.mpf("1e-20")
            r = mp.sqrt(u)
            return (f(r) / r - lead) / u
        poly, err = mp.chebyfit(g, [mp.mpf("1e-8"), mp.mpf(1) / 4], 1, error=True)
        return float(lead), float(poly[0]), err / 4 / lead
    w0, w1, ew = cubic(lambda r: mp.sin(r * step), step)
    t0, t1, et = cubic(lambda r: mp.tan(r * step / 2), step / 2)
    k, q2 = 1 / step, mp.sqrt(2)
    khi, qhi = float(k), float(q2)
    return (w0, w1, ew), (t0, t1, et), (khi, float(k - khi)), (qhi, float(q2 - qhi)), float(step)


def device_sincos_node(a, tab, w, t):
    """(sin, cos) of a pi/2048 as the kernels compute them."""
    m = a + MAGIC
    q = m - MAGIC
    return turn(tab, ((lo32(m) << 4) & 0xFFFF) >> 4, a - q, w, t)


def constants():
    """The table, the shear coefficients and the radian reduction's constants,
    with the fit errors: (tab, [(W0, W1)], (T0, T1), inv, pa, pb, errw, errt)."""
    (w0, w1, ew), (t0, t1, et), kk, _, _ = node_constants()
    tab = []
    for k in range(N_TAB):
        a = k * mp.pi / 2048
        tab += [float(mp.sin(a)), float(mp.cos(a))]
    pi_a = float(mp.pi)
    pi_b = float(mp.pi - pi_a)
    pa, pb = pi_a / 2048.0, pi_b / 2048.0      # exact: division by a power of two
    return tab, [(w0, w1)], (t0, t1), kk[0], pa, pb, ew, et


def z_constants():
    """The same coefficients for device_zterms: ([(W0, W1)], (T0, T1), errw, errt)."""
    _, ps, pc, _, _, _, ew, et = constants()
    return ps, pc, ew, et


def main():
    tab, ps, pc, inv, pa, pb, _, _ = constants()
    nw, nt, kk, q2, rpn = node_constants()
    rnd = random.Random(5)
    ns = [rnd.uniform(-5e3, 5e3) for _ in range(4000)] + [rnd.uniform(-1e9, 1e9) for _ in range(2000)]
    ns += [(k + 0.5) * (1 + s * 1e-15) for k in range(-4200, 4200, 7) for s in (-1, 0, 1)]
    es = ec = 0.0
    for a in ns:
        s, c = device_sincos_node(a, tab, nw, nt)
        x = mp.mpf(a) * mp.pi / 2048
        es = max(es, abs(s - float(mp.sin(x))))
        ec = max(ec, abs(c - float(mp.cos(x))))
    # The kick's z factors from the doubled angle, over radians up to 1e6.
    ez2 = ezs = 0.0
    zs = [rnd.uniform(-7.0, 7.0) for _ in range(3000)] + [rnd.uniform(-1e6, 1e6) for _ in range(1500)]
    zs += [float((k + 0.5) * mp.pi / 4096) * (1 + s * 1e-15) for k in range(-4200, 4200, 7) for s in (-1, 1)]
    for z in zs:
        zsz, z2 = device_zterms(z, tab, ps[0], pc, inv, pa, pb)
        cz, sz = mp.cos(mp.mpf(z)), mp.sin(mp.mpf(z))
        ez2 = max(ez2, abs(z2 - float(cz * cz)))
        ezs = max(ezs, abs(zsz - float(cz * sz)))
    out = sys.stdout
    out.write("/* Generated by gen_sincos_tab.py -- do not edit. */\n#pragma once\n")
    out.write(f"/* w = r (W0 + W1 r^2), t = r (T0 + T1 r^2), |r| <= 1/2 node: fit errors {mp.nstr(nw[2], 3)} and "
              f"{mp.nstr(nt[2], 3)} of the angle; device sequence replayed with single-rounding FMAs over {len(ns)} "
              f"arguments up to 1e9 nodes: max abs error sin {es:.3e}, cos {ec:.3e} */\n")
    out.write(f"/* from the doubled angle, replayed over {len(zs)} arguments up to 1e6: max abs error cos^2 z {ez2:.3e}, "
              f"cos z sin z {ezs:.3e} */\n")
    out.write(f"#define AW_TAB_N {N_TAB}\n")
    out.write(f"static constexpr double AW_NODE_W[2] = {{{nw[0].hex()}, {nw[1].hex()}}};\n")
    out.write(f"static constexpr double AW_NODE_T[2] = {{{nt[0].hex()}, {nt[1].hex()}}};\n")
    out.write(f"static constexpr double AW_NODES_PER_RAD[2] = {{{kk[0].hex()}, {kk[1].hex()}}};  /* 2048/pi, two parts */\n")
    out.write(f"static constexpr double AW_RAD_PER_NODE = {rpn.hex()};\n")
    out.write(f"static constexpr double AW_PI2K_A = {pa.hex()};  /* pi/2048, two parts */\n")
    out.write(f"static constexpr double AW_PI2K_B = {pb.hex()};\n")
    out.write(f"static constexpr double AW_SQRT2[2] = {{{q2[0].hex()}, {q2[1].hex()}}};  /* two parts */\n")
    out.write("/* (sin, cos)(k pi/2048), k = 0..4095, interleaved */\n")
    out.write("static constexpr double AW_TAB_SC[2 * AW_TAB_N] = {\n")
    for k in range(N_TAB):
        out.write(f"  {tab[2 * k].hex()}, {tab[2 * k + 1].hex()},\n")
    out.write("};\n")


if __name__ == "__main__":
    main()
