// aw_device.hpp -- device-side arithmetic of the ensemble mapper (gfx950, FP64).
//
// Model (arXiv:1107.4107, eqs. 1-2): H = |P|^2/2 + eps Hp(X),
// Hp = cos x cos y (1 + cos 2z) = 2 cx cy cz^2.
//   grad Hp = (-2 sx cy cz^2, -2 cx sy cz^2, -4 cx cy cz sz)
//   Hess Hp: xx = yy = -2 cx cy cz^2, zz = -4 cx cy (cz^2 - sz^2),
//            xy = 2 sx sy cz^2, xz = 4 sx cy cz sz, yz = 4 cx sy cz sz.
// Kick K(t): P -= t eps grad Hp(X), dP -= t eps Hess(X) dX.
// Drift D(t): X += t P, dX += t dP.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "aw_sincos_coef.h"
#include "aw_sincos_tab.h"

namespace aw {

// ---------------------------------------------------------------------------
// sin and cos of an unwrapped angle.
// x = q pi + r with q = nearest integer to x/pi (by adding 1.5*2^52, whose
// low mantissa word then holds q), r reduced with a two-part pi: the first
// fused step is exact for |x| < 2^20 pi and the neglected tail of pi adds at
// most 1e-27 to r there.  sin x = (-1)^q sin r, cos x = (-1)^q cos r.  The
// sign (-1)^q is NOT applied here: `par` returns q's low bit in bit 0 so that
// callers can fold signs of products together.
// ---------------------------------------------------------------------------
struct SinCos {
  double c, s;     // cos r, sin r
  uint32_t par;    // low word of (q + 1.5*2^52): bit 0 = q mod 2
};

__device__ __forceinline__ SinCos sincos_red(double x) {
  const double t = __builtin_fma(x, AW_INV_PI, AW_ROUND_MAGIC);
  const double q = t - AW_ROUND_MAGIC;
  double r = __builtin_fma(-q, AW_PI_A, x);
  r = __builtin_fma(-q, AW_PI_B, r);
  const double u = r * r;
  double ps = AW_SIN_C[AW_SIN_NC - 1];
#pragma unroll
  for (int i = AW_SIN_NC - 2; i >= 0; --i) ps = __builtin_fma(ps, u, AW_SIN_C[i]);
  double pc = AW_COS_C[AW_COS_NC - 1];
#pragma unroll
  for (int i = AW_COS_NC - 2; i >= 0; --i) pc = __builtin_fma(pc, u, AW_COS_C[i]);
  SinCos o;
  o.s = __builtin_fma(r * u, ps, r);
  o.c = __builtin_fma(u, pc, 1.0);
  o.par = (uint32_t)__double2loint(t);
  return o;
}

// Flip the sign of v when bit 31 of `sgn` is set.
__device__ __forceinline__ double flip(double v, uint32_t sgn) {
  return __hiloint2double(__double2hiint(v) ^ (int)sgn, __double2loint(v));
}

// ---------------------------------------------------------------------------
// Table-driven sin and cos of an unwrapped angle (the propagation and adjoint
// kernels), from a 4096-entry table of (S, C) = (sin, cos)(k pi/2048) in LDS
// (64 KB) whose entries carry every quadrant's signs.  The kernels hold their
// angles in units of the table's nodes, a = 2048 x/pi (the drifts' weights
// carry the factor).  The reduction is then
// exact and takes three additions: q = nearest integer to a (the low mantissa
// word of a + 1.5*2^52 holds it), r = a - q, |r| <= 1/2.  The table entry
// (S, C) of node q mod 4096 is turned by the angle r pi/2048 with three
// shears,
//   c1 = C - t S,  s = S + w c1,  c = c1 - t s,
// t = tan(r pi/4096) and w = sin(r pi/2048), one coefficient each beyond the
// leading one.  5 FMA, 3 MUL, 3 ADD in place of the radian form's 8, 4 and 1
// plus the products that a doubled angle needed, and no reduction constants.
// Error over random arguments: sin at most 1.12e-16 (rms 3.8e-17), cos 1.66e-16
// (4.8e-17); the radian form's are 1.63e-16 (4.3e-17) and 1.64e-16 (4.6e-17).
//
// The table's byte offset, the low word shifted left by 4 and cut to 16 bits,
// is one 16-bit shift, which clears the upper half of its result: whatever m
// holds, the read stays inside the table.  Declared as a kernel's first LDS
// object, the table sits at address 0 and the offset is the address.  A simple
// 32-bit or 16-bit instruction takes 2.6 cycles of a SIMD with two waves
// where an SDWA form, like every FP64 instruction, takes 4.5.
// ---------------------------------------------------------------------------
struct NodeSC {
  double s, c;
};

__device__ __forceinline__ uint32_t node_offset(double t) {
  uint32_t a;
  asm("v_lshlrev_b16_e32 %0, 4, %1" : "=v"(a) : "v"((uint32_t)__double2loint(t)));
  return a;
}

// The table entries e turned by rem(k) nodes, at most 1/2: remainders and
// coefficients, then the shears of all angles in step.
template <int K, class Rem>
__device__ __forceinline__ void turn_nodes(const double2 (&e)[K], Rem &&rem, NodeSC (&o)[K]) {
  double r[K], w[K], t[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    r[k] = rem(k);
    const double u = r[k] * r[k];
    w[k] = r[k] * __builtin_fma(AW_NODE_W[1], u, AW_NODE_W[0]);
    t[k] = r[k] * __builtin_fma(AW_NODE_T[1], u, AW_NODE_T[0]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < K; ++k) o[k].c = __builtin_fma(-t[k], e[k].x, e[k].y);
#pragma unroll
  for (int k = 0; k < K; ++k) o[k].s = __builtin_fma(w[k], o[k].c, e[k].x);
#pragma unroll
  for (int k = 0; k < K; ++k) o[k].c = __builtin_fma(-t[k], o[k].s, o[k].c);
}

// The sines and cosines of K angles, in three phases that the instruction
// scheduler may not mix: every angle's table read, then the remainders and
// coefficients while the reads are on their way, then the shears of all angles
// in step.  Left to itself it serialises the angles to save registers, which
// costs a wave that has its SIMD to itself the read's latency per angle and 8.7
// cycles per dependent instruction instead of 5.3 per independent one.  4096
// orbits x 900 steps: 1.22 -> 1.01 ms; four waves per SIMD gain 2-7%.
// ALIGN puts the remainders, a run of 8-byte instructions, at a multiple of 8
// bytes: a wave that has its SIMD to itself takes 6% longer per step where the
// step loop happens to start 4 bytes off (1.17 against 1.10 us per S6 step with
// the tangent).  Without the tangent the padding costs as much as it gains.
template <int K, bool ALIGN = false>
__device__ __forceinline__ void sincos_nodes(const double (&a)[K], NodeSC (&o)[K], const double2 *__restrict__ tab) {
  double m[K];
  double2 e[K];
#pragma unroll
  for (int k = 0; k < K; ++k) m[k] = a[k] + AW_ROUND_MAGIC;
#pragma unroll
  for (int k = 0; k < K; ++k) e[k] = *(const double2 *)((const char *)tab + node_offset(m[k]));
  __builtin_amdgcn_sched_barrier(0);
  if (ALIGN) asm volatile(".p2align 3");
  turn_nodes<K>(e, [&](int k) { return a[k] - (m[k] - AW_ROUND_MAGIC); }, o);
}

// x times a constant held in two parts, rounded once (to within 2^-100).
__device__ __forceinline__ double times2(double x, const double (&k)[2]) {
#pragma clang fp contract(off)
  const double p = x * k[0];
  const double e = __builtin_fma(x, k[0], -p);
  return p + __builtin_fma(x, k[1], e);
}

__device__ __forceinline__ double to_nodes(double x) { return times2(x, AW_NODES_PER_RAD); }
__device__ __forceinline__ double times_sqrt2(double x) { return times2(x, AW_SQRT2); }
constexpr double AW_SQRT1_2 = 0x1.6a09e667f3bcdp-1;

// Fill a block's LDS copy of the (sin, cos)(k pi/2048) table; every thread of
// the block must call this before any of them returns.
__device__ __forceinline__ void load_sincos_table(double2 *tab) {
  for (int i = threadIdx.x; i < AW_TAB_N; i += blockDim.x) tab[i] = make_double2(AW_TAB_SC[2 * i], AW_TAB_SC[2 * i + 1]);
  __syncthreads();
}

// True signed cos/sin (used outside the hot loop).
__device__ __forceinline__ void sincos_full(double x, double &s, double &c) {
  SinCos a = sincos_red(x);
  uint32_t sg = a.par << 31;
  s = flip(a.s, sg);
  c = flip(a.c, sg);
}

// Hp(X) = 2 cx cy cz^2.
__device__ __forceinline__ double hp_value(double x, double y, double z) {
  SinCos X = sincos_red(x), Y = sincos_red(y), Z = sincos_red(z);
  uint32_t sg = (X.par ^ Y.par) << 31;
  return flip(2.0 * X.c * Y.c * (Z.c * Z.c), sg);
}

// ---------------------------------------------------------------------------
// Per-orbit register state.
// ---------------------------------------------------------------------------
struct Orbit {
  double x, y, z, px, py, pz;          // state (X unwrapped)
  double dx, dy, dz, dpx, dpy, dpz;    // tangent vector, scaled by 2^-kexp
  double p0x, p0y, p0z;                // initial momentum
  double jsum;                         // sum_k |P_k - P_0|^2
  int kexp;                            // tangent scale exponent (|w| true = |w| 2^kexp)
};

// The kernels step the rotated frame u = x + y, v = x - y, scaled:
// the Orbit's x, y, z hold u, v and 2 z in table nodes; px, py, pz hold
// p_u = p_x + p_y, p_v = p_x - p_y and sqrt 2 p_z; the tangent's dx, dy, dz,
// dpx, dpy, dpz hold du, dv, sqrt 2 dz and the same of its momenta, in plain
// units.  Eq. 2's H_p = 2 cx cy cz^2 is (cos u + cos v) cz^2, so the force and
// its Jacobian do not couple u and v, and the factor sqrt 2 on z makes the
// Jacobian symmetric: with a = t eps, e1 = a (1 + cos 2z), e2 = sqrt 2 a sin 2z
// and cs = cos u + cos v,
//   p_u += e1 sin u,  p_v += e1 sin v,  p_z += e2 cs,
//   dp_u += e1 cos u du - e2 sin u dz,
//   dp_v += e1 cos v dv - e2 sin v dz,
//   dp_z += -e2 (sin u du + sin v dv) + 2 a cos 2z cs dz.
// 52 FP64 instructions and three offsets with the tangent (39 without), where
// the unscaled form took 59 (46): bound by VALU issue, an S6 step is 563 VALU
// instructions instead of 627 (415 instead of 470).  The 1024 x 1024 slice over
// 1000 steps takes 18.9 ms instead of 21.3, 2e6 state-only orbits over 200
// steps 5.45 ms instead of 6.35.
template <bool TAN>
__device__ __forceinline__ void kick_node(Orbit &o, double a, double b, const double2 *__restrict__ tab) {
  NodeSC sc[3];
  const double ang[3] = {o.x, o.y, o.z};
  sincos_nodes<3, TAN>(ang, sc, tab);
  const NodeSC U = sc[0], V = sc[1], Z = sc[2];
  const double e1 = __builtin_fma(a, Z.c, a);
  const double e2 = b * Z.s;
  const double cs = U.c + V.c;
  if (TAN) {
    const double du = o.dx, dv = o.dy, dz = o.dz;
    const double fu = e1 * du, fv = e1 * dv, h = e2 * dz;
    const double g = __builtin_fma(U.s, du, V.s * dv);
    const double mz = cs * __builtin_fma(2.0, e1, -2.0 * a);
    o.dpx = __builtin_fma(U.c, fu, __builtin_fma(-U.s, h, o.dpx));
    o.dpy = __builtin_fma(V.c, fv, __builtin_fma(-V.s, h, o.dpy));
    o.dpz = __builtin_fma(mz, dz, __builtin_fma(-e2, g, o.dpz));
  }
  o.px = __builtin_fma(e1, U.s, o.px);
  o.py = __builtin_fma(e1, V.s, o.py);
  o.pz = __builtin_fma(e2, cs, o.pz);
}

// A drift of time t: wu = t in nodes per unit of p_u, wz = sqrt 2 wu (2 z in
// nodes per unit of sqrt 2 p_z).
template <bool TAN>
__device__ __forceinline__ void drift_node(Orbit &o, double wu, double wz, double t) {
  o.x = __builtin_fma(wu, o.px, o.x);
  o.y = __builtin_fma(wu, o.py, o.y);
  o.z = __builtin_fma(wz, o.pz, o.z);
  if (TAN) {
    o.dx = __builtin_fma(t, o.dpx, o.dx);
    o.dy = __builtin_fma(t, o.dpy, o.dy);
    o.dz = __builtin_fma(t, o.dpz, o.dz);
  }
}

// Into the scaled rotated frame (p0 alike).
__device__ __forceinline__ void to_node(Orbit &o) {
#pragma clang fp contract(off)
  const double x = o.x, y = o.y, px = o.px, py = o.py;
  o.x = to_nodes(x + y); o.y = to_nodes(x - y); o.z = to_nodes(2.0 * o.z);
  o.px = px + py; o.py = px - py; o.pz = times_sqrt2(o.pz);
  const double p0x = o.p0x, p0y = o.p0y;
  o.p0x = p0x + p0y; o.p0y = p0x - p0y; o.p0z = times_sqrt2(o.p0z);
  const double dx = o.dx, dy = o.dy, dpx = o.dpx, dpy = o.dpy;
  o.dx = dx + dy; o.dy = dx - dy; o.dz = times_sqrt2(o.dz);
  o.dpx = dpx + dpy; o.dpy = dpx - dpy; o.dpz = times_sqrt2(o.dpz);
}

// Back to the original frame, as displacements from the initial state s0
// (x, y, z, px, py, pz), whose scaled form is recomputed here exactly as
// to_node formed it: what the steps did not change comes back unchanged (at
// eps = 0 the momenta exactly).
__device__ __forceinline__ void from_node(Orbit &o, const double (&s0)[6]) {
#pragma clang fp contract(off)
  const double du0 = (o.x - to_nodes(s0[0] + s0[1])) * AW_RAD_PER_NODE;
  const double dv0 = (o.y - to_nodes(s0[0] - s0[1])) * AW_RAD_PER_NODE;
  const double dz0 = (o.z - to_nodes(2.0 * s0[2])) * (0.5 * AW_RAD_PER_NODE);
  const double dpu0 = o.px - (s0[3] + s0[4]), dpv0 = o.py - (s0[3] - s0[4]);
  const double dpz0 = (o.pz - times_sqrt2(s0[5])) * AW_SQRT1_2;
  o.x = s0[0] + 0.5 * (du0 + dv0); o.y = s0[1] + 0.5 * (du0 - dv0); o.z = s0[2] + dz0;
  o.px = s0[3] + 0.5 * (dpu0 + dpv0); o.py = s0[4] + 0.5 * (dpu0 - dpv0); o.pz = s0[5] + dpz0;
  const double du = o.dx, dv = o.dy, dpu = o.dpx, dpv = o.dpy;
  o.dx = 0.5 * (du + dv); o.dy = 0.5 * (du - dv); o.dz = o.dz * AW_SQRT1_2;
  o.dpx = 0.5 * (dpu + dpv); o.dpy = 0.5 * (dpu - dpv); o.dpz = o.dpz * AW_SQRT1_2;
}

// In the scaled frame |P - P0|^2 is half the sum of the three squares: jsum
// collects twice the step sum.
__device__ __forceinline__ void accum_j_node(Orbit &o) {
  const double eu = o.px - o.p0x, ev = o.py - o.p0y, ez = o.pz - o.p0z;
  o.jsum = __builtin_fma(eu, eu, o.jsum);
  o.jsum = __builtin_fma(ev, ev, o.jsum);
  o.jsum = __builtin_fma(ez, ez, o.jsum);
}

// Rescale the tangent by an exact power of two so that |w|^2 lies in
// [0.5, 2); the scale is accumulated in kexp.  Exact: it changes no mantissa.
// In the scaled frame |w|^2 is half the sum of the six squares.
__device__ __forceinline__ void renorm_node(Orbit &o) {
  double a = o.dx * o.dx;
  a = __builtin_fma(o.dy, o.dy, a);
  a = __builtin_fma(o.dz, o.dz, a);
  a = __builtin_fma(o.dpx, o.dpx, a);
  a = __builtin_fma(o.dpy, o.dpy, a);
  a = __builtin_fma(o.dpz, o.dpz, a);
  const int s = (__builtin_amdgcn_frexp_exp(a) - 1) >> 1;
  o.dx = __builtin_amdgcn_ldexp(o.dx, -s);
  o.dy = __builtin_amdgcn_ldexp(o.dy, -s);
  o.dz = __builtin_amdgcn_ldexp(o.dz, -s);
  o.dpx = __builtin_amdgcn_ldexp(o.dpx, -s);
  o.dpy = __builtin_amdgcn_ldexp(o.dpy, -s);
  o.dpz = __builtin_amdgcn_ldexp(o.dpz, -s);
  o.kexp += s;
}

// ---------------------------------------------------------------------------
// Counter-based SplitMix64 (Steele, Lea & Flood 2014): output number c of the
// stream seeded with `seed` is mix(seed + (c + 1) * 0x9E3779B97F4A7C15).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t c) {
  uint64_t z = seed + (c + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double u01(uint64_t seed, uint64_t c) {
  return (double)(splitmix64(seed, c) >> 11) * 0x1.0p-53;
}

}  // namespace aw
