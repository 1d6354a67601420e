// aw_ftle_adj.hip -- reverse-mode gradient of the tangent-growth indicator
// L = ln(|w_T| / |w_0|) (the finite-time Lyapunov indicator) with respect to
// the initial state and eps, for the maps of aw_fwd.hip: a second-order
// adjoint, since L is a function of the tangent map itself.
//
// The state of one orbit is s = (X, P) and its tangent w = (dX, dP); the
// adjoint carries (Xbar, Pbar, dXbar, dPbar) and epsbar.  With
// M(X) = -t eps Hess Hp(X) for a kick of weight t, the stages and their
// transposes are
//   drift D(t):  X += t P, dX += t dP
//                Pbar += t Xbar, dPbar += t dXbar
//   kick  K(t):  P += -t eps grad Hp(X), dP += M(X) dX
//                Xbar  += M(X) Pbar - t eps T3(X)[dX, dPbar]
//                dXbar += M(X) dPbar
//                epsbar += -t grad Hp(X) . Pbar - t (Hess Hp(X) dX) . dPbar
// where T3 is the third-derivative tensor of Hp (symmetric), contracted
// with dX and dPbar.  The end condition is dL/dw_T = w_T / |w_T|^2.
// The kernels step in the scaled rotated frame of the forward kernels
// (kick_node; tangent and adjoint in (u, v, sqrt 2 z) and their momenta): there
// the kick's Jacobian has 7 non-zero entries and is symmetric, |w|^2 is half
// the sum of the six squares, and the gradient is taken back to (x, y, z) at
// the end.
//
// The tangent is rescaled by exact powers of two after every 8th step
// (global step count), as in the forward kernel.  A rescale w <- 2^-k w is
// linear, so its transpose rescales the adjoint of w by the same 2^-k; the
// exponent is recomputed in the reverse sweep from the stored pre-rescale
// tangent, so it matches the forward pass exactly.
//
// Forward kernel: one lane per orbit, or two for few orbits, runs the map with its tangent, stores
// (s, w) at the start of every segment of `ckpt` steps and writes L.  In the
// last segments, as many as the workspace has room for, it also keeps (s, w)
// at the end of every ADJ_SUB-th step and of the segment's last step (before
// any rescale).
// Backward kernel: it walks the segments from the last; a
// segment whose states were not kept it recomputes from its checkpoint, keeping
// the same ones, then it sweeps the steps backwards, undoing each stage by its exact
// inverse (drift: X -= t P, dX -= t dP; kick: P -= the kick's increment,
// dP -= M dX) from the kept state at the end of each group of steps, while the
// adjoint above is propagated.  Each lane only reads back what it wrote itself.
//
// Reversible sweep (k_ftle_bwd_rev): no recompute and no stored step states.
// Each segment is swept back from the exact state at its end (the next
// checkpoint; the final state for the last segment), inverting the stages of
// state and tangent step after step.  The exponent of every rescale cannot be
// recovered from the rescaled tangent, so the forward pass records it (one
// 16-bit integer per orbit per 8 steps) and the sweep applies it to the tangent and,
// inversely, to its adjoint.
#include <hip/hip_runtime.h>

#include "aw_device.hpp"
#include "aw_internal.hpp"
#include "aw_launch.hpp"
#include "aw_step.hpp"

namespace aw {

namespace {

constexpr double LN2_D = 0.693147180559945309417232121458176568;
constexpr int64_t RESCALE_MASK = 7;  // rescale after steps k with (k + 1) % 8 == 0
static_assert(((RESCALE_MASK + 1) % ADJ_SUB) == 0, "every rescale step must be a kept step");

template <int FORM>
__device__ __forceinline__ void tan_step(Orbit &o, const AdjDesc &d, const double2 *__restrict__ tab) {
  Orbit t[1] = {o};
  map_step<FORM, true, 1>(t, d.w, tab);
  o = t[0];
}

struct Adjoint2 {
  double xb, yb, zb, pxb, pyb, pzb;        // state adjoint
  double dxb, dyb, dzb, dpxb, dpyb, dpzb;  // tangent adjoint
  double eb;                               // eps adjoint
};

// Undo D(t) and apply its transpose.
__device__ __forceinline__ void rev_drift2(Orbit &o, Adjoint2 &a, double wu, double wz, double t) {
  o.x = __builtin_fma(-wu, o.px, o.x);
  o.y = __builtin_fma(-wu, o.py, o.y);
  o.z = __builtin_fma(-wz, o.pz, o.z);
  o.dx = __builtin_fma(-t, o.dpx, o.dx);
  o.dy = __builtin_fma(-t, o.dpy, o.dy);
  o.dz = __builtin_fma(-t, o.dpz, o.dz);
  a.pxb = __builtin_fma(t, a.xb, a.pxb);
  a.pyb = __builtin_fma(t, a.yb, a.pyb);
  a.pzb = __builtin_fma(t, a.zb, a.pzb);
  a.dpxb = __builtin_fma(t, a.dxb, a.dpxb);
  a.dpyb = __builtin_fma(t, a.dyb, a.dpyb);
  a.dpzb = __builtin_fma(t, a.dzb, a.dpzb);
}

// Undo K(t) and apply its transpose, in the scaled frame (the Adjoint2's x, y,
// z, px, py, pz fields hold the adjoints of (u, v, sqrt 2 z) and their momenta
// and of their tangents).  With a = t eps, e1 = a (1 + cos 2z),
// e2 = sqrt 2 a sin 2z, g = 2 a cos 2z and cs = cos u + cos v -- in
// w = sqrt 2 z: de1/dw = -e2, de2/dw = g, dg/dw = -2 e2 -- the kick is
// F = (e1 sin u, e1 sin v, e2 cs) with the symmetric Jacobian
//   M = [[e1 cos u, 0, -e2 sin u], [0, e1 cos v, -e2 sin v],
//        [-e2 sin u, -e2 sin v, g cs]],
// and the tangent kick dP += M dX.  Its transpose gives
//   Xbar  += M Pbar + S,   S_k = sum_ij dPbar_i (dM_ij/dX_k) dX_j,
//   dXbar += M dPbar,      epsbar += (F . Pbar + (M dX) . dPbar) / eps.
// With the symmetric products of tangent and adjoint tangent
//   auu = dPbar_u du, avv alike, azz = dPbar_z dz,
//   auz = dPbar_u dz + dPbar_z du, avz alike,
// and q = sin u Pbar_u + sin v Pbar_v, kc = cos u auu + cos v avv,
// ks = sin u auz + sin v avz, A = cs Pbar_z - ks, the terms collect to
//   Xbar_u += cos u (e1 Pbar_u - e2 auz) - sin u (e2 Pbar_z + g azz + e1 auu),
//   Xbar_z += g A - e2 (q + kc + 2 cs azz),
//   eps epsbar += e1 (q + kc) + e2 A + g cs azz.
// 98 FP64 instructions where the unscaled, unsymmetric frame took 112.
// F and M carry the factor eps.  For eps != 0 (EPS0 false) a.eb collects eps
// epsbar and the kernel divides by eps once at the end.  For eps = 0 (EPS0
// true) the same sums are taken with the kick's time t in the place of a.
// Sines and cosines from the same table as the forward kick.
template <bool EPS0>
__device__ __forceinline__ void rev_kick2(Orbit &o, Adjoint2 &a, double ka, double kb, double kt, double ktb,
                                          const double2 *__restrict__ tab) {
  NodeSC sc[3];
  const double ang[3] = {o.x, o.y, o.z};
  sincos_nodes<3, true>(ang, sc, tab);
  const NodeSC U = sc[0], V = sc[1], Z = sc[2];
  const double e1 = __builtin_fma(ka, Z.c, ka);
  const double e2 = kb * Z.s;
  const double g = __builtin_fma(2.0, e1, -2.0 * ka);
  const double cs = U.c + V.c;
  const double du = o.dx, dv = o.dy, dz = o.dz;
  const double pub = a.pxb, pvb = a.pyb, pzb = a.pzb;
  const double dpub = a.dpxb, dpvb = a.dpyb, dpzb = a.dpzb;
  const double mzz = cs * g;

  const double auu = dpub * du, avv = dpvb * dv, azz = dpzb * dz;
  const double auz = __builtin_fma(dpub, dz, dpzb * du);
  const double avz = __builtin_fma(dpvb, dz, dpzb * dv);
  const double q = __builtin_fma(U.s, pub, V.s * pvb);
  const double kc = __builtin_fma(U.c, auu, V.c * avv);
  const double ks = __builtin_fma(U.s, auz, V.s * avz);
  const double A = __builtin_fma(cs, pzb, -ks);
  const double csz = cs * azz;
  const double qk = q + kc;

  if constexpr (EPS0) {
    const double f1 = __builtin_fma(kt, Z.c, kt), f2 = ktb * Z.s, gf = __builtin_fma(2.0, f1, -2.0 * kt);
    a.eb = __builtin_fma(f1, qk, a.eb);
    a.eb = __builtin_fma(f2, A, a.eb);
    a.eb = __builtin_fma(gf, csz, a.eb);
  } else {
    a.eb = __builtin_fma(e1, qk, a.eb);
    a.eb = __builtin_fma(e2, A, a.eb);
    a.eb = __builtin_fma(g, csz, a.eb);
  }

  // Xbar += M Pbar + S.
  const double hb = __builtin_fma(e2, pzb, g * azz);
  a.xb = __builtin_fma(U.c, __builtin_fma(-e2, auz, e1 * pub), __builtin_fma(-U.s, __builtin_fma(e1, auu, hb), a.xb));
  a.yb = __builtin_fma(V.c, __builtin_fma(-e2, avz, e1 * pvb), __builtin_fma(-V.s, __builtin_fma(e1, avv, hb), a.yb));
  a.zb = __builtin_fma(g, A, __builtin_fma(-e2, __builtin_fma(2.0, csz, qk), a.zb));

  // dXbar += M dPbar.
  const double hd = e2 * dpzb;
  a.dxb = __builtin_fma(U.c, e1 * dpub, __builtin_fma(-U.s, hd, a.dxb));
  a.dyb = __builtin_fma(V.c, e1 * dpvb, __builtin_fma(-V.s, hd, a.dyb));
  a.dzb = __builtin_fma(mzz, dpzb, __builtin_fma(-e2, __builtin_fma(U.s, dpub, V.s * dpvb), a.dzb));

  // Undo the kick: dP -= M dX, P -= F.
  const double h = e2 * dz;
  o.dpx = __builtin_fma(-U.c, e1 * du, __builtin_fma(U.s, h, o.dpx));
  o.dpy = __builtin_fma(-V.c, e1 * dv, __builtin_fma(V.s, h, o.dpy));
  o.dpz = __builtin_fma(-mzz, dz, __builtin_fma(e2, __builtin_fma(U.s, du, V.s * dv), o.dpz));
  o.px = __builtin_fma(-e1, U.s, o.px);
  o.py = __builtin_fma(-e1, V.s, o.py);
  o.pz = __builtin_fma(-e2, cs, o.pz);
}

template <int FORM, bool EPS0>
__device__ __forceinline__ void rev_tan_step(Orbit &o, Adjoint2 &a, const AdjDesc &d, const double2 *__restrict__ tab) {
  using F = FormPattern<FORM>;
  constexpr int NK = F::NK;
  auto drift = [&](int q) { rev_drift2(o, a, d.w.dnode[q], d.w.dnodez[q], d.w.drift[q]); };
  auto kick = [&](int q) { rev_kick2<EPS0>(o, a, d.w.ka[q], d.w.kb[q], d.kt[q], d.ktb[q], tab); };
  if constexpr (F::LEAD) {
    drift(F::drift_idx[NK]);
#pragma unroll
    for (int i = NK - 1; i >= 0; --i) {
      kick(F::kick_idx[i]);
      drift(F::drift_idx[i]);
    }
  } else {
    drift(0);
    kick(0);
  }
}

__device__ __forceinline__ void load12(const double *p, int64_t N, int64_t n, Orbit &o) {
  o.x = p[0 * N + n]; o.y = p[1 * N + n]; o.z = p[2 * N + n];
  o.px = p[3 * N + n]; o.py = p[4 * N + n]; o.pz = p[5 * N + n];
  o.dx = p[6 * N + n]; o.dy = p[7 * N + n]; o.dz = p[8 * N + n];
  o.dpx = p[9 * N + n]; o.dpy = p[10 * N + n]; o.dpz = p[11 * N + n];
}

__device__ __forceinline__ void store12(double *p, int64_t N, int64_t n, const Orbit &o) {
  p[0 * N + n] = o.x; p[1 * N + n] = o.y; p[2 * N + n] = o.z;
  p[3 * N + n] = o.px; p[4 * N + n] = o.py; p[5 * N + n] = o.pz;
  p[6 * N + n] = o.dx; p[7 * N + n] = o.dy; p[8 * N + n] = o.dz;
  p[9 * N + n] = o.dpx; p[10 * N + n] = o.dpy; p[11 * N + n] = o.dpz;
}

// The sum of the tangent's six squares: 2 |w|^2 in the scaled frame.
__device__ __forceinline__ double tan_sum2(const Orbit &o) {
  double a = o.dx * o.dx;
  a = __builtin_fma(o.dy, o.dy, a);
  a = __builtin_fma(o.dz, o.dz, a);
  a = __builtin_fma(o.dpx, o.dpx, a);
  a = __builtin_fma(o.dpy, o.dpy, a);
  return __builtin_fma(o.dpz, o.dpz, a);
}

// The initial-state gradient, back from the scaled frame (d/dx = d/du + d/dv,
// d/dy = d/du - d/dv, d/dz = sqrt 2 d/d(sqrt 2 z); momenta alike).
__device__ __forceinline__ void store_grad2(const FtleDesc &d, int64_t n, const Adjoint2 &a) {
  const int64_t N = d.N;
  d.gic[0 * N + n] = a.xb + a.yb;
  d.gic[1 * N + n] = a.xb - a.yb;
  d.gic[2 * N + n] = times_sqrt2(a.zb);
  d.gic[3 * N + n] = a.pxb + a.pyb;
  d.gic[4 * N + n] = a.pxb - a.pyb;
  d.gic[5 * N + n] = times_sqrt2(a.pzb);
  d.geps[n] = a.eb;
}

// One orbit's state, tangent and adjoint as the kernels below hold them: on one
// lane, or on the two lanes of a pair (HalfOrbit; the adjoint is split the same
// way, and the even lane's eb is the orbit's).  The sums over u and v and what they
// enter (zb, dzb, dp_z, eb) are formed in the even lane as rev_kick2 forms them and
// handed to the odd one, so both ways give the same bits.
// Bound by VALU issue: a step back is 903 VALU instructions on two lanes (162 of
// them the hand-overs) and 1024 on one, a step forward 449 and 559; 16384 orbits
// over 200 steps take 600 us and 679, 4096 orbits 584 and 665.
struct OneLane {
  Orbit o;
  Adjoint2 a{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double n0;  // |w_0|^2

  static __device__ __forceinline__ int64_t orbit() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }
  __device__ __forceinline__ void begin() {
    o.p0x = o.p0y = o.p0z = 0.0;
    o.jsum = 0.0;
    o.kexp = 0;
  }
  __device__ __forceinline__ void start(const FtleDesc &d, int64_t n) {
    const int64_t N = d.N;
    begin();
    o.x = d.ic[0 * N + n]; o.y = d.ic[1 * N + n]; o.z = d.ic[2 * N + n];
    o.px = d.ic[3 * N + n]; o.py = d.ic[4 * N + n]; o.pz = d.ic[5 * N + n];
    o.dx = d.w0[0 * N + n]; o.dy = d.w0[1 * N + n]; o.dz = d.w0[2 * N + n];
    o.dpx = d.w0[3 * N + n]; o.dpy = d.w0[4 * N + n]; o.dpz = d.w0[5 * N + n];
    n0 = tan_sum2(o);   // before the frame
    to_node(o);
  }
  __device__ __forceinline__ void load(const double *p, int64_t N, int64_t n) { load12(p, N, n, o); }
  __device__ __forceinline__ void store(double *p, int64_t N, int64_t n) const { store12(p, N, n, o); }
  template <int FORM>
  __device__ __forceinline__ void fwd(const FtleDesc &d, const double2 *__restrict__ tab) { tan_step<FORM>(o, d, tab); }
  __device__ __forceinline__ double sum2() const { return tan_sum2(o); }
  // The power-of-two exponent of the forward rescale of this tangent, and w <- 2^-k w.
  __device__ __forceinline__ int exponent() const {
    Orbit t = o;
    t.kexp = 0;
    renorm_node(t);
    return t.kexp;
  }
  __device__ __forceinline__ int rescale() {
    const int k0 = o.kexp;
    renorm_node(o);
    return o.kexp - k0;
  }
  __device__ __forceinline__ void unscale(int k) {
    o.dx = __builtin_amdgcn_ldexp(o.dx, k);
    o.dy = __builtin_amdgcn_ldexp(o.dy, k);
    o.dz = __builtin_amdgcn_ldexp(o.dz, k);
    o.dpx = __builtin_amdgcn_ldexp(o.dpx, k);
    o.dpy = __builtin_amdgcn_ldexp(o.dpy, k);
    o.dpz = __builtin_amdgcn_ldexp(o.dpz, k);
  }
  __device__ __forceinline__ void rescale_adjoint(int k) {
    a.dxb = __builtin_amdgcn_ldexp(a.dxb, -k);
    a.dyb = __builtin_amdgcn_ldexp(a.dyb, -k);
    a.dzb = __builtin_amdgcn_ldexp(a.dzb, -k);
    a.dpxb = __builtin_amdgcn_ldexp(a.dpxb, -k);
    a.dpyb = __builtin_amdgcn_ldexp(a.dpyb, -k);
    a.dpzb = __builtin_amdgcn_ldexp(a.dpzb, -k);
  }
  __device__ __forceinline__ bool writes() const { return true; }
  __device__ __forceinline__ int kexp() const { return o.kexp; }
  // dL/dw_T in the scaled frame: w_T over the sum of its squares, scaled by the
  // upstream gradient gl.
  __device__ __forceinline__ void end_condition(double gl) {
    const double c = gl / sum2();
    a.dxb = c * o.dx; a.dyb = c * o.dy; a.dzb = c * o.dz;
    a.dpxb = c * o.dpx; a.dpyb = c * o.dpy; a.dpzb = c * o.dpz;
  }
  template <int FORM, bool EPS0>
  __device__ __forceinline__ void rev(const FtleDesc &d, const double2 *__restrict__ tab) {
    rev_tan_step<FORM, EPS0>(o, a, d, tab);
  }
  template <bool EPS0>
  __device__ __forceinline__ void finish(const FtleDesc &d, int64_t n) {
    if (!EPS0) a.eb /= d.eps;   // the kicks collected eps epsbar
    store_grad2(d, n, a);
  }
};

struct TwoLanes {
  HalfOrbit h;
  double wb = 0.0, zb = 0.0, pwb = 0.0, pzb = 0.0;      // state adjoint
  double dwb = 0.0, dzb = 0.0, dpwb = 0.0, dpzb = 0.0;  // tangent adjoint
  double eb = 0.0, n0;
  int odd;

  static __device__ __forceinline__ int64_t orbit() {
    return ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 1;
  }
  __device__ __forceinline__ void begin() {
    odd = (int)(threadIdx.x & 1u);
    h.p0w = h.p0z = h.jsum = 0.0;
    h.kexp = 0;
  }
  __device__ __forceinline__ void start(const FtleDesc &d, int64_t n) {
    OneLane whole;
    whole.start(d, n);
    begin();
    n0 = whole.n0;
    h.w = odd ? whole.o.y : whole.o.x;
    h.pw = odd ? whole.o.py : whole.o.px;
    h.dw = odd ? whole.o.dy : whole.o.dx;
    h.dpw = odd ? whole.o.dpy : whole.o.dpx;
    h.z = whole.o.z; h.pz = whole.o.pz;
    h.dz = whole.o.dz; h.dpz = whole.o.dpz;
  }
  // Both lanes store z's rows, so that a lane reads back what it wrote itself.
  __device__ __forceinline__ void load(const double *p, int64_t N, int64_t n) {
    h.w = p[(0 + odd) * N + n]; h.z = p[2 * N + n];
    h.pw = p[(3 + odd) * N + n]; h.pz = p[5 * N + n];
    h.dw = p[(6 + odd) * N + n]; h.dz = p[8 * N + n];
    h.dpw = p[(9 + odd) * N + n]; h.dpz = p[11 * N + n];
  }
  __device__ __forceinline__ void store(double *p, int64_t N, int64_t n) const {
    p[(0 + odd) * N + n] = h.w; p[2 * N + n] = h.z;
    p[(3 + odd) * N + n] = h.pw; p[5 * N + n] = h.pz;
    p[(6 + odd) * N + n] = h.dw; p[8 * N + n] = h.dz;
    p[(9 + odd) * N + n] = h.dpw; p[11 * N + n] = h.dpz;
  }
  template <int FORM>
  __device__ __forceinline__ void fwd(const FtleDesc &d, const double2 *__restrict__ tab) {
    pair_step<FORM, true>(h, d.w, tab);
  }
  __device__ __forceinline__ double sum2() const { return pair_tan_sum2(h); }
  __device__ __forceinline__ int exponent() const { return pair_rescale_exponent(h); }
  __device__ __forceinline__ int rescale() {
    const int k = exponent();
    pair_rescale(h, k);
    return k;
  }
  __device__ __forceinline__ void unscale(int k) { pair_rescale(h, -k); }
  __device__ __forceinline__ void rescale_adjoint(int k) {
    dwb = __builtin_amdgcn_ldexp(dwb, -k);
    dzb = __builtin_amdgcn_ldexp(dzb, -k);
    dpwb = __builtin_amdgcn_ldexp(dpwb, -k);
    dpzb = __builtin_amdgcn_ldexp(dpzb, -k);
  }
  __device__ __forceinline__ bool writes() const { return !odd; }
  __device__ __forceinline__ int kexp() const { return h.kexp; }
  __device__ __forceinline__ void end_condition(double gl) {
    const double c = gl / sum2();
    dwb = c * h.dw; dzb = c * h.dz;
    dpwb = c * h.dpw; dpzb = c * h.dpz;
  }
  __device__ __forceinline__ void drift(double wu, double wz, double t) {
    h.w = __builtin_fma(-wu, h.pw, h.w);
    h.z = __builtin_fma(-wz, h.pz, h.z);
    h.dw = __builtin_fma(-t, h.dpw, h.dw);
    h.dz = __builtin_fma(-t, h.dpz, h.dz);
    pwb = __builtin_fma(t, wb, pwb);
    pzb = __builtin_fma(t, zb, pzb);
    dpwb = __builtin_fma(t, dwb, dpwb);
    dpzb = __builtin_fma(t, dzb, dpzb);
  }
  // rev_kick2's sums over u and v; right in the even lane.
  static __device__ __forceinline__ double both(double f, double x) {
    return __builtin_fma(f, x, dpp_pair<DPP_SWAP>(f * x));
  }
  template <bool EPS0>
  __device__ __forceinline__ void kick(double ka, double kb, double kt, double ktb, const double2 *__restrict__ tab) {
    NodeSC sc[2];
    const double ang[2] = {h.w, h.z};
    sincos_nodes<2, true>(ang, sc, tab);
    const NodeSC W = sc[0], Z = sc[1];
    const double e1 = __builtin_fma(ka, Z.c, ka);
    const double e2 = kb * Z.s;
    const double g = __builtin_fma(2.0, e1, -2.0 * ka);
    const double cs = W.c + dpp_pair<DPP_SWAP>(W.c);
    const double mzz = cs * g;

    const double aww = dpwb * h.dw, azz = dpzb * h.dz;
    const double awz = __builtin_fma(dpwb, h.dz, dpzb * h.dw);
    const double q = both(W.s, pwb), kc = both(W.c, aww), ks = both(W.s, awz);
    const double A = __builtin_fma(cs, pzb, -ks);
    const double csz = cs * azz;
    const double qk = q + kc;
    if constexpr (EPS0) {
      const double f1 = __builtin_fma(kt, Z.c, kt), f2 = ktb * Z.s, gf = __builtin_fma(2.0, f1, -2.0 * kt);
      eb = __builtin_fma(f1, qk, eb);
      eb = __builtin_fma(f2, A, eb);
      eb = __builtin_fma(gf, csz, eb);
    } else {
      eb = __builtin_fma(e1, qk, eb);
      eb = __builtin_fma(e2, A, eb);
      eb = __builtin_fma(g, csz, eb);
    }

    const double hb = __builtin_fma(e2, pzb, g * azz);
    wb = __builtin_fma(W.c, __builtin_fma(-e2, awz, e1 * pwb), __builtin_fma(-W.s, __builtin_fma(e1, aww, hb), wb));
    zb = dpp_pair<DPP_EVEN>(__builtin_fma(g, A, __builtin_fma(-e2, __builtin_fma(2.0, csz, qk), zb)));

    const double hd = e2 * dpzb;
    dwb = __builtin_fma(W.c, e1 * dpwb, __builtin_fma(-W.s, hd, dwb));
    dzb = dpp_pair<DPP_EVEN>(__builtin_fma(mzz, dpzb, __builtin_fma(-e2, both(W.s, dpwb), dzb)));

    const double r = e2 * h.dz;
    h.dpw = __builtin_fma(-W.c, e1 * h.dw, __builtin_fma(W.s, r, h.dpw));
    h.dpz = dpp_pair<DPP_EVEN>(__builtin_fma(-mzz, h.dz, __builtin_fma(e2, both(W.s, h.dw), h.dpz)));
    h.pw = __builtin_fma(-e1, W.s, h.pw);
    h.pz = __builtin_fma(-e2, cs, h.pz);
  }
  template <int FORM, bool EPS0>
  __device__ __forceinline__ void rev(const FtleDesc &d, const double2 *__restrict__ tab) {
    using F = FormPattern<FORM>;
    constexpr int NK = F::NK;
    auto undrift = [&](int q) { drift(d.w.dnode[q], d.w.dnodez[q], d.w.drift[q]); };
    auto unkick = [&](int q) { kick<EPS0>(d.w.ka[q], d.w.kb[q], d.kt[q], d.ktb[q], tab); };
    if constexpr (F::LEAD) {
      undrift(F::drift_idx[NK]);
#pragma unroll
      for (int i = NK - 1; i >= 0; --i) {
        unkick(F::kick_idx[i]);
        undrift(F::drift_idx[i]);
      }
    } else {
      undrift(0);
      unkick(0);
    }
  }
  template <bool EPS0>
  __device__ __forceinline__ void finish(const FtleDesc &d, int64_t n) {
    if (!EPS0) eb /= d.eps;   // the kicks collected eps epsbar
    Adjoint2 a{};
    a.xb = wb; a.yb = dpp_pair<DPP_SWAP>(wb); a.zb = zb;
    a.pxb = pwb; a.pyb = dpp_pair<DPP_SWAP>(pwb); a.pzb = pzb;
    a.eb = eb;
    if (!odd) store_grad2(d, n, a);
  }
};

template <int FORM, class LANES>
__global__ __launch_bounds__(512) void k_ftle_fwd(FtleDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  const int64_t N = d.N;
  LANES l;
  l.start(d, n);
  for (int64_t s = 0; s < d.n_seg; ++s) {
    l.store(d.ckpts + s * 12 * N, N, n);
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    const bool keep = s >= d.keep_from;
    double *steps = d.steps + adj_steps_at(d, s) * 12 * N;
    for (int64_t g = g0; g < g1; ++g) {
      l.template fwd<FORM>(d, s_tab);
      if (keep && adj_kept(g, g1)) l.store(steps + adj_slot(g, g0) * 12 * N, N, n);
      if (((g + 1) & RESCALE_MASK) == 0) {
        const int k = l.rescale();
        if (l.writes()) d.exps[((g + 1) / (RESCALE_MASK + 1) - 1) * N + n] = (int16_t)k;
      }
    }
  }
  l.store(d.ckpts + d.n_seg * 12 * N, N, n);   // the final state (after any last rescale)
  if (d.L) {
    const double n2 = 0.5 * l.sum2();
    const int e = __builtin_amdgcn_frexp_exp(n2);
    const double mant = __builtin_amdgcn_frexp_mant(n2);
    if (l.writes()) d.L[n] = 0.5 * ((double)(2 * l.kexp() + e) * LN2_D + log(mant)) - 0.5 * log(l.n0);
  }
}

template <int FORM, bool EPS0, class LANES>
__global__ __launch_bounds__(512) void k_ftle_bwd(FtleDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  const int64_t N = d.N;
  const double gl = d.gL ? d.gL[n] : 1.0;
  LANES l;
  l.begin();
  for (int64_t s = d.n_seg - 1; s >= 0; --s) {
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    double *steps = d.steps + adj_steps_at(d, s) * 12 * N;
    if (s < d.keep_from) {  // else the forward pass has kept the step states already
      l.load(d.ckpts + s * 12 * N, N, n);
      for (int64_t g = g0; g < g1; ++g) {
        l.template fwd<FORM>(d, s_tab);
        if (adj_kept(g, g1)) l.store(steps + adj_slot(g, g0) * 12 * N, N, n);
        if (((g + 1) & RESCALE_MASK) == 0) l.rescale();
      }
    }
    for (int64_t g = g1 - 1; g >= g0; --g) {
      // end of step g, before any rescale: kept (every rescale step is kept,
      // since ADJ_SUB divides 8), or rebuilt by the inverse of step g + 1
      if (adj_kept(g, g1)) l.load(steps + adj_slot(g, g0) * 12 * N, N, n);
      if (g == d.T - 1) l.end_condition(gl);  // dL/dw_T = w_T / |w_T|^2 (scaled by the upstream gradient)
      else if (((g + 1) & RESCALE_MASK) == 0) l.rescale_adjoint(l.exponent());
      l.template rev<FORM, EPS0>(d, s_tab);
    }
  }
  l.template finish<EPS0>(d, n);
}

template <int FORM, bool EPS0, class LANES>
__global__ __launch_bounds__(512) void k_ftle_bwd_rev(FtleDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  const int64_t N = d.N;
  const double gl = d.gL ? d.gL[n] : 1.0;
  LANES l;
  l.begin();
  for (int64_t s = d.n_seg - 1; s >= 0; --s) {
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    // Exact state at the end of step g1 - 1, after any rescale there.
    l.load(d.ckpts + (s + 1) * 12 * N, N, n);
    for (int64_t g = g1 - 1; g >= g0; --g) {
      // here: the state at the end of step g, after any rescale that followed it
      if (g == d.T - 1) l.end_condition(gl);
      if (((g + 1) & RESCALE_MASK) == 0) {
        // the forward set w_post = 2^-k w_pre: restore w_pre, and wbar_pre = 2^-k wbar_post
        const int k = d.exps[((g + 1) / (RESCALE_MASK + 1) - 1) * N + n];
        l.unscale(k);
        l.rescale_adjoint(k);
      }
      l.template rev<FORM, EPS0>(d, s_tab);   // the state at the start of step g
    }
  }
  l.template finish<EPS0>(d, n);
}

template <bool EPS0>
hipError_t launch_bwd(const FtleDesc &d, bool rev, int form, const Tuning &t, hipStream_t s) {
  return for_form(form, [&](auto f) {
    constexpr int F = decltype(f)::value;
    const bool two = two_lanes(t, d.N, n_cus());
    if (two && rev) launch_lanes(k_ftle_bwd_rev<F, EPS0, TwoLanes>, 2 * d.N, d, t, s);
    else if (two) launch_lanes(k_ftle_bwd<F, EPS0, TwoLanes>, 2 * d.N, d, t, s);
    else if (rev) launch_lanes(k_ftle_bwd_rev<F, EPS0, OneLane>, d.N, d, t, s);
    else launch_lanes(k_ftle_bwd<F, EPS0, OneLane>, d.N, d, t, s);
  });
}

}  // namespace

hipError_t launch_ftle_forward(const FtleDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return for_form(form, [&](auto f) {
    constexpr int F = decltype(f)::value;
    if (two_lanes(t, d.N, n_cus())) launch_lanes(k_ftle_fwd<F, TwoLanes>, 2 * d.N, d, t, s);
    else launch_lanes(k_ftle_fwd<F, OneLane>, d.N, d, t, s);
  });
}

hipError_t launch_ftle_backward_reversible(const FtleDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return d.eps == 0.0 ? launch_bwd<true>(d, true, form, t, s) : launch_bwd<false>(d, true, form, t, s);
}

hipError_t launch_ftle_backward(const FtleDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return d.eps == 0.0 ? launch_bwd<true>(d, false, form, t, s) : launch_bwd<false>(d, false, form, t, s);
}

}  // namespace aw
