// aw_adj.hip -- reverse-mode (adjoint) gradient of the step-averaged momentum
// drift J = (1/T) sum_{k=1..T} |P_k - P_0|^2 with respect to the initial
// state and eps, for the maps of aw_fwd.hip.
//
// Forward kernel: one lane per orbit, or two for few orbits, runs the map (no tangent), accumulates J
// and stores the state at the start of every segment of `ckpt` steps.  In the
// last segments, as many as the workspace has room for, it also keeps the end
// state of every ADJ_SUB-th step (and of the segment's last step).
// Backward kernel: it walks the segments from the last one; a
// segment whose states were not kept it recomputes from its checkpoint, keeping
// the same ones, then it sweeps the steps backwards.  The stages are undone in reverse order by inverting
// them exactly in exact arithmetic (drift: X -= t P; kick: P += t eps grad
// Hp(X)), starting from the kept state at the end of each group of ADJ_SUB
// steps and carrying the rebuilt state through the group, while the adjoint
// is propagated:
//   drift  D(t):  Pbar += t Xbar
//   kick   K(t):  Xbar -= t eps Hess(X) Pbar,  epsbar -= t grad Hp(X) . Pbar
// and the source of J, (2 gJ / T)(P_k - P_0), enters Pbar at every step
// boundary k >= 1.  The explicit P_0 dependence of J adds
// -(2 gJ / T) sum_k (P_k - P_0) to the initial-momentum gradient.
// All of it runs in the scaled rotated frame of the forward kernels
// (kick_node), where the kick's Jacobian has 7 non-zero entries and is
// symmetric; the checkpoints and step states hold scaled states, the adjoint
// that of (u, v, sqrt 2 z) and their momenta, and the gradient is taken back to
// (x, y, z) at the end.
// Each lane only reads back what it wrote itself, so no synchronisation
// between lanes is needed.
//
// Reversible sweep (k_adj_bwd_rev): the same reverse pass without the
// recompute and without storing step states.  Each segment is swept back from
// the exact state at its end (the next checkpoint; the final state for the
// last segment), undoing the steps one after the other by inverting their
// stages.  The reconstructed states carry the rounding of the inversion,
// which restarts from an exact state at every checkpoint.
#include <hip/hip_runtime.h>

#include "aw_device.hpp"
#include "aw_internal.hpp"
#include "aw_launch.hpp"
#include "aw_step.hpp"

namespace aw {

namespace {

template <int FORM>
__device__ __forceinline__ void adj_step_fwd(Orbit &o, const AdjDesc &d, const double2 *__restrict__ tab) {
  Orbit t[1] = {o};
  map_step<FORM, false, 1>(t, d.w, tab);
  o = t[0];
}

struct Adjoint {
  double xb, yb, zb, pxb, pyb, pzb, eb;
};

// Undo D(t) on the state and apply its transpose to the adjoint.
__device__ __forceinline__ void rev_drift(Orbit &o, Adjoint &a, double wu, double wz, double t) {
  o.x = __builtin_fma(-wu, o.px, o.x);
  o.y = __builtin_fma(-wu, o.py, o.y);
  o.z = __builtin_fma(-wz, o.pz, o.z);
  a.pxb = __builtin_fma(t, a.xb, a.pxb);
  a.pyb = __builtin_fma(t, a.yb, a.pyb);
  a.pzb = __builtin_fma(t, a.zb, a.pzb);
}

// Undo K(t) on the state and apply its transpose to the adjoint, in the scaled
// frame of the forward kernels (the Adjoint's fields hold the adjoints of u, v,
// sqrt 2 z and their momenta).  With a = t eps, e1 = a (1 + cos 2z),
// e2 = sqrt 2 a sin 2z and cs = cos u + cos v the kick is
// F = (e1 sin u, e1 sin v, e2 cs) and its symmetric Jacobian
//   [[e1 cos u, 0, -e2 sin u], [0, e1 cos v, -e2 sin v],
//    [-e2 sin u, -e2 sin v, 2 a cos 2z cs]]
// acts on Pbar; dF/deps = F / eps.  For eps != 0 (EPS0 false) a.eb collects
// eps epsbar = F . Pbar and the kernel divides by eps once at the end; for
// eps = 0 (EPS0 true) F / eps is formed from the kick's time t, sqrt 2 t.
// Sines and cosines from the same table as the forward kick, so the undone
// kick matches it.  54 FP64 instructions (62 in the unscaled frame).
template <bool EPS0>
__device__ __forceinline__ void rev_kick(Orbit &o, Adjoint &a, double ka, double kb, double kt, double ktb,
                                         const double2 *__restrict__ tab) {
  NodeSC sc[3];
  const double ang[3] = {o.x, o.y, o.z};
  sincos_nodes<3, true>(ang, sc, tab);
  const NodeSC U = sc[0], V = sc[1], Z = sc[2];
  const double e1 = __builtin_fma(ka, Z.c, ka);
  const double e2 = kb * Z.s;
  const double cs = U.c + V.c;
  const double pub = a.pxb, pvb = a.pyb, pzb = a.pzb;
  const double q = __builtin_fma(U.s, pub, V.s * pvb);   // sin u pu_bar + sin v pv_bar
  const double h = e2 * pzb;
  if constexpr (EPS0) {
    a.eb = __builtin_fma(__builtin_fma(kt, Z.c, kt), q, a.eb);
    a.eb = __builtin_fma((ktb * Z.s) * pzb, cs, a.eb);
  } else {
    a.eb = __builtin_fma(e1, q, a.eb);
    a.eb = __builtin_fma(h, cs, a.eb);
  }
  const double fu = e1 * pub, fv = e1 * pvb;
  a.xb = __builtin_fma(U.c, fu, __builtin_fma(-U.s, h, a.xb));
  a.yb = __builtin_fma(V.c, fv, __builtin_fma(-V.s, h, a.yb));
  const double mz = cs * __builtin_fma(2.0, e1, -2.0 * ka);
  a.zb = __builtin_fma(mz, pzb, __builtin_fma(-e2, q, a.zb));
  // P before the kick.
  o.px = __builtin_fma(-e1, U.s, o.px);
  o.py = __builtin_fma(-e1, V.s, o.py);
  o.pz = __builtin_fma(-e2, cs, o.pz);
}

template <int FORM, bool EPS0>
__device__ __forceinline__ void adj_step_rev(Orbit &o, Adjoint &a, const AdjDesc &d, const double2 *__restrict__ tab) {
  using F = FormPattern<FORM>;
  constexpr int NK = F::NK;
  auto drift = [&](int q) { rev_drift(o, a, d.w.dnode[q], d.w.dnodez[q], d.w.drift[q]); };
  auto kick = [&](int q) { rev_kick<EPS0>(o, a, d.w.ka[q], d.w.kb[q], d.kt[q], d.ktb[q], tab); };
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

__device__ __forceinline__ void load6(const double *p, int64_t N, int64_t n, Orbit &o) {
  o.x = p[0 * N + n]; o.y = p[1 * N + n]; o.z = p[2 * N + n];
  o.px = p[3 * N + n]; o.py = p[4 * N + n]; o.pz = p[5 * N + n];
}

__device__ __forceinline__ void store6(double *p, int64_t N, int64_t n, const Orbit &o) {
  p[0 * N + n] = o.x; p[1 * N + n] = o.y; p[2 * N + n] = o.z;
  p[3 * N + n] = o.px; p[4 * N + n] = o.py; p[5 * N + n] = o.pz;
}

// The initial-state gradient: the explicit P_0 share of J, then back from the
// scaled frame (u = x + y, v = x - y, so d/dx = d/du + d/dv and
// d/dy = d/du - d/dv; d/dz = sqrt 2 d/d(sqrt 2 z); momenta alike).
__device__ __forceinline__ void store_grad(const AdjDesc &d, int64_t n, const Adjoint &a, double c,
                                           double su, double sv, double sz) {
  const int64_t N = d.N;
  const double pub = __builtin_fma(-c, su, a.pxb), pvb = __builtin_fma(-c, sv, a.pyb);
  d.gic[0 * N + n] = a.xb + a.yb;
  d.gic[1 * N + n] = a.xb - a.yb;
  d.gic[2 * N + n] = times_sqrt2(a.zb);
  d.gic[3 * N + n] = pub + pvb;
  d.gic[4 * N + n] = pub - pvb;
  d.gic[5 * N + n] = times_sqrt2(__builtin_fma(-c, sz, a.pzb));
  d.geps[n] = a.eb;
}

// One orbit's state, adjoint and sums as the kernels below hold them: on one lane,
// or on the two lanes of a pair (HalfOrbit; the adjoint is split the same way, and
// eb and the sums of the even lane are the orbit's).  The sum
// q = sin u pu_bar + sin v pv_bar is formed in the even lane as rev_kick forms it
// and handed to the odd one, so both ways give the same bits.
// Bound by VALU issue: a step back is 473 VALU instructions on two lanes and 586
// on one, a step forward 310 and 418; 16384 orbits over 200 steps take 378 us and
// 464, 4096 orbits 361 and 444.
struct OneLane {
  Orbit o;
  Adjoint a{0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  double sx = 0.0, sy = 0.0, sz = 0.0;  // sum_k (P_k - P_0)

  static __device__ __forceinline__ int64_t orbit() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }
  __device__ __forceinline__ void start(const AdjDesc &d, int64_t n) {
    load6(d.ic, d.N, n, o);
    o.p0x = o.px; o.p0y = o.py; o.p0z = o.pz;
    o.dx = o.dy = o.dz = o.dpx = o.dpy = o.dpz = 0.0;
    o.jsum = 0.0;
    o.kexp = 0;
    to_node(o);
  }
  __device__ __forceinline__ void load(const double *p, int64_t N, int64_t n) { load6(p, N, n, o); }
  __device__ __forceinline__ void store(double *p, int64_t N, int64_t n) const { store6(p, N, n, o); }
  template <int FORM>
  __device__ __forceinline__ void fwd(const AdjDesc &d, const double2 *__restrict__ tab) { adj_step_fwd<FORM>(o, d, tab); }
  __device__ __forceinline__ void accum_j() { accum_j_node(o); }
  __device__ __forceinline__ void store_j(const AdjDesc &d, int64_t n) const { d.J[n] = (0.5 * o.jsum) / (double)d.T; }
  __device__ __forceinline__ void source(double c) {
    const double ex = o.px - o.p0x, ey = o.py - o.p0y, ez = o.pz - o.p0z;
    a.pxb = __builtin_fma(c, ex, a.pxb);
    a.pyb = __builtin_fma(c, ey, a.pyb);
    a.pzb = __builtin_fma(c, ez, a.pzb);
    sx += ex; sy += ey; sz += ez;
  }
  template <int FORM, bool EPS0>
  __device__ __forceinline__ void rev(const AdjDesc &d, const double2 *__restrict__ tab) {
    adj_step_rev<FORM, EPS0>(o, a, d, tab);
  }
  template <bool EPS0>
  __device__ __forceinline__ void finish(const AdjDesc &d, int64_t n, double c) {
    if (!EPS0) a.eb /= d.eps;   // the kicks collected eps epsbar
    store_grad(d, n, a, c, sx, sy, sz);
  }
};

struct TwoLanes {
  HalfOrbit h;
  double wb = 0.0, zb = 0.0, pwb = 0.0, pzb = 0.0, eb = 0.0;
  double sw = 0.0, sz = 0.0;
  int odd;

  static __device__ __forceinline__ int64_t orbit() {
    return ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 1;
  }
  __device__ __forceinline__ void start(const AdjDesc &d, int64_t n) {
    OneLane whole;
    whole.start(d, n);
    odd = (int)(threadIdx.x & 1u);
    h.w = odd ? whole.o.y : whole.o.x;
    h.pw = h.p0w = odd ? whole.o.py : whole.o.px;
    h.z = whole.o.z;
    h.pz = h.p0z = whole.o.pz;
    h.dw = h.dpw = h.dz = h.dpz = 0.0;
    h.jsum = 0.0;
    h.kexp = 0;
  }
  // Both lanes store z's rows, so that a lane reads back what it wrote itself.
  __device__ __forceinline__ void load(const double *p, int64_t N, int64_t n) {
    h.w = p[(0 + odd) * N + n]; h.z = p[2 * N + n];
    h.pw = p[(3 + odd) * N + n]; h.pz = p[5 * N + n];
  }
  __device__ __forceinline__ void store(double *p, int64_t N, int64_t n) const {
    p[(0 + odd) * N + n] = h.w; p[2 * N + n] = h.z;
    p[(3 + odd) * N + n] = h.pw; p[5 * N + n] = h.pz;
  }
  template <int FORM>
  __device__ __forceinline__ void fwd(const AdjDesc &d, const double2 *__restrict__ tab) {
    pair_step<FORM, false>(h, d.w, tab);
  }
  __device__ __forceinline__ void accum_j() { pair_accum_j(h); }
  __device__ __forceinline__ void store_j(const AdjDesc &d, int64_t n) const {
    if (!odd) d.J[n] = (0.5 * h.jsum) / (double)d.T;
  }
  __device__ __forceinline__ void source(double c) {
    const double ew = h.pw - h.p0w, ez = h.pz - h.p0z;
    pwb = __builtin_fma(c, ew, pwb);
    pzb = __builtin_fma(c, ez, pzb);
    sw += ew; sz += ez;
  }
  __device__ __forceinline__ void drift(double wu, double wz, double t) {
    h.w = __builtin_fma(-wu, h.pw, h.w);
    h.z = __builtin_fma(-wz, h.pz, h.z);
    pwb = __builtin_fma(t, wb, pwb);
    pzb = __builtin_fma(t, zb, pzb);
  }
  template <bool EPS0>
  __device__ __forceinline__ void kick(double ka, double kb, double kt, double ktb, const double2 *__restrict__ tab) {
    NodeSC sc[2];
    const double ang[2] = {h.w, h.z};
    sincos_nodes<2, true>(ang, sc, tab);
    const NodeSC W = sc[0], Z = sc[1];
    const double e1 = __builtin_fma(ka, Z.c, ka);
    const double e2 = kb * Z.s;
    const double cs = W.c + dpp_pair<DPP_SWAP>(W.c);
    const double q = dpp_pair<DPP_EVEN>(__builtin_fma(W.s, pwb, dpp_pair<DPP_SWAP>(W.s * pwb)));
    const double r = e2 * pzb;
    if constexpr (EPS0) {
      eb = __builtin_fma(__builtin_fma(kt, Z.c, kt), q, eb);
      eb = __builtin_fma((ktb * Z.s) * pzb, cs, eb);
    } else {
      eb = __builtin_fma(e1, q, eb);
      eb = __builtin_fma(r, cs, eb);
    }
    wb = __builtin_fma(W.c, e1 * pwb, __builtin_fma(-W.s, r, wb));
    const double mz = cs * __builtin_fma(2.0, e1, -2.0 * ka);
    zb = __builtin_fma(mz, pzb, __builtin_fma(-e2, q, zb));
    h.pw = __builtin_fma(-e1, W.s, h.pw);
    h.pz = __builtin_fma(-e2, cs, h.pz);
  }
  template <int FORM, bool EPS0>
  __device__ __forceinline__ void rev(const AdjDesc &d, const double2 *__restrict__ tab) {
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
  __device__ __forceinline__ void finish(const AdjDesc &d, int64_t n, double c) {
    if (!EPS0) eb /= d.eps;   // the kicks collected eps epsbar
    const Adjoint a{wb, dpp_pair<DPP_SWAP>(wb), zb, pwb, dpp_pair<DPP_SWAP>(pwb), pzb, eb};
    const double sv = dpp_pair<DPP_SWAP>(sw);
    if (!odd) store_grad(d, n, a, c, sw, sv, sz);
  }
};

template <int FORM, class LANES>
__global__ __launch_bounds__(512) void k_adj_fwd(AdjDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  LANES l;
  l.start(d, n);
  for (int64_t s = 0; s < d.n_seg; ++s) {
    l.store(d.ckpts + s * 6 * d.N, d.N, n);
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    const bool keep = s >= d.keep_from;
    double *steps = d.steps + adj_steps_at(d, s) * 6 * d.N;
    for (int64_t g = g0; g < g1; ++g) {
      l.template fwd<FORM>(d, s_tab);
      l.accum_j();
      if (keep && adj_kept(g, g1)) l.store(steps + adj_slot(g, g0) * 6 * d.N, d.N, n);
    }
  }
  l.store(d.ckpts + d.n_seg * 6 * d.N, d.N, n);   // the final state
  if (d.J) l.store_j(d, n);
}

// P_0 comes from the initial state, in the scaled frame and rounded as the
// forward pass formed it.  J is half the step average of the three squared
// displacements: the source is c (P_k - P_0).
template <int FORM, bool EPS0, class LANES>
__global__ __launch_bounds__(512) void k_adj_bwd_rev(AdjDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  const int64_t N = d.N;
  const double c = (d.gJ ? d.gJ[n] : 1.0) / (double)d.T;
  LANES l;
  l.start(d, n);
  for (int64_t s = d.n_seg - 1; s >= 0; --s) {
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    l.load(d.ckpts + (s + 1) * 6 * N, N, n);          // exact state after step g1 - 1
    for (int64_t g = g1 - 1; g >= g0; --g) {
      l.source(c);
      l.template rev<FORM, EPS0>(d, s_tab);           // state now at the start of step g
    }
  }
  l.template finish<EPS0>(d, n, c);
}

template <int FORM, bool EPS0, class LANES>
__global__ __launch_bounds__(512) void k_adj_bwd(AdjDesc d) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n = LANES::orbit();
  if (n >= d.N) return;
  const int64_t N = d.N;
  const double c = (d.gJ ? d.gJ[n] : 1.0) / (double)d.T;
  LANES l;
  l.start(d, n);
  for (int64_t s = d.n_seg - 1; s >= 0; --s) {
    const int64_t g0 = s * d.ckpt;
    const int64_t g1 = g0 + d.ckpt < d.T ? g0 + d.ckpt : d.T;
    double *steps = d.steps + adj_steps_at(d, s) * 6 * N;
    if (s < d.keep_from) {  // else the forward pass has kept the step states already
      l.load(d.ckpts + s * 6 * N, N, n);
      for (int64_t g = g0; g < g1; ++g) {
        l.template fwd<FORM>(d, s_tab);
        if (adj_kept(g, g1)) l.store(steps + adj_slot(g, g0) * 6 * N, N, n);
      }
    }
    for (int64_t g = g1 - 1; g >= g0; --g) {
      // state after step g: kept, or rebuilt by the inverse of step g + 1
      if (adj_kept(g, g1)) l.load(steps + adj_slot(g, g0) * 6 * N, N, n);
      l.source(c);
      l.template rev<FORM, EPS0>(d, s_tab);
    }
  }
  l.template finish<EPS0>(d, n, c);
}

template <bool EPS0>
hipError_t launch_bwd(const AdjDesc &d, bool rev, int form, const Tuning &t, hipStream_t s) {
  return for_form(form, [&](auto f) {
    constexpr int F = decltype(f)::value;
    const bool two = two_lanes(t, d.N, n_cus());
    if (two && rev) launch_lanes(k_adj_bwd_rev<F, EPS0, TwoLanes>, 2 * d.N, d, t, s);
    else if (two) launch_lanes(k_adj_bwd<F, EPS0, TwoLanes>, 2 * d.N, d, t, s);
    else if (rev) launch_lanes(k_adj_bwd_rev<F, EPS0, OneLane>, d.N, d, t, s);
    else launch_lanes(k_adj_bwd<F, EPS0, OneLane>, d.N, d, t, s);
  });
}

}  // namespace

hipError_t launch_adj_forward(const AdjDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return for_form(form, [&](auto f) {
    constexpr int F = decltype(f)::value;
    if (two_lanes(t, d.N, n_cus())) launch_lanes(k_adj_fwd<F, TwoLanes>, 2 * d.N, d, t, s);
    else launch_lanes(k_adj_fwd<F, OneLane>, d.N, d, t, s);
  });
}

hipError_t launch_adj_backward_reversible(const AdjDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return d.eps == 0.0 ? launch_bwd<true>(d, true, form, t, s) : launch_bwd<false>(d, true, form, t, s);
}

hipError_t launch_adj_backward(const AdjDesc &d, int form, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  return d.eps == 0.0 ? launch_bwd<true>(d, false, form, t, s) : launch_bwd<false>(d, false, form, t, s);
}

}  // namespace aw
