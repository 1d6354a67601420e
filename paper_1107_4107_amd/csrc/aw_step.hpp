// aw_step.hpp -- one map step of the propagation and adjoint kernels.
#pragma once

#include "aw_device.hpp"
#include "aw_internal.hpp"

namespace aw {

// One map step: NK kicks, each preceded by a drift, and a closing drift
// (symmetric compositions), or kick-then-drift (coupled standard map).  The
// kicks take their sines and cosines from the block's LDS table `tab`.  OPL
// orbits are interleaved stage by stage.
template <int FORM, bool TAN, int OPL>
__device__ __forceinline__ void map_step(Orbit (&o)[OPL], const StepWeights &d, const double2 *__restrict__ tab) {
  using F = FormPattern<FORM>;
  constexpr int NK = F::NK;
  auto drift = [&](int q) {
#pragma unroll
    for (int j = 0; j < OPL; ++j) drift_node<TAN>(o[j], d.dnode[q], d.dnodez[q], d.drift[q]);
  };
  auto kick = [&](int q) {
#pragma unroll
    for (int j = 0; j < OPL; ++j) kick_node<TAN>(o[j], d.ka[q], d.kb[q], tab);
  };
  if constexpr (F::LEAD) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      drift(F::drift_idx[i]);
      kick(F::kick_idx[i]);
    }
    drift(F::drift_idx[NK]);
  } else {
    kick(0);
    drift(0);
  }
}

// Two lanes per orbit.  In the scaled frame neither the force nor its Jacobian
// couples u and v, so lane 2m of a pair holds u, p_u and their tangent, lane
// 2m + 1 holds v's, and both hold z's.  A kick takes one table sine and cosine of
// the lane's own coordinate and the z factors, swaps the cosine with the partner
// lane (cs = cos u + cos v is the same sum in both lanes: IEEE addition commutes),
// and advances the lane's own momenta and p_z; a drift advances the lane's
// coordinate and z.  The sums that round differently by order, such as
// sin u du + sin v dv, are formed in the even lane and handed to the odd one.
// Every value is formed and rounded as with one lane per orbit, so every result is
// the same bit for bit.

// Lanes 2m and 2m + 1 exchange v (DPP quad_perm [1, 0, 3, 2]), or both take lane
// 2m's (quad_perm [0, 0, 2, 2]).  A lane takes from its own pair only, whose lanes
// run the same orbit and leave together.
constexpr int DPP_SWAP = 0xB1, DPP_EVEN = 0xA0;

template <int CTRL>
__device__ __forceinline__ double dpp_pair(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

struct HalfOrbit {
  double w, pw;          // own coordinate (u or v, in nodes) and its momentum
  double z, pz;          // 2 z in nodes, sqrt 2 p_z
  double dw, dpw, dz, dpz;  // their tangent
  double p0w, p0z;
  double jsum;           // meaningful in the pair's even lane
  int kexp;
};

template <bool TAN>
__device__ __forceinline__ void pair_kick(HalfOrbit &h, double a, double b, const double2 *__restrict__ tab) {
  NodeSC sc[2];
  const double ang[2] = {h.w, h.z};
  sincos_nodes<2, true>(ang, sc, tab);
  const NodeSC W = sc[0], Z = sc[1];
  const double e1 = __builtin_fma(a, Z.c, a);
  const double e2 = b * Z.s;
  const double cs = W.c + dpp_pair<DPP_SWAP>(W.c);
  if (TAN) {
    const double f = e1 * h.dw, q = e2 * h.dz;
    const double g = dpp_pair<DPP_EVEN>(__builtin_fma(W.s, h.dw, dpp_pair<DPP_SWAP>(W.s * h.dw)));
    const double mz = cs * __builtin_fma(2.0, e1, -2.0 * a);
    h.dpw = __builtin_fma(W.c, f, __builtin_fma(-W.s, q, h.dpw));
    h.dpz = __builtin_fma(mz, h.dz, __builtin_fma(-e2, g, h.dpz));
  }
  h.pw = __builtin_fma(e1, W.s, h.pw);
  h.pz = __builtin_fma(e2, cs, h.pz);
}

template <bool TAN>
__device__ __forceinline__ void pair_drift(HalfOrbit &h, double wu, double wz, double t) {
  h.w = __builtin_fma(wu, h.pw, h.w);
  h.z = __builtin_fma(wz, h.pz, h.z);
  if (TAN) {
    h.dw = __builtin_fma(t, h.dpw, h.dw);
    h.dz = __builtin_fma(t, h.dpz, h.dz);
  }
}

template <int FORM, bool TAN>
__device__ __forceinline__ void pair_step(HalfOrbit &h, const StepWeights &d, const double2 *__restrict__ tab) {
  using F = FormPattern<FORM>;
  constexpr int NK = F::NK;
  auto drift = [&](int q) { pair_drift<TAN>(h, d.dnode[q], d.dnodez[q], d.drift[q]); };
  auto kick = [&](int q) { pair_kick<TAN>(h, d.ka[q], d.kb[q], tab); };
  if constexpr (F::LEAD) {
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      drift(F::drift_idx[i]);
      kick(F::kick_idx[i]);
    }
    drift(F::drift_idx[NK]);
  } else {
    kick(0);
    drift(0);
  }
}

// J as accum_j_node accumulates it, in the even lane: the u, v and z squares in
// that order.
__device__ __forceinline__ void pair_accum_j(HalfOrbit &h) {
  const double e = h.pw - h.p0w;
  const double ep = dpp_pair<DPP_SWAP>(e);
  const double ez = h.pz - h.p0z;
  h.jsum = __builtin_fma(e, e, h.jsum);
  h.jsum = __builtin_fma(ep, ep, h.jsum);
  h.jsum = __builtin_fma(ez, ez, h.jsum);
}

// The sum of the tangent's six squares (renorm_node's order, formed in the even
// lane), and the power-of-two exponent renorm_node takes from it.
__device__ __forceinline__ double pair_tan_sum2(const HalfOrbit &h) {
  const double dv = dpp_pair<DPP_SWAP>(h.dw), dpv = dpp_pair<DPP_SWAP>(h.dpw);
  double a = h.dw * h.dw;
  a = __builtin_fma(dv, dv, a);
  a = __builtin_fma(h.dz, h.dz, a);
  a = __builtin_fma(h.dpw, h.dpw, a);
  a = __builtin_fma(dpv, dpv, a);
  return dpp_pair<DPP_EVEN>(__builtin_fma(h.dpz, h.dpz, a));
}

__device__ __forceinline__ int pair_rescale_exponent(const HalfOrbit &h) {
  return (__builtin_amdgcn_frexp_exp(pair_tan_sum2(h)) - 1) >> 1;
}

__device__ __forceinline__ void pair_rescale(HalfOrbit &h, int s) {
  h.dw = __builtin_amdgcn_ldexp(h.dw, -s);
  h.dz = __builtin_amdgcn_ldexp(h.dz, -s);
  h.dpw = __builtin_amdgcn_ldexp(h.dpw, -s);
  h.dpz = __builtin_amdgcn_ldexp(h.dpz, -s);
  h.kexp += s;
}

}  // namespace aw
