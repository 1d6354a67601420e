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

}  // namespace aw
