// aw_launch.hpp -- host-side launchers of the kernels (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "aw_internal.hpp"

namespace aw {

struct Tuning {
  int block = 0;  // 0: automatic (block_for)
  int opl = 1;
  int unroll = 1;
  int renorm = 8;
  int pwgs = 0;
  int lpo = 0;    // lanes per orbit: 0 auto (two_lanes, fwd_two_lanes), 1 or 2
};

int n_cus();  // compute units of the current device

// Whether n orbits run on two lanes each: when asked for (lanes_per_orbit 2) or,
// by default, while every pair's wave has a SIMD of its own.  200 S6 steps in us,
// one lane and two: 32768 orbits 238 and 211 (188 and 148 without the tangent);
// past that two waves share a SIMD, 33000 orbits 234 and 333 (187 and 237).  The
// gradient of J, 16384 orbits 464 and 378, 32761 466 and 404, 33000 458 and 594;
// of L, 16384 679 and 600, 32761 691 and 656, 33000 682 and 988.
inline bool two_lanes(const Tuning &t, int64_t n, int64_t cus) {
  return n > 0 && (t.lpo ? t.lpo == 2 : n <= cus * 4 * 32);
}

// The same for the propagation without the window test.  The pair kernel has one
// shape, so by default it does not take the place of a block, a number of orbits
// per lane or an unrolling that the caller asked for -- but for part, a
// tangent-free launch that ends before n_steps or bins a time window, whose
// automatic choice has always been made from n alone.
inline bool fwd_two_lanes(const Tuning &t, int64_t n, bool part, int64_t cus) {
  const bool shaped = t.block != 0 || t.opl != 1 || t.unroll != 1;
  return two_lanes(t, n, cus) && (t.lpo == 2 || part || !shaped);
}

// Lanes per block of the adjoint kernels for n lanes in all.  A block set in the
// tuning is used as is.  Automatic: 256, one wave per SIMD of a CU, while every
// CU holds at most one such block, else 512 (a block holds the 64 KB sine/cosine
// table, so two blocks share a CU, and it takes two of 512 lanes to fill it at
// four waves per SIMD).  Smaller blocks would spread over more CUs but share
// SIMDs when two land on one CU: the gradient of J for 40000 orbits over 200
// steps takes 472 us in blocks of 256 and took 780 in blocks of 128, for 257 orbits
// 511 and 524 in blocks of 64.  No result depends on the block.
int block_for(const Tuning &t, int64_t n);

inline int block_512(const Tuning &t) { return t.block ? t.block : 512; }

// Propagation.
hipError_t launch_fwd(const FwdDesc &d, const Tuning &t, int form, bool tan, hipStream_t s);
// descs sorted by their step counts, longest first; ends[e]: tiles of 64 opl
// orbits in descs[0..e].  n_wg = 0 clears the counters only.
hipError_t launch_fwd_batched(const FwdDesc *descs_dev, const int64_t *ends_dev, int32_t n_descs,
                              unsigned long long *head_dev, const Tuning &t, int form, bool tan, int n_wg,
                              hipStream_t s);
int persistent_blocks_per_cu(int form, bool tan, const Tuning &t);
hipError_t launch_gen_ic(const FwdDesc &d, double *ic, double *w0, hipStream_t s);
hipError_t launch_zero_u32(uint32_t *p, int32_t n, hipStream_t s);
void step_op_counts(int form, bool tan, int64_t *fma, int64_t *mul, int64_t *add);

// Histogram reduction.
struct HistPlan {
  int W = 0, H = 0, tiles_x = 0, n_tiles = 0;
  int32_t G = 0;
  int64_t chunk = 0;       // items per accumulation chunk
  int64_t max_chunks = 0;  // accumulation workgroups launched: n_tiles + ceil(N / chunk)
};
struct HistKeys {
  const double *a = nullptr, *b = nullptr;
  double lo0 = 0, hi0 = 0, lo1 = 0, hi1 = 0;
  int32_t closed = 0;  // the upper edges belong to the last bins
};
struct HistScratch {
  uint32_t *block_counts = nullptr;
  uint32_t *block_dropped = nullptr;
  uint32_t *tile_start = nullptr;   // n_tiles + 1 entries
  uint32_t *tile_total = nullptr;   // n_tiles entries (in the same buffer, after tile_start)
  uint32_t *chunk_first = nullptr;  // n_tiles + 1: first chunk of each tile; [n_tiles] = chunks in all
  uint32_t *part_first = nullptr;   // n_tiles + 1: first partial-tile slot of each tile of several chunks
  uint32_t *chunk_tile = nullptr;   // the tile of each chunk
  uint32_t *part_counts = nullptr;  // [slots][TILE_BINS] partial counts
  double *part_sums = nullptr;      // [slots][TILE_BINS] partial sums (with values only)
  uint16_t *sorted_local = nullptr;
  double *sorted_val = nullptr;
};
HistPlan hist_plan(int64_t N, int W, int H);
hipError_t launch_vdir_keys(int64_t N, const double *V, double *phi, double *mu, hipStream_t s);
// Items by their bins, or by a caller's keys if keys != nullptr: bins is then
// scratch.  accumulate != 0: counts are added to counts_out instead of written.
hipError_t launch_hist_reduce(int64_t N, const HistKeys *keys, uint32_t *bins, const double *vals, const HistPlan &p,
                              const HistScratch &w, int mode, double norm, uint32_t *counts_out,
                              double *f_out, uint64_t *dropped_out, hipStream_t s, int accumulate = 0);

// Adjoint kernels: `lanes` lanes in blocks of block_for, and the call f(form) with
// the map form as a compile-time constant.
template <class D>
void launch_lanes(void (*kernel)(D), int64_t lanes, const D &d, const Tuning &t, hipStream_t s) {
  const int tb = block_for(t, lanes);
  hipLaunchKernelGGL(kernel, dim3((unsigned)((lanes + tb - 1) / tb)), dim3((unsigned)tb), 0, s, d);
}

template <class Fn>
hipError_t for_form(int form, Fn &&f) {
  switch (form) {
  case 1: f(std::integral_constant<int, 1>{}); break;
  case 2: f(std::integral_constant<int, 2>{}); break;
  case 4: f(std::integral_constant<int, 4>{}); break;
  case 6: f(std::integral_constant<int, 6>{}); break;
  case 7: f(std::integral_constant<int, 7>{}); break;
  default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_adj_forward(const AdjDesc &d, int form, const Tuning &t, hipStream_t s);
hipError_t launch_adj_backward(const AdjDesc &d, int form, const Tuning &t, hipStream_t s);
hipError_t launch_adj_backward_reversible(const AdjDesc &d, int form, const Tuning &t, hipStream_t s);

// Gradient of the tangent-growth indicator L: the adjoint descriptor, whose
// checkpoint and step buffers then hold 12 rows (state and tangent) per
// orbit, plus the tangent start, the upstream gradient and L.
struct FtleDesc : AdjDesc {
  const double *w0;  // [6][N]
  const double *gL;  // [N] or null (ones)
  double *L;         // [N] or null
  int16_t *exps;     // [floor(T/8)][N]: exponent of each tangent rescale
};
hipError_t launch_ftle_forward(const FtleDesc &d, int form, const Tuning &t, hipStream_t s);
hipError_t launch_ftle_backward(const FtleDesc &d, int form, const Tuning &t, hipStream_t s);
hipError_t launch_ftle_backward_reversible(const FtleDesc &d, int form, const Tuning &t, hipStream_t s);

}  // namespace aw
