// aw_fwd.hip -- ensemble propagation kernels (gfx950, FP64).
//
// One orbit per lane (or two, interleaved, for instruction-level
// parallelism; or, for small ensembles, one orbit on two lanes);
// the state, the tangent vector and the accumulators stay in
// VGPRs for the whole run; initial conditions are generated in registers from
// the ensemble descriptor, so the only HBM traffic is the coalesced
// structure-of-arrays store of the per-orbit results (and of the resumable
// carry when a run is split into several launches).
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "aw_device.hpp"
#include "aw_internal.hpp"
#include "aw_launch.hpp"
#include "aw_step.hpp"

namespace aw {

// ---------------------------------------------------------------------------
// Initial conditions and tangent start.  GRID2, BOX, EXPLICIT and the tangent
// start use exact or correctly rounded operations only, so the values are
// bitwise those of any IEEE implementation of the same formulas; SPHERE also
// takes a cosine, a sine and Hp(X), so it agrees to a few ulps.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void gen_ic(const FwdDesc &d, int64_t n, double s[6]) {
#pragma clang fp contract(off)
  if (d.ic_kind == 0) {
    const int64_t i = n % d.nx, j = n / d.nx;
    const double v0 = d.lo0 + (double)i * d.d0;
    const double v1 = d.lo1 + (double)j * d.d1;
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = (k == d.ax0) ? v0 : ((k == d.ax1) ? v1 : d.base[k]);
  } else if (d.ic_kind == 1) {
#pragma unroll
    for (int k = 0; k < 6; ++k)
      s[k] = d.box_lo[k] + d.box_span[k] * u01(d.seed_ic, 16ull * (uint64_t)n + (uint64_t)k);
  } else if (d.ic_kind == 3) {
    // Fixed energy: X on the torus, direction uniform in area on the (phi, mu)
    // segment, |P| from H(P, X) = E.
    const uint64_t c = 16ull * (uint64_t)n;
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = d.box_lo[k] + d.box_span[k] * u01(d.seed_ic, c + (uint64_t)k);
    const double mu = d.win[2] + (d.win[3] - d.win[2]) * u01(d.seed_ic, c + 3ull);
    const double phi = d.win[0] + (d.win[1] - d.win[0]) * u01(d.seed_ic, c + 4ull);
    const double st = sqrt(1.0 - mu * mu);
    const double p = sqrt(2.0 * (d.energy - d.eps * hp_value(s[0], s[1], s[2])));
    double sp, cp;
    sincos_full(phi, sp, cp);
    s[3] = p * st * cp;
    s[4] = p * st * sp;
    s[5] = p * mu;
  } else if (d.ic_kind == 4) {
    // Fig. 4 cloud: Gaussian (vx, vy) by Box-Muller, X on the torus by
    // rejection until the energy condition leaves a real vz.
    const uint64_t c = 128ull * (uint64_t)n;
    const double u1 = u01(d.seed_ic, c + 120ull), u2 = u01(d.seed_ic, c + 121ull);
    const double rr = sqrt(-2.0 * log(1.0 - u1));
    double sg, cg;
    sincos_full(2.0 * M_PI * u2, sg, cg);
    const double vx = d.cloud[0] + d.cloud[2] * (rr * cg);
    const double vy = d.cloud[1] + d.cloud[3] * (rr * sg);
    double R = -1.0;
    for (int a = 0; a < 40 && R < 0.0; ++a) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        s[k] = d.box_lo[k] + d.box_span[k] * u01(d.seed_ic, c + 3ull * (uint64_t)a + (uint64_t)k);
      R = 2.0 * (d.energy - d.eps * hp_value(s[0], s[1], s[2])) - vx * vx - vy * vy;
    }
    const double vz = sqrt(R > 0.0 ? R : 0.0);
    s[3] = vx;
    s[4] = vy;
    s[5] = u01(d.seed_ic, c + 122ull) < 0.5 ? -vz : vz;
  } else {
#pragma unroll
    for (int k = 0; k < 6; ++k) s[k] = d.ic[k * d.N + n];
  }
}

__device__ __forceinline__ void gen_w0(uint64_t seed, int64_t n, double w[6]) {
#pragma clang fp contract(off)
  double u[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) u[k] = 2.0 * u01(seed, 16ull * (uint64_t)n + (uint64_t)k) - 1.0;
  double n2 = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) n2 = n2 + u[k] * u[k];
  const double nu = sqrt(n2);
#pragma unroll
  for (int k = 0; k < 6; ++k) w[k] = u[k] / nu;
}

// Select row r of the nine per-orbit results by masking bit patterns.  A
// chain of selects over the array's elements is folded by the optimizer into
// one load at a selected offset, which keeps the array in memory (private
// scratch, or LDS sized for the whole block); AND/OR of the bits leaves
// nothing to fold.
__device__ __forceinline__ double pick9(const double (&v)[9], int r) {
  uint64_t o = 0;
#pragma unroll
  for (int k = 0; k < 9; ++k) o |= (uint64_t)__double_as_longlong(v[k]) & (0ull - (uint64_t)(r == k));
  return __longlong_as_double((long long)o);
}

__device__ __forceinline__ uint32_t bin_of(double a, double b, double lo0, double hi0, double lo1,
                                           double hi1, int W, int H, bool closed) {
#pragma clang fp contract(off)
  if (!isfinite(a) || !isfinite(b)) return BIN_DROP;
  double fi = floor((a - lo0) / (hi0 - lo0) * (double)W);
  double fj = floor((b - lo1) / (hi1 - lo1) * (double)H);
  if (closed) {
    if (fi == (double)W && a == hi0) fi = (double)(W - 1);
    if (fj == (double)H && b == hi1) fj = (double)(H - 1);
  }
  if (!(fi >= 0.0) || fi >= (double)W || !(fj >= 0.0) || fj >= (double)H) return BIN_DROP;
  return (uint32_t)fj * (uint32_t)W + (uint32_t)fi;
}

__device__ __forceinline__ void vdir_key(double vx, double vy, double vz, double &phi, double &mu) {
#pragma clang fp contract(off)
  const double r = sqrt(vx * vx + vy * vy + vz * vz);
  if (r == 0.0) {
    phi = __builtin_nan("");
    mu = __builtin_nan("");
    return;
  }
  phi = atan2(vy, vx);
  mu = vz / r;
}

constexpr double LN2 = 0x1.62e42fefa39efp-1;

// Is the direction of P inside the closed window phi in [phi_lo, phi_hi],
// mu = pz/|P| in [mu_lo, mu_hi]?  The phi test uses half-plane (cross
// product) tests against the edge directions e0, e1 instead of atan2: for a
// window of width w <= pi, phi is inside iff e0 x d >= 0 and d x e1 >= 0; for
// w > pi, iff d is not strictly inside the complementary sector.
__device__ __forceinline__ bool in_phi(double px, double py, const FwdDesc &d) {
#pragma clang fp contract(off)
  if (d.win_phi == 0) return true;
  const double c0 = d.e0x * py - d.e0y * px;   // e0 x d
  const double c1 = px * d.e1y - py * d.e1x;   // d x e1
  return d.win_phi == 1 ? (c0 >= 0.0 && c1 >= 0.0) : !(c0 < 0.0 && c1 < 0.0);
}

// The initial momentum, as it was given.
__device__ __forceinline__ bool in_window0(double px, double py, double pz, const FwdDesc &d) {
#pragma clang fp contract(off)
  bool ok = in_phi(px, py, d);
  if (d.win_mu != 0) {
    const double r = sqrt(px * px + py * py + pz * pz);
    ok = ok && pz >= d.win[2] * r && pz <= d.win[3] * r;
  }
  return ok;
}

// After a step, on the scaled momenta (p_u, p_v, sqrt 2 p_z), whose squares add
// up to 2 |P|^2; the phi test takes 2 P.  The mu test compares p |p| against
// mu |mu| times the sum of squares, which needs no square root: the whole test
// is 14 FP64 instructions where the rotated-back momentum, its norm and their
// products took about 100.  The squares of a momentum that lies on an edge, or
// within the rounding of in_window0, come out up to 17 half-ulps beyond it;
// the edges' squares are moved out by 32, so that a momentum which does not
// change stays in.
__device__ __forceinline__ bool in_window(double pu, double pv, double pz, const FwdDesc &d) {
#pragma clang fp contract(off)
  bool ok = in_phi(pu + pv, pu - pv, d);
  if (d.win_mu != 0) {
    const double r2 = __builtin_fma(pu, pu, __builtin_fma(pv, pv, pz * pz));
    const double q = pz * fabs(pz);
    ok = ok && q >= d.mu2_lo * r2 && q <= d.mu2_hi * r2;
  }
  return ok;
}

// Row 21 of the resumable carry: whether the orbit has left the window, and
// whether rows 0-20 hold the scaled frame.  A carry without the second flag
// was written in the unscaled rotated frame (u, v, z and their momenta, z and
// p_z not scaled) and is taken over.
constexpr int CARRY_LEFT = 1, CARRY_NODES = 2;

__device__ __forceinline__ void carry_to_nodes(Orbit &o) {
  o.x = to_nodes(o.x);
  o.y = to_nodes(o.y);
  o.z = to_nodes(2.0 * o.z);
  o.pz = times_sqrt2(o.pz);
  o.p0z = times_sqrt2(o.p0z);
  o.dz = times_sqrt2(o.dz);
  o.dpz = times_sqrt2(o.dpz);
}

// The descriptor a kernel was launched with, read where it lies in the kernel
// arguments (it is the first one), and any descriptor read anew: what follows
// the step loop loads its fields again instead of holding them in scalar
// registers across the loop, where they would push the stage weights out into
// vector lanes (24 v_readlane and 8 v_writelane per step with the window test).
typedef const __attribute__((address_space(4))) FwdDesc *ConstDesc;

__device__ __forceinline__ const FwdDesc &launched_desc() {
  return *(const FwdDesc *)(ConstDesc)__builtin_amdgcn_kernarg_segment_ptr();
}

__device__ __forceinline__ const FwdDesc &reread(const FwdDesc &d) {
  uint64_t p = (uint64_t)(uintptr_t)&d;
  asm volatile("" : "+s"(p));
  return *(const FwdDesc *)(ConstDesc)p;
}

// After the step loop: the resumable carry of an intermediate launch (or a
// time window), or the outputs of the final one.
template <bool TAN, int OPL, bool WINV>
__device__ __forceinline__ void finish_orbits(const FwdDesc &d, Orbit (&o)[OPL], const int64_t (&n)[OPL],
                                              const bool (&act)[OPL], const bool (&left)[OPL],
                                              const double (&xs)[OPL], const double (&ys)[OPL],
                                              const double (&zs)[OPL], int64_t k0, int64_t k1) {
  if (k1 < d.T || WINV) {
    // Intermediate launch (or a time window): store the resumable carry.
#pragma unroll
    for (int j = 0; j < OPL; ++j) {
      if (!act[j]) continue;
      if (WINV) {
#pragma clang fp contract(off)
        double phi, mu;
        const double du = (o[j].x - xs[j]) * AW_RAD_PER_NODE, dv = (o[j].y - ys[j]) * AW_RAD_PER_NODE;
        const double dz = (o[j].z - zs[j]) * (0.5 * AW_RAD_PER_NODE);
        vdir_key(0.5 * (du + dv) / d.wdt, 0.5 * (du - dv) / d.wdt, dz / d.wdt, phi, mu);
        d.bins[n[j]] = left[j] ? BIN_DROP : bin_of(phi, mu, d.klo0, d.khi0, d.klo1, d.khi1, d.W, d.H, true);
      }
      double *c = d.carry;
      const int64_t N = d.N, m = n[j];
      if (k0 == 0) {  // what the steps do not change
        double s0[6];
        gen_ic(d, m, s0);
        c[12 * N + m] = s0[0]; c[13 * N + m] = s0[1]; c[14 * N + m] = s0[2];
      }
      c[0 * N + m] = o[j].x; c[1 * N + m] = o[j].y; c[2 * N + m] = o[j].z;
      c[3 * N + m] = o[j].px; c[4 * N + m] = o[j].py; c[5 * N + m] = o[j].pz;
      c[6 * N + m] = o[j].dx; c[7 * N + m] = o[j].dy; c[8 * N + m] = o[j].dz;
      c[9 * N + m] = o[j].dpx; c[10 * N + m] = o[j].dpy; c[11 * N + m] = o[j].dpz;
      c[15 * N + m] = o[j].p0x; c[16 * N + m] = o[j].p0y; c[17 * N + m] = o[j].p0z;
      c[18 * N + m] = o[j].jsum;
      c[19 * N + m] = (double)o[j].kexp;
      c[20 * N + m] = (double)k1;
      c[21 * N + m] = (double)(CARRY_NODES | (left[j] ? CARRY_LEFT : 0));
    }
    return;
  }

  // Final launch: per-orbit observables.  Contraction is off so that every
  // kernel variant rounds the sums of products below (L, dP^2, the energies)
  // the same way: whether the compiler fuses a*b + c depends on the code
  // around it, and the results are to be bitwise independent of the launch
  // shape and of batching.
  uint32_t n_chaotic = 0;
#pragma unroll
  for (int j = 0; j < OPL; ++j) {
#pragma clang fp contract(off)
    const int64_t N = d.N, m = n[j];
    double s0[6];
    gen_ic(d, m, s0);
    from_node(o[j], s0);
    double res[9];
    double wn = 1.0;
    if (TAN) {
      double n2 = o[j].dx * o[j].dx;
      n2 = __builtin_fma(o[j].dy, o[j].dy, n2);
      n2 = __builtin_fma(o[j].dz, o[j].dz, n2);
      n2 = __builtin_fma(o[j].dpx, o[j].dpx, n2);
      n2 = __builtin_fma(o[j].dpy, o[j].dpy, n2);
      n2 = __builtin_fma(o[j].dpz, o[j].dpz, n2);
      const int e = __builtin_amdgcn_frexp_exp(n2);
      const double mant = __builtin_amdgcn_frexp_mant(n2);
      const double L = 0.5 * ((double)(2 * o[j].kexp + e) * LN2 + log(mant));
      res[0] = L;
      res[1] = L / d.th;
      res[2] = L / d.lth;
      wn = sqrt(n2);
    } else {
      res[0] = res[1] = res[2] = __builtin_nan("");
    }
    res[3] = (o[j].x - s0[0]) / d.th;
    res[4] = (o[j].y - s0[1]) / d.th;
    res[5] = (o[j].z - s0[2]) / d.th;
    const double ex = o[j].px - s0[3], ey = o[j].py - s0[4], ez = o[j].pz - s0[5];
    res[6] = ex * ex + ey * ey + ez * ez;
    res[7] = (0.5 * o[j].jsum) / (double)d.T;
    const double E1 = 0.5 * (o[j].px * o[j].px + o[j].py * o[j].py + o[j].pz * o[j].pz) +
                      d.eps * hp_value(o[j].x, o[j].y, o[j].z);
    const double E0 = 0.5 * (s0[3] * s0[3] + s0[4] * s0[4] + s0[5] * s0[5]) +
                      d.eps * hp_value(s0[0], s0[1], s0[2]);
    res[8] = E1 - E0;
    const bool chaotic = TAN && (res[2] > d.chi_thr);
    n_chaotic += (uint32_t)__popcll(__ballot(act[j] && chaotic));
    if (!act[j]) continue;
    if (d.out) {
      double *out = d.out;
      out[0 * N + m] = res[0]; out[1 * N + m] = res[1]; out[2 * N + m] = res[2];
      out[3 * N + m] = res[3]; out[4 * N + m] = res[4]; out[5 * N + m] = res[5];
      out[6 * N + m] = res[6]; out[7 * N + m] = res[7]; out[8 * N + m] = res[8];
    }
    if (d.state) {
      double *st = d.state;
      st[0 * N + m] = o[j].x; st[1 * N + m] = o[j].y; st[2 * N + m] = o[j].z;
      st[3 * N + m] = o[j].px; st[4 * N + m] = o[j].py; st[5 * N + m] = o[j].pz;
      st[6 * N + m] = o[j].dx / wn; st[7 * N + m] = o[j].dy / wn; st[8 * N + m] = o[j].dz / wn;
      st[9 * N + m] = o[j].dpx / wn; st[10 * N + m] = o[j].dpy / wn; st[11 * N + m] = o[j].dpz / wn;
    }
    if (d.cls) d.cls[m] = (uint8_t)((chaotic ? 1 : 0) | (left[j] ? 2 : 0));
    if (d.epi == EPI_IC_GRID) {
      d.img[m] = pick9(res, d.field);
    } else if (d.epi == EPI_HIST_P0) {
      double a = s0[0], b = s0[0];
#pragma unroll
      for (int k = 1; k < 6; ++k) {
        a = (d.key0 == k) ? s0[k] : a;
        b = (d.key1 == k) ? s0[k] : b;
      }
      d.bins[m] = left[j] ? BIN_DROP : bin_of(a, b, d.klo0, d.khi0, d.klo1, d.khi1, d.W, d.H, false);
      d.vals[m] = pick9(res, d.field);
    } else if (d.epi == EPI_HIST_VDIR) {
      double phi, mu;
      vdir_key(res[3], res[4], res[5], phi, mu);
      d.bins[m] = left[j] ? BIN_DROP : bin_of(phi, mu, d.klo0, d.khi0, d.klo1, d.khi1, d.W, d.H, true);
    }
  }
  // Class count of the IC-grid image: one ballot and popcount per wave and
  // slot (above), one atomic per wave from its lowest active lane.
  if (d.epi == EPI_IC_GRID && d.n_class != nullptr && TAN) {
    const uint64_t active = __ballot(1);
    if ((int)__lane_id() == __ffsll((unsigned long long)active) - 1 && n_chaotic != 0)
      atomicAdd(d.n_class, n_chaotic);
  }
}

// Orbit m at step k_begin in the scaled frame: its initial state, or the
// carry as the loop left it.
template <bool TAN, bool FILT>
__device__ __forceinline__ void start_orbit(const FwdDesc &d, int64_t m, Orbit &o, bool &left) {
  left = false;
  if (d.k_begin == 0) {
    double s[6];
    gen_ic(d, m, s);
    o.x = s[0]; o.y = s[1]; o.z = s[2];
    o.px = s[3]; o.py = s[4]; o.pz = s[5];
    o.p0x = s[3]; o.p0y = s[4]; o.p0z = s[5];
    o.jsum = 0.0;
    o.kexp = 0;
    if (TAN) {
      double w[6];
      gen_w0(d.seed_tan, m, w);
      o.dx = w[0]; o.dy = w[1]; o.dz = w[2];
      o.dpx = w[3]; o.dpy = w[4]; o.dpz = w[5];
    } else {
      o.dx = o.dy = o.dz = o.dpx = o.dpy = o.dpz = 0.0;
    }
    if (FILT) left = !in_window0(s[3], s[4], s[5], d);
    to_node(o);
  } else {
    const double *c = d.carry;
    const int64_t N = d.N;
    const int flags = (int)c[21 * N + m];
    o.x = c[0 * N + m]; o.y = c[1 * N + m]; o.z = c[2 * N + m];
    o.px = c[3 * N + m]; o.py = c[4 * N + m]; o.pz = c[5 * N + m];
    o.dx = c[6 * N + m]; o.dy = c[7 * N + m]; o.dz = c[8 * N + m];
    o.dpx = c[9 * N + m]; o.dpy = c[10 * N + m]; o.dpz = c[11 * N + m];
    o.p0x = c[15 * N + m]; o.p0y = c[16 * N + m]; o.p0z = c[17 * N + m];
    o.jsum = c[18 * N + m];
    o.kexp = (int)c[19 * N + m];
    if (FILT) left = (flags & CARRY_LEFT) != 0;
    if (!(flags & CARRY_NODES)) carry_to_nodes(o);
  }
}

// ---------------------------------------------------------------------------
// Run one wave's tile of 64 OPL orbits, (tile OPL + j) 64 + lane for j < OPL,
// over global steps [k_begin, k_end).  FILT: test the window after every step.
// `tab` is the block's LDS copy of the sine/cosine table (filled by the caller).
// ---------------------------------------------------------------------------
template <int FORM, bool TAN, int OPL, int UNR, bool FILT = false, bool WINV = false>
__device__ __forceinline__ void run_orbits(const FwdDesc &d, int64_t tile, const double2 *__restrict__ tab) {
  int64_t n[OPL];
  bool act[OPL];
#pragma unroll
  for (int j = 0; j < OPL; ++j) {
    const int64_t m = (tile * OPL + j) * 64 + (int)__lane_id();
    act[j] = m < d.N;
    n[j] = act[j] ? m : d.N - 1;  // inactive slots repeat a valid orbit, never stored
  }
  if (tile * 64 * OPL >= d.N || !act[0]) return;

  Orbit o[OPL];
  bool left[OPL];
#pragma unroll
  for (int j = 0; j < OPL; ++j) {
    start_orbit<TAN, FILT>(d, n[j], o[j], left[j]);
  }

  // Positions at the start of this launch (time-window velocity; scaled frame).
  double xs[OPL], ys[OPL], zs[OPL];
  if (WINV) {
#pragma unroll
    for (int j = 0; j < OPL; ++j) {
      xs[j] = o[j].x;
      ys[j] = o[j].y;
      zs[j] = o[j].z;
    }
  }

  // Hot loop.  The trip count and the renormalisation test are uniform.
  // UNR = 2 runs steps in pairs plus a one-step tail, written out: the table
  // offset is inline assembly, which the compiler treats as convergent and
  // will not unroll with a remainder.
  const int64_t k0 = d.k_begin, k1 = d.k_end;
  const int64_t mask = d.renorm_mask;
  // Stage weights.  In the plain tangent kernel they move into VGPRs (an empty
  // asm the compiler must treat as producing per-lane values): left in SGPRs,
  // which the epilogue's descriptor fields hold across the loop, they are
  // spilled and read back every step.  A block of 512 leaves 256 VGPRs a lane.
  // The unrolled, two-orbit and window variants would lose occupancy and keep
  // them in SGPRs.
  constexpr bool kVregW = TAN && OPL == 1 && UNR == 1 && !FILT && !WINV;
  StepWeights sw = d.w;
  if (kVregW) {
#pragma unroll
    for (int q = 0; q < MAX_UNIQUE; ++q)
      asm volatile("" : "+v"(sw.drift[q]), "+v"(sw.dnode[q]), "+v"(sw.dnodez[q]), "+v"(sw.ka[q]), "+v"(sw.kb[q]));
  }
  auto one_step = [&](int64_t k) {
    map_step<FORM, TAN, OPL>(o, sw, tab);
#pragma unroll
    for (int j = 0; j < OPL; ++j) accum_j_node(o[j]);
    if (FILT) {
#pragma unroll
      for (int j = 0; j < OPL; ++j) left[j] = left[j] || !in_window(o[j].px, o[j].py, o[j].pz, d);
    }
    if (TAN && ((k + 1) & mask) == 0) {
#pragma unroll
      for (int j = 0; j < OPL; ++j) renorm_node(o[j]);
    }
  };
  int64_t k = k0;
  if (UNR == 2) {
#pragma nounroll
    for (; k + 1 < k1; k += 2) {
      one_step(k);
      one_step(k + 1);
    }
  }
#pragma nounroll
  for (; k < k1; ++k) one_step(k);

  finish_orbits<TAN, OPL, WINV>(reread(d), o, n, act, left, xs, ys, zs, k0, k1);
}

// A wave runs one tile of 64 OPL orbits; a block's waves share only the 64 KB
// table.  The first full_blocks blocks, whole rounds of what the chip holds at
// once, run nw consecutive tiles each.  The tiles of the last, partial round
// are dealt one to a block in turn over as many blocks as there are CUs (or
// slots), so that they spread over the CUs' SIMDs instead of filling a few CUs
// while the others idle.
__device__ __forceinline__ int64_t tile_of_wave(int64_t full_blocks) {
  const int64_t nw = blockDim.x >> 6, b = blockIdx.x;
  const int64_t wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return b < full_blocks ? b * nw + wave : full_blocks * nw + wave * (gridDim.x - full_blocks) + (b - full_blocks);
}

// Without the tangent two blocks of 512 share a CU at up to 128 VGPRs, four
// waves per SIMD; with it, or with two orbits per lane, a wave may take 256, one
// block and two waves per SIMD, which issue 97% of the slots.  300007 orbits in
// chunks of 100 steps took 2.05 ms with the last round in whole blocks and take
// 1.79 now, 1e6 orbits x 400 steps 7.45 and 7.21 ms.
constexpr bool two_blocks(bool tan, int opl) { return !tan && opl == 1; }

template <int FORM, bool TAN, int OPL, int UNR, bool FILT = false, bool WINV = false>
__global__ __launch_bounds__(512, two_blocks(TAN, OPL) ? 4 : 2) void k_fwd(FwdDesc, int64_t full_blocks) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  run_orbits<FORM, TAN, OPL, UNR, FILT, WINV>(launched_desc(), tile_of_wave(full_blocks), s_tab);
}

// ---------------------------------------------------------------------------
// Two lanes per orbit (pair_step), for ensembles too small to give every SIMD a
// wave at one lane per orbit (Fig. 4's 3.2e4 orbits make 500 waves for 1024
// SIMDs).  The window test runs one lane per orbit.
// A lone wave is bound by its own issue and by the chain of its kicks, ten
// dependent operations and a table read each.  An S6 step is 454 VALU instructions
// instead of 563 with the tangent, 307 instead of 415 without: 4096 orbits over
// 200 steps take 197 us instead of 235, and 134 instead of 184.
// ---------------------------------------------------------------------------
template <int FORM, bool TAN, bool WINV>
__global__ __launch_bounds__(512, 2) void k_fwd_pair(FwdDesc, int64_t full_blocks) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const FwdDesc &d = launched_desc();
  const int64_t tile = tile_of_wave(full_blocks);   // of 32 orbits
  if (tile * 32 >= d.N) return;
  const int64_t m = tile * 32 + ((int)__lane_id() >> 1);
  const bool odd = (threadIdx.x & 1u) != 0;
  const int64_t n[1] = {m < d.N ? m : d.N - 1};     // past the end: repeat a valid orbit, never stored
  const bool act[1] = {m < d.N && !odd};            // the even lane stores the orbit
  Orbit o[1];
  bool left[1];
  start_orbit<TAN, false>(d, n[0], o[0], left[0]);
  const double xs[1] = {o[0].x}, ys[1] = {o[0].y}, zs[1] = {o[0].z};
  HalfOrbit h;
  h.w = odd ? o[0].y : o[0].x;
  h.pw = odd ? o[0].py : o[0].px;
  h.z = o[0].z;
  h.pz = o[0].pz;
  h.dw = odd ? o[0].dy : o[0].dx;
  h.dpw = odd ? o[0].dpy : o[0].dpx;
  h.dz = o[0].dz;
  h.dpz = o[0].dpz;
  h.p0w = odd ? o[0].p0y : o[0].p0x;
  h.p0z = o[0].p0z;
  h.jsum = o[0].jsum;
  h.kexp = o[0].kexp;
  const StepWeights sw = d.w;
  const int64_t k0 = d.k_begin, k1 = d.k_end, mask = d.renorm_mask;
#pragma nounroll
  for (int64_t k = k0; k < k1; ++k) {
    pair_step<FORM, TAN>(h, sw, s_tab);
    pair_accum_j(h);
    if (TAN && ((k + 1) & mask) == 0) pair_rescale(h, pair_rescale_exponent(h));
  }
  // The whole orbit again, as the even lane stores it.
  o[0].x = h.w;
  o[0].y = dpp_pair<DPP_SWAP>(h.w);
  o[0].z = h.z;
  o[0].px = h.pw;
  o[0].py = dpp_pair<DPP_SWAP>(h.pw);
  o[0].pz = h.pz;
  o[0].dx = h.dw;
  o[0].dy = dpp_pair<DPP_SWAP>(h.dw);
  o[0].dz = h.dz;
  o[0].dpx = h.dpw;
  o[0].dpy = dpp_pair<DPP_SWAP>(h.dpw);
  o[0].dpz = h.dpz;
  o[0].p0x = h.p0w;
  o[0].p0y = dpp_pair<DPP_SWAP>(h.p0w);
  o[0].p0z = h.p0z;
  o[0].jsum = h.jsum;
  o[0].kexp = h.kexp;
  finish_orbits<TAN, 1, WINV>(reread(d), o, n, act, left, xs, ys, zs, k0, k1);
}

// Persistent batched propagation: every wave starts on a tile of 64 OPL orbits of
// its own, the first waves of all blocks before their second ones, and then takes
// the next tile from a device counter until the tiles of all ensembles, the longest
// runs first, are done.  descs[e] are sorted by their step counts, and
// ends[e] is the number of tiles of descs[0..e]; the tile's ensemble is found
// by bisection.  Waves share nothing but the table: a tile of the longest run
// keeps one wave and not the whole block from the next tile.  With the first tiles
// from the counter too the first blocks' waves took them all, two to a SIMD, and
// every take cost 11 ns on the one counter: 18 slices of up to 39 x 39 orbits over up to
// 579 steps took 1228 us and take 706, two of up to 300 x 300 over 900 steps of the
// standard map 83 and 59.
// Two orbits per lane take about 266 VGPRs; held to 256 (two waves per SIMD
// instead of one, the spills outside the step loop) the batch runs a fifth
// faster.  One orbit per lane without the tangent is held to 128, four waves per
// SIMD, and spills 72 VGPRs per tile, outside the step loop: two slices of 1024 x
// 1024 over 200 and 100 steps of the standard map take 595 us (613 at 256 VGPRs,
// without spills; 650 in blocks of 256 lanes that pulled tiles of 256), 200 slices
// of 40 x 40 152 (159; 197), 16 of up to 256 x 256 over up to 900 S6 steps 3.71 ms
// (3.40; 3.92).
template <int FORM, bool TAN, int OPL>
__global__ __launch_bounds__(512, (TAN || OPL > 1) ? 2 : 4) void k_fwd_persist(const FwdDesc *__restrict__ descs,
                                                                               const int64_t *__restrict__ ends,
                                                                               int32_t n_descs,
                                                                               unsigned long long *head) {
  __shared__ double2 s_tab[AW_TAB_N];
  load_sincos_table(s_tab);
  const int64_t n_tiles = ends[n_descs - 1], n_waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  int64_t t = (int64_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * gridDim.x + blockIdx.x;
  while (t < n_tiles) {
    int32_t lo = 0, hi = n_descs - 1;   // the first e with ends[e] > t
    while (lo < hi) {
      const int32_t mid = (lo + hi) >> 1;
      if (ends[mid] > t) hi = mid;
      else lo = mid + 1;
    }
    const int32_t e = __builtin_amdgcn_readfirstlane(lo);
    run_orbits<FORM, TAN, OPL, 1>(descs[e], t - (e > 0 ? ends[e - 1] : 0), s_tab);
    if (n_tiles <= n_waves) break;
    unsigned long long t0 = 0;
    if (__lane_id() == 0) t0 = atomicAdd(head, 1ull);
    t = n_waves + (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(t0 >> 32)) << 32) |
                            (uint32_t)__builtin_amdgcn_readfirstlane((int)t0));
  }
}

// Clears what a batched launch counts in: the queue's head and, for IC-grid
// images, every ensemble's counter of class-1 orbits.
__global__ void k_batch_clear(const FwdDesc *__restrict__ descs, int32_t n_descs, unsigned long long *head) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *head = 0ull;
  if (i < n_descs && descs[i].epi == EPI_IC_GRID && descs[i].n_class) *descs[i].n_class = 0u;
}

__global__ void k_zero_u32(uint32_t *p, int32_t n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0u;
}

__global__ void k_gen_ic(FwdDesc d, double *ic, double *w0) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= d.N) return;
  double s[6];
  if (ic) {
    gen_ic(d, n, s);
#pragma unroll
    for (int k = 0; k < 6; ++k) ic[k * d.N + n] = s[k];
  }
  if (w0) {
    gen_w0(d.seed_tan, n, s);
#pragma unroll
    for (int k = 0; k < 6; ++k) w0[k * d.N + n] = s[k];
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers.
// ---------------------------------------------------------------------------
int n_cus() {
  int dev = 0, ncu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
    ncu = 256;
  return ncu;
}

int block_for(const Tuning &t, int64_t n) {
  if (t.block) return t.block;
  return n <= (int64_t)n_cus() * 256 ? 256 : 512;
}

// The grid for n_tiles tiles, one per wave, in blocks of `lanes` lanes: whole
// rounds of the blocks the chip holds at once, then the rest (see
// tile_of_wave) four to a CU, one per SIMD, while there are CUs, then one more
// per SIMD, then over every slot.  A CU holds two blocks (the table), or one of
// 512 lanes where a wave may take 256 VGPRs.  Four waves on a CU run 6-8%
// faster than four waves on four CUs: the clock falls with the CUs in use.
struct TileGrid {
  int64_t full_blocks;
  unsigned blocks;
};

static TileGrid tile_grid(int64_t n_tiles, int lanes, bool two_of_512) {
  const int64_t ncu = n_cus(), nw = lanes >> 6, per = std::min<int64_t>(nw, 4);
  const int64_t slots = lanes < 512 || two_of_512 ? 2 * ncu : ncu;
  const int64_t full = n_tiles / (slots * nw) * slots, rest = n_tiles - full * nw;
  const int64_t tail = rest <= ncu * nw ? std::min(ncu, (rest + per - 1) / per) : slots;
  return {full, (unsigned)(full + tail)};
}

static bool use_pair(const FwdDesc &d, const Tuning &t, bool tan) {
  return !d.filter && fwd_two_lanes(t, d.N, !tan && (d.window_v || d.k_end < d.T), n_cus());
}

template <int FORM, bool TAN>
static hipError_t fwd_dispatch_opl(const FwdDesc &d, const Tuning &t, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  if (use_pair(d, t, TAN)) {
    const TileGrid g = tile_grid((d.N + 31) / 32, 512, false);
    if (d.window_v) hipLaunchKernelGGL((k_fwd_pair<FORM, TAN, true>), dim3(g.blocks), dim3(512), 0, s, d, g.full_blocks);
    else hipLaunchKernelGGL((k_fwd_pair<FORM, TAN, false>), dim3(g.blocks), dim3(512), 0, s, d, g.full_blocks);
    return hipGetLastError();
  }
  // The window test and the time-window velocity run with one orbit per lane
  // and no unrolling.
  const int opl = d.filter || d.window_v ? 1 : t.opl;
  const int lanes = block_512(t);
  const TileGrid g = tile_grid((d.N + 64 * opl - 1) / (64 * opl), lanes, two_blocks(TAN, opl));
  const dim3 grid(g.blocks), block((unsigned)lanes);
  const int64_t fb = g.full_blocks;
  if (d.filter && d.window_v) hipLaunchKernelGGL((k_fwd<FORM, TAN, 1, 1, true, true>), grid, block, 0, s, d, fb);
  else if (d.filter) hipLaunchKernelGGL((k_fwd<FORM, TAN, 1, 1, true, false>), grid, block, 0, s, d, fb);
  else if (d.window_v) hipLaunchKernelGGL((k_fwd<FORM, TAN, 1, 1, false, true>), grid, block, 0, s, d, fb);
  else if (opl == 1 && t.unroll == 1) hipLaunchKernelGGL((k_fwd<FORM, TAN, 1, 1>), grid, block, 0, s, d, fb);
  else if (opl == 1) hipLaunchKernelGGL((k_fwd<FORM, TAN, 1, 2>), grid, block, 0, s, d, fb);
  else if (t.unroll == 1) hipLaunchKernelGGL((k_fwd<FORM, TAN, 2, 1>), grid, block, 0, s, d, fb);
  else hipLaunchKernelGGL((k_fwd<FORM, TAN, 2, 2>), grid, block, 0, s, d, fb);
  return hipGetLastError();
}

hipError_t launch_fwd(const FwdDesc &d, const Tuning &t, int form, bool tan, hipStream_t s) {
  switch (form) {
  case 1: return tan ? fwd_dispatch_opl<1, true>(d, t, s) : fwd_dispatch_opl<1, false>(d, t, s);
  case 2: return tan ? fwd_dispatch_opl<2, true>(d, t, s) : fwd_dispatch_opl<2, false>(d, t, s);
  case 4: return tan ? fwd_dispatch_opl<4, true>(d, t, s) : fwd_dispatch_opl<4, false>(d, t, s);
  case 6: return tan ? fwd_dispatch_opl<6, true>(d, t, s) : fwd_dispatch_opl<6, false>(d, t, s);
  case 7: return tan ? fwd_dispatch_opl<7, true>(d, t, s) : fwd_dispatch_opl<7, false>(d, t, s);
  default: return hipErrorInvalidValue;
  }
}

template <int FORM, bool TAN>
static hipError_t persist_dispatch(const FwdDesc *descs, const int64_t *ends, int32_t n_descs,
                                   unsigned long long *head, const Tuning &t, int n_wg, hipStream_t s) {
  const dim3 grid((unsigned)n_wg), block((unsigned)block_512(t));
  if (t.opl == 1) hipLaunchKernelGGL((k_fwd_persist<FORM, TAN, 1>), grid, block, 0, s, descs, ends, n_descs, head);
  else hipLaunchKernelGGL((k_fwd_persist<FORM, TAN, 2>), grid, block, 0, s, descs, ends, n_descs, head);
  return hipGetLastError();
}

hipError_t launch_fwd_batched(const FwdDesc *descs, const int64_t *ends, int32_t n_descs, unsigned long long *head,
                              const Tuning &t, int form, bool tan, int n_wg, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_clear, dim3((unsigned)((n_descs + 255) / 256)), dim3(256), 0, s, descs, n_descs, head);
  if (n_wg <= 0) return hipGetLastError();
#define AW_PERSIST(F)                                                                      \
  case F: return tan ? persist_dispatch<F, true>(descs, ends, n_descs, head, t, n_wg, s)   \
                     : persist_dispatch<F, false>(descs, ends, n_descs, head, t, n_wg, s);
  switch (form) {
    AW_PERSIST(1) AW_PERSIST(2) AW_PERSIST(4) AW_PERSIST(6) AW_PERSIST(7)
  default: return hipErrorInvalidValue;
  }
#undef AW_PERSIST
}

int persistent_blocks_per_cu(int form, bool tan, const Tuning &t) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
#define AW_OCC(F)                                                                                 \
  if (form == F) {                                                                                \
    if (tan) e = t.opl == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd_persist<F, true, 1>, block_512(t), 0) \
                            : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd_persist<F, true, 2>, block_512(t), 0); \
    else e = t.opl == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd_persist<F, false, 1>, block_512(t), 0) \
                        : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_fwd_persist<F, false, 2>, block_512(t), 0); \
  }
  AW_OCC(1) AW_OCC(2) AW_OCC(4) AW_OCC(6) AW_OCC(7)
#undef AW_OCC
  return (e == hipSuccess && nb > 0) ? nb : 1;
}

hipError_t launch_gen_ic(const FwdDesc &d, double *ic, double *w0, hipStream_t s) {
  if (d.N <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((d.N + 255) / 256);
  hipLaunchKernelGGL(k_gen_ic, dim3(blocks), dim3(256), 0, s, d, ic, w0);
  return hipGetLastError();
}

hipError_t launch_zero_u32(uint32_t *p, int32_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

// FP64 operations per map step in the unscaled rotated frame, a fixed unit of
// work (amortised renormalisation excluded): a sincos takes 8 FMA, 4 MUL
// and 1 ADD, the z factors 9, 3 and 1, the rest of a kick 3, 2 and 1 and with
// the tangent 8 FMA and 6 MUL more; a drift 3 FMA, 6 with the tangent; the J
// accumulator 3 FMA and 4 ADD.  kick_node and drift_node take fewer.
void step_op_counts(int form, bool tan, int64_t *fma, int64_t *mul, int64_t *add) {
  int nk = 0, nd = 0;
  switch (form) {
  case 1: nk = 1; nd = 1; break;
  case 2: nk = 1; nd = 2; break;
  case 4: nk = 3; nd = 4; break;
  case 6: nk = 9; nd = 10; break;
  case 7: nk = 7; nd = 8; break;
  default: break;
  }
  const int kf = 2 * 8 + 9 + 3 + (tan ? 8 : 0);
  const int km = 2 * 4 + 3 + 2 + (tan ? 6 : 0);
  *fma = (int64_t)nk * kf + (int64_t)nd * (tan ? 6 : 3) + 3;
  *mul = (int64_t)nk * km;
  *add = (int64_t)nk * 4 + 4;
}

}  // namespace aw
