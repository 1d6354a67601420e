// aw_hist.hip -- image reductions of per-orbit (bin, value) items.
//
// The W x H image (512 x 512 for the large ensemble: 3 MB of counts and
// sums) does not fit in the 160 KB LDS of a CU, so the image is cut into tiles
// of TILE_W x TILE_H bins, whose counts (ds_add_u32) and sums (ds_add_f64) do,
// and the items are brought to their tiles, in one of three ways:
//   few items (hist_small): one workgroup per tile reads every item's bin and
//     keeps its own, in one launch (k_hist_small);
//   images of at most SEG_MAX_TILES tiles: each block sorts its segment of
//     SEG_ITEMS items by tile in LDS and writes it in place (k_tile_segments);
//     the tiles' totals are added up (k_segment_totals); one workgroup per
//     chunk of a tile's items gathers its runs from all segments
//     (k_segment_accum);
//   larger images, whose runs would be a few items each: a sort by tile over
//     the whole range, by counts per block (k_tile_count), their scans
//     (k_tile_scan_rows, k_tile_scan_tiles) and a scatter (k_tile_scatter);
//     one workgroup per chunk of a tile's range (k_tile_accum), and one per
//     tile of several chunks (k_tile_merge).
// A tile of few items is one chunk; a tile of several leaves partial tiles,
// which one workgroup adds up in chunk order: no global atomics on the image.
// Counts are exact and independent of scheduling; the order of the float
// additions inside a chunk is not, so sums can differ in the last bits.
#include <hip/hip_runtime.h>
#include <math.h>

#include "aw_hist.hpp"
#include "aw_internal.hpp"
#include "aw_launch.hpp"

namespace aw {

static_assert(ACC_BLOCK == TILE_BINS, "the merge runs one lane per bin, as many as the accumulation's lanes");

// The column and row of keys (a, b); false if they fall outside.
__device__ __forceinline__ bool column_row(double a, double b, const HistKeys &q, int W, int H, uint32_t &i,
                                           uint32_t &j) {
#pragma clang fp contract(off)
  if (!isfinite(a) || !isfinite(b)) return false;
  double fi = floor((a - q.lo0) / (q.hi0 - q.lo0) * (double)W);
  double fj = floor((b - q.lo1) / (q.hi1 - q.lo1) * (double)H);
  if (q.closed) {
    if (fi == (double)W && a == q.hi0) fi = (double)(W - 1);
    if (fj == (double)H && b == q.hi1) fj = (double)(H - 1);
  }
  if (!(fi >= 0.0) || fi >= (double)W || !(fj >= 0.0) || fj >= (double)H) return false;
  i = (uint32_t)fi;
  j = (uint32_t)fj;
  return true;
}

// The items' values are read where the caller keeps them, by the scatter.
__global__ void k_hist_bins(int64_t N, HistKeys q, int W, int H, uint32_t *__restrict__ bins) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  uint32_t i, j;
  bins[n] = column_row(q.a[n], q.b[n], q, W, H, i, j) ? j * (uint32_t)W + i : BIN_DROP;
}

__global__ void k_vdir_keys(int64_t N, const double *__restrict__ V, double *__restrict__ phi,
                            double *__restrict__ mu) {
#pragma clang fp contract(off)
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const double vx = V[n], vy = V[N + n], vz = V[2 * N + n];
  const double r = sqrt(vx * vx + vy * vy + vz * vz);
  if (r == 0.0) {
    phi[n] = __builtin_nan("");
    mu[n] = __builtin_nan("");
    return;
  }
  phi[n] = atan2(vy, vx);
  mu[n] = vz / r;
}

struct TileGeom {
  int W, H, tiles_x, n_tiles;
};

__device__ __forceinline__ void tile_of(uint32_t bin, const TileGeom &g, int &tile, int &local) {
  const int i = (int)(bin % (uint32_t)g.W), j = (int)(bin / (uint32_t)g.W);
  tile = (j / TILE_H) * g.tiles_x + i / TILE_W;
  local = (j % TILE_H) * TILE_W + (i % TILE_W);
}

// Both per-block kernels hold one LDS word per tile, sized at launch to the
// image (n_tiles + 1 words), so that a small image leaves room for more
// blocks per CU.
extern __shared__ uint32_t tile_words[];

// 1. Per-block tile counts; dropped items per block.
__global__ __launch_bounds__(HIST_BLOCK) void k_tile_count(int64_t N, const uint32_t *__restrict__ bins,
                                                           TileGeom g, int32_t G,
                                                           uint32_t *__restrict__ block_counts,
                                                           uint32_t *__restrict__ block_dropped) {
  uint32_t *cnt = tile_words;
  uint32_t &drop = tile_words[g.n_tiles];
  for (int t = threadIdx.x; t < g.n_tiles; t += blockDim.x) cnt[t] = 0u;
  if (threadIdx.x == 0) drop = 0u;
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * HIST_ITEMS_PER_BLOCK;
  const int64_t end = beg + HIST_ITEMS_PER_BLOCK < N ? beg + HIST_ITEMS_PER_BLOCK : N;
  const int64_t bd = blockDim.x;
  uint32_t my_drop = 0;
  auto count = [&](uint32_t bin) {
    if (bin == BIN_DROP) {
      ++my_drop;
      return;
    }
    int tile, local;
    tile_of(bin, g, tile, local);
    atomicAdd(&cnt[tile], 1u);
  };
  int64_t n = beg + threadIdx.x;
  for (; n + 3 * bd < end; n += 4 * bd) {  // four loads in flight per lane
    uint32_t b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = bins[n + k * bd];
#pragma unroll
    for (int k = 0; k < 4; ++k) count(b[k]);
  }
  for (; n < end; n += bd) count(bins[n]);
  if (my_drop) atomicAdd(&drop, my_drop);
  __syncthreads();
  for (int t = threadIdx.x; t < g.n_tiles; t += blockDim.x)
    block_counts[(int64_t)t * G + blockIdx.x] = cnt[t];
  if (threadIdx.x == 0) block_dropped[blockIdx.x] = drop;
}

// 2a. Exclusive scan of one tile's row of per-block counts, in place (one
//     workgroup per tile; the row is read and written in coalesced chunks of
//     SCAN_BLOCK entries, scanned by wave shuffles); the row total goes to
//     tile_total[t].
__global__ __launch_bounds__(SCAN_BLOCK) void k_tile_scan_rows(uint32_t *__restrict__ counts, int32_t G,
                                                               uint32_t *__restrict__ tile_total) {
  constexpr int NW = SCAN_BLOCK / 64;
  __shared__ uint32_t wsum[NW];
  uint32_t *row = counts + (int64_t)blockIdx.x * G;
  const int lane = (int)__lane_id(), wv = (int)(threadIdx.x >> 6);
  uint32_t carry = 0;
  for (int32_t base = 0; base < G; base += SCAN_BLOCK) {
    const int32_t e = base + (int32_t)threadIdx.x;
    const uint32_t v = e < G ? row[e] : 0u;
    uint32_t x = v;  // inclusive scan within the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wv] = x;
    __syncthreads();
    uint32_t before = carry, total = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      before += k < wv ? wsum[k] : 0u;
      total += wsum[k];
    }
    if (e < G) row[e] = before + x - v;
    carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) tile_total[blockIdx.x] = carry;
}

// Accumulation chunks of a tile of c items (at least one, so that every tile
// is written out).
__device__ __forceinline__ uint32_t n_chunks(uint32_t c, uint32_t chunk) {
  return c == 0u ? 1u : (c + chunk - 1u) / chunk;
}

// 2b. Exclusive scans of the tile totals, of the tiles' chunk counts and of
//     the partial-tile slots of tiles of several chunks, and the count of
//     dropped items (one workgroup of 1024 lanes): tile_start[t] = first
//     sorted position of tile t, tile_start[n_tiles] = items kept;
//     chunk_first[t] = first chunk of tile t, chunk_first[n_tiles] = chunks in
//     all; part_first[t] = first partial slot of tile t; chunk_tile[c] = the
//     tile of chunk c.
__global__ __launch_bounds__(1024) void k_tile_scan_tiles(const uint32_t *__restrict__ tile_total, int32_t n_tiles,
                                                          const uint32_t *__restrict__ block_dropped, int32_t G,
                                                          uint32_t chunk, uint32_t *__restrict__ tile_start,
                                                          uint32_t *__restrict__ chunk_first,
                                                          uint32_t *__restrict__ part_first,
                                                          uint32_t *__restrict__ chunk_tile,
                                                          uint64_t *__restrict__ dropped_out) {
  __shared__ uint32_t part[1024], pch[1024], ppt[1024];
  __shared__ uint64_t dsum[1024];
  const int tid = threadIdx.x;
  const int per = (n_tiles + 1023) / 1024;
  const int beg = tid * per;
  const int end = beg + per < n_tiles ? beg + per : n_tiles;
  uint32_t s = 0, sc = 0, sp = 0;
  for (int t = beg; t < end; ++t) {
    const uint32_t c = tile_total[t], k = n_chunks(c, chunk);
    s += c;
    sc += k;
    sp += k > 1u ? k : 0u;
  }
  part[tid] = s;
  pch[tid] = sc;
  ppt[tid] = sp;
  uint64_t d = 0;
  for (int b = tid; b < G; b += 1024) d += block_dropped[b];
  dsum[tid] = d;
  __syncthreads();
  // Hillis-Steele inclusive scans of the 1024 partial sums.
  for (int off = 1; off < 1024; off <<= 1) {
    const uint32_t v = tid >= off ? part[tid - off] : 0u;
    const uint32_t vc = tid >= off ? pch[tid - off] : 0u;
    const uint32_t vp = tid >= off ? ppt[tid - off] : 0u;
    __syncthreads();
    part[tid] += v;
    pch[tid] += vc;
    ppt[tid] += vp;
    __syncthreads();
  }
  uint32_t run = tid > 0 ? part[tid - 1] : 0u;
  uint32_t runc = tid > 0 ? pch[tid - 1] : 0u;
  uint32_t runp = tid > 0 ? ppt[tid - 1] : 0u;
  for (int t = beg; t < end; ++t) {
    const uint32_t c = tile_total[t], k = n_chunks(c, chunk);
    tile_start[t] = run;
    chunk_first[t] = runc;
    part_first[t] = runp;
    for (uint32_t q = 0; q < k; ++q) chunk_tile[runc + q] = (uint32_t)t;
    run += c;
    runc += k;
    runp += k > 1u ? k : 0u;
  }
  if (tid == 1023) {
    tile_start[n_tiles] = part[1023];
    chunk_first[n_tiles] = pch[1023];
    part_first[n_tiles] = ppt[1023];
  }
  // Tree sum of the dropped counts.
  for (int off = 512; off > 0; off >>= 1) {
    if (tid < off) dsum[tid] += dsum[tid + off];
    __syncthreads();
  }
  if (tid == 0 && dropped_out) *dropped_out = dsum[0];
}

// 3. Move each block's items to their tile ranges.
__global__ __launch_bounds__(HIST_BLOCK) void k_tile_scatter(int64_t N, const uint32_t *__restrict__ bins,
                                                             const double *__restrict__ vals, TileGeom g,
                                                             int32_t G, const uint32_t *__restrict__ offsets,
                                                             const uint32_t *__restrict__ tile_start,
                                                             uint16_t *__restrict__ sorted_local,
                                                             double *__restrict__ sorted_val) {
  uint32_t *cur = tile_words;
  for (int t = threadIdx.x; t < g.n_tiles; t += blockDim.x)
    cur[t] = tile_start[t] + offsets[(int64_t)t * G + blockIdx.x];
  __syncthreads();
  const int64_t beg = (int64_t)blockIdx.x * HIST_ITEMS_PER_BLOCK;
  const int64_t end = beg + HIST_ITEMS_PER_BLOCK < N ? beg + HIST_ITEMS_PER_BLOCK : N;
  const int64_t bd = blockDim.x;
  auto place = [&](int64_t n, uint32_t bin) {
    if (bin == BIN_DROP) return;
    int tile, local;
    tile_of(bin, g, tile, local);
    const uint32_t pos = atomicAdd(&cur[tile], 1u);
    sorted_local[pos] = (uint16_t)local;
    if (vals) sorted_val[pos] = vals[n];
  };
  int64_t n = beg + threadIdx.x;
  for (; n + 3 * bd < end; n += 4 * bd) {  // four loads in flight per lane
    uint32_t b[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) b[k] = bins[n + k * bd];
#pragma unroll
    for (int k = 0; k < 4; ++k) place(n + k * bd, b[k]);
  }
  for (; n < end; n += bd) place(n, bins[n]);
}

// Bin k of tile t, from its count and sum.  mode 0: counts + sums;
// 1: counts + mean; 2: counts + density (count * norm).  accumulate: counts
// are added to what counts_out holds.
__device__ __forceinline__ void write_bin(const TileGeom &g, int t, int k, uint32_t cc, double sk, int32_t mode,
                                          double norm, int32_t accumulate, uint32_t *__restrict__ counts_out,
                                          double *__restrict__ f_out) {
  const int tx = t % g.tiles_x, ty = t / g.tiles_x;
  const int i = tx * TILE_W + (k % TILE_W), j = ty * TILE_H + (k / TILE_W);
  if (i >= g.W || j >= g.H) return;
  const int64_t o = (int64_t)j * g.W + i;
  if (counts_out) counts_out[o] = accumulate ? counts_out[o] + cc : cc;
  if (f_out) {
    double f;
    if (mode == 0) f = sk;
    else if (mode == 1) f = cc ? sk / (double)cc : 0.0;
    else f = (double)cc * norm;
    f_out[o] = f;
  }
}

// 4. One workgroup per chunk: LDS accumulation of the chunk's items, then the
//    tile is written out (a tile of one chunk) or left as the chunk's partial
//    tile (a tile of several).  Each lane takes four items per pass so that
//    four loads are in flight.
__global__ __launch_bounds__(ACC_BLOCK) void k_tile_accum(const uint32_t *__restrict__ tile_start,
                                                           const uint32_t *__restrict__ chunk_first,
                                                           const uint32_t *__restrict__ part_first,
                                                           const uint32_t *__restrict__ chunk_tile, uint32_t chunk,
                                                           const uint16_t *__restrict__ sorted_local,
                                                           const double *__restrict__ sorted_val,
                                                           TileGeom g, int32_t mode, double norm, int32_t accumulate,
                                                           uint32_t *__restrict__ counts_out,
                                                           double *__restrict__ f_out,
                                                           uint32_t *__restrict__ part_counts,
                                                           double *__restrict__ part_sums) {
  __shared__ uint32_t c[TILE_BINS];
  __shared__ double s[TILE_BINS];
  const uint32_t w = blockIdx.x;
  if (w >= chunk_first[g.n_tiles]) return;  // the grid bounds the chunk count from above
  const int t = (int)chunk_tile[w];
  const uint32_t c0 = chunk_first[t], nch = chunk_first[t + 1] - c0;
  const uint32_t te = tile_start[t + 1];
  const uint32_t beg = tile_start[t] + (w - c0) * chunk;
  const uint32_t end = te - beg > chunk ? beg + chunk : te;
  for (int k = threadIdx.x; k < TILE_BINS; k += blockDim.x) {
    c[k] = 0u;
    s[k] = 0.0;
  }
  __syncthreads();
  const bool have_vals = sorted_val != nullptr;
  const uint32_t bd = blockDim.x;
  uint32_t p = beg + threadIdx.x;
  for (; p + 3 * bd < end; p += 4 * bd) {
    int loc[4];
    double val[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k) loc[k] = sorted_local[p + k * bd];
    if (have_vals) {
#pragma unroll
      for (int k = 0; k < 4; ++k) val[k] = sorted_val[p + k * bd];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      atomicAdd(&c[loc[k]], 1u);
      if (have_vals) atomicAdd(&s[loc[k]], val[k]);
    }
  }
  for (; p < end; p += bd) {
    const int loc = sorted_local[p];
    atomicAdd(&c[loc], 1u);
    if (have_vals) atomicAdd(&s[loc], sorted_val[p]);
  }
  __syncthreads();
  if (nch == 1u) {
    for (int k = threadIdx.x; k < TILE_BINS; k += blockDim.x)
      write_bin(g, t, k, c[k], s[k], mode, norm, accumulate, counts_out, f_out);
  } else {
    const int64_t slot = (int64_t)(part_first[t] + (w - c0)) * TILE_BINS;
    for (int k = threadIdx.x; k < TILE_BINS; k += blockDim.x) {
      part_counts[slot + k] = c[k];
      if (have_vals) part_sums[slot + k] = s[k];
    }
  }
}

// 5. One workgroup of TILE_BINS lanes per tile; tiles of several chunks add
//    their partial tiles in chunk order (lane k: bin k) and write the tile out.
__global__ __launch_bounds__(TILE_BINS) void k_tile_merge(const uint32_t *__restrict__ chunk_first,
                                                           const uint32_t *__restrict__ part_first, TileGeom g,
                                                           int32_t mode, double norm, int32_t accumulate,
                                                           const uint32_t *__restrict__ part_counts,
                                                           const double *__restrict__ part_sums,
                                                           uint32_t *__restrict__ counts_out,
                                                           double *__restrict__ f_out) {
  const int t = blockIdx.x, k = threadIdx.x;
  const uint32_t nch = chunk_first[t + 1] - chunk_first[t];
  if (nch < 2u) return;
  const int64_t p0 = part_first[t];
  uint32_t cc = 0;
  double sk = 0.0;
  for (uint32_t q = 0; q < nch; ++q) {
    const int64_t o = (p0 + q) * TILE_BINS + k;
    cc += part_counts[o];
    if (part_sums) sk += part_sums[o];
  }
  write_bin(g, t, k, cc, sk, mode, norm, accumulate, counts_out, f_out);
}

// Few items: one workgroup per tile reads all N bins (N / 1024 coalesced loads
// per lane, from the L2 after the first reader) and accumulates those of its
// own tile in LDS.  Bound by launch and load latency while the items spread
// over many tiles (32000 items and 512 x 512 bins with the keys 18.5 us, 34.4
// sorted), by the LDS adds of one CU where a tile holds most of them (65536
// items in 64 x 64 bins 27.6 us, 38.2 sorted; all within 1/50 of either
// width 42.6, 67.5).
__global__ __launch_bounds__(ACC_BLOCK) void k_hist_small(int64_t N, const uint32_t *__restrict__ bins,
                                                           const double *__restrict__ vals, TileGeom g, int32_t mode,
                                                           double norm, int32_t accumulate,
                                                           uint32_t *__restrict__ counts_out,
                                                           double *__restrict__ f_out,
                                                           uint64_t *__restrict__ dropped_out) {
  __shared__ uint32_t c[TILE_BINS];
  __shared__ double s[TILE_BINS];
  __shared__ uint32_t drop;
  const int t = blockIdx.x, tid = threadIdx.x;
  c[tid] = 0u;
  s[tid] = 0.0;
  if (tid == 0) drop = 0u;
  __syncthreads();
  const uint32_t W = (uint32_t)g.W, tx = (uint32_t)(t % g.tiles_x), j0 = (uint32_t)(t / g.tiles_x) * TILE_H;
  const uint32_t first = j0 * W, span = ((uint32_t)g.H - j0 < TILE_H ? (uint32_t)g.H - j0 : TILE_H) * W;
  const bool count_drops = t == 0 && dropped_out != nullptr;
  uint32_t my_drop = 0;
  auto add = [&](int64_t n, uint32_t bin) {
    if (count_drops && bin == BIN_DROP) ++my_drop;
    const uint32_t d = bin - first;   // BIN_DROP stays above every span
    if (d >= span) return;
    const uint32_t j = d / W, i = d - j * W;
    if (i / TILE_W != tx) return;
    const uint32_t k = j * TILE_W + i % TILE_W;
    atomicAdd(&c[k], 1u);
    if (vals) atomicAdd(&s[k], vals[n]);
  };
  int64_t n = tid;
  for (; n + 7 * ACC_BLOCK < N; n += 8 * ACC_BLOCK) {  // eight loads in flight per lane
    uint32_t b[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k] = bins[n + k * ACC_BLOCK];
#pragma unroll
    for (int k = 0; k < 8; ++k) add(n + k * ACC_BLOCK, b[k]);
  }
  for (; n < N; n += ACC_BLOCK) add(n, bins[n]);
  if (my_drop) atomicAdd(&drop, my_drop);
  __syncthreads();
  write_bin(g, t, tid, c[tid], s[tid], mode, norm, accumulate, counts_out, f_out);
  if (count_drops && tid == 0) *dropped_out = drop;
}

// Segments: images of at most SEG_MAX_TILES tiles.  One pass reads each item
// once (its keys, or its bin where the propagation left one), sorts it by tile
// within its block's segment of SEG_ITEMS in LDS, and writes the sorted
// segment in place with the end of every tile's run; no item waits for
// another block's counts.  The accumulation gathers a tile's runs from all
// segments.  Against the sort by tile over the whole range, this drops the
// bins' write and two reads of them, the two scans and their launches.
// Bound by memory: 72 MB of keys and values read and 30 MB written in 24.3 us
// with the launch where the inputs are new (4.2 TB/s; a large copy reaches 5.0),
// in 21.9 where repeated calls leave them in the Infinity Cache.  3000001 items
// into 512 x 512 bins, all launches, inputs new / repeated: 72 / 68 us sorted over
// the whole range, 44 / 42 in segments; repeated, into 64 x 64 78 / 55, into
// 1024 x 512 72 / 49; all within 1/50 of either width of 512 x 512 84 / 62; 98304
// items into 512 x 512 34 / 21.  Blocks of 512 lanes: three per CU hold 3e6
// items at once; 6144 items on 1024 lanes took 28 us in place of 22.
template <bool KEYS, bool VALS>
__global__ __launch_bounds__(SEG_BLOCK) void k_tile_segments(int64_t N, HistKeys q,
                                                             const uint32_t *__restrict__ bins,
                                                             const double *__restrict__ vals, TileGeom g,
                                                             uint16_t *__restrict__ seg_end,
                                                             uint16_t *__restrict__ sorted_local,
                                                             double *__restrict__ sorted_val) {
  constexpr int NW = SEG_BLOCK / 64;
  constexpr int IPL = SEG_ITEMS / SEG_BLOCK;      // items per lane
  constexpr int TPL = SEG_MAX_TILES / SEG_BLOCK;  // tiles per lane in the scan
  static_assert(IPL * SEG_BLOCK == SEG_ITEMS && TPL * SEG_BLOCK == SEG_MAX_TILES, "whole numbers per lane");
  __shared__ double st_val[VALS ? SEG_ITEMS : 1];
  __shared__ alignas(4) uint16_t st_local[SEG_ITEMS];
  __shared__ uint32_t cnt[SEG_MAX_TILES];
  __shared__ uint32_t wsum[NW];
  const int nt = g.n_tiles, tid = threadIdx.x, lane = (int)__lane_id(), wv = tid >> 6;
  const int64_t beg = (int64_t)blockIdx.x * SEG_ITEMS;
  const int32_t n_here = N - beg < SEG_ITEMS ? (int32_t)(N - beg) : SEG_ITEMS;
  double a[IPL], b[IPL], val[IPL];
  uint32_t bin[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    const int32_t o = tid + k * SEG_BLOCK;
    const bool in = o < n_here;
    if constexpr (KEYS) {
      a[k] = in ? q.a[beg + o] : __builtin_nan("");
      b[k] = in ? q.b[beg + o] : 0.0;
    } else {
      bin[k] = in ? bins[beg + o] : BIN_DROP;
    }
  }
  if constexpr (VALS) {
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
      const int32_t o = tid + k * SEG_BLOCK;
      val[k] = o < n_here ? vals[beg + o] : 0.0;
    }
  }
#pragma unroll
  for (int k = 0; k < TPL; ++k) cnt[tid * TPL + k] = 0u;
  __syncthreads();
  // Each item's tile, local bin and rank among the block's items of its tile.
  uint32_t at[IPL], rank[IPL];
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    uint32_t i = 0, j = 0;
    bool in;
    if constexpr (KEYS) {
      in = column_row(a[k], b[k], q, g.W, g.H, i, j);
    } else {
      in = bin[k] != BIN_DROP;
      j = bin[k] / (uint32_t)g.W;
      i = bin[k] - j * (uint32_t)g.W;
    }
    at[k] = BIN_DROP;
    if (!in) continue;
    const uint32_t t = j / TILE_H * (uint32_t)g.tiles_x + i / TILE_W;
    at[k] = t * TILE_BINS + j % TILE_H * TILE_W + i % TILE_W;
    rank[k] = atomicAdd(&cnt[t], 1u);
  }
  __syncthreads();
  // Exclusive scan of the tile counts, in place; the ends go out.
  uint32_t v[TPL], mine = 0;
#pragma unroll
  for (int k = 0; k < TPL; ++k) {
    v[k] = cnt[tid * TPL + k];
    mine += v[k];
  }
  uint32_t x = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  uint32_t before = x - mine, kept = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    before += k < wv ? wsum[k] : 0u;
    kept += wsum[k];
  }
#pragma unroll
  for (int k = 0; k < TPL; ++k) {
    const int t = tid * TPL + k;
    cnt[t] = before;
    before += v[k];
    if (t < nt) seg_end[(int64_t)blockIdx.x * nt + t] = (uint16_t)before;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPL; ++k) {
    if (at[k] == BIN_DROP) continue;
    const uint32_t slot = cnt[at[k] / TILE_BINS] + rank[k];
    st_local[slot] = (uint16_t)(at[k] % TILE_BINS);
    if constexpr (VALS) st_val[slot] = val[k];
  }
  __syncthreads();
  // Two local bins per store: the second of an odd count's last pair lies in
  // the segment, or in the padding after the last one.
  uint32_t *out = (uint32_t *)(sorted_local + beg);
  for (uint32_t i = tid; 2 * i < kept; i += SEG_BLOCK) out[i] = ((const uint32_t *)st_local)[i];
  if constexpr (VALS)
    for (uint32_t i = tid; i < kept; i += SEG_BLOCK) sorted_val[beg + i] = st_val[i];
}

// Inclusive scan over the block's ACC_BLOCK lanes; total = the sum.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wsum, uint32_t &total) {
  constexpr int NW = ACC_BLOCK / 64;
  const int lane = (int)__lane_id(), wv = (int)(threadIdx.x >> 6);
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  __syncthreads();  // an earlier scan's sums have been read
  if (lane == 63) wsum[wv] = x;
  __syncthreads();
  total = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    x += k < wv ? wsum[k] : 0u;
    total += wsum[k];
  }
  return x;
}

// The tile of workgroup w: workgroups go round the 8 XCDs, and each XCD takes a
// contiguous range of tiles, whose runs share lines in its L2 (a run of 16 local
// bins is a quarter of one).
__device__ __forceinline__ int tile_of_group(int w, int nt) {
  const int x = w % 8, q = nt / 8, r = nt % 8;
  return x * q + (x < r ? x : r) + w / 8;
}

// Items of tile t in segment `seg`: their number and the first one's place.
__device__ __forceinline__ uint32_t run_of(const uint16_t *__restrict__ seg_end, int nt, int t, int32_t seg,
                                           uint32_t &first) {
  const uint16_t *row = seg_end + (int64_t)seg * nt;
  const uint32_t f = t ? row[t - 1] : 0u, len = row[t] - f;
  first = (uint32_t)seg * SEG_ITEMS + f;
  return len;
}

// Every tile's total over the segments, one workgroup each.
__global__ __launch_bounds__(SCAN_BLOCK) void k_segment_totals(int32_t n_segs, int nt,
                                                               const uint16_t *__restrict__ seg_end,
                                                               uint32_t *__restrict__ tile_total,
                                                               uint32_t *__restrict__ tile_done) {
  __shared__ uint32_t sum;
  const int t = tile_of_group((int)blockIdx.x, nt);
  if (threadIdx.x == 0) sum = 0u;
  __syncthreads();
  uint32_t mine = 0, first;
#pragma unroll 4
  for (int32_t seg = (int32_t)threadIdx.x; seg < n_segs; seg += SCAN_BLOCK) mine += run_of(seg_end, nt, t, seg, first);
  atomicAdd(&sum, mine);
  __syncthreads();
  if (threadIdx.x == 0) {
    tile_total[t] = sum;
    tile_done[t] = 0u;
  }
}

// Accumulation over segments.  Workgroups [0, n_tiles) take the first chunk of
// their tile; the rest find the tile of their further chunk in a scan of the
// totals, and leave if there is none.  A chunk is a range of the tile's items
// in segment order: per batch of ACC_BLOCK segments the runs' lengths are
// scanned, and in windows of ACC_WINDOW items every run marks its first item
// and a running maximum gives each item its run (a binary search per item cost
// 7 us more at 3000001 items into 512 x 512 bins).  A tile of several chunks
// leaves partial tiles, which the workgroup that finishes last adds up in chunk
// order.  Bound by latency: runs, marks, items, adds one after the other, 15 us
// with the launch at those sizes (21 in windows of 4096 and without
// tile_of_group); all items within one tile 35 us.
__global__ __launch_bounds__(ACC_BLOCK) void k_segment_accum(int64_t N, int32_t n_segs, uint32_t chunk, TileGeom g,
                                                             const uint16_t *__restrict__ seg_end,
                                                             const uint32_t *__restrict__ tile_total,
                                                             uint32_t *__restrict__ tile_done,
                                                             const uint16_t *__restrict__ sorted_local,
                                                             const double *__restrict__ sorted_val, int32_t mode,
                                                             double norm, int32_t accumulate,
                                                             uint32_t *__restrict__ counts_out,
                                                             double *__restrict__ f_out, uint32_t *part_counts,
                                                             double *part_sums, uint64_t *__restrict__ dropped_out) {
  __shared__ uint32_t c[TILE_BINS];
  __shared__ double s[TILE_BINS];
  __shared__ uint32_t src[ACC_BLOCK], wsum[ACC_BLOCK / 64], found[4];
  __shared__ alignas(16) uint16_t own[ACC_WINDOW];
  using ushort8 = uint16_t __attribute__((ext_vector_type(8)));
  constexpr int MARKS = ACC_WINDOW / ACC_BLOCK / 8;  // 16-byte words of marks per lane, at most
  static_assert(SEG_MAX_TILES <= ACC_BLOCK, "one lane per tile in the scans");
  const int nt = g.n_tiles, tid = threadIdx.x, lane = (int)__lane_id(), wv = tid >> 6;
  int t = (int)blockIdx.x < nt ? tile_of_group((int)blockIdx.x, nt) : (int)blockIdx.x;
  uint32_t q = 0, slot0 = 0, nch = 1;
  // The first batch's run of the tile, read ahead of what only further chunks need.
  uint32_t first = 0, len = 0;
  if (t < nt && tid < n_segs) len = run_of(seg_end, nt, t, tid, first);
  const uint32_t tot = tid < nt ? tile_total[tid] : 0u;
  if (blockIdx.x == 0 && dropped_out) {
    uint32_t kept;
    block_scan(tot, wsum, kept);
    if (tid == 0) *dropped_out = (uint64_t)(N - (int64_t)kept);
  }
  if (t < nt) nch = n_chunks(tile_total[t], chunk);
  if (t >= nt || nch > 1u) {
    const uint32_t k = tid < nt ? n_chunks(tot, chunk) : 1u;
    uint32_t total, parts;
    const uint32_t more = block_scan(k - 1u, wsum, total);          // further chunks up to and with this tile
    const uint32_t slots = block_scan(k > 1u ? k : 0u, wsum, parts);  // partial tiles likewise
    if (t >= nt) {
      const uint32_t e = (uint32_t)t - (uint32_t)nt;
      if (e >= total) return;
      if (e < more && e >= more - (k - 1u)) {
        found[0] = (uint32_t)tid;
        found[1] = e - (more - (k - 1u)) + 1u;
        found[2] = slots - k;
        found[3] = k;
      }
    } else if (tid == t) {
      found[0] = (uint32_t)t;
      found[1] = 0u;
      found[2] = slots - k;
      found[3] = k;
    }
    __syncthreads();
    if (t >= nt && tid < n_segs) len = run_of(seg_end, nt, (int)found[0], tid, first);
    t = (int)found[0];
    q = found[1];
    slot0 = found[2];
    nch = found[3];
  }
  const uint32_t items = tile_total[t];
  const uint32_t c0 = q * chunk, c1 = items - c0 > chunk ? c0 + chunk : items;
  c[tid] = 0u;
  s[tid] = 0.0;
  const bool have_vals = sorted_val != nullptr;
  uint32_t done = 0;  // the tile's items in earlier batches
  for (int32_t b0 = 0; b0 < n_segs && done < c1; b0 += ACC_BLOCK) {
    const int32_t seg = b0 + tid;
    uint32_t in_batch;
    if (b0 > 0) len = seg < n_segs ? run_of(seg_end, nt, t, seg, first) : 0u;
    const uint32_t at = block_scan(len, wsum, in_batch) - len;
    src[tid] = first - at;
    const uint32_t lo = c0 > done ? c0 - done : 0u, hi = c1 - done < in_batch ? c1 - done : in_batch;
    for (uint32_t w0 = lo; w0 < hi; w0 += ACC_WINDOW) {
      const uint32_t n = hi - w0 < ACC_WINDOW ? hi - w0 : ACC_WINDOW;
      const int marks = n <= 8 * ACC_BLOCK ? 1 : MARKS;
      ushort8 m[MARKS];
#pragma unroll
      for (int p = 0; p < MARKS; ++p)
        if (p < marks) *(ushort8 *)&own[8 * (marks * tid + p)] = ushort8{};
      __syncthreads();
      if (len != 0u && at < w0 + n && at + len > w0) own[at > w0 ? at - w0 : 0u] = (uint16_t)tid;
      __syncthreads();
      uint16_t x = 0;
#pragma unroll
      for (int p = 0; p < MARKS; ++p) {
        if (p >= marks) break;
        m[p] = *(const ushort8 *)&own[8 * (marks * tid + p)];
#pragma unroll
        for (int k = 0; k < 8; ++k) m[p][k] = x = m[p][k] > x ? m[p][k] : x;
      }
      uint32_t y = x;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t z = __shfl_up(y, off, 64);
        y = lane >= off && z > y ? z : y;
      }
      if (lane == 63) wsum[wv] = y;
      uint32_t before = __shfl_up(y, 1, 64);  // the largest mark before this lane's
      if (lane == 0) before = 0u;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < ACC_BLOCK / 64; ++k) before = k < wv && wsum[k] > before ? wsum[k] : before;
#pragma unroll
      for (int p = 0; p < MARKS; ++p) {
        if (p >= marks) break;
#pragma unroll
        for (int k = 0; k < 8; ++k) m[p][k] = m[p][k] > before ? m[p][k] : (uint16_t)before;
        *(ushort8 *)&own[8 * (marks * tid + p)] = m[p];
      }
      __syncthreads();
      constexpr int U = 8;
      for (uint32_t i0 = tid; i0 < n; i0 += U * ACC_BLOCK) {  // eight items in flight per lane
        uint32_t loc[U];
        double val[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const uint32_t i = i0 + k * ACC_BLOCK;
          if (i >= n) continue;
          const uint32_t from = src[own[i]] + w0 + i;
          loc[k] = sorted_local[from];
          if (have_vals) val[k] = sorted_val[from];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
          if (i0 + k * ACC_BLOCK >= n) continue;
          atomicAdd(&c[loc[k]], 1u);
          if (have_vals) atomicAdd(&s[loc[k]], val[k]);
        }
      }
      __syncthreads();
    }
    done += in_batch;
  }
  __syncthreads();
  if (nch == 1u) {
    write_bin(g, t, tid, c[tid], s[tid], mode, norm, accumulate, counts_out, f_out);
    return;
  }
  const int64_t o = ((int64_t)slot0 + q) * TILE_BINS + tid;
  part_counts[o] = c[tid];
  if (have_vals) part_sums[o] = s[tid];
  // Every wave waits until its own stores have reached the L2: the barrier waits
  // for LDS operations only, and the release below for the stores of its own
  // wave.  Then one lane's release writes the L2 back for the whole workgroup,
  // and its acquire covers the loads after the next barrier (a fence on every
  // wave would write the L2 back 16 times).
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) found[0] = __hip_atomic_fetch_add(&tile_done[t], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (found[0] != nch - 1u) return;
  uint32_t cc = 0;
  double sk = 0.0;
  for (uint32_t p0 = 0; p0 < nch; p0 += 8) {  // eight partial tiles in flight
    uint32_t pc[8];
    double ps[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const int64_t op = ((int64_t)slot0 + p0 + k) * TILE_BINS + tid;
      pc[k] = p0 + k < nch ? part_counts[op] : 0u;
      ps[k] = p0 + k < nch && have_vals ? part_sums[op] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      cc += pc[k];
      sk += ps[k];
    }
  }
  write_bin(g, t, tid, cc, sk, mode, norm, accumulate, counts_out, f_out);
}

hipError_t launch_vdir_keys(int64_t N, const double *V, double *phi, double *mu, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_vdir_keys, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, N, V, phi, mu);
  return hipGetLastError();
}

HistPlan hist_plan(int64_t N, int W, int H) {
  HistPlan p;
  p.W = W;
  p.H = H;
  p.tiles_x = (W + TILE_W - 1) / TILE_W;
  p.n_tiles = p.tiles_x * ((H + TILE_H - 1) / TILE_H);
  p.G = (int32_t)((N + HIST_ITEMS_PER_BLOCK - 1) / HIST_ITEMS_PER_BLOCK);
  if (p.G < 1) p.G = 1;
  const int64_t n = N > 0 ? N : 0;
  p.chunk = acc_chunk(n, p.n_tiles);
  p.max_chunks = p.n_tiles + (n + p.chunk - 1) / p.chunk;
  return p;
}

// launch_hist_reduce through segments, for images of at most SEG_MAX_TILES
// tiles.  The ends take the place of the block counts, the totals and the
// counts of finished chunks that of the tile starts.
static hipError_t launch_segments(int64_t N, const HistKeys *keys, const uint32_t *bins, const double *vals,
                                  const HistPlan &p, const HistScratch &w, const TileGeom &g, int mode, double norm,
                                  uint32_t *counts_out, double *f_out, uint64_t *dropped_out, hipStream_t s,
                                  int accumulate) {
  static_assert(2 * SEG_ITEMS >= HIST_ITEMS_PER_BLOCK && SEG_ITEMS <= 65535, "the ends fit the block counts' room");
  const int32_t n_segs = (int32_t)((N + SEG_ITEMS - 1) / SEG_ITEMS);
  uint16_t *ends = (uint16_t *)w.block_counts;
  uint32_t *total = w.tile_start, *done = total + p.n_tiles;
  const HistKeys q = keys ? *keys : HistKeys{};
#define AW_SEGMENTS(K, V)                                                                                      \
  hipLaunchKernelGGL((k_tile_segments<K, V>), dim3((unsigned)n_segs), dim3(SEG_BLOCK), 0, s, N, q, bins, vals, \
                     g, ends, w.sorted_local, w.sorted_val)
  if (keys && vals) AW_SEGMENTS(true, true);
  else if (keys) AW_SEGMENTS(true, false);
  else if (vals) AW_SEGMENTS(false, true);
  else AW_SEGMENTS(false, false);
#undef AW_SEGMENTS
  hipLaunchKernelGGL(k_segment_totals, dim3((unsigned)p.n_tiles), dim3(SCAN_BLOCK), 0, s, n_segs, p.n_tiles, ends,
                     total, done);
  hipLaunchKernelGGL(k_segment_accum, dim3((unsigned)p.max_chunks), dim3(ACC_BLOCK), 0, s, N, n_segs,
                     (uint32_t)p.chunk, g, ends, total, done, w.sorted_local, vals ? w.sorted_val : nullptr, mode,
                     norm, accumulate, counts_out, f_out, w.part_counts, vals ? w.part_sums : nullptr, dropped_out);
  return hipGetLastError();
}

hipError_t launch_hist_reduce(int64_t N, const HistKeys *keys, uint32_t *bins, const double *vals, const HistPlan &p,
                              const HistScratch &w, int mode, double norm, uint32_t *counts_out,
                              double *f_out, uint64_t *dropped_out, hipStream_t s, int accumulate) {
  TileGeom g{p.W, p.H, p.tiles_x, p.n_tiles};
  if (!hist_small(N, p.n_tiles) && p.n_tiles <= SEG_MAX_TILES)
    return launch_segments(N, keys, bins, vals, p, w, g, mode, norm, counts_out, f_out, dropped_out, s, accumulate);
  if (keys && N > 0)
    hipLaunchKernelGGL(k_hist_bins, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, N, *keys, p.W, p.H, bins);
  if (hist_small(N, p.n_tiles)) {
    hipLaunchKernelGGL(k_hist_small, dim3((unsigned)p.n_tiles), dim3(ACC_BLOCK), 0, s, N, bins, vals, g, mode, norm,
                       accumulate, counts_out, f_out, dropped_out);
    return hipGetLastError();
  }
  const unsigned tile_lds = (unsigned)(sizeof(uint32_t) * ((size_t)p.n_tiles + 1));  // <= 32 KB + 4 B
  hipLaunchKernelGGL(k_tile_count, dim3((unsigned)p.G), dim3(HIST_BLOCK), tile_lds, s, N, bins, g, p.G,
                     w.block_counts, w.block_dropped);
  hipLaunchKernelGGL(k_tile_scan_rows, dim3((unsigned)p.n_tiles), dim3(SCAN_BLOCK), 0, s, w.block_counts, p.G,
                     w.tile_total);
  hipLaunchKernelGGL(k_tile_scan_tiles, dim3(1), dim3(1024), 0, s, w.tile_total, p.n_tiles, w.block_dropped, p.G,
                     (uint32_t)p.chunk, w.tile_start, w.chunk_first, w.part_first, w.chunk_tile, dropped_out);
  hipLaunchKernelGGL(k_tile_scatter, dim3((unsigned)p.G), dim3(HIST_BLOCK), tile_lds, s, N, bins, vals, g, p.G,
                     w.block_counts, w.tile_start, w.sorted_local, vals ? w.sorted_val : nullptr);
  double *psums = vals ? w.part_sums : nullptr;
  hipLaunchKernelGGL(k_tile_accum, dim3((unsigned)p.max_chunks), dim3(ACC_BLOCK), 0, s, w.tile_start,
                     w.chunk_first, w.part_first, w.chunk_tile, (uint32_t)p.chunk, w.sorted_local,
                     vals ? w.sorted_val : nullptr, g, mode, norm, accumulate, counts_out, f_out, w.part_counts,
                     psums);
  if (N > p.chunk)  // else no tile has several chunks
    hipLaunchKernelGGL(k_tile_merge, dim3((unsigned)p.n_tiles), dim3(TILE_BINS), 0, s, w.chunk_first, w.part_first,
                       g, mode, norm, accumulate, w.part_counts, psums, counts_out, f_out);
  return hipGetLastError();
}

}  // namespace aw
