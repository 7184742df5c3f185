// lc_launch.h -- which kernel and launch shape a grid takes: the rules of the
// dispatch, on sizes and element sizes alone.  Host arithmetic in plain C++.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/lc.h"

namespace lc {

constexpr int NUM_CU = 256;  // compute units of the chip

// A two-dimensional grid of N sites as a launch with one block per tile sees
// it: the tiles of the columns from xb on.
struct TileDims {
  int nx, ny, xb;
  int64_t N;
};

// launch(blocks_x, blocks_y, xb, before) for the launches that take the tiles of
// tx x ty sites of a two-dimensional grid, `threads` threads each: the columns
// from xb on, after `before` blocks.  One launch, but where its threads along x
// do not fit the runtime's 32 bits (1024 per tile of 32 columns: from 2^27
// columns on), where several take a range of columns each.
template <typename LAUNCH>
inline void tile_launches(const lc_grid& g, int tx, int ty, int threads, LAUNCH launch) {
  const int64_t most = ((int64_t(1) << 32) - 1) / threads;
  const int64_t ntx = (int64_t(g.nx) + tx - 1) / tx, nty = (g.ny + ty - 1) / ty;
  for (int64_t t = 0; t < ntx; t += most)
    launch(unsigned(std::min(most, ntx - t)), unsigned(nty), int(t * tx), t * nty);
}

// Whether the coordinates x0 - 2 .. x0 + t + 1 of a tile of t >= 2 sites from x0
// on (a multiple of t within the grid) are in -n .. 2n - 1, so that they wrap at
// most once.
constexpr bool region_wraps_once(int n, int t) { return n >= 2 && 2 * int64_t(n) >= t + 2; }

// Chunks of `planes` planes cut evenly: as many of them, as long as each other.
// XCDs take contiguous ranges of blocks, so a short last chunk leaves one of
// them with little to do: single pass on 150x150x200, FP64, 33 planes 1572 us
// per step in launch order and 1860 in ranges, 128 planes 1772 and 2211; cut
// evenly 1614 and 1737.
inline int even_chunk(int nz, int planes) {
  const int longest = std::min(planes, nz), chunks = nz / longest + (nz % longest != 0);
  return nz / chunks + (nz % chunks != 0);
}

// Planes per block along z for a sweep of `tiles` column tiles on a grid of
// nz planes, at most `most`.  A block of zc planes marches zc + `extra`
// planes, one after another, so a grid with few tiles is bound by that serial
// chain while most CUs idle: there shorter chunks win in spite of the planes
// they compute twice.  The estimate counts, per CU, the marches that run one
// after another; a march that shares its CU with one other takes 1.4 times as
// long as alone (measured 1.3-1.6), with two others 1.85 times (Q sweep,
// 1.8-1.9).
// Measured on the stress/LB and Q sweeps, long default chunks against the
// chosen ones: 24^3 FP32 67.7 -> 14.7 and 56.9 -> 11.7 us, 64^3 FP64
// 80 -> 32 and 147 -> 24 us, 129x100x75 FP32 isotropic 186 -> 95 and
// 474 -> 111 us.  On large grids it stays near the longest: 16 of 16 and 86 of
// 128 planes on 256^3, 15 and 54 on 270^3 (FP32).
// `resident` is what the sweep's registers and LDS allow on a CU: two blocks of
// the stress/LB sweep, three of the Q sweep (two with the isotropic stencils),
// one of the single pass; a kernel that changes those needs it changed.
// `margin`: chunks that make more blocks than the longest do must be estimated
// that much faster; the longest are at least cut evenly.
inline int pick_chunk(int nz, int64_t tiles, int most, int extra, int resident = 2, double margin = 0.0) {
  constexpr double BESIDE[4] = {0.0, 1.0, 1.4, 1.85};  // by blocks on the CU
  auto cost = [&](int zc) {
    const int64_t blocks = tiles * ((nz + zc - 1) / zc);
    const int64_t full = blocks / (NUM_CU * resident), rest = blocks % (NUM_CU * resident);
    const double rounds = double(full) * BESIDE[resident] + BESIDE[(rest + NUM_CU - 1) / NUM_CU];
    return rounds * (zc + extra);
  };
  const int longest = std::min(most, nz);
  int best = 1;
  for (int zc = 2; zc <= longest; zc++)
    if (cost(zc) <= cost(best)) best = zc;
  if (cost(best) > (1.0 - margin) * cost(longest)) best = std::max(best, even_chunk(nz, longest));
  return best;
}

// Shapes of the single pass on two-dimensional grids (lc_fused2d.h): tiles of
// TX x TY sites, all with 1024 threads.  A step of a small grid is a chain of
// stages with a barrier between them, and a CU that holds one block spends the
// chain once; so a grid takes the smallest tile of those with which the chip
// goes through the fewest rounds of one tile per CU (16x8 up to 32x20, whose
// radius-3 rectangle of 38x26 points still has one thread per point).  Measured per step in the mixed form on 301x419
// sites: 15.4 us with 530 tiles of 32x8 sites and 512 threads (two rounds of
// blocks), 9.7 us with 210 tiles of 32x20; on 256^2 sites (32x8 tiles)
// 7.4 -> 7.1 us in FP64 and 5.9 -> 5.6 us in FP32, on 128x16 (16x8) 6.0 -> 4.9
// us in FP64, against the same tiles without the overlap of their stages.  With
// more tiles than CUs, smallest with the fewest rounds against 32x20: 20000x7
// (32x8) FP32 10.0 and 12.3 us, 400^2 (32x12) FP64 15.0 and 18.9, 448^2 (32x16)
// FP64 18.8 and 20.6, FP32 9.4 and 10.6.
constexpr int FUSED2D_NTHR = 1024;
constexpr int FUSED2D_PAIR_TX = 16, FUSED2D_PAIR_TY = 8;  // tiles of two steps per launch
constexpr int FUSED2D_NV = 5;
constexpr int fused2d_tx(int v) { return v == 0 ? 16 : 32; }
constexpr int fused2d_ty(int v) { return v < 2 ? 8 : (v == 2 ? 12 : (v == 3 ? 16 : 20)); }

inline int64_t fused2d_tiles(const lc_grid& g, int v) {
  return int64_t((g.nx + fused2d_tx(v) - 1) / fused2d_tx(v)) * ((g.ny + fused2d_ty(v) - 1) / fused2d_ty(v));
}
inline int fused2d_shape(const lc_grid& g) {
  auto rounds = [&](int v) { return (fused2d_tiles(g, v) + NUM_CU - 1) / NUM_CU; };
  int best = 0;
  for (int v = 1; v < FUSED2D_NV; v++)
    if (rounds(v) < rounds(best)) best = v;
  return best;
}
inline bool fused2d_fits(const lc_grid& g) { return fused2d_tiles(g, FUSED2D_NV - 1) <= NUM_CU; }

// The marching single pass (lc_march2d.h): columns of a strip.
constexpr int MARCH_HALO = 4, MARCH_COLS = 64 - 2 * MARCH_HALO;

inline int64_t march_strips(const lc_grid& g) { return (g.nx + MARCH_COLS - 1) / MARCH_COLS; }

// Waves of the march that the chip holds at once: two per SIMD where Q is
// float, one where it is double (the registers set it).  Chunks are cut so
// that a launch has at most that many, in one round, unless the strips alone are
// more; measured per step on 2048^2 sites, FP32: 130 us with 1998 waves of 38
// rows, 160 with 2368 waves of 32 rows (a second round for the rest), 178 with
// 814 waves of 96 rows.
constexpr int march_waves(bool double_q) { return (double_q ? 4 : 8) * NUM_CU; }
inline bool double_q(const lc_grid& g) { return g.precision == LC_FP64 || g.precision == LC_MIXED; }

// Rows per chunk of the marching single pass for n grids of one precision
// together: the fewest whose waves are on the chip at once (all, where the
// strips alone are more).
inline int march_rows(int n, const lc_grid* g) {
  auto waves = [&](int64_t rows) {
    int64_t w = 0;
    for (int k = 0; k < n; k++) w += march_strips(g[k]) * ((g[k].ny + rows - 1) / rows);
    return w;
  };
  int most = 1;
  for (int k = 0; k < n; k++) most = std::max(most, int(g[k].ny));
  int lo = 1, hi = most;  // waves() falls with the rows
  while (lo < hi) {
    const int mid = lo + (hi - lo) / 2;
    if (waves(mid) <= march_waves(double_q(g[0])))
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

// Whether the marching single pass takes n 2D grids (one, or the grids of a
// batch) of at least MARCH_MIN_SITES sites together.  Below that its waves
// have too few rows each to be worth the eight they repeat: 512^2 in FP32
// 15.0 us per step against 10.7 in tiles and 13.5 in two sweeps, in FP64 24.1
// against 19.8 and 20.2; 700^2 18.0 against 21.2 in two sweeps, and 28.4
// against 32.7; 1000^2 27.1 against 35.9, and 45.7 against 58.8.  A strip is 56
// columns wide: grids that fill less than three quarters of their strips stay
// in the other forms, and so do components beyond 32-bit byte offsets.
constexpr int64_t MARCH_MIN_SITES = 640 * 640;
inline bool march_offsets_fit(int n, const lc_grid* g) {
  for (int k = 0; k < n; k++)
    if (int64_t(g[k].nx) * g[k].ny > (int64_t(1) << 32) / 8) return false;
  return true;
}
inline bool march_takes(int n, const lc_grid* g) {
  if (!march_offsets_fit(n, g)) return false;
  int64_t sites = 0, lanes = 0;
  for (int k = 0; k < n; k++) {
    sites += int64_t(g[k].nx) * g[k].ny;
    lanes += march_strips(g[k]) * MARCH_COLS * g[k].ny;
  }
  return sites >= MARCH_MIN_SITES && 4 * sites >= 3 * lanes;
}

// Whether the strips are expected to take at most as long as the two sweeps on
// the grids they take.  The strips go through their chunks in rounds of
// march_waves, and a round that is not full costs `part` of a full one at least;
// a chunk repeats some rows (`more`), and tiles of the sweeps compute rows beyond
// the grid (`idle`, their share of a row's time).  So where the strips alone
// nearly fill the chip, and chunks can not be cut to fill it, the sweeps win.
// Fitted to strips / sweeps measured on 4 to 96 rows, per part of the waves the
// chip holds (FP64): 1.05 rounds 1.32 (8 rows), 1.19 (16), 1.09 (64); half a
// round 1.13 (16), 1.20 (64); full rounds 0.89 (8), 0.77 (16), 0.72 (64).  FP32
// with the compact stencils 0.43 to 1.03 everywhere.  Within 3% the strips stay.
inline bool march_beats_sweeps(int n, const lc_grid* g, bool isotropic) {
  const bool dq = double_q(g[0]);
  if (!dq && g[0].precision != LC_FP32_SR && !isotropic) return true;
  const double part = dq ? 0.59 : 0.51, more = dq ? 2.7 : 1.8, row = dq ? 0.67 : 0.64, idle = 0.5;
  const int rows = march_rows(n, g);
  double waves = 0.0, marched = 0.0, swept = 0.0;
  for (int k = 0; k < n; k++) {
    const double strips = double(march_strips(g[k])), chunks = (g[k].ny + rows - 1) / rows;
    waves += strips * chunks;
    marched += strips * g[k].ny;
    swept += strips * (g[k].ny + idle * ((g[k].ny + 7) / 8 * 8 - g[k].ny));
  }
  const double most = march_waves(dq);
  const double full = double(int64_t(waves / most)), rest = waves / most - full;
  const double rounds = full + (rest > 0.0 ? part + (1.0 - part) * rest : 0.0);
  return row * rounds * most * (marched / waves + more) <= 1.03 * swept;
}

// The form of a step of a two-dimensional grid in the single pass.
enum Form2d { FORM_TILES, FORM_PAIRS, FORM_STRIPS };
inline Form2d fused2d_form(const lc_grid& g, bool isotropic, bool timed) {
  if (march_takes(1, &g)) return FORM_STRIPS;
  // two steps go in a launch where every 16x8 tile has a CU; not where
  // launches are timed one by one, nor in FP64 with the isotropic stencils,
  // whose larger first step spills (64^2 6.6 us per step in pairs against 6.2)
  if (fused2d_tiles(g, 0) <= NUM_CU && !timed && !(g.precision == LC_FP64 && isotropic)) return FORM_PAIRS;
  return FORM_TILES;
}

// Whether the tiles of the single pass are expected to take at most as long as
// the two sweeps on a grid with more tiles than CUs, below the strips' sites: the
// tiles go through the chip in rounds, a part of a round at `part` of a whole one
// at least; the sweeps' time grows with their blocks of 32x8 sites.  Fitted to
// 2184 measured grids of 70 000 to 405 000 sites (1 to 600 rows or columns),
// tiles / sweeps: Q float 0.55 to 0.96 in two rounds (512^2 FP32 10.7 and 13.5
// us), 0.61 to 1.15 in three and four, 0.83 to 1.76 in more (300000x1 1.67); Q
// double 0.58 to 1.16 in two rounds (448^2 FP64 18.8 and 18.4 us, 33x4454 0.87),
// 0.74 to 1.35 in three and four, up to 2.2 in more.  On average the choice costs
// 0.2% over the faster one (0.6% in FP32), at most 19%.
inline bool tiles_beat_sweeps(const lc_grid& g) {
  const bool dq = double_q(g);
  const double launch = dq ? 0.20 : -0.09, part = dq ? 0.61 : 0.62, block = (dq ? 1.54 : 2.64) / 1024;
  const double round[2][FUSED2D_NV] = {{0.93, 0.93, 1.13, 1.44, 1.67}, {0.74, 0.74, 0.90, 1.10, 1.25}};  // by shape
  const int v = fused2d_shape(g);
  const double tiles = double(fused2d_tiles(g, v)) / NUM_CU, full = double(int64_t(tiles)), rest = tiles - full;
  const double rounds = full + (rest > 0.0 ? part + (1.0 - part) * rest : 0.0);
  const double blocks = double((g.nx + 31) / 32) * ((g.ny + 7) / 8);
  return launch + round[dq][v] * rounds <= 1.0 + block * blocks;
}

// The variant AUTO runs (bit-identical results).  The two sweeps in 3D.  In 2D
// the single pass, in tiles where each has a CU of its own (launches are
// latency bound there: 256^2 5.6 us per step in FP32 against 9.0 in two sweeps,
// 7.1 against 10.0 in FP64; 384^2 8.0 against 11.1 and 11.5 against 14.7),
// marching on large grids; it or the two sweeps, whichever is expected to be
// faster, in between and where the strips are many.
inline int auto_variant(const lc_grid& g, bool isotropic) {
  if (g.lattice != LC_D2Q9) return LC_VARIANT_SPLIT;
  if (fused2d_fits(g)) return LC_VARIANT_FUSED;
  const bool single = int64_t(g.nx) * g.ny < MARCH_MIN_SITES
                          ? tiles_beat_sweeps(g)
                          : march_takes(1, &g) && march_beats_sweeps(1, &g, isotropic);
  return single ? LC_VARIANT_FUSED : LC_VARIANT_SPLIT;
}

// Tiles of the reverse step (lc_vjp.h), one block of REV_NTHR threads each:
// 16x16 sites, or 40x4 on grids of few rows, the one with fewer rounds of one
// tile per CU.  A step of a segment on 30000x3 sites: 116.9 us in 16x16, 56.7 in
// 40x4 (60.2 in the 64x4 blocks of three kernels).
constexpr int REV_NTHR = 768, REV_NV = 2;
constexpr int rev_tx(int v) { return v == 0 ? 16 : 40; }
constexpr int rev_ty(int v) { return v == 0 ? 16 : 4; }
inline int64_t rev_tiles(const lc_grid& g, int v) {
  return (int64_t(g.nx) + rev_tx(v) - 1) / rev_tx(v) * ((g.ny + rev_ty(v) - 1) / rev_ty(v));
}
inline int rev_shape(const lc_grid& g) {
  auto rounds = [&](int v) { return (rev_tiles(g, v) + NUM_CU - 1) / NUM_CU; };
  return rounds(1) < rounds(0) ? 1 : 0;
}

}  // namespace lc
