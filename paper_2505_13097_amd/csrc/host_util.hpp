// host_util.hpp -- host-side helpers shared by the translation units of
// the library: kernel variant table, type dispatch, error macro, device
// guard and small launch wrappers.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <type_traits>

#include "kernels.hpp"
#include "lbm_stefan.h"
#include "sweep2d.hpp"

namespace irebm {

// A kernel variant: block of bx x by threads, each thread updating npt
// nodes bx apart along x; the tile is (bx * npt) x by nodes, and one block
// sweeps `rows` tiles stacked along y.  nt: stores bypass the caches
// (non-temporal); rev: the item order is reversed on every other step, so
// that the rows written last (still in the memory-side cache) are read
// first.  tb: two steps per launch (step2_kernel): a window of bx columns
// (bx - 4 written), by rows per pass, `rows` rows per block, non-temporal
// stores; where the lattice is large enough, and in the batched form, up to
// four steps by sweeping waves instead (sweep_kernel, segments of `rows`
// rows).  res: D1Q3 lattices of at most kResident1D nodes run many steps
// per launch in one workgroup (resident1d_kernel); others take the default
// one-step tiling.  tb = 2: as tb = 1, more segment lengths.  lib: what the
// library takes by itself (params.variant = -1): several steps per launch or
// a one-step tiling, by lattice.
struct Variant {
  int bx, by, npt, nt, rev, rows, tb, res, lib;
};

inline const Variant *variants(int q, int *n) {
  static const Variant v1[] = {{256, 1, 1, 0, 0, 1, 0}, {128, 1, 1, 0, 0, 1, 0},
                               {64, 1, 1, 0, 0, 1, 0},  {256, 1, 2, 0, 0, 1, 0},
                               {1024, 1, 2, 0, 0, 1, 0, 1}};
  static const Variant v2[] = {
      {64, 4, 1, 0, 0, 1, 0}, {256, 1, 1, 0, 0, 1, 0}, {128, 2, 1, 0, 0, 1, 0},
      {64, 4, 2, 0, 0, 1, 0}, {128, 2, 2, 0, 0, 1, 0}, {256, 1, 2, 0, 0, 1, 0},
      {64, 2, 2, 0, 0, 1, 0}, {64, 4, 4, 0, 0, 1, 0},  {64, 4, 2, 1, 0, 1, 0},
      {64, 4, 2, 0, 1, 1, 0}, {64, 4, 2, 1, 1, 1, 0},  {128, 2, 2, 0, 1, 1, 0},
      {64, 4, 2, 1, 0, 2, 0}, {64, 4, 2, 1, 0, 4, 0},  {64, 4, 2, 1, 0, 8, 0},
      {64, 4, 2, 0, 0, 4, 0}, {64, 4, 1, 1, 0, 4, 0},  {64, 4, 2, 1, 1, 4, 0},
      {128, 2, 2, 1, 0, 4, 0}, {64, 4, 2, 1, 0, 16, 0}, {64, 1, 1, 0, 0, 1, 0},
      {64, 2, 1, 0, 0, 1, 0},
      {256, 2, 1, 1, 0, 32, 1},  {256, 2, 1, 1, 0, 64, 1},
      {128, 2, 1, 1, 0, 16, 1},  {128, 2, 1, 1, 0, 24, 1},
      {128, 2, 1, 1, 0, 32, 1},  {128, 2, 1, 1, 0, 64, 1},
      {128, 4, 1, 1, 0, 32, 1},  {128, 4, 1, 1, 0, 64, 1},
      {128, 2, 1, 1, 0, 16, 2},  {128, 2, 1, 1, 0, 24, 2},
      {128, 2, 1, 1, 0, 32, 2},  {128, 2, 1, 1, 0, 64, 2},
      {128, 4, 1, 1, 0, 32, 2},  {128, 2, 1, 1, 0, 96, 2},
      {128, 2, 1, 1, 0, 128, 2},
      {64, 4, 2, 0, 0, 1, 0, 0, 1}};
  if (q == 3) {
    *n = (int)(sizeof(v1) / sizeof(Variant));
    return v1;
  }
  *n = (int)(sizeof(v2) / sizeof(Variant));
  return v2;
}
constexpr int kDefaultVariant1D = 0;
constexpr int kResidentVariant1D = 4;
constexpr int kDefaultVariant2D = 3;
constexpr int kLibraryVariant2D = 37;
// 128x2/t2s/r32/nt: the batched form's default (sweeping waves)
constexpr int kSweepVariant2D = 32;

inline int64_t tiles_x_for(const Variant &v, int64_t nx) {
  const int64_t tw = (int64_t)v.bx * v.npt;
  return (nx + tw - 1) / tw;
}
inline int64_t tiles_y_for(const Variant &v, int64_t ny) {
  return (ny + v.by - 1) / v.by;
}
// work items (one block each) of an nx x ny lattice
inline int64_t items_for(const Variant &v, int64_t nx, int64_t ny) {
  if (v.tb)
    return ((nx + v.bx - 5) / (v.bx - 4)) * ((ny + v.rows - 1) / v.rows);
  return tiles_x_for(v, nx) * ((tiles_y_for(v, ny) + v.rows - 1) / v.rows);
}
// tile grid and work items of A for variant v
// (two-step variants: tiles_x strips of bx - 4 columns, tiles_y segments
// of `rows` rows, group = rows)
inline void set_tiling(StepArgs *A, const Variant &v) {
  if (v.tb) {
    A->tiles_x = (A->nx + v.bx - 5) / (v.bx - 4);
    A->tiles_y = (A->ny + v.rows - 1) / v.rows;
  } else {
    A->tiles_x = (int32_t)tiles_x_for(v, A->nx);
    A->tiles_y = (int32_t)tiles_y_for(v, A->ny);
  }
  A->group = v.rows;
  A->nitems = (int32_t)items_for(v, A->nx, A->ny);
  A->per_xcd = (A->nitems + 7) / 8;
}

// LDS a block of tile_kernel may take: what a launch gets unasked (the
// largest tile, 20 x 20 nodes of D2Q9 FP64, takes 29 KB)
constexpr size_t kTileLds = 64 * 1024;

// The library's choice for tile_kernel on an nx x ny lattice (q populations
// of s bytes), where sweep_kernel is not taken: steps per launch k and the
// side of a tile.  Measured on square lattices (us per step, the one-step
// kernel's best tiling -> tile_kernel, D2Q5 FP64 freezing; D2Q9, FP32 and the
// melting set-up alike):
//   IREBM: a step is one Newton solve long, so small tiles that put a block
//   on every CU and few halo nodes win, and the kernel stops paying where
//   the halo's solves outweigh the launch: 60^2 8.9 -> 5.4, 151^2 8.9 -> 5.6
//   (k 4, side 8), 201^2 9.1 -> 6.2, 301^2 9.7 -> 7.8 (3, 10), 351^2 10.0 ->
//   8.8 (2, 12), 401^2 10.4 -> 10.8.
//   EEBM: no solve, so more steps: 101^2 4.5 -> 2.5 (6, 8), 201^2 4.8 -> 2.7
//   (4, 8); larger ones sweep.
// Lattices too thin for a strip, above 60000 nodes: their tiles are mostly
// wall.  With solves single steps (tiles / so: 33 x 2946 melted 12.4 / 9.0, 35
// x 2878 freezing 11.4 / 10.5, 25812 x 4 12.1 / 10.9); without, tiles of 14 a
// side up to 100000 nodes in rows of the lattice's length (3250 x 20 D2Q9 FP32
// 4.4 / 5.5, 6500 x 20 6.8 / 6.1, 22757 x 11 12.5 / 7.4) and to 200000 where
// rows are short and a wave's loads with them (20 x 6500 8.7 / 9.9, 57 x 1136
// 4.3 / 6.8, 30 x 10000 15.8 / 12.9).
inline TilePlan tile_plan(int q, size_t s, bool eebm, int64_t nx,
                          int64_t ny) {
  const int64_t n = nx * ny;
  int k = 0, side = 0;
  if (n > 60000 && (nx < 64 || ny < 64)) {
    if (eebm && n <= (nx < 64 ? 200000 : 100000)) k = 4, side = 14;
  } else if (!eebm) {
    if (n <= 30000) k = 4, side = 8;
    else if (n <= 110000) k = 3, side = 10;
    else if (n <= 130000) k = 2, side = 12;
  } else {
    if (n <= 15000) k = 6, side = 8;
    else if (n <= 60000) k = 4, side = 8;
  }
  TilePlan P;
  if (k == 0) return P;
  P.k = k;
  P.ntx = (int32_t)((nx + side - 1) / side);
  P.nty = (int32_t)((ny + side - 1) / side);
  // tiles of nearly equal sizes, at least two nodes wide
  P.rx = (int32_t)((nx + P.ntx - 1) / P.ntx) + 2 * k;
  P.ry = (int32_t)((ny + P.nty - 1) / P.nty) + 2 * k;
  if (P.rx * P.ry > 1024 || (size_t)P.rx * P.ry * q * s > kTileLds ||
      nx / P.ntx < 2 || ny / P.nty < 2)
    return TilePlan();
  return P;
}

// bit i: an IREBM front starts at wall i: a Dirichlet wall that is hot (a
// profile, or a temperature off phi's lower plateau), or any Dirichlet wall
// where none is hot (a melt that freezes)
inline int front_walls(const lbm_stefan_params &p, bool *hot) {
  int h = 0, d = 0;
  for (int i = 0; i < 4; ++i)
    if (p.bc[i] == LBM_BC_DIRICHLET) {
      d |= 1 << i;
      if (p.wall_profile[i] || p.wall_T[i] >= p.t_m - 20.0 * p.delta)
        h |= 1 << i;
    }
  *hot = h != 0;
  return h ? h : d;
}

// The partition of a 2D lattice for sweep_kernel at up to k steps per
// launch, segments of `rows` rows; an empty plan when the lattice is too
// small for the frame and a strip.  The frame is two tiles deep where a
// front starts (a strip that reaches the front solves in every row: the
// 8192^2 cavity took 380 us per step with one tile, 324 with two, 347 and 330
// with three and four, segments of 32 rows everywhere), one at the other
// walls.  The strip next to it
// goes in segments of `frows` rows, for a front that has left the frame:
// 8 in a batch (the one named at batch_plan takes 622 us with segments as
// everywhere, 505 with 8, 520 with 4), 2 in a single lattice that sweeps
// wherever its front is (route_lattice).
inline SweepPlan sweep_plan(const lbm_stefan_params &p, int k, int rows,
                            int frows, bool nt) {
  SweepPlan P;
  const int T = frame_tile(k), w = 64 - 2 * k;
  const int nx = (int)p.nx, ny = (int)p.ny;
  const bool px = p.bc[0] == LBM_BC_PERIODIC, py = p.bc[2] == LBM_BC_PERIODIC;
  bool hot;
  const int front = p.scheme == LBM_SCHEME_IREBM ? front_walls(p, &hot) : 0;
  auto band = [&](int i) { return front >> i & 1 ? 2 : 1; };
  P.tile = T;
  P.xb = nx;
  P.yb = ny;
  if (!px) {
    P.nleft = band(0);
    P.nright = band(1);
    P.nside = (ny + T - 1) / T;
    P.xa = P.nleft * T;
    P.xb = nx - P.nright * T;
  }
  if (!py) {
    P.nbottom = band(2);
    P.ntop = band(3);
    P.ya = P.nbottom * T;
    P.yb = ny - P.ntop * T;
  }
  if (P.xb - P.xa < 64 || P.yb - P.ya < 16) return SweepPlan();
  P.nacross = (P.xb - P.xa + T - 1) / T;
  P.fl = front & 1;
  P.fr = front >> 1 & 1;
  P.cut(w);
  P.rows = rows;
  P.frows = frows < rows ? frows : rows;
  P.fseg = (P.yb - P.ya + P.frows - 1) / P.frows;
  P.nseg = (P.yb - P.ya + rows - 1) / rows;
  P.nt = nt ? 1 : 0;
  P.k = k;
  return P;
}

// Where a front stands off the walls, the waves that hold it solve in every
// row, one after the other, 2 to 4 us a row at the slowest lane, on top of the
// sweep's own time: a chain of k rows + k (k - 1) of them per launch, against
// k single steps that each pass over the state at 5 TB/s.  The sweep itself
// takes 0.37 of those on lattices of 60 us a step and more, 0.5 to 0.6 below,
// which leaves 0.16 and 0.105 rows for every us.  us per step, sweeps with the
// front in the frame / at column 100 / half way / single steps, half way: 900
// x 700 D2Q9 FP64 10 / 40 / 47 / 21, 2048^2 D2Q5 FP32 18 / 58 / 71 / 38,
// 4096^2 68 / 142 / 199 / 151, 2048^2 D2Q9 FP64 50 / 98 / 129 / 134, 8192^2
// D2Q9 FP32 344 / 464 / 601 / 925.  So a lattice on which such a chain costs more than the
// single steps leaves the sweeps where a wave holds more rows with solves
// than they pay for (RouteCtl), and one on which it does not sweeps always.
// The strip next to a wall where a front starts goes in segments of `frows`
// rows where they are short enough for that.
inline void route_lattice(SweepPlan *P, const lbm_stefan_params &p, int frows) {
  if (P->k == 0 || p.scheme != LBM_SCHEME_IREBM) return;
  const double step_us = 2.0 * p.q * (p.storage == LBM_STORE_F64 ? 8 : 4) *
                         (double)p.nx * (double)p.ny / 5e6;
  const double rows = P->k * step_us * (step_us >= 60.0 ? 0.16 : 0.105);
  P->chain_max = (int32_t)(rows < 1e6 ? rows : 1e6);
  P->gated = P->k * P->rows + P->k * (P->k - 1) > P->chain_max;
  if (P->k * frows + P->k * (P->k - 1) > P->chain_max) {
    P->fl = P->fr = 0;
    P->cut(64 - 2 * P->k);
  } else {
    P->frows = frows < P->rows ? frows : P->rows;
    P->fseg = (P->yb - P->ya + P->frows - 1) / P->frows;
  }
}

// nodes above which the two routes' launches go on streams of their own
// (advance_routed)
constexpr int64_t kRouteBeside = 2000000;

// IREBM lattices (and batches) of fewer nodes do not sweep: the launches of
// the route not taken are too large a part of a step (front half way, default
// with them / single steps: 900 x 700 D2Q9 FP64 24.6 / 23.6 us, 1001 x 777
// D2Q5 FP32 14.1 / 13.2), and in a batch of small lattices most nodes lie in
// the frame (48 FP32 D2Q5 lattices of 64^2 to 256^2, 1.4M nodes, 28.6 us per
// step, 37.6 in sweeps).
inline int64_t sweep_nodes(int storage) {
  return storage == LBM_STORE_F64 ? 600000 : 1500000;
}

// rows per segment: enough waves for the chip, few halo rows (8 on 512^2, 16
// on 2048^2, 32 on 8192^2)
inline int sweep_rows(int64_t ny) {
  const int64_t rows = (ny / 128 + 3) / 4 * 4;
  return (int)(rows < 8 ? 8 : (rows > 32 ? 32 : rows));
}

// sweep_kernel under the library default (an empty plan: tile_kernel or
// single steps).  Measured (us per step, the best one-step tiling -> here):
// IREBM heated at a wall, the front in the frame (beyond it: route_lattice),
// 1001 x 777 D2Q9 FP64 21.3 -> 12.9, 2048^2 D2Q5 FP32 31.6 -> 20.3, D2Q9 FP64
// 134 -> 50, 8192^2 D2Q9 FP32 921 -> 345; EEBM 201^2 D2Q9 FP64 5.8 -> 3.4
// (tile_kernel 4.2), 801^2 18.2 -> 7.9, 2048^2 D2Q5 FP32 28.0 -> 11.4.  A
// freezing IREBM lattice (no hot wall) keeps single steps: its bulk is
// liquid, so the solves of a wave, one after the other, cost more than the
// traffic saved (801^2 D2Q5 21.2 -> 22.4).
// Three steps instead of four on FP32 lattices that the memory-side cache
// holds (2048^2 D2Q9 31.9 against 34.6).
// With walls above and below, few rows are left between the tiles at them, and
// below 56 rows in FP64, 96 in FP32, single steps are ahead (front in the
// frame / so, D2Q9: FP64 700000 nodes in 48 rows 27.4 / 21.2, 2M in 48 70.2 /
// 71.6, in 63 60.6 / 68.7; FP32 1.55M in 48 37.3 / 24.7, in 80 27.5 / 23.1, 4M
// in 80 65.3 / 67.3, in 120 54.3 / 70.2).
inline SweepPlan sweep_default(const lbm_stefan_params &p) {
  const int64_t n = p.nx * p.ny;
  if (p.dim != 2 || p.scheme == LBM_SCHEME_ILFBM) return SweepPlan();
  const bool eebm = p.scheme == LBM_SCHEME_EEBM;
  bool hot;
  front_walls(p, &hot);
  if (n <= (eebm ? 30000 : sweep_nodes(p.storage)) || (!eebm && !hot))
    return SweepPlan();
  if (!eebm && p.bc[2] != LBM_BC_PERIODIC &&
      p.ny < (p.storage == LBM_STORE_F64 ? 56 : 96))
    return SweepPlan();
  const int k = !eebm && p.storage == LBM_STORE_F32 && n < 6000000 ? 3 : 4;
  SweepPlan P = sweep_plan(p, k, sweep_rows(p.ny), sweep_rows(p.ny),
                           n > (1 << 24));
  route_lattice(&P, p, 2);
  return P;
}

// Rows per segment in a batch of `nodes` nodes under a two-step variant: its
// own, at most 32 (48 FP32 D2Q5 lattices of 64^2 to 1024^2 take 505 us per four
// steps with 32 and 64 rows, 560 with 16 and 128; two-step launches of
// step2_kernel, split by quiet and solving items, took 1040), and fewer in
// small batches, which leave the chip short of waves otherwise (6 EEBM lattices
// of 600 x 45, 9.0 us per step with 32 rows, 3.8 with 8, single steps 6.8).
inline int batch_rows(const Variant &v, int64_t nodes) {
  const int64_t most = nodes / 229376 / 4 * 4;   // (56 columns, 4096 waves)
  const int64_t rows = most < 8 ? 8 : (most > 32 ? 32 : most);
  return (int)(v.rows < rows ? v.rows : rows);
}

// An instance of such a batch: its plan, or tiles alone where no strip fits.
inline SweepPlan batch_plan(const lbm_stefan_params &p, const Variant &v,
                            int64_t nodes) {
  SweepPlan P = sweep_plan(p, 4, batch_rows(v, nodes), 8, v.nt != 0);
  if (P.k > 0) return P;
  P.k = 4;
  P.tile = frame_tile(4);
  P.nleft = (int32_t)((p.nx + P.tile - 1) / P.tile);
  P.nside = (int32_t)((p.ny + P.tile - 1) / P.tile);
  P.xa = P.xb = (int32_t)p.nx;
  P.yb = (int32_t)p.ny;
  P.nacross = P.strips = P.rows = 1;
  return P;
}

// sweep_kernel under a two-step variant, in segments of at most its rows
inline SweepPlan sweep_variant(const lbm_stefan_params &p, const Variant &v) {
  if (p.dim != 2 || p.scheme == LBM_SCHEME_ILFBM || !v.tb) return SweepPlan();
  for (int i = 0; i < 4; ++i)
    if (p.bc[i] == LBM_BC_NEUMANN) return SweepPlan();
  if (p.scheme == LBM_SCHEME_IREBM && p.nx * p.ny <= sweep_nodes(p.storage))
    return SweepPlan();
  const int rows = v.rows < sweep_rows(p.ny) ? v.rows : sweep_rows(p.ny);
  SweepPlan P = sweep_plan(p, 4, rows, rows, v.nt != 0);
  route_lattice(&P, p, 2);
  return P;
}

// The one-step tiling of the library default: one node per thread and 64 x
// 1 blocks (index 20) while the lattice leaves the chip short of waves (one
// node's chain per wave: 201^2 D2Q5 FP64 freezing 12.4 -> 9.2 us per step,
// 512^2 D2Q9 FP64 14.0 -> 11.5, 1001 x 777 23.3 -> 21.5; FP32 512^2 D2Q5
// 8.3 -> 7.5, 1001 x 777 11.5 against 13.1), 128 x 4 tiles with two nodes
// per thread (kDefaultVariant2D) above, and where there are many rows: those
// deal the columns at x = 0 out, so that a front there falls into one wave of
// four rows instead of one a row (64 x 1 against 128 x 4: 215 x 1838 D2Q5 FP32
// 11.5 / 9.2, 100 x 3000 11.8 / 10.4, 300 x 700 7.9 / 8.0, melted 9.0 / 8.6;
// FP64 D2Q9 11 x 22757 56 / 42, 130 x 6000 43.7 / 39.0 freezing, 62 x 1951 15.9
// / 13.8 freezing, 64 x 4000 17.3 / 18.8).
inline int one_step_default(size_t s, int64_t nodes, int64_t ny) {
  const bool small = s == 8 ? nodes <= 1200000 && ny <= 1500
                            : nodes <= 350000 && ny <= 600;
  return small ? 20 : kDefaultVariant2D;
}

// doubles of scratch that stats_async needs for n slots
inline int64_t stats_partials(int64_t n) {
  return 5 * ((n + kStatsChunk - 1) / kStatsChunk);
}

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

inline unsigned blocks_for(int64_t n, int t) {
  return (unsigned)((n + t - 1) / t);
}

struct DeviceGuard {
  int prev = -1;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess || prev == dev ||
        hipSetDevice(dev) != hipSuccess)
      prev = -1;
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

template <int Q>
using QT = std::integral_constant<int, Q>;
template <typename T>
struct TT {
  using type = T;
};

// calls f(QT<Q>{}, TT<S>{}) for a lattice and a storage type
template <typename F>
hipError_t dispatch_qs(int q, int storage, F &&f) {
  const bool f32 = storage == LBM_STORE_F32;
  switch (q) {
    case 3:
      return f32 ? f(QT<3>{}, TT<float>{}) : f(QT<3>{}, TT<double>{});
    case 5:
      return f32 ? f(QT<5>{}, TT<float>{}) : f(QT<5>{}, TT<double>{});
    default:
      return f32 ? f(QT<9>{}, TT<float>{}) : f(QT<9>{}, TT<double>{});
  }
}

// as dispatch_qs, also for the 3D lattices (q = 7, 19): for the kernels
// that only loop over the q planes (fields, energy, front)
template <typename F>
hipError_t dispatch_qs_all(int q, int storage, F &&f) {
  const bool f32 = storage == LBM_STORE_F32;
  if (q == 7) return f32 ? f(QT<7>{}, TT<float>{}) : f(QT<7>{}, TT<double>{});
  if (q == 19)
    return f32 ? f(QT<19>{}, TT<float>{}) : f(QT<19>{}, TT<double>{});
  return dispatch_qs(q, storage, f);
}

// nodes of a lattice, and its rows along x
inline int64_t lattice_nodes(const lbm_stefan_params &p) {
  return p.nx * p.ny * (p.dim == 3 ? p.nz : 1);
}
inline int64_t lattice_rows(const lbm_stefan_params &p) {
  return p.ny * (p.dim == 3 ? p.nz : 1);
}

#define QS_TYPES(qt, tt)                  \
  constexpr int Q = decltype(qt)::value; \
  using S = typename decltype(tt)::type

inline hipError_t zero_async(void *p, size_t bytes, hipStream_t s) {
  const int64_t n = (int64_t)(bytes / 8);
  if (n <= 0) return hipSuccess;
  zero_kernel<<<blocks_for(n, 256), 256, 0, s>>>((uint64_t *)p, n);
  return hipGetLastError();
}

// E = sum [T + phi(T)/Ste] (EEBM: sum H) of the state `src` of a lattice
// with params p into *out (device), using `partials` (>= ceil(nodes /
// kEnergyChunk) doubles) as scratch
inline hipError_t energy_async(const lbm_stefan_params &p, const void *src,
                               double *partials, double *out,
                               hipStream_t stream,
                               const double *lf = nullptr) {
  const int64_t n = lattice_nodes(p);
  return dispatch_qs_all(p.q, p.storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    const int64_t parts = (n + kEnergyChunk - 1) / kEnergyChunk;
    energy_partial_kernel<Q, S><<<(unsigned)parts, 256, 0, stream>>>(
        (const S *)src, n, p.scheme == LBM_SCHEME_EEBM, p.t_m, 1.0 / p.delta,
        1.0 / p.ste, lf, partials);
    sum_kernel<<<1, 256, 0, stream>>>(partials, parts, out);
    return hipGetLastError();
  });
}

// per-row front of the state `src` of a lattice with params p (p.dx > 0)
// into out[0..rows) (device; rows ny, or nz * ny in 3D); lf: the ILFBM
// liquid fraction plane
inline hipError_t front_async(const lbm_stefan_params &p, const void *src,
                              int mode, double *out, hipStream_t stream,
                              const double *lf = nullptr) {
  const int eebm = p.scheme == LBM_SCHEME_EEBM;
  const int64_t n = lattice_nodes(p);
  const unsigned rows = (unsigned)lattice_rows(p);
  return dispatch_qs_all(p.q, p.storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    if (mode == LBM_FRONT_LIQUID_INTEGRAL)
      front_integral_kernel<Q, S><<<rows, 256, 0, stream>>>(
          (const S *)src, n, (int)p.nx, eebm, p.t_m, 1.0 / p.delta, p.ste,
          lf, p.dx, out);
    else
      front_crossing_kernel<Q, S><<<rows, 256, 0, stream>>>(
          (const S *)src, n, (int)p.nx, eebm, p.t_m, 1.0 / p.ste, p.dx, out);
    return hipGetLastError();
  });
}

// temperature of every node of the state `src` into T (device doubles)
inline hipError_t temperature_async(const lbm_stefan_params &p,
                                    const void *src, double *T,
                                    hipStream_t stream) {
  const int64_t n = lattice_nodes(p);
  return dispatch_qs_all(p.q, p.storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    temp_kernel<Q, S><<<blocks_for(n, 256), 256, 0, stream>>>(
        (const S *)src, n, p.scheme == LBM_SCHEME_EEBM, p.t_m, 1.0 / p.ste,
        T);
    return hipGetLastError();
  });
}

// liquid fraction of every node of the state `src` into out (device)
inline hipError_t liquid_async(const lbm_stefan_params &p, const void *src,
                               const double *lf, double *out,
                               hipStream_t stream) {
  const int64_t n = lattice_nodes(p);
  return dispatch_qs_all(p.q, p.storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    liquid_kernel<Q, S><<<blocks_for(n, 256), 256, 0, stream>>>(
        (const S *)src, n, p.scheme == LBM_SCHEME_EEBM, p.t_m, 1.0 / p.delta,
        p.ste, lf, out);
    return hipGetLastError();
  });
}

// equilibrium initial state of the lattice described by A (A.dst), and
// the ILFBM liquid fraction into lf when given
inline hipError_t init_async(int q, int storage, const StepArgs &A,
                             const double *T0, hipStream_t stream,
                             double *lf = nullptr) {
  return dispatch_qs(q, storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    init_kernel<Q, S><<<blocks_for(A.plane, 256), 256, 0, stream>>>(A, T0,
                                                                     lf);
    return hipGetLastError();
  });
}

}  // namespace irebm

#define HIPCHK(h, expr)                                                   \
  do {                                                                    \
    hipError_t e_ = (expr);                                               \
    if (e_ != hipSuccess)                                                 \
      return irebm::fail((h), LBM_STEFAN_EDEVICE,                         \
                         std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)
