// sweep2d.hpp -- K time steps of a large 2D lattice per launch: waves that
// sweep strips of columns upward with every level's rows in registers, and
// a frame of small tiles in LDS along the walls.
//
// What bounds a large lattice is the traffic of one state in and one out
// per step, so K steps share one pass.  Level l of the sweep is the state l
// steps on, and its row y needs rows y - 1, y and y + 1 of level l - 1.  A
// wave owns a window of 64 columns, a lane each, and loads one row at a
// time; with row r of level 0 it computes row r - 1 of level 1, r - 2 of
// level 2, ..., r - K of level K, which it stores.  What a level keeps for
// the next one fits in registers: of its last row the populations that stay
// in the row and the sum T, of that row and the one before those that move
// up; those that move down are used at once.  Neighbours along x are the
// next lanes (DPP wave shifts).  So there is no LDS traffic and no barrier,
// and a wave that runs Newton solves holds up no other.  The window loses a
// column a side per level and a segment of rows K rows a side, which the
// neighbouring waves compute as well: 64 - 2 K columns and the segment's
// rows are stored and counted.
//
// The sweep knows no walls.  The frame (one or two tiles along the walls of an
// axis that is not periodic) is advanced by blocks of the same launch as tiles
// of 16 x 16 nodes with their halo (tile_body): the closures stay out of the
// sweep's registers, and the front of a heated wall, a Newton solve per row
// and level there, is worked on by many waves at once instead of row after row
// by one.  A front that has left the frame is that serial chain again, and
// more so the longer a wave's segment: on lattices where it costs more than
// the traffic saved, a group of steps is issued as sweeps and as single steps,
// and the device's RouteCtl, from what the last sweep (or a scan of the state)
// held, says which of them leaves at once (900 x 700 D2Q9 FP64, front half
// way: 47 us per step in sweeps, 24 so; route_lattice has the line).
// Every update is the code and the operands of the one-step kernel, so the
// states are those of K single steps bit for bit.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "kernels.hpp"

namespace irebm {

// the value of the lane one below or above (0 at the wave's ends)
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                         0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  union { double d; int i[2]; } u{v};
  u.i[0] = __builtin_amdgcn_update_dpp(0, u.i[0], CTRL, 0xf, 0xf, true);
  u.i[1] = __builtin_amdgcn_update_dpp(0, u.i[1], CTRL, 0xf, 0xf, true);
  return u.d;
}
constexpr int kLaneBelow = 0x138, kLaneAbove = 0x130;  // wave_shr, wave_shl

// side of a frame tile's region and columns (rows) it advances k steps
constexpr int kFrameSide = 16;
constexpr int frame_tile(int k) { return kFrameSide - 2 * k; }

// what level l - 1 keeps for level l: of its last row the populations that
// stay in the row (directions 0, 1, 3), those that move up (2, 5, 6) and
// the sum T, of the row before those that move up
template <int Q, typename S>
struct SweepRow {
  static constexpr int UP = Q == 9 ? 3 : 1;
  S mid[3], up[UP], up1[UP];
  double th;
};
// what nband rows with a node in or near the band and nliquid rows of solid
// and liquid nodes cost the chip, in units of 0.45 ns (measured on batches of
// 12 to 400 lattices: 0.45 ns a liquid row, 0.7 to 2.2 ns one with the band)
__host__ __device__ constexpr int route_units(int nband, int nliquid) {
  return 5 * nband + nliquid;
}

// index of direction i among those kept (rest, +x, -x; the upward ones)
constexpr int sweep_mid(int i) { return i == 0 ? 0 : (i == 1 ? 1 : 2); }
constexpr int sweep_up(int i) { return i == 2 ? 0 : (i == 5 ? 1 : 2); }

// Work of one lattice at up to k steps per launch: the frame's tiles, a
// block of 256 threads each, then the strips of [xa, xb) x [ya, yb) in
// segments of `rows` rows, a wave each, strip-fastest, so that neighbouring
// strips share halo lines in an L2.  The strip next to a side band where a
// front starts (nfl, nfr: the first, the last) is cut into shorter segments
// and goes first: a front that has left the band puts a solve into every row
// of it, one after the other.  Each XCD takes one contiguous part of
// either list, the frame's (which hold the solves and take longest) first.
struct SweepPlan {
  int32_t k = 0;                       // 0: the lattice takes another kernel
  int32_t xa = 0, xb = 0, ya = 0, yb = 0;
  int32_t tile = 0;                    // side of a frame tile
  int32_t nleft = 0, nright = 0;       // tile columns of the side bands
  int32_t nside = 0;                   // tile rows of the side bands (whole
                                       // height)
  int32_t nbottom = 0, ntop = 0;       // tile rows of the other bands
  int32_t nacross = 0;                 // their tile columns, over [xa, xb)
  int32_t strips = 0, rows = 0, nseg = 0;
  int32_t fl = 0, fr = 0;              // a front starts at x = 0, at nx - 1
  int32_t nfl = 0, nfr = 0, frows = 1, fseg = 0;
  int32_t nt = 0;
  // 1: the lattice (the batch) goes by single steps where a sweep holds a
  // wave of more than chain_max rows with solves
  int32_t gated = 0, chain_max = 0;
  RouteCtl *ctl = nullptr;             // null: the launch always runs
  // strips of w columns
  void cut(int w) {
    strips = (xb - xa + w - 1) / w;
    nfl = fl && strips > 0 ? 1 : 0;
    nfr = fr && strips > nfl ? 1 : 0;
  }
  __host__ __device__ int64_t tiles() const {
    return (int64_t)(nleft + nright) * nside +
           (int64_t)(nbottom + ntop) * nacross;
  }
  __host__ __device__ int64_t waves() const {
    return (int64_t)(nfl + nfr) * fseg + (int64_t)(strips - nfl - nfr) * nseg;
  }
  __host__ __device__ int64_t slots() const { return tiles() + waves(); }
};

// One wave: columns [x0, x1) (at most 64 - 2 K), rows [y0, y1), K steps
// from src to dst.  The K columns and rows around them are lattice nodes
// (the frame, or wrapped on a periodic axis).  nt: stores bypass the
// caches.  MID: level l < K is also stored at mid + l * mid_stride bytes
// (the reverse mode's recomputed states).  plan.ctl: when given, takes the rows
// that held a solve.
template <int Q, typename S, int MODE, int K, bool MID>
__device__ __forceinline__ void sweep_body(const StepArgs &A,
                                           const SweepPlan &plan,
                                           gptr<const S> __restrict__ src,
                                           gptr<S> __restrict__ dst, int x0,
                                           int x1, int y0, int y1, bool nt,
                                           char *mid, int64_t mid_stride,
                                           StatSlot *slot) {
  constexpr bool PLAIN = base_mode(MODE) == kPlain;
  constexpr bool EEBM = base_mode(MODE) == kEebm;
  const int lane = (int)(threadIdx.x & 63);
  const int nx = A.nx, ny = A.ny;
  const int64_t P = A.plane;
  const int w = x1 - x0 + 2 * K;  // lanes in use
  int x = x0 - K + min(lane, w - 1);
  if (x < 0) x += nx;
  if (x >= nx) x -= nx;
  const bool own = lane >= K && lane < w - K;
  auto lrow = [&](int r) { return r < 0 ? r + ny : (r >= ny ? r - ny : r); };
  auto load = [&](int r, S (&d)[Q]) {
    const gptr<const S> row = src + (int64_t)lrow(r) * nx;
#pragma unroll
    for (int j = 0; j < Q; ++j) d[j] = (row + j * P)[(uint32_t)x];
  };
  S pf[Q], v[Q];
  // v as row y of a state
  auto store = [&](gptr<S> to, int y) {
    if (y < y0 || y >= y1 || !own) return;
    const gptr<S> row = to + (int64_t)y * nx;
#pragma unroll
    for (int j = 0; j < Q; ++j) {
      const gptr<S> a = (row + j * P) + (uint32_t)x;
      if (nt) __builtin_nontemporal_store(v[j], a);
      else *a = v[j];
    }
  };
  SweepRow<Q, S> ring[K];
#pragma unroll
  for (int l = 0; l < K; ++l) {
#pragma unroll
    for (int k = 0; k < 3; ++k) ring[l].mid[k] = (S)0;
#pragma unroll
    for (int k = 0; k < SweepRow<Q, S>::UP; ++k)
      ring[l].up[k] = ring[l].up1[k] = (S)0;
    ring[l].th = 0.0;
  }
  const int re = y1 - 1 + K;   // last row loaded
  NodeStats st;
  uint64_t saw = 0, saw2 = 0;  // quiet nodes; those of two iterations
  int rows_solved = 0;  // those in the band times 2^16, those above it only
#pragma unroll
  for (int j = 0; j < Q; ++j) v[j] = (S)0;
  load(y0 - K, pf);
  for (int r = y0 - K; r <= re; ++r) {
    // Loads and stores share one counter and are waited for in order: the
    // row asked for a whole iteration ago is waited for first, then the row
    // the last iteration left in v is stored, then the next one asked for,
    // so neither wait meets a young access.
#pragma unroll
    for (int j = 0; j < Q; ++j) asm volatile("" : "+v"(pf[j]));
    store(dst, r - 1 - K);
#pragma unroll
    for (int j = 0; j < Q; ++j) v[j] = pf[j];
    if (r < re) load(r + 1, pf);
#pragma unroll
    for (int l = 1; l <= K; ++l) {
      SweepRow<Q, S> &R = ring[l - 1];
      const int y = r - l;
      if (MID && l > 1)  // v: row y + 1 of level l - 1
        store(to_global((S *)(mid + (l - 1) * mid_stride)), y + 1);
      S p[Q];  // what row y of level l pulls
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const S a = cy<Q>(i) == 0   ? R.mid[sweep_mid(i)]
                    : cy<Q>(i) == 1 ? R.up1[cy<Q>(i) == 1 ? sweep_up(i) : 0]
                                    : v[i];
        p[i] = cx<Q>(i) == 0   ? a
               : cx<Q>(i) == 1 ? lane_shift<kLaneBelow>(a)
                               : lane_shift<kLaneAbove>(a);
      }
      const double th = R.th;
      // row r - l + 1 of level l - 1 (v) into what level l keeps
#pragma unroll
      for (int i = 1; i < Q; ++i)
        if (cy<Q>(i) == 1) {
          R.up1[sweep_up(i)] = R.up[sweep_up(i)];
          R.up[sweep_up(i)] = v[i];
        }
      R.mid[0] = v[0];
      R.mid[1] = v[1];
      R.mid[2] = v[3];
      if constexpr (!EEBM) {
        double t = 0.0;
#pragma unroll
        for (int j = 0; j < Q; ++j) t += (double)v[j];
        R.th = t;
      }
      if (y < y0 - (K - l) || y >= y1 + (K - l)) continue;
      // row y of level l into v
      double q[Q], m0 = 0.0;
#pragma unroll
      for (int i = 0; i < Q; ++i) q[i] = (double)p[i];
#pragma unroll
      for (int i = 0; i < Q; ++i) m0 += q[i];
      if constexpr (EEBM) {
        update_pulled<Q, S, MODE>(A, 0.0, q, st, v);
      } else {
        // the quiet test and update of update_pulled, for the whole row
        const bool valid = lane >= l && lane < w - l;
        const double d = th - m0;
        const double dx0 = m0 - (m0 - A.inv_ste);
        const bool quiet =
            (int)((th - A.tm) * A.inv_delta < -20.0) &
            (int)((m0 - A.tm) * A.inv_delta < -20.0) & (int)(th - d == m0) &
            (PLAIN ? 1 : (int)(2.0 * fabs(d) <= fabs(dx0)));
        const bool row = y >= y0 && y < y1;
        if (__builtin_amdgcn_ballot_w64(valid && !quiet) == 0) {
          const bool two = !(fabs(d) <= A.tol);
          saw |= __builtin_amdgcn_ballot_w64(valid);
          saw2 |= __builtin_amdgcn_ballot_w64(valid && two);
          if (A.max_it < 2 && row && own && two) ++st.nonconv;
#pragma unroll
          for (int i = 0; i < Q; ++i)
            v[i] = (S)(A.a * q[i] + A.wtau[wclass<Q>(i)] * m0);
        } else {
          // a row without the band: solid nodes far below it and liquid ones
          // far above, whose new populations are the same sum (phi does not
          // change); the liquid nodes' solves only count
          bool solve = true;
          if constexpr (!PLAIN) {
            const bool liquid = (int)((th - A.tm) * A.inv_delta > 20.0) &
                                (int)((m0 - A.tm) * A.inv_delta > 20.5);
            if (__builtin_amdgcn_ballot_w64(valid && !quiet && !liquid) ==
                0) {
              double tn = 0.0;
              int it = 0;
              bool conv = true, above = true;
              if (valid && liquid)
                above = newton_liquid(m0, th, A, tn, it, conv);
              if (__builtin_amdgcn_ballot_w64(!above) == 0) {
                solve = false;
                rows_solved += 1;
                const bool two = !(fabs(d) <= A.tol);
                saw |= __builtin_amdgcn_ballot_w64(valid && quiet);
                saw2 |= __builtin_amdgcn_ballot_w64(valid && quiet && two);
                if (row && own)
                  st.nonconv += quiet ? (int)(A.max_it < 2 && two)
                                      : (int)!conv;
                st.max_it = max(st.max_it, it);
                if (it > 0)
                  st.max_res = fmax(st.max_res, fabs(tn + A.inv_ste -
                                                     (m0 + A.inv_ste)));
#pragma unroll
                for (int i = 0; i < Q; ++i)
                  v[i] = (S)(A.a * q[i] + A.wtau[wclass<Q>(i)] * m0);
              }
            }
          }
          if (!solve) continue;
          rows_solved += 1 << 16;
          // a row with a solve in or near the band (the arguments read
          // again: see step_item)
          int z = 0;
          asm volatile("" : "+s"(z));
          const StepArgs &B = (&A)[z];
          if (valid) {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
              // keeps the FP64 copies of the test above from staying live
              asm volatile("" : "+v"(p[i]));
              q[i] = (double)p[i];
            }
            NodeStats one;
            update_pulled<Q, S, MODE>(B, th, q, one, v);
            // (a halo node's solve is counted by its own wave as well)
            st.max_it = max(st.max_it, one.max_it);
            st.max_res = fmax(st.max_res, one.max_res);
            if (row && own) st.nonconv += one.nonconv;
          }
        }
      }
    }
  }
  store(dst, re - K);
  if constexpr (!EEBM) {
    const int quiet = saw2 && A.max_it >= 2 ? 2 : (saw ? 1 : 0);
    const int it = wave_max_i(max(st.max_it, quiet));
    const int nc = wave_sum_i(st.nonconv);
    const double res = wave_max(st.max_res);
    if (lane == 0) {
      StatSlot s = *slot;
      s.max_it = max(s.max_it, it);
      s.nonconv += nc;
      s.max_res = fmax(s.max_res, res);
      *slot = s;
      // (read here: held through the sweep it would cost registers)
      int z = 0;
      asm volatile("" : "+s"(z));
      RouteCtl *ctl = (&plan)[z].ctl;
      if (ctl && rows_solved > 0) {
        const int nband = rows_solved >> 16, nliquid = rows_solved & 0xffff;
        atomicMax(&ctl->chain, nband + nliquid);
        atomicAdd(&ctl->units,
                  (unsigned long long)route_units(nband, nliquid));
      }
    }
  }
}

// the tile t of the frame
__device__ __forceinline__ void frame_tile_of(const SweepPlan &P, int nx,
                                              int ny, int t, int &x0, int &x1,
                                              int &y0, int &y1) {
  const int T = P.tile, ns = (P.nleft + P.nright) * P.nside;
  if (t < ns) {
    const int c = t % (P.nleft + P.nright), r = t / (P.nleft + P.nright);
    x0 = c < P.nleft ? c * T : P.xb + (c - P.nleft) * T;
    x1 = min(x0 + T, c < P.nleft ? P.xa : nx);
    y0 = (int)((int64_t)r * ny / P.nside);
    y1 = (int)((int64_t)(r + 1) * ny / P.nside);
  } else {
    const int c = (t - ns) % P.nacross, r = (t - ns) / P.nacross;
    x0 = P.xa + (int)((int64_t)c * (P.xb - P.xa) / P.nacross);
    x1 = P.xa + (int)((int64_t)(c + 1) * (P.xb - P.xa) / P.nacross);
    y0 = r < P.nbottom ? r * T : P.yb + (r - P.nbottom) * T;
    y1 = min(y0 + T, r < P.nbottom ? P.ya : ny);
  }
}

// the wave k of the strips of w columns: its own nodes
__device__ __forceinline__ void sweep_wave_of(const SweepPlan &P, int k, int w,
                                              int &x0, int &x1, int &y0,
                                              int &y1) {
  const int nf = P.nfl + P.nfr, m = P.strips - nf;
  int strip, rows;
  if (k < nf * P.fseg) {
    strip = k % nf < P.nfl ? 0 : P.strips - 1;
    rows = P.frows;
    y0 = P.ya + k / nf * rows;
  } else {
    k -= nf * P.fseg;
    strip = P.nfl + k % m;
    rows = P.rows;
    y0 = P.ya + k / m * rows;
  }
  x0 = P.xa + strip * w;
  x1 = min(x0 + w, P.xb);
  y1 = min(y0 + rows, P.yb);
}

namespace {

// waves per SIMD asked for: what the registers allow without spilling
constexpr int sweep_waves(int q, int bytes, int k) {
  return q == 9 && bytes == 8 && k > 2 ? 2 : 3;
}

template <int Q, typename S, int MODE, int K, bool MID>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sweep_waves(Q, sizeof(S), K))))
void sweep_kernel(StepArgs A, SweepPlan P, char *mid, int64_t mid_stride) {
  __shared__ S lds[Q * kFrameSide * kFrameSide];
  if (P.ctl && !on_route(P.ctl, 0)) return;
  const int xcd = (int)(blockIdx.x & 7), j = (int)(blockIdx.x >> 3);
  const int nt = (int)P.tiles(), nw = (int)P.waves();
  const int ct = (nt + 7) >> 3, cw = (((nw + 7) >> 3) + 3) & ~3;
  if (j < ct) {
    const int t = xcd * ct + j;
    if (t >= nt) return;
    int x0, x1, y0, y1;
    frame_tile_of(P, A.nx, A.ny, t, x0, x1, y0, y1);
    tile_body<Q, S, MODE>(A, to_global((const S *)A.src),
                          to_global((S *)A.dst), K, x0, x1, y0, y1, kFrameSide,
                          kFrameSide * kFrameSide,
                          t < (P.nleft + P.nright) * P.nside, lds, MID ? mid : nullptr, mid_stride,
                          A.slots + t);
    return;
  }
  const int i = (j - ct) * 4 +
                __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int k = xcd * cw + i;
  if (i >= cw || k >= nw) return;
  int x0, x1, y0, y1;
  sweep_wave_of(P, k, 64 - 2 * K, x0, x1, y0, y1);
  sweep_body<Q, S, base_mode(MODE), K, MID>(
      A, P, to_global((const S *)A.src), to_global((S *)A.dst), x0, x1, y0, y1,
      P.nt != 0, mid, mid_stride, A.slots + nt + k);
}

// The same over a batch of lattices (descriptor, plan): tiles and waves are
// listed in two tables of (instance, item), each cut into one contiguous
// part per XCD; strips are as wide as K = 4 allows at every K, so that the
// tables do not depend on it.
template <int Q, typename S, int MODE, int K>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sweep_waves(Q, sizeof(S), K))))
void batch_sweep_kernel(const StepArgs *__restrict__ descs,
                        const SweepPlan *__restrict__ plans,
                        const int2 *__restrict__ tiles, int32_t nt,
                        const int2 *__restrict__ waves, int32_t nw,
                        int32_t parity, RouteCtl *ctl) {
  __shared__ S lds[Q * kFrameSide * kFrameSide];
  if (ctl && !on_route(ctl, 0)) return;
  const int xcd = (int)(blockIdx.x & 7), j = (int)(blockIdx.x >> 3);
  const int ct = (nt + 7) >> 3, cw = (((nw + 7) >> 3) + 3) & ~3;
  if (j < ct) {
    const int i = xcd * ct + j;
    if (i >= nt) return;
    const int2 e = tiles[i];
    const int inst = __builtin_amdgcn_readfirstlane(e.x);
    const int t = __builtin_amdgcn_readfirstlane(e.y);
    const StepArgs &A = descs[inst];
    int x0, x1, y0, y1;
    frame_tile_of(plans[inst], A.nx, A.ny, t, x0, x1, y0, y1);
    tile_body<Q, S, MODE>(A, to_global((const S *)(parity ? A.dst : A.src)),
                          to_global((S *)(parity ? A.src : A.dst)), K, x0, x1,
                          y0, y1, kFrameSide, kFrameSide * kFrameSide,
                          t < (plans[inst].nleft + plans[inst].nright) *
                                  plans[inst].nside,
                          lds, nullptr, 0, A.slots + t);
    return;
  }
  const int i = (j - ct) * 4 +
                __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (i >= cw || xcd * cw + i >= nw) return;
  const int2 e = waves[xcd * cw + i];
  const int inst = __builtin_amdgcn_readfirstlane(e.x);
  const int k = __builtin_amdgcn_readfirstlane(e.y);
  const StepArgs &A = descs[inst];
  const SweepPlan &P = plans[inst];
  int x0, x1, y0, y1;
  sweep_wave_of(P, k, 64 - 2 * P.k, x0, x1, y0, y1);
  sweep_body<Q, S, MODE, K, false>(
      A, P, to_global((const S *)(parity ? A.dst : A.src)),
      to_global((S *)(parity ? A.src : A.dst)), x0, x1, y0, y1, P.nt != 0,
      nullptr, 0, A.slots + (int)P.tiles() + k);
}

// ---------------------------------------------------------------------
// the route of a state that the lattice was given

// What a sweep of K steps over rows [y0, y1) of columns [x0, x1) of `src`
// would count, from its temperatures: the rows off phi's lower plateau, at
// every level.
template <int Q, typename S>
__device__ __forceinline__ void route_scan(const StepArgs &A, const S *src,
                                           int x0, int x1, int y0, int y1,
                                           int K, RouteCtl *ctl) {
  const int lane = (int)(threadIdx.x & 63);
  const int x = min(x0 + lane, x1 - 1);
  int nband = 0, nliquid = 0;
  for (int y = y0; y < y1; ++y) {
    double T = 0.0;
#pragma unroll
    for (int j = 0; j < Q; ++j)
      T += (double)src[j * A.plane + (int64_t)y * A.nx + x];
    const double u = (T - A.tm) * A.inv_delta;
    if (__builtin_amdgcn_ballot_w64(!(u < -20.0)) == 0) continue;
    if (__builtin_amdgcn_ballot_w64(!(u < -20.0) && !(u > 20.0)) == 0)
      ++nliquid;
    else
      ++nband;
  }
  if (lane == 0 && nband + nliquid > 0) {
    // the rows around them too: level l has 2 (K - l) more
    atomicMax(&ctl->chain, K * (nband + nliquid) + K * (K - 1));
    atomicAdd(&ctl->units,
              (unsigned long long)route_units(K * nband, K * nliquid));
  }
}

template <int Q, typename S>
__global__ __launch_bounds__(256) void route_scan_kernel(StepArgs A,
                                                         SweepPlan P,
                                                         RouteCtl *ctl) {
  const int k = (int)blockIdx.x * 4 +
                __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (k >= P.waves()) return;
  int x0, x1, y0, y1;
  sweep_wave_of(P, k, 64 - 2 * P.k, x0, x1, y0, y1);
  route_scan<Q, S>(A, (const S *)A.src, x0, x1, y0, y1, P.k, ctl);
}

// the same over a batch's waves
template <int Q, typename S>
__global__ __launch_bounds__(256) void batch_route_scan_kernel(
    const StepArgs *__restrict__ descs, const SweepPlan *__restrict__ plans,
    const int2 *__restrict__ waves, int32_t nw, int32_t parity,
    RouteCtl *ctl) {
  const int i = (int)blockIdx.x * 4 +
                __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (i >= nw) return;
  const int2 e = waves[i];
  const int inst = __builtin_amdgcn_readfirstlane(e.x);
  const int k = __builtin_amdgcn_readfirstlane(e.y);
  const StepArgs &A = descs[inst];
  const SweepPlan &P = plans[inst];
  int x0, x1, y0, y1;
  sweep_wave_of(P, k, 64 - 2 * P.k, x0, x1, y0, y1);
  route_scan<Q, S>(A, (const S *)(parity ? A.dst : A.src), x0, x1, y0, y1,
                   P.k, ctl);
}

// groups of single steps after which a sweep is tried again (of up to 32 K
// steps each: a try in a state that does not suit a sweep costs 1% or so)
constexpr int kRouteRetry = 128;

// The route of the next group, from what the last one's sweeps counted (scan:
// from what the scan of a new state counted), after all of its launches.
__global__ void route_decide_kernel(RouteCtl *ctl, int32_t scan,
                                    int32_t chain_max,
                                    unsigned long long units_max) {
  RouteCtl c = *ctl;
  if (scan || c.route == 0) {
    c.route = c.chain > chain_max || c.units > units_max;
    c.age = 0;
  } else if (++c.age >= kRouteRetry) {
    c.route = 0;
  }
  c.chain = 0;
  c.units = 0;
  *ctl = c;
}

}  // namespace
}  // namespace irebm
