// ilfbm.hip -- the implicit liquid fraction based method (ILFBM, Section
// 3.3, Algorithm 1) on gfx950, the inner-loop scheme the paper compares
// IREBM with.
//
// The state is the post-collision population planes Omega0 (collision
// without source, as for the other schemes) and the liquid fraction plane
// l.  One step runs the inner loop of Algorithm 1: iteration k pulls
//   f_i^(k)(x) = Omega0_i(x - e_i) + (w_i/Ste)(l - l^(k-1))(x - e_i)
// (the collision with source of the upstream node, then streaming),
// closes the unknown populations (Section 4.2 on the streamed populations,
// Dirichlet target T_D), and forms H^(k) = M0(f^(k)) + l^(k-1)/Ste and
// l^(k) = clamp(Ste (H^(k) - T_m), 0, 1).  The source term reaches across
// nodes; but Omega0 and l do not change during the inner loop, so a block
// holds the pulled Omega0 of a tile and its halo in registers and takes
// several iterations per launch on it (at most kTileIt), l - l^(k-1) in LDS
// (ilfbm_tile_kernel).  Every iteration with a change above tol sets a flag
// of its own; a launch whose predecessor has an unset one returns.  The host
// reads the flags after every few launches, and the launch that holds the
// last iteration is run once more up to it, now writing the next state, the
// boundary fluxes and the largest change.  Tolerance and cap: the params'
// newton_tol and newton_max_it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "host_util.hpp"
#include "kernels.hpp"
#include "lbm_stefan.h"
#include "lbm_stefan_internal.hpp"

using namespace irebm;

namespace {

constexpr int kTileIt = 8;       // inner iterations per launch, at most
constexpr int kTileThreads = 1024;
constexpr int kTileRow = 32;     // 2D tiles: 32 x 32 with the halo
constexpr int kBurst = 8;        // launches between two host checks
constexpr int kSets = 2 * kBurst;

// device control block of one step's inner loop
struct IlfCtrl {
  // of a step's last iteration, summed over its tiles
  double dl, flux_in, flux_out;
  // launch j, iteration m: open[j % kSets][m] is set when l changed by more
  // than tol somewhere
  int32_t open[kSets][kTileIt];
};

// tiles of a launch of kk iterations: own nodes per tile along x and y at
// most (the rest of a block's threads hold the halo)
constexpr int tile_x(int q, int kk) {
  return q == 3 ? kTileThreads - 2 * kk : kTileRow - 2 * kk;
}
constexpr int tile_y(int q, int kk) {
  return q == 3 ? 1 : kTileThreads / kTileRow - 2 * kk;
}

struct IlfArgs {
  StepArgs A;            // lattice; A.src = Omega0, A.dst = next state
  const double *l;       // liquid fraction of the state
  const double *lprev;   // l^(k-1)
  double *lout;          // l^(k)
  double ste;
};

// Omega^(k)_i at node k: the collision with source of Algorithm 1
template <int Q, typename S>
__device__ __forceinline__ double omega_k(const IlfArgs &G, int i,
                                          int64_t node) {
  const S *src = (const S *)G.A.src;
  return (double)src[i * G.A.plane + node] +
         wt<Q>(i) * G.A.inv_ste * (G.l[node] - G.lprev[node]);
}

// lattice node of the pull source x - e_i (wrapped on periodic axes; the
// caller knows from the masks that it is one)
template <int Q>
__device__ __forceinline__ int64_t source_node(const StepArgs &A, int x, int y,
                                               int i) {
  int sx = x - cx<Q>(i), sy = y - cy<Q>(i);
  if (sx < 0) sx += A.nx;
  if (sx >= A.nx) sx -= A.nx;
  if (sy < 0) sy += A.ny;
  if (sy >= A.ny) sy -= A.ny;
  return (int64_t)sy * A.nx + sx;
}

// inner iteration at node k: writes l^(k) and the collision of f^(k), adds
// |l^(k) - l^(k-1)| (max), the closure inflow and the outflow
template <int Q, typename S>
__device__ __forceinline__ void ilfbm_node(const IlfArgs &G, int64_t k,
                                           double &dl, double &fin,
                                           double &fout) {
  const StepArgs &A = G.A;
  {
    const int x = (int)(k % A.nx), y = (int)(k / A.nx);
    uint32_t known, out;
    node_masks<Q>(A, x, y, known, out);
    double om[Q], q[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) om[j] = omega_k<Q, S>(G, j, k);
#pragma unroll
    for (int i = 0; i < Q; ++i)
      q[i] = (known >> i & 1u) ? omega_k<Q, S>(G, i, source_node<Q>(A, x, y, i))
                               : 0.0;
    if (known != (1u << Q) - 1u) {
      double mirror = 0.0;
      int mx, my;
      if (neumann_mirror<Q>(A, x, y, mx, my)) {
        // M0 of the populations streamed into the mirror node; every
        // source is a lattice node (no bounce-back beside Neumann walls)
#pragma unroll
        for (int i = 0; i < Q; ++i)
          mirror += omega_k<Q, S>(G, i, source_node<Q>(A, mx, my, i));
      }
      fin += close_node<Q, SCHEME_ILFBM, true>(A, x, y, 0.0, om, q, known,
                                                mirror);
    }
#pragma unroll
    for (int i = 1; i < Q; ++i)
      if (out >> i & 1u) fout += om[i];
    double m0 = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) m0 += q[i];
    const double H = m0 + G.lprev[k] * A.inv_ste;
    double ln = G.ste * (H - A.tm);
    ln = ln < 0.0 ? 0.0 : (ln > 1.0 ? 1.0 : ln);
    G.lout[k] = ln;
    dl = fmax(dl, fabs(ln - G.lprev[k]));
    // the collision of f^(k): the next state if k is the last iteration
    S *dst = (S *)A.dst;
#pragma unroll
    for (int i = 0; i < Q; ++i)
      dst[i * A.plane + k] = (S)(A.a * q[i] + A.wtau[wclass<Q>(i)] * m0);
  }
}

// kk (at most kTileIt) inner iterations on the tiles of the lattice, G.lprev
// -> G.lout.  The region a block holds shrinks by one node a side and
// iteration, as in tile_body; nodes of a halo are computed by their
// neighbours as well, by the same code from the same values.  open: this
// launch's flags; prev: those of the launch before (nprev of them, 0 for the
// first launch);
// clear: a set that a later launch will use.  FINAL: the last iteration also
// writes the next state to G.A.dst and per tile (pend) the largest change
// and the boundary fluxes.
//
// A launch per iteration and one to check it took 14 us per iteration of a
// 201^2 D2Q9 FP64 lattice, latency of launches and global memory all of it.
// 8 iterations of a block take 20 us, most of it the closures of the wall
// nodes (29 us while those reloaded their Omega0 in every iteration), and a
// step of 114 iterations 450 us with the host reads, before 1600.
template <int Q, typename S, bool FINAL>
__global__ __launch_bounds__(kTileThreads) void ilfbm_tile_kernel(
    IlfArgs G, int32_t ntx, int32_t nty, int32_t kk, const int32_t *prev,
    int32_t nprev, int32_t *open, int32_t *clear, double tol, double *pend) {
  constexpr int RX = Q == 3 ? kTileThreads : kTileRow;
  __shared__ double lds[2][kTileThreads];
  __shared__ int32_t s_open[kTileIt];
  const int t = (int)threadIdx.x;
  if (!FINAL) {
    int all = 1;
    for (int m = 0; m < nprev; ++m) all &= prev[m];
    if (!all) return;                // an earlier iteration converged
  }
  const int tiles = ntx * nty, per_xcd = (tiles + 7) >> 3;
  const int tile = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (blockIdx.x == 0 && t < kTileIt) clear[t] = 0;
  if (tile >= tiles) return;
  const StepArgs &A = G.A;
  const int nx = A.nx, ny = A.ny;
  const int64_t PL = A.plane;
  const gptr<const S> src = to_global((const S *)A.src);
  const int tx = tile % ntx, ty = tile / ntx;
  const int x0 = (int)((int64_t)tx * nx / ntx);
  const int x1 = (int)((int64_t)(tx + 1) * nx / ntx);
  const int y0 = (int)((int64_t)ty * ny / nty);
  const int y1 = (int)((int64_t)(ty + 1) * ny / nty);
  const int hy = Q == 3 ? 0 : kk;    // halo rows (D1Q3: one row, no y)
  const int lx = t % RX, ly = t / RX;
  const int x = x0 - kk + lx, y = y0 - hy + ly;
  const int w = x1 - x0 + 2 * kk, h = y1 - y0 + 2 * hy;
  int gx = x, gy = y;
  if (A.periodic_x) gx = ((x % nx) + nx) % nx;
  if (A.periodic_y) gy = ((y % ny) + ny) % ny;
  const bool node = lx < w && ly < h && gx >= 0 && gx < nx && gy >= 0 &&
                    gy < ny;
  const bool own = node && x >= x0 && x < x1 && y >= y0 && y < y1;
  const int64_t at = node ? (int64_t)gy * nx + gx : 0;
  // static over the inner loop: the pulled Omega0, l, masks, and on an edge
  // node its own Omega0 and what its mirror node pulls
  const double lo = G.l[at];
  double lp = G.lprev[at];
  lds[0][t] = lo - lp;
  if (t < kTileIt) s_open[t] = 0;
  uint32_t known = 0, out = 0;
  S p[Q], own_om[Q], pm[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) p[i] = own_om[i] = pm[i] = (S)0;
  if (node) {
    node_masks<Q>(A, gx, gy, known, out);
#pragma unroll
    for (int i = 0; i < Q; ++i)
      if (known >> i & 1u) p[i] = src[i * PL + source_node<Q>(A, gx, gy, i)];
  }
  const bool edge = node && (known != (1u << Q) - 1u || out);
  bool mirrored = false;
  int mt = 0;
  if (edge) {
    int mx, my;
    mirrored = known != (1u << Q) - 1u && neumann_mirror<Q>(A, gx, gy, mx, my);
    if (mirrored) mt = t + (mx - gx) + (my - gy) * RX;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      own_om[i] = src[i * PL + at];
      if (mirrored) pm[i] = src[i * PL + source_node<Q>(A, mx, my, i)];
    }
  }
  double dl = 0.0, fin = 0.0, fout = 0.0;
  for (int m = 1; m <= kk; ++m) {
    __syncthreads();
    const double *D = lds[(m - 1) & 1];
    const bool act = node && lx >= m && lx < w - m &&
                     (Q == 3 || (ly >= m && ly < h - m));
    bool big = false;
    if (act) {
      double q[Q];
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const double o = (double)p[i] + wt<Q>(i) * A.inv_ste *
                                            D[t - cx<Q>(i) - cy<Q>(i) * RX];
        q[i] = (known >> i & 1u) ? o : 0.0;
      }
      if (edge) {
        double om[Q];
#pragma unroll
        for (int j = 0; j < Q; ++j)
          om[j] = (double)own_om[j] + wt<Q>(j) * A.inv_ste * D[t];
        if (known != (1u << Q) - 1u) {
          double mirror = 0.0;
          if (mirrored) {
            // M0 of the populations streamed into the mirror node; every
            // source is a lattice node (no bounce-back beside Neumann walls)
#pragma unroll
            for (int i = 0; i < Q; ++i)
              mirror += (double)pm[i] + wt<Q>(i) * A.inv_ste *
                                            D[mt - cx<Q>(i) - cy<Q>(i) * RX];
          }
          const double f = close_node<Q, SCHEME_ILFBM, true>(
              A, gx, gy, 0.0, om, q, known, mirror);
          if (FINAL && own && m == kk) fin += f;
        }
        if (FINAL && own && m == kk) {
#pragma unroll
          for (int i = 1; i < Q; ++i)
            if (out >> i & 1u) fout += om[i];
        }
      }
      double m0 = 0.0;
#pragma unroll
      for (int i = 0; i < Q; ++i) m0 += q[i];
      const double H = m0 + lp * A.inv_ste;
      double ln = G.ste * (H - A.tm);
      ln = ln < 0.0 ? 0.0 : (ln > 1.0 ? 1.0 : ln);
      const double ch = fabs(ln - lp);
      big = own && ch > tol;
      lp = ln;
      lds[m & 1][t] = lo - ln;
      if (m == kk && own) {
        G.lout[at] = ln;
        if (FINAL) {
          dl = fmax(dl, ch);
          // the collision of f^(k): the next state
          const gptr<S> dst = to_global((S *)A.dst);
#pragma unroll
          for (int i = 0; i < Q; ++i)
            dst[i * PL + at] = (S)(A.a * q[i] + A.wtau[wclass<Q>(i)] * m0);
        }
      }
    }
    if (__any(big) && (t & 63) == 0) s_open[m - 1] = 1;
  }
  __syncthreads();
  if (t < kk && s_open[t]) open[t] = 1;
  if constexpr (FINAL) {
    // (lds is free: the barrier above)
    double *sh = &lds[0][0];
    dl = wave_max(dl);
    fin = wave_sum(fin);
    fout = wave_sum(fout);
    if ((t & 63) == 0) {
      sh[3 * (t >> 6)] = dl;
      sh[3 * (t >> 6) + 1] = fin;
      sh[3 * (t >> 6) + 2] = fout;
    }
    __syncthreads();
    if (t == 0) {
      for (int v = 1; v < kTileThreads / 64; ++v) {
        dl = fmax(dl, sh[3 * v]);
        fin += sh[3 * v + 1];
        fout += sh[3 * v + 2];
      }
      pend[3 * tile] = dl;
      pend[3 * tile + 1] = fin;
      pend[3 * tile + 2] = fout;
    }
  }
}

// largest change and fluxes of a step, over its tiles in a fixed order; the
// flags are clear again for the next step
__global__ __launch_bounds__(256) void ilfbm_sum_kernel(const double *pend,
                                                        int64_t ntiles,
                                                        IlfCtrl *ctrl) {
  if (threadIdx.x < kSets * kTileIt)
    ctrl->open[threadIdx.x / kTileIt][threadIdx.x % kTileIt] = 0;
  double m = 0.0, fin = 0.0, fout = 0.0;
  for (int64_t b = threadIdx.x; b < ntiles; b += 256) {
    m = fmax(m, pend[3 * b]);
    fin += pend[3 * b + 1];
    fout += pend[3 * b + 2];
  }
  __shared__ double s_m[4];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  const double sfin = block_sum_256(fin);
  const double sfout = block_sum_256(fout);
  if (threadIdx.x == 0) {
    ctrl->dl = fmax(fmax(s_m[0], s_m[1]), fmax(s_m[2], s_m[3]));
    ctrl->flux_in = sfin;
    ctrl->flux_out = sfout;
  }
}

// Small D1Q3 lattices (at most kResidentNodes nodes): one workgroup runs
// `nsteps` whole steps in one launch, block barriers in place of launches
// and host reads.  (256 nodes, 48 iterations a step: 110 us per step either
// way, 2000 nodes 280 here against 112 in tiles; a 2D iteration takes 14 us
// here at any size, 24^2 D2Q9 1736 us per step against 486; only tiny ones that
// take an iteration or two per step would be faster here, 45 x 20 19 us against
// 36.)  Node updates and convergence decisions are those of the multi-launch
// path (same ilfbm_node, exact max), so the states are the same; only the flux
// sums are reduced in another order.  L[0] is the
// state's l plane, L[1] and L[2] the inner-loop planes; planes and buffers
// rotate in registers, and the final assignment and statistics are
// written to `res` for the host.
constexpr int kResident = 1024;         // threads of the resident block
constexpr int64_t kResidentNodes = 512;

struct IlfResident {
  IlfArgs G;            // lattice, ste; l/lprev/lout unused
  void *buf[2];
  double *L[3];
  int32_t cur, nsteps, cap;
  double tol;
  double *res;          // out: cur, L roles (3), max_it, capped steps,
                        // max residual, flux in, flux out
};

// Block reductions with one barrier each: consecutive reductions use
// alternate halves of sh (`r` counts them), and the barrier of reduction
// r + 1 separates the reads of reduction r from the writes of r + 2.
// Every thread calls them in the same order.
__device__ __forceinline__ double block_max_1024(double v, double *sh,
                                                 int &r) {
  double *b = sh + (r++ & 1) * (kResident / 64);
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) b[threadIdx.x >> 6] = v;
  __syncthreads();
  double m = b[0];
  for (int w = 1; w < kResident / 64; ++w) m = fmax(m, b[w]);
  return m;
}

__device__ __forceinline__ double block_sum_1024(double v, double *sh,
                                                 int &r) {
  double *b = sh + (r++ & 1) * (kResident / 64);
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) b[threadIdx.x >> 6] = v;
  __syncthreads();
  double m = b[0];
  for (int w = 1; w < kResident / 64; ++w) m += b[w];
  return m;
}

template <int Q, typename S>
__global__ __launch_bounds__(kResident) void ilfbm_resident_kernel(
    IlfResident R) {
  __shared__ double sh[2 * (kResident / 64)];
  int red = 0;
  IlfArgs G = R.G;
  int cur = R.cur;
  int li = 0, la = 1, lb = 2;       // state, and the two inner planes
  int max_it = 0, capped = 0;
  double max_res = 0.0, fin_tot = 0.0, fout_tot = 0.0;
  const int64_t n = G.A.plane;
  for (int s = 0; s < R.nsteps; ++s) {
    G.A.src = R.buf[cur];
    G.A.dst = R.buf[cur ^ 1];
    G.l = R.L[li];
    int k = 0;
    bool done = false;
    double dl = 0.0, a = 0.0, b = 0.0;
    while (k < R.cap && !done) {
      ++k;
      G.lprev = k == 1 ? R.L[li] : R.L[(k - 1) & 1 ? la : lb];
      G.lout = R.L[k & 1 ? la : lb];
      double d = 0.0;
      a = 0.0;
      b = 0.0;
      for (int64_t j = threadIdx.x; j < n; j += kResident)
        ilfbm_node<Q, S>(G, j, d, a, b);
      // the barrier inside the reduction also orders this iteration's
      // writes before the next iteration's reads
      dl = block_max_1024(d, sh, red);
      done = dl <= R.tol;
    }
    // fluxes of the last iteration
    const double fin = block_sum_1024(a, sh, red);
    const double fout = block_sum_1024(b, sh, red);
    // l^(k) becomes the state's plane
    const int lk = k & 1 ? la : lb;
    if (lk == la) {
      la = li;
    } else {
      lb = li;
    }
    li = lk;
    cur ^= 1;
    max_it = max(max_it, k);
    if (!done) {
      capped++;
      max_res = fmax(max_res, dl);
    }
    fin_tot += fin;
    fout_tot += fout;
  }
  if (threadIdx.x == 0) {
    R.res[0] = cur;
    R.res[1] = li;
    R.res[2] = la;
    R.res[3] = lb;
    R.res[4] = max_it;
    R.res[5] = capped;
    R.res[6] = max_res;
    R.res[7] = fin_tot;
    R.res[8] = fout_tot;
  }
}

static_assert(kSets * kTileIt <= 256, "ilfbm_sum_kernel clears the flags");

int64_t tiles_of(int64_t n, int side) { return (n + side - 1) / side; }
int64_t iter_tiles(const lbm_stefan_params *p, int kk = kTileIt) {
  return tiles_of(p->nx, tile_x(p->q, kk)) * tiles_of(p->ny, tile_y(p->q, kk));
}

}  // namespace

size_t irebm::ilfbm_bytes(const lbm_stefan_params *p) {
  if (p->scheme != LBM_SCHEME_ILFBM) return 0;
  const int64_t n = p->nx * p->ny;
  return 3 * align256((size_t)n * 8) + align256((size_t)iter_tiles(p) * 24) +
         align256(sizeof(IlfCtrl));
}

hipError_t irebm::ilfbm_attach(lbm_stefan_t *h, char *base) {
  const int64_t n = h->p.nx * h->p.ny;
  const size_t plane = align256((size_t)n * 8);
  h->lf = (double *)base;
  h->lscr[0] = (double *)(base + plane);
  h->lscr[1] = (double *)(base + 2 * plane);
  h->pend = (double *)(base + 3 * plane);
  h->ctrl = base + 3 * plane + align256((size_t)iter_tiles(&h->p) * 24);
  ilfbm_reset_stats(h);
  return zero_async(h->ctrl, sizeof(IlfCtrl), h->stream);
}

void irebm::ilfbm_reset_stats(lbm_stefan_t *h) {
  h->ilf_max_it = 0;
  h->ilf_nonconv = 0;
  h->ilf_max_res = 0.0;
  h->ilf_fin = 0.0;
  h->ilf_fout = 0.0;
}

namespace {

// nsteps steps of a small lattice in launches of the resident kernel
hipError_t ilfbm_advance_resident(lbm_stefan_t *h, int64_t nsteps) {
  const lbm_stefan_params &p = h->p;
  constexpr int64_t kChunk = 2048;    // steps per launch
  IlfResident R;
  fill_step_args(h, &R.G.A);
  R.G.ste = p.ste;
  R.buf[0] = h->buf[0];
  R.buf[1] = h->buf[1];
  R.cap = p.newton_max_it;
  R.tol = p.newton_tol;
  R.res = h->pend;                    // >= 256 bytes: reuse the pending area
  for (int64_t left = nsteps; left > 0;) {
    const int32_t chunk = (int32_t)std::min(left, kChunk);
    double *Lp[3] = {h->lf, h->lscr[0], h->lscr[1]};
    for (int j = 0; j < 3; ++j) R.L[j] = Lp[j];
    R.cur = h->cur;
    R.nsteps = chunk;
    if (p.storage == LBM_STORE_F32)
      ilfbm_resident_kernel<3, float><<<1, kResident, 0, h->stream>>>(R);
    else
      ilfbm_resident_kernel<3, double><<<1, kResident, 0, h->stream>>>(R);
    hipError_t e = hipGetLastError();
    double res[9];
    if (e == hipSuccess)
      e = hipMemcpyAsync(res, h->pend, sizeof(res), hipMemcpyDeviceToHost,
                         h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return e;
    h->cur = (int)res[0];
    h->lf = Lp[(int)res[1]];
    h->lscr[0] = Lp[(int)res[2]];
    h->lscr[1] = Lp[(int)res[3]];
    h->ilf_max_it = std::max(h->ilf_max_it, (int32_t)res[4]);
    h->ilf_nonconv += (int64_t)res[5];
    if (res[5] > 0) h->ilf_max_res = std::max(h->ilf_max_res, res[6]);
    h->ilf_fin += res[7];
    h->ilf_fout += res[8];
    h->steps += chunk;
    left -= chunk;
  }
  return hipSuccess;
}

}  // namespace

hipError_t irebm::ilfbm_advance(lbm_stefan_t *h, int64_t nsteps) {
  const lbm_stefan_params &p = h->p;
  if (p.q == 3 && p.nx <= kResidentNodes)
    return ilfbm_advance_resident(h, nsteps);
  IlfCtrl *ctrl = (IlfCtrl *)h->ctrl;
  IlfArgs G;
  fill_step_args(h, &G.A);
  G.ste = p.ste;
  const int cap = p.newton_max_it;
  IlfCtrl hc{};
  bool pending = false, capped = false;   // a step's sums are still on their way
  auto take = [&] {
    if (!pending) return;
    if (capped) h->ilf_max_res = std::max(h->ilf_max_res, hc.dl);
    h->ilf_fin += hc.flux_in;
    h->ilf_fout += hc.flux_out;
    pending = false;
  };
  auto read = [&] {
    hipError_t e = hipMemcpyAsync(&hc, ctrl, sizeof(hc), hipMemcpyDeviceToHost,
                                  h->stream);
    return e == hipSuccess ? hipStreamSynchronize(h->stream) : e;
  };
  for (int64_t s = 0; s < nsteps; ++s) {
    G.A.src = h->buf[h->cur];
    G.A.dst = h->buf[h->cur ^ 1];
    G.l = h->lf;
    // Launch j: iterations from(j) + 1 to from(j + 1), at most cap; the first
    // as many as the last step took, if those are few: on wider tiles, and as
    // the step's end if its guess holds (us per step, 8 always / so: 1601^2
    // D2Q9 FP64 that converges in 3 907 / 210, at a cap of 2 604 / 182, 501^2
    // 106 / 56; a launch per iteration 467, 306, 63).
    const int k0 = h->ilf_last > 0 && h->ilf_last < kTileIt ? h->ilf_last
                                                            : kTileIt;
    auto from = [&](int64_t j) -> int64_t {
      return j == 0 ? 0 : std::min<int64_t>(cap, k0 + (j - 1) * kTileIt);
    };
    auto launch = [&](int64_t j, int kk, bool final) {
      const int32_t ntx = (int32_t)tiles_of(p.nx, tile_x(p.q, kk));
      const int32_t nty = (int32_t)tiles_of(p.ny, tile_y(p.q, kk));
      const unsigned grid = (unsigned)(8 * (((int64_t)ntx * nty + 7) / 8));
      G.lprev = j == 0 ? h->lf : h->lscr[(j - 1) & 1];
      G.lout = h->lscr[j & 1];
      int32_t *open = ctrl->open[j % kSets];
      const int32_t *prev = ctrl->open[(j + kSets - 1) % kSets];
      const int32_t np = (int32_t)(j == 0 ? 0 : from(j) - from(j - 1));
      int32_t *clear = ctrl->open[(j + kBurst) % kSets];
      return dispatch_qs(p.q, p.storage, [&](auto qt, auto tt) {
        QS_TYPES(qt, tt);
        if (final)
          ilfbm_tile_kernel<Q, S, true><<<grid, kTileThreads, 0, h->stream>>>(
              G, ntx, nty, kk, prev, np, open, clear, p.newton_tol, h->pend);
        else
          ilfbm_tile_kernel<Q, S, false><<<grid, kTileThreads, 0, h->stream>>>(
              G, ntx, nty, kk, prev, np, open, clear, p.newton_tol, h->pend);
        return hipGetLastError();
      });
    };
    hipError_t e = hipSuccess;
    int64_t kf = 0, jf = 0;          // the last iteration and its launch
    bool done = false;
    for (int64_t j = 0; e == hipSuccess && !done && kf < cap;) {
      const int64_t j0 = j;
      // (one launch where the last step's iterations fit into it, and one
      // more where they just did not: 300^2 D2Q9 that takes 3 and 2 in turn
      // 96 us per step, 80 so)
      const int64_t burst = j <= 1 && k0 < kTileIt ? 1 : kBurst;
      for (; j < j0 + burst && from(j) < cap && e == hipSuccess; ++j)
        e = launch(j, (int)(from(j + 1) - from(j)), j == 0 && k0 < kTileIt);
      if (e == hipSuccess) e = read();
      if (e != hipSuccess) break;
      take();
      for (int64_t i = j0; i < j && !done; ++i)
        for (int64_t k = from(i); k < from(i + 1) && !done; ++k) {
          kf = k + 1;
          jf = i;
          done = !hc.open[i % kSets][k - from(i)];
        }
    }
    if (e != hipSuccess) return e;
    // the launch that holds it again, up to it (unless that was the guess)
    const int kk = (int)(kf - from(jf));
    if (k0 == kTileIt || jf > 0 || kk < from(1)) e = launch(jf, kk, true);
    if (e != hipSuccess) return e;
    h->ilf_last = (int32_t)kf;
    ilfbm_sum_kernel<<<1, 256, 0, h->stream>>>(h->pend, iter_tiles(&p, kk),
                                               ctrl);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    std::swap(h->lf, h->lscr[jf & 1]);
    h->cur ^= 1;
    h->steps++;
    h->ilf_max_it = std::max(h->ilf_max_it, (int32_t)kf);
    if (!done) h->ilf_nonconv++;
    pending = true;
    capped = !done;
  }
  if (pending) {
    hipError_t e = read();
    if (e != hipSuccess) return e;
    take();
  }
  return hipSuccess;
}
