// batch.hip -- many independent IREBM lattices of uneven sizes and
// parameters advanced by one persistent kernel launch per time step.
//
// Every instance gets a descriptor (its StepArgs: sizes, physics,
// boundaries, buffers, statistics base) and its work items (stacks of
// tiles, see step_item) are listed in one flat table, instance by
// instance and row by row within an instance.  A grid of one block per
// item, or a persistent grid of (compute units x blocks per CU) blocks,
// walks that table: the table is cut into eight contiguous chunks, one per
// XCD (block b runs on XCD b mod 8), so neighbouring tiles of an instance
// are swept by the same XCD and share its L2.  The node update is the one of
// the single-lattice step (step_item), so a batch member evolves exactly
// as the same lattice run alone, IREBM or EEBM alike.  Steps can be
// captured in a hipGraph; the autotuner picks the tile variant and the
// grid size.  Under a two-step variant a launch takes up to four steps by
// sweeping waves, the walls and fronts of every instance as a frame of small
// tiles in LDS (batch_sweep_kernel, sweep2d.hpp); where too many of their
// rows hold solves, single steps instead (RouteCtl).  This unit is the host
// side; the kernels and their launches are in launch.hpp and
// launch_sweep.hpp (instantiated by k_batch_<mode>.hip, k_bsweep_<mode>.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "host_util.hpp"
#include "kernels.hpp"
#include "lbm_stefan.h"
#include "lbm_stefan_internal.hpp"

using namespace irebm;

struct lbm_stefan_batch {
  std::vector<lbm_stefan_params> ps;
  int count = 0, q = 0, storage = 0;
  int mode = kSafeguarded;  // node-update mode shared by the instances
  int device = 0, cus = 0;
  hipStream_t stream = nullptr, cap_stream = nullptr;
  // sweeps of IREBM lattices: the single steps' launches of a large batch go
  // on a stream of their own, forked from and joined into the launching one
  hipStream_t side = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
  char *ws = nullptr;
  StepArgs *descs = nullptr;
  int2 *items = nullptr;
  StatSlot *slots = nullptr;
  SweepPlan *plans = nullptr;  // two-step variants
  BatchQuery *query = nullptr; // count + 1 entries
  RouteCtl *route = nullptr;
  int2 *singles = nullptr;     // the single steps' items beside sweeps
  int64_t nsingles = 0;
  bool beside = false;         // ... on a stream of their own (kRouteBeside)
  int32_t chain_max = 0;       // what sweeps may hold (RouteCtl)
  unsigned long long units_max = 0;
  int64_t nparts = 0;          // energy chunks of all instances
  double *profs = nullptr, *partials = nullptr, *small = nullptr;
  char *state[2] = {nullptr, nullptr};
  size_t state_bytes = 0;
  int graph_flip = 0;          // does a graph end in the other buffer?
  int64_t nslots = 0, ntiles = 0;
  std::vector<size_t> off;          // instance offset in a state region
  std::vector<size_t> prof_off;     // instance offset in the profiles
  std::vector<int64_t> first_item, nitems_inst;
  int64_t max_items = 0, nitems = 0;
  int cur = 0;
  int variant = kDefaultVariant2D, blocks_per_cu = 0, graph_steps = 0;
  int run = kDefaultVariant2D; // what the variant runs as (run_variant)
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  int64_t steps = 0;
  std::string err;
};

namespace {

struct BLayout {
  size_t descs, items, singles, slots, plans, query, route, profs, partials,
      small, stateA, stateB, total;
  size_t state_bytes;
  int64_t max_items, max_parts, small_len;
  std::vector<size_t> off, prof_off;
};

// work items (and statistics slots) of an instance under variant v
int64_t batch_items(const Variant &v, const lbm_stefan_params &p,
                    int64_t nodes) {
  return v.tb ? batch_plan(p, v, nodes).slots() : items_for(v, p.nx, p.ny);
}

int64_t batch_nodes(const lbm_stefan_params *ps, int count) {
  int64_t nodes = 0;
  for (int k = 0; k < count; ++k) nodes += ps[k].nx * ps[k].ny;
  return nodes;
}

// do batches of p sweep by groups (RouteCtl)?
bool routed(const Variant &v, const lbm_stefan_params &p) {
  return v.tb && p.scheme == LBM_SCHEME_IREBM;
}
// statistics slots of an instance under variant v
int64_t batch_slots(const Variant &v, const lbm_stefan_params &p,
                    int64_t nodes) {
  int nv;
  const int64_t n = batch_items(v, p, nodes);
  if (!routed(v, p)) return n;
  return std::max(n, items_for(variants(p.q, &nv)[kDefaultVariant2D], p.nx,
                               p.ny));
}

// Do two-step variants of a batch sweep?  The frame's tiles compute each node
// up to four times over, and lattices too small for a strip are all tiles, so
// the batch takes single steps (the default tiling) where more than 0.3 of its
// nodes lie in frames, EEBM 0.35 (us per step, single steps / sweeps: 1000
// FP32 D2Q5 lattices of 64^2 80 / 205, EEBM 46 / 66; 600 FP64 D2Q9 ones 131 /
// 269; 500 FP32 D2Q9 ones of 87^2 119 / 204; 100 FP64 D2Q5 ones of 150^2, 0.26
// in frames, 58 / 49; 60 FP64 D2Q9 ones of 200^2 107 / 73; EEBM 110^2, 0.27,
// 40 / 22, 70 FP64 D2Q5 ones of about 1600 x 30, 0.4, 42 / 47).
bool batch_sweeps(const lbm_stefan_params *ps, int count) {
  int nv;
  const Variant &v = variants(ps[0].q, &nv)[kSweepVariant2D];
  const int64_t all = batch_nodes(ps, count);
  double strips = 0.0;
  for (int k = 0; k < count; ++k) {
    const SweepPlan P = batch_plan(ps[k], v, all);
    strips += (double)(P.xb - P.xa) * (P.yb - P.ya);
  }
  return all - strips <= (ps[0].scheme == LBM_SCHEME_EEBM ? 0.35 : 0.3) * all;
}

// what variant v of a batch runs as
int run_variant(const lbm_stefan_params *ps, int count, int v) {
  int nv;
  return variants(ps[0].q, &nv)[v].tb && !batch_sweeps(ps, count)
             ? kDefaultVariant2D
             : v;
}

// the variant a batch starts with (and -1 selects): sweeping waves, unless the
// batch is small or of small lattices, or a member is an IREBM melt that
// freezes (see sweep_nodes, sweep_default)
int default_variant(const lbm_stefan_params *ps, int count) {
  if (ps[0].q == 3) return kDefaultVariant1D;
  const int64_t nodes = batch_nodes(ps, count);
  if (ps[0].scheme == LBM_SCHEME_IREBM && nodes <= sweep_nodes(ps[0].storage))
    return kDefaultVariant2D;
  for (int k = 0; k < count; ++k) {
    bool hot;
    front_walls(ps[k], &hot);
    if (ps[k].scheme == LBM_SCHEME_IREBM && !hot) return kDefaultVariant2D;
  }
  return run_variant(ps, count, kSweepVariant2D);
}

int bfail(lbm_stefan_batch_t *b, int code, const std::string &msg) {
  if (b) b->err = msg;
  else set_global_error(msg);
  return code;
}

#define BCHK(b, expr)                                                    \
  do {                                                                   \
    hipError_t e_ = (expr);                                              \
    if (e_ != hipSuccess)                                                \
      return bfail((b), LBM_STEFAN_EDEVICE,                              \
                   std::string(#expr) + ": " + hipGetErrorString(e_));   \
  } while (0)

std::string validate_batch(const lbm_stefan_params *ps, int32_t count) {
  if (!ps) return "params is NULL";
  if (count < 1 || count > (1 << 20)) return "count must be in 1..2^20";
  for (int k = 0; k < count; ++k) {
    const std::string e = validate_params(&ps[k]);
    if (!e.empty()) return "instance " + std::to_string(k) + ": " + e;
    if (ps[k].dim == 3)
      return "instance " + std::to_string(k) +
             ": the batched form takes 1D and 2D lattices";
    if (ps[k].q != ps[0].q || ps[k].storage != ps[0].storage ||
        ps[k].newton_mode != ps[0].newton_mode ||
        ps[k].scheme != ps[0].scheme)
      return "instances must share lattice, storage, newton_mode and scheme";
    if (has_neumann(ps[k]))
      return "instance " + std::to_string(k) +
             ": the batched form has no Neumann closure";
    if (ps[k].scheme == LBM_SCHEME_ILFBM)
      return "instance " + std::to_string(k) +
             ": the batched form runs IREBM and EEBM only";
  }
  return "";
}

BLayout batch_layout(const lbm_stefan_params *ps, int32_t count) {
  BLayout L;
  const size_t s = ps[0].storage == LBM_STORE_F64 ? 8 : 4;
  int nv;
  const Variant *v = variants(ps[0].q, &nv);
  const int64_t nodes = batch_nodes(ps, count);
  L.max_items = 0;
  for (int i = 0; i < nv; ++i) {
    int64_t t = 0;
    for (int k = 0; k < count; ++k) t += batch_slots(v[i], ps[k], nodes);
    L.max_items = std::max(L.max_items, t);
  }
  L.max_parts = 0;
  L.state_bytes = 0;
  L.off.resize(count);
  L.prof_off.resize(count);
  size_t prof_total = 0;
  int64_t max_ny = 16;
  for (int k = 0; k < count; ++k) {
    const int64_t n = ps[k].nx * ps[k].ny;
    L.off[k] = L.state_bytes;
    L.state_bytes += align256((size_t)ps[k].q * n * s);
    L.prof_off[k] = prof_total;
    prof_total += 4 * (size_t)std::max(ps[k].nx, ps[k].ny);
    max_ny = std::max(max_ny, ps[k].ny);
    L.max_parts += (n + kEnergyChunk - 1) / kEnergyChunk;
  }
  L.max_parts = std::max(L.max_parts, stats_partials(L.max_items));
  L.small_len = 16 * (int64_t)count + max_ny + 16;
  size_t o = 0;
  L.descs = o;
  o += align256(count * sizeof(StepArgs));
  L.items = o;
  o += align256(L.max_items * sizeof(int2));
  L.singles = o;
  for (int k = 0; k < count && ps[0].q != 3; ++k)
    o += items_for(v[kDefaultVariant2D], ps[k].nx, ps[k].ny) * sizeof(int2);
  o = align256(o);
  L.slots = o;
  o += align256(L.max_items * sizeof(StatSlot));
  L.plans = o;
  o += align256(count * sizeof(SweepPlan));
  L.query = o;
  o += align256((count + 1) * sizeof(BatchQuery));
  L.route = o;
  o += align256(sizeof(RouteCtl));
  L.profs = o;
  o += align256(prof_total * 8);
  L.partials = o;
  o += align256(L.max_parts * 8);
  L.small = o;
  o += align256(L.small_len * 8);
  L.stateA = o;
  o += L.state_bytes;
  L.stateB = o;
  o += L.state_bytes;
  L.total = o;
  return L;
}

void drop_side(lbm_stefan_batch_t *b) {
  if (b->fork) (void)hipEventDestroy(b->fork);
  if (b->join) (void)hipEventDestroy(b->join);
  if (b->side) (void)hipStreamDestroy(b->side);
  b->fork = b->join = nullptr;
  b->side = nullptr;
}

void drop_graphs(lbm_stefan_batch_t *b) {
  for (int k = 0; k < 2; ++k)
    if (b->graph[k]) {
      (void)hipGraphExecDestroy(b->graph[k]);
      b->graph[k] = nullptr;
    }
}

// What the sweeps of up to K steps may hold before the batch goes by single
// steps, which pass over the states (`bytes` in and out) at 4 TB/s: in one
// wave 0.105 (FP64) or 0.155 (FP32) rows with solves for every us of those
// (route_lattice); all such rows together may come to 0.65 of those steps'
// time (route_units; at 0.5 the first batch below leaves the sweeps at column
// 64, at 0.9 it never does).  us per step, single steps / sweeps with the front
// at column 8, 24, 64, 100, half way: 48 FP32 D2Q5 lattices of 64^2 to 1024^2
// 272 / 121, 158, 213, 267, 310; 12 D2Q9 ones of 512^2 to 1024^2 150 / 65, 89,
// 146, 171, 189; 400 D2Q5 ones of 64^2 to 256^2 188 to 231 / 178, 241, 361,
// 343, 364; 24 FP64 D2Q9 ones of 64^2 to 1024^2 384 / 156, 167, 203, 288, 376;
// 43 FP64 D2Q5 ones of up to 753 x 690, half way, 245 / 313; 11 of about 1200
// x 900 235 / 280.
void set_batch_route(lbm_stefan_batch_t *b, int K, double bytes) {
  const double us = K * bytes / 4e6;
  // ns of a unit (route_units)
  const double ns = b->storage == LBM_STORE_F64 ? 0.65 : 0.45;
  const double rows = us * (b->storage == LBM_STORE_F64 ? 0.105 : 0.155);
  b->chain_max = (int32_t)std::min(rows, 1e6);
  b->units_max = (unsigned long long)(0.65 * us * 1e3 / ns);
}

// descriptors and item table for the current variant; uploads both and
// zeroes the statistics (the item -> slot map changes with the items).
// The statistics slots of instance k are contiguous.
int build_schedule(lbm_stefan_batch_t *b) {
  int nv;
  const Variant *vt = variants(b->q, &nv);
  b->run = run_variant(b->ps.data(), b->count, b->variant);
  const Variant &v = vt[b->run];
  const bool two = routed(v, b->ps[0]);   // (also laid out for single steps)
  std::vector<StepArgs> d(b->count);
  std::vector<SweepPlan> pl(b->count);
  std::vector<BatchQuery> qu(b->count + 1);
  std::vector<int2> t, wv, sg;
  t.reserve(b->max_items);
  b->first_item.assign(b->count, 0);
  b->nitems_inst.assign(b->count, 0);
  int64_t sbase = 0;
  b->nparts = 0;
  double bytes = 0.0;
  const int64_t nodes = batch_nodes(b->ps.data(), b->count);
  for (int k = 0; k < b->count; ++k) {
    const lbm_stefan_params &p = b->ps[k];
    double *prof[4];
    for (int w = 0; w < 4; ++w)
      prof[w] = p.wall_profile[w] ? b->profs + b->prof_off[k] +
                                        w * std::max(p.nx, p.ny)
                                  : nullptr;
    fill_args(p, prof, &d[k]);
    d[k].src = b->state[0] + b->off[k];
    d[k].dst = b->state[1] + b->off[k];
    set_tiling(&d[k], two ? vt[kDefaultVariant2D] : v);
    bytes += 2.0 * p.q * (p.storage == LBM_STORE_F64 ? 8 : 4) * p.nx * p.ny;
    for (int i = 0; two && i < d[k].nitems; ++i) sg.push_back(make_int2(k, i));
    const int64_t n = batch_slots(v, p, nodes);
    d[k].slots = b->slots + sbase;
    b->first_item[k] = sbase;
    if (v.tb) {
      pl[k] = batch_plan(p, v, nodes);
      pl[k].ctl = two ? b->route : nullptr;
      for (int64_t i = 0; i < pl[k].tiles(); ++i)
        t.push_back(make_int2(k, (int)i));
      for (int64_t i = 0; i < pl[k].waves(); ++i)
        wv.push_back(make_int2(k, (int)i));
    } else {
      for (int64_t i = 0; i < n; ++i) t.push_back(make_int2(k, (int)i));
    }
    b->nitems_inst[k] = n;
    sbase += n;
    qu[k].part = b->nparts;
    qu[k].nslots = n;
    b->nparts += (p.nx * p.ny + kEnergyChunk - 1) / kEnergyChunk;
  }
  qu[b->count].part = b->nparts;
  qu[b->count].nslots = 0;
  b->ntiles = (int64_t)t.size();
  t.insert(t.end(), wv.begin(), wv.end());
  b->nitems = (int64_t)t.size();
  b->nsingles = (int64_t)sg.size();
  b->beside = nodes > kRouteBeside;
  set_batch_route(b, 4, bytes);
  BCHK(b, hipMemcpyAsync(b->descs, d.data(), d.size() * sizeof(StepArgs),
                         hipMemcpyHostToDevice, b->stream));
  BCHK(b, hipMemcpyAsync(b->items, t.data(), t.size() * sizeof(int2),
                         hipMemcpyHostToDevice, b->stream));
  if (two)
    BCHK(b, hipMemcpyAsync(b->singles, sg.data(), sg.size() * sizeof(int2),
                           hipMemcpyHostToDevice, b->stream));
  if (two && b->beside && !b->side) {
    BCHK(b, hipStreamCreateWithFlags(&b->side, hipStreamNonBlocking));
    BCHK(b, hipEventCreateWithFlags(&b->fork, hipEventDisableTiming));
    BCHK(b, hipEventCreateWithFlags(&b->join, hipEventDisableTiming));
  }
  BCHK(b, zero_async(b->route, sizeof(RouteCtl), b->stream));
  BCHK(b, hipMemcpyAsync(b->plans, pl.data(), pl.size() * sizeof(SweepPlan),
                         hipMemcpyHostToDevice, b->stream));
  BCHK(b, hipMemcpyAsync(b->query, qu.data(), qu.size() * sizeof(BatchQuery),
                         hipMemcpyHostToDevice, b->stream));
  BCHK(b, zero_async(b->slots, b->nslots * sizeof(StatSlot), b->stream));
  BCHK(b, hipStreamSynchronize(b->stream));
  drop_graphs(b);
  return LBM_STEFAN_OK;
}

bool routed(const lbm_stefan_batch_t *b) {
  int nv;
  return routed(variants(b->q, &nv)[b->run], b->ps[0]);
}

// one launch of k steps (at most steps_per_launch) from buffer `parity`
hipError_t launch_batch(const lbm_stefan_batch_t *b, hipStream_t stream,
                        int parity, int k, RouteCtl *ctl = nullptr) {
  int nv;
  const Variant *vt = variants(b->q, &nv);
  const Variant &v = vt[b->run];
  BatchLaunch L;
  L.descs = b->descs;
  L.items = b->items;
  L.nitems = b->nitems;
  L.cus = b->cus;
  L.blocks_per_cu = b->run == b->variant ? b->blocks_per_cu : 0;
  L.parity = parity;
  L.ctl = ctl;
  if (!v.tb) return batch_launch(b->mode, b->q, b->storage, L, v, stream);
  L.plans = b->plans;
  L.ntiles = b->ntiles;
  return batch_sweep(b->mode, b->q, b->storage, L, k, stream);
}

// a single step beside the sweeps
hipError_t launch_single(const lbm_stefan_batch_t *b, hipStream_t stream,
                         int parity, RouteCtl *ctl) {
  int nv;
  BatchLaunch L;
  L.descs = b->descs;
  L.items = b->singles;
  L.nitems = b->nsingles;
  L.cus = b->cus;
  L.blocks_per_cu = 0;
  L.parity = parity;
  L.ctl = ctl;
  return batch_launch(b->mode, b->q, b->storage, L,
                      variants(b->q, &nv)[kDefaultVariant2D], stream);
}

// time steps one launch advances at most under the current variant
int steps_per_launch(const lbm_stefan_batch_t *b) {
  int nv;
  return variants(b->q, &nv)[b->run].tb ? 4 : 1;
}

// nsteps steps from buffer `parity`, which follows them; sweeps that are
// routed go by groups, as in advance_routed
hipError_t advance_batch(const lbm_stefan_batch_t *b, hipStream_t stream,
                         int *parity, int64_t nsteps) {
  const int64_t K = steps_per_launch(b);
  hipError_t e = hipSuccess;
  if (!routed(b)) {
    while (nsteps > 0 && e == hipSuccess) {
      const int64_t m = (nsteps + K - 1) / K;
      const int64_t k = (nsteps + m - 1) / m;
      e = launch_batch(b, stream, *parity, (int)k);
      *parity ^= 1;
      nsteps -= k;
    }
    return e;
  }
  while (nsteps > 0 && e == hipSuccess) {
    const int64_t n = nsteps >= 32 * K ? 16 * K : nsteps;
    int64_t m = (n + K - 1) / K;
    m += (m ^ n) & 1;
    if (n / m < 2) {
      e = launch_single(b, stream, *parity, nullptr);
      *parity ^= 1;
      nsteps--;
      continue;
    }
    if (b->beside) e = hipEventRecord(b->fork, stream);
    if (b->beside && e == hipSuccess)
      e = hipStreamWaitEvent(b->side, b->fork, 0);
    int p = *parity, c = *parity;
    for (int64_t i = 0, left = n; i < m && e == hipSuccess; ++i, p ^= 1) {
      const int64_t k = (left + m - i - 1) / (m - i);
      e = launch_batch(b, stream, p, (int)k, b->route);
      for (int64_t j = 0; j < k && e == hipSuccess; ++j, c ^= 1)
        e = launch_single(b, b->beside ? b->side : stream, c, b->route);
      left -= k;
    }
    if (b->beside && e == hipSuccess) e = hipEventRecord(b->join, b->side);
    if (b->beside && e == hipSuccess)
      e = hipStreamWaitEvent(stream, b->join, 0);
    if (e != hipSuccess) break;
    // (units add up over the group's launches)
    route_decide_kernel<<<1, 1, 0, stream>>>(b->route, 0, b->chain_max,
                                             b->units_max * m);
    e = hipGetLastError();
    *parity ^= n & 1;
    nsteps -= n;
  }
  return e;
}

// the route of the batch's current states
hipError_t scan_route(lbm_stefan_batch_t *b) {
  if (!routed(b)) return hipSuccess;
  const int64_t nw = b->nitems - b->ntiles;
  hipError_t e = hipSuccess;
  if (nw > 0)
    e = dispatch_qs(b->q, b->storage, [&](auto qt, auto tt) {
      QS_TYPES(qt, tt);
      batch_route_scan_kernel<Q, S><<<(unsigned)((nw + 3) / 4), 256, 0,
                                      b->stream>>>(
          b->descs, b->plans, b->items + b->ntiles, (int32_t)nw, b->cur,
          b->route);
      return hipGetLastError();
    });
  if (e != hipSuccess) return e;
  route_decide_kernel<<<1, 1, 0, b->stream>>>(b->route, 1, b->chain_max,
                                              b->units_max);
  return hipGetLastError();
}

// graph of the launches of graph_steps steps starting at parity `par`
int ensure_graph(lbm_stefan_batch_t *b, int par) {
  if (b->graph[par]) return LBM_STEFAN_OK;
  if (!b->cap_stream)
    BCHK(b, hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
  BCHK(b, hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
  int p = par;
  const hipError_t le = advance_batch(b, b->cap_stream, &p, b->graph_steps);
  b->graph_flip = p ^ par;
  hipGraph_t g = nullptr;
  const hipError_t ee = hipStreamEndCapture(b->cap_stream, &g);
  if (le != hipSuccess || ee != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    return bfail(b, LBM_STEFAN_EDEVICE,
                 std::string("graph capture failed: ") +
                     hipGetErrorString(le != hipSuccess ? le : ee));
  }
  const hipError_t ie = hipGraphInstantiate(&b->graph[par], g, nullptr,
                                            nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ie != hipSuccess) {
    b->graph[par] = nullptr;
    return bfail(b, LBM_STEFAN_EDEVICE,
                 std::string("hipGraphInstantiate: ") + hipGetErrorString(ie));
  }
  return LBM_STEFAN_OK;
}

}  // namespace

extern "C" {

const char *lbm_stefan_batch_last_error(const lbm_stefan_batch_t *b) {
  return b ? b->err.c_str() : lbm_stefan_last_error(nullptr);
}

int lbm_stefan_batch_workspace_bytes(const lbm_stefan_params *ps,
                                     int32_t count, size_t *bytes) {
  const std::string e = validate_batch(ps, count);
  if (!e.empty()) return bfail(nullptr, LBM_STEFAN_EINVAL, e);
  if (!bytes) return bfail(nullptr, LBM_STEFAN_EINVAL, "bytes is NULL");
  *bytes = batch_layout(ps, count).total;
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_init(const lbm_stefan_params *ps, int32_t count,
                          const double *const *T0, void *workspace,
                          size_t bytes, void *stream,
                          lbm_stefan_batch_t **out) {
  const std::string e = validate_batch(ps, count);
  if (!e.empty()) return bfail(nullptr, LBM_STEFAN_EINVAL, e);
  if (!out) return bfail(nullptr, LBM_STEFAN_EINVAL, "out is NULL");
  *out = nullptr;
  const BLayout L = batch_layout(ps, count);
  if (!workspace || bytes < L.total)
    return bfail(nullptr, LBM_STEFAN_EINVAL, "workspace too small");
  if ((uintptr_t)workspace % 256)
    return bfail(nullptr, LBM_STEFAN_EINVAL, "workspace not 256-byte aligned");
  lbm_stefan_batch_t *b = new (std::nothrow) lbm_stefan_batch_t();
  if (!b) return bfail(nullptr, LBM_STEFAN_EDEVICE, "out of host memory");
  auto bail = [&](int code) {
    set_global_error(b->err);
    drop_graphs(b);
    drop_side(b);
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    delete b;
    return code;
  };
  b->ps.assign(ps, ps + count);
  b->count = count;
  b->q = ps[0].q;
  b->storage = ps[0].storage;
  b->mode = mode_of(ps[0]);
  b->stream = (hipStream_t)stream;
  if (hipGetDevice(&b->device) != hipSuccess ||
      hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount,
                            b->device) != hipSuccess)
    return bail(bfail(b, LBM_STEFAN_EDEVICE, "device query failed"));
  b->variant = default_variant(ps, count);
  char *ws = (char *)workspace;
  b->ws = ws;
  b->descs = (StepArgs *)(ws + L.descs);
  b->items = (int2 *)(ws + L.items);
  b->slots = (StatSlot *)(ws + L.slots);
  b->nslots = L.max_items;
  b->singles = (int2 *)(ws + L.singles);
  b->route = (RouteCtl *)(ws + L.route);
  b->plans = (SweepPlan *)(ws + L.plans);
  b->query = (BatchQuery *)(ws + L.query);
  b->profs = (double *)(ws + L.profs);
  b->partials = (double *)(ws + L.partials);
  b->small = (double *)(ws + L.small);
  b->state[0] = ws + L.stateA;
  b->state[1] = ws + L.stateB;
  b->state_bytes = L.state_bytes;
  b->off = L.off;
  b->prof_off = L.prof_off;
  b->max_items = L.max_items;
  for (int k = 0; k < count; ++k) {
    lbm_stefan_params &p = b->ps[k];
    if (p.dx == 0.0) p.dx = 1.0 / (double)(p.nx - 1);
    if (p.dim == 1) p.bc[2] = p.bc[3] = LBM_BC_PERIODIC;
    const int64_t plen = std::max(p.nx, p.ny);
    for (int w = 0; w < 4; ++w) {
      if (!ps[k].wall_profile[w] || (p.dim == 1 && w >= 2)) {
        p.wall_profile[w] = nullptr;
        continue;
      }
      const int64_t len = w < 2 ? p.ny : p.nx;
      for (int64_t j = 0; j < len; ++j)
        if (!std::isfinite(ps[k].wall_profile[w][j]))
          return bail(bfail(b, LBM_STEFAN_EINVAL, "wall profile not finite"));
      if (hipMemcpy(b->profs + L.prof_off[k] + w * plen, ps[k].wall_profile[w],
                    len * 8, hipMemcpyHostToDevice) != hipSuccess)
        return bail(bfail(b, LBM_STEFAN_EDEVICE, "copy of a wall profile failed"));
      p.wall_profile[w] = b->profs + L.prof_off[k] + w * plen;  // marker only
    }
  }
  if (build_schedule(b) != LBM_STEFAN_OK) return bail(LBM_STEFAN_EDEVICE);
  // initial states; T0 of instance k is staged through its B buffer
  std::vector<StepArgs> d(count);
  if (hipMemcpy(d.data(), b->descs, count * sizeof(StepArgs),
                hipMemcpyDeviceToHost) != hipSuccess)
    return bail(bfail(b, LBM_STEFAN_EDEVICE, "descriptor readback failed"));
  for (int k = 0; k < count; ++k) {
    const double *t0 = T0 ? T0[k] : nullptr;
    const int64_t n = b->ps[k].nx * b->ps[k].ny;
    double *stage = (double *)(b->state[1] + b->off[k]);
    if (t0 && hipMemcpy(stage, t0, n * 8, hipMemcpyHostToDevice) != hipSuccess)
      return bail(bfail(b, LBM_STEFAN_EDEVICE, "copy of T0 failed"));
    StepArgs A = d[k];
    A.dst = b->state[0] + b->off[k];
    if (init_async(b->q, b->storage, A, t0 ? stage : nullptr, b->stream) !=
        hipSuccess)
      return bail(bfail(b, LBM_STEFAN_EDEVICE, "init kernel failed"));
  }
  if (scan_route(b) != hipSuccess ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return bail(bfail(b, LBM_STEFAN_EDEVICE, "init failed"));
  *out = b;
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_set_schedule(lbm_stefan_batch_t *b, int32_t variant,
                                  int32_t blocks_per_cu, int32_t graph_steps) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  int nv;
  const Variant *vt = variants(b->q, &nv);
  if (variant < -1 || variant >= nv)
    return bfail(b, LBM_STEFAN_EINVAL, "unknown kernel variant");
  if (variant >= 0 && vt[variant].res)
    return bfail(b, LBM_STEFAN_EINVAL,
                 "the resident variant runs single lattices only");
  if (blocks_per_cu < 0 || blocks_per_cu > 32)
    return bfail(b, LBM_STEFAN_EINVAL, "blocks_per_cu must be in 0..32");
  if (graph_steps < 0 || graph_steps % 2 || graph_steps > 100000)
    return bfail(b, LBM_STEFAN_EINVAL,
                 "graph_steps must be even and in 0..100000");
  const int nvar = variant < 0 || vt[variant].lib
                       ? default_variant(b->ps.data(), b->count)
                       : variant;
  DeviceGuard g(b->device);
  b->blocks_per_cu = blocks_per_cu;
  b->graph_steps = graph_steps;
  drop_graphs(b);
  if (nvar != b->variant) {
    b->variant = nvar;
    const int rc = build_schedule(b);
    if (rc != LBM_STEFAN_OK) return rc;
    BCHK(b, scan_route(b));
  }
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_launches(const lbm_stefan_batch_t *b,
                              const char **kernel, int32_t *steps,
                              int32_t *routed_out) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  const int k = steps_per_launch(b);
  if (kernel)
    *kernel = k > 1 ? "batch_sweep_kernel"
              : b->blocks_per_cu > 0 && b->run == b->variant
                  ? "batch_persistent_kernel"
                  : "batch_step_kernel";
  if (steps) *steps = k;
  if (routed_out) *routed_out = routed(b);
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_step(lbm_stefan_batch_t *b, int64_t nsteps) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  if (nsteps < 0) return bfail(b, LBM_STEFAN_EINVAL, "nsteps < 0");
  DeviceGuard g(b->device);
  int64_t left = nsteps;
  if (b->graph_steps > 0) {
    while (left >= b->graph_steps) {
      const int rc = ensure_graph(b, b->cur);
      if (rc) return rc;
      BCHK(b, hipGraphLaunch(b->graph[b->cur], b->stream));
      left -= b->graph_steps;
      b->steps += b->graph_steps;
      b->cur ^= b->graph_flip;
    }
  }
  BCHK(b, advance_batch(b, b->stream, &b->cur, left));
  b->steps += left;
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_reset_stats(lbm_stefan_batch_t *b) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  DeviceGuard g(b->device);
  BCHK(b, zero_async(b->slots, b->nslots * sizeof(StatSlot), b->stream));
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_stats(lbm_stefan_batch_t *b, lbm_stefan_stats *out) {
  if (!b || !out) return bfail(b, LBM_STEFAN_EINVAL, "NULL argument");
  DeviceGuard g(b->device);
  std::vector<double> hs((size_t)b->count * 16);
  BCHK(b, dispatch_qs(b->q, b->storage, [&](auto qt, auto tt) {
         QS_TYPES(qt, tt);
         batch_energy_kernel<Q, S><<<(unsigned)b->nparts, 256, 0, b->stream>>>(
             b->descs, b->query, b->count, b->cur, b->mode == kEebm,
             b->partials);
         return hipGetLastError();
       }));
  batch_stats_kernel<<<(unsigned)b->count, 256, 0, b->stream>>>(
      b->descs, b->query, b->partials, b->small);
  BCHK(b, hipGetLastError());
  for (int k = 0; k < b->count; ++k)
    if (b->nitems_inst[k] > kStatsChunk)
      BCHK(b, stats_async(b->slots + b->first_item[k], b->nitems_inst[k],
                          b->partials, stats_partials(b->nitems_inst[k]),
                          b->small + 16 * k, b->stream));
  BCHK(b, hipMemcpyAsync(hs.data(), b->small, hs.size() * 8,
                         hipMemcpyDeviceToHost, b->stream));
  BCHK(b, hipStreamSynchronize(b->stream));
  bool finite = true;
  for (int k = 0; k < b->count; ++k) {
    const double *h = &hs[16 * (size_t)k];
    lbm_stefan_stats &s = out[k];
    s.steps = b->steps;
    s.max_newton_it = (int32_t)h[0];
    s.reserved = 0;
    s.nonconverged = (int64_t)h[1];
    s.max_residual = h[2];
    s.flux_in = h[3];
    s.flux_out = h[4];
    s.energy = h[8];
    finite = finite && std::isfinite(s.energy);
  }
  if (!finite) return bfail(b, LBM_STEFAN_ENAN, "an energy is not finite");
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_query_front(lbm_stefan_batch_t *b, int32_t inst,
                                 int32_t mode, double *front, double *energy) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  if (inst < 0 || inst >= b->count)
    return bfail(b, LBM_STEFAN_EINVAL, "instance out of range");
  if (mode != LBM_FRONT_LIQUID_INTEGRAL && mode != LBM_FRONT_ZERO_CROSSING)
    return bfail(b, LBM_STEFAN_EINVAL, "unknown front mode");
  DeviceGuard g(b->device);
  const lbm_stefan_params &p = b->ps[inst];
  const char *src = b->state[b->cur] + b->off[inst];
  double *fr = b->small + 16 * (int64_t)b->count + 16;
  if (front) {
    BCHK(b, front_async(p, src, mode, fr, b->stream));
    BCHK(b, hipMemcpyAsync(front, fr, p.ny * 8, hipMemcpyDeviceToHost,
                           b->stream));
  }
  double e = 0.0;
  if (energy) {
    BCHK(b, energy_async(p, src, b->partials,
                         b->small + 16 * (int64_t)b->count, b->stream));
    BCHK(b, hipMemcpyAsync(&e, b->small + 16 * (int64_t)b->count, 8,
                           hipMemcpyDeviceToHost, b->stream));
  }
  BCHK(b, hipStreamSynchronize(b->stream));
  if (energy) {
    *energy = e;
    if (!std::isfinite(e)) return bfail(b, LBM_STEFAN_ENAN, "energy not finite");
  }
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_get_field(lbm_stefan_batch_t *b, int32_t inst,
                               int32_t what, void *host) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  if (inst < 0 || inst >= b->count || !host)
    return bfail(b, LBM_STEFAN_EINVAL, "bad instance or host pointer");
  DeviceGuard g(b->device);
  const lbm_stefan_params &p = b->ps[inst];
  const int64_t n = p.nx * p.ny;
  const char *src = b->state[b->cur] + b->off[inst];
  if (what == LBM_FIELD_STATE) {
    const size_t s = b->storage == LBM_STORE_F64 ? 8 : 4;
    BCHK(b, hipMemcpyAsync(host, src, p.q * n * s, hipMemcpyDeviceToHost,
                           b->stream));
  } else if (what == LBM_FIELD_T) {
    // the instance's idle buffer holds >= 12 n bytes
    double *T = (double *)(b->state[b->cur ^ 1] + b->off[inst]);
    BCHK(b, temperature_async(p, src, T, b->stream));
    BCHK(b, hipMemcpyAsync(host, T, n * 8, hipMemcpyDeviceToHost, b->stream));
  } else {
    return bfail(b, LBM_STEFAN_EINVAL, "unknown field");
  }
  BCHK(b, hipStreamSynchronize(b->stream));
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_state_bytes(const lbm_stefan_batch_t *b, size_t *bytes) {
  if (!b || !bytes) return bfail(nullptr, LBM_STEFAN_EINVAL, "NULL argument");
  *bytes = b->state_bytes;
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_autotune(lbm_stefan_batch_t *b, void *scratch,
                              size_t scratch_bytes, int32_t steps,
                              int32_t *best_variant, int32_t *best_blocks_per_cu,
                              double *best_ms_per_step) {
  if (!b) return bfail(nullptr, LBM_STEFAN_EINVAL, "batch is NULL");
  if (!scratch || scratch_bytes < b->state_bytes)
    return bfail(b, LBM_STEFAN_EINVAL, "scratch smaller than the state");
  if (steps < 1 || steps > 10000)
    return bfail(b, LBM_STEFAN_EINVAL, "steps must be in 1..10000");
  DeviceGuard g(b->device);
  const int cur0 = b->cur;
  BCHK(b, hipMemcpyAsync(scratch, b->state[cur0], b->state_bytes,
                         hipMemcpyDeviceToDevice, b->stream));
  hipEvent_t e0, e1;
  BCHK(b, hipEventCreate(&e0));
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return bfail(b, LBM_STEFAN_EDEVICE, "hipEventCreate failed");
  }
  int nv;
  const Variant *vt = variants(b->q, &nv);
  const int bpcs[] = {0, 2, 4, 8};
  const int64_t nodes = batch_nodes(b->ps.data(), b->count);
  const int v0 = b->variant, bpc0 = b->blocks_per_cu;
  int best_v = v0, best_bpc = bpc0;
  float best_ms = -1.0f;
  int rc = LBM_STEFAN_OK;
  hipError_t err = hipSuccess;
  for (int v = 0; v < nv && rc == LBM_STEFAN_OK && err == hipSuccess; ++v) {
    // (single lattices only; one of the others)
    if (vt[v].res || vt[v].lib) continue;
    if (run_variant(b->ps.data(), b->count, v) != v) continue;
    // two-step variants differ by their segments' rows alone
    bool tried = false;
    for (int u = 0; u < v && vt[v].tb; ++u)
      tried |= vt[u].tb &&
               batch_rows(vt[u], nodes) == batch_rows(vt[v], nodes) &&
               vt[u].nt == vt[v].nt;
    if (tried) continue;
    if (v != b->variant) {
      b->variant = v;
      rc = build_schedule(b);
    }
    if (rc == LBM_STEFAN_OK) err = scan_route(b);
    // a sweeping launch covers four steps; the persistent grid is for
    // one-step variants only
    const int spl = steps_per_launch(b);
    const int launches = (steps + spl - 1) / spl;
    for (int bpc : bpcs) {
      if (rc != LBM_STEFAN_OK || err != hipSuccess) break;
      if (vt[v].tb && bpc > 0) break;
      b->blocks_per_cu = bpc;
      err = advance_batch(b, b->stream, &b->cur, 2 * spl);
      if (err == hipSuccess) err = hipEventRecord(e0, b->stream);
      if (err == hipSuccess)
        err = advance_batch(b, b->stream, &b->cur, (int64_t)launches * spl);
      if (err == hipSuccess) err = hipEventRecord(e1, b->stream);
      if (err == hipSuccess) err = hipEventSynchronize(e1);
      float ms = 0.0f;
      if (err == hipSuccess) err = hipEventElapsedTime(&ms, e0, e1);
      ms /= (float)(launches * spl);
      if (err == hipSuccess && (best_ms < 0.0f || ms < best_ms)) {
        best_ms = ms;
        best_v = v;
        best_bpc = bpc;
      }
      b->cur = cur0;
      if (err == hipSuccess)
        err = hipMemcpyAsync(b->state[cur0], scratch, b->state_bytes,
                             hipMemcpyDeviceToDevice, b->stream);
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  b->cur = cur0;
  if (rc != LBM_STEFAN_OK) return rc;
  if (err != hipSuccess)
    return bfail(b, LBM_STEFAN_EDEVICE,
                 std::string("autotune: ") + hipGetErrorString(err));
  b->blocks_per_cu = best_bpc;
  if (best_v != b->variant) {
    b->variant = best_v;
    rc = build_schedule(b);
    if (rc) return rc;
    BCHK(b, scan_route(b));
  } else {
    BCHK(b, zero_async(b->slots, b->nslots * sizeof(StatSlot), b->stream));
  }
  drop_graphs(b);
  BCHK(b, hipStreamSynchronize(b->stream));
  if (best_variant) *best_variant = best_v;
  if (best_blocks_per_cu) *best_blocks_per_cu = best_bpc;
  if (best_ms_per_step) *best_ms_per_step = best_ms;
  return LBM_STEFAN_OK;
}

int lbm_stefan_batch_destroy(lbm_stefan_batch_t *b) {
  if (!b) return LBM_STEFAN_OK;
  DeviceGuard g(b->device);
  hipError_t e = hipStreamSynchronize(b->stream);
  if (e == hipSuccess && b->side) e = hipStreamSynchronize(b->side);
  drop_graphs(b);
  drop_side(b);
  if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
  delete b;
  if (e != hipSuccess) return bfail(nullptr, LBM_STEFAN_EDEVICE, hipGetErrorString(e));
  return LBM_STEFAN_OK;
}

}  // extern "C"
