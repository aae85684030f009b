// launch_sweep.hpp -- launches of sweep_kernel and batch_sweep_kernel for one
// node-update mode, instantiated by the k_sweep_<mode>.hip and
// k_bsweep_<mode>.hip units and reached through sweep_launch and
// batch_sweep (lbm_stefan_internal.hpp).
#pragma once

#include <hip/hip_runtime.h>

#include "host_util.hpp"
#include "lbm_stefan_internal.hpp"
#include "sweep2d.hpp"

namespace irebm {
namespace {

template <int Q, typename S, int MODE>
hipError_t launch_sweep_t(const StepArgs &A, const SweepPlan &P, int k,
                          char *mid, int64_t mid_stride, hipStream_t stream) {
  if constexpr (Q == 3) {
    return hipErrorInvalidValue;
  } else {
    if (k < 2 || k > P.k) return hipErrorInvalidValue;
    // strips as wide as k steps allow
    SweepPlan R = P;
    R.cut(64 - 2 * k);
    const int64_t ct = (R.tiles() + 7) / 8;
    const int64_t cw = (((R.waves() + 7) / 8) + 3) / 4;
    const unsigned grid = (unsigned)(8 * (ct + cw));
#define SWEEP(K, MID) \
  sweep_kernel<Q, S, MODE, K, MID><<<grid, 256, 0, stream>>>(A, R, mid, mid_stride)
#define SWEEP_K(MID)           \
  do {                         \
    if (k == 4) SWEEP(4, MID); \
    else if (k == 3) SWEEP(3, MID); \
    else SWEEP(2, MID);        \
  } while (0)
    if (k > 4) return hipErrorInvalidValue;
    // the states in between: the reverse mode's recomputation (IREBM)
    if (mid) {
      if constexpr (MODE == kSafeguarded || MODE == kPlain) SWEEP_K(true);
      else return hipErrorInvalidValue;
    } else {
      SWEEP_K(false);
    }
#undef SWEEP_K
#undef SWEEP
    return hipGetLastError();
  }
}

// k steps (1 to 4) of a batch (see BatchLaunch)
template <int Q, typename S, int MODE>
hipError_t launch_batch_sweep_t(const BatchLaunch &b, int k,
                                hipStream_t stream) {
  if constexpr (Q == 3) {
    return hipErrorInvalidValue;
  } else {
    const int64_t ct = (b.ntiles + 7) / 8;
    const int64_t cw = (((b.nitems - b.ntiles + 7) / 8) + 3) / 4;
    const unsigned grid = (unsigned)(8 * (ct + cw));
#define BSWEEP(K)                                                         \
  batch_sweep_kernel<Q, S, MODE, K><<<grid, 256, 0, stream>>>(            \
      b.descs, b.plans, b.items, (int32_t)b.ntiles, b.items + b.ntiles,   \
      (int32_t)(b.nitems - b.ntiles), b.parity, b.ctl)
    if (k == 4) BSWEEP(4);
    else if (k == 3) BSWEEP(3);
    else if (k == 2) BSWEEP(2);
    else if (k == 1) BSWEEP(1);
    else return hipErrorInvalidValue;
#undef BSWEEP
    return hipGetLastError();
  }
}

}  // namespace

template <int MODE>
hipError_t batch_sweep_mode(int q, int storage, const BatchLaunch &b, int k,
                            hipStream_t stream) {
  return dispatch_qs(q, storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    return launch_batch_sweep_t<Q, S, MODE>(b, k, stream);
  });
}

template <int MODE>
hipError_t sweep_launch_mode(int q, int storage, const StepArgs &A,
                             const SweepPlan &P, int k, char *mid,
                             int64_t mid_stride, hipStream_t stream) {
  return dispatch_qs(q, storage, [&](auto qt, auto tt) {
    QS_TYPES(qt, tt);
    return launch_sweep_t<Q, S, MODE>(A, P, k, mid, mid_stride, stream);
  });
}

}  // namespace irebm

#define IREBM_INSTANTIATE_SWEEP(M)                                         \
  template hipError_t irebm::sweep_launch_mode<M>(                         \
      int, int, const irebm::StepArgs &, const irebm::SweepPlan &, int,    \
      char *, int64_t, hipStream_t)

#define IREBM_INSTANTIATE_BATCH_SWEEP(M)                                   \
  template hipError_t irebm::batch_sweep_mode<M>(                          \
      int, int, const irebm::BatchLaunch &, int, hipStream_t)
