// k_bsweep_plain.hip -- batched sweep kernels of one node-update mode.
#include "launch_sweep.hpp"

IREBM_INSTANTIATE_BATCH_SWEEP(irebm::kPlain);
