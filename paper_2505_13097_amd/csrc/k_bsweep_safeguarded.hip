// k_bsweep_safeguarded.hip -- batched sweep kernels of one node-update mode.
#include "launch_sweep.hpp"

IREBM_INSTANTIATE_BATCH_SWEEP(irebm::kSafeguarded);
