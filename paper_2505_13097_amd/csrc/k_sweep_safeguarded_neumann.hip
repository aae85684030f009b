// k_sweep_safeguarded_neumann.hip -- sweep kernels of one node-update mode.
#include "launch_sweep.hpp"

IREBM_INSTANTIATE_SWEEP(irebm::kSafeguarded | irebm::kNeumann);
