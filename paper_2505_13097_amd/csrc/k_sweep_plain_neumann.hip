// k_sweep_plain_neumann.hip -- sweep kernels of one node-update mode.
#include "launch_sweep.hpp"

IREBM_INSTANTIATE_SWEEP(irebm::kPlain | irebm::kNeumann);
