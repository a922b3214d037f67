// Kernel instantiations for the FCFS policy, prompt prefilled at admission.
#include "sim_kernel.hpp"

namespace fs {
hipError_t launch_sim_fcfs_prefill(const SimArgs& a, int K, int NW, int waves_per_block,
                                   size_t lds_bytes, hipStream_t s) {
  return launch_sim<POL_FCFS, false, true>(a, K, NW, waves_per_block, lds_bytes, s);
}
}  // namespace fs
