// md_step.hip -- instantiation of the persistent step kernel (md_step_kernel.h)
// with the nominal constants for every drone.
// Compiled once per action type (MD_ACT).
#include "md_step_kernel.h"

namespace md {

template <>
hipError_t launch_step<MD_ACT>(const StepArgs &a, uint32_t mask, const LaunchCfg &cfg,
                               int n_bins, int slots, hipStream_t stream) {
    return launch_step_t<MD_ACT, 0>(a, mask, cfg, n_bins, slots, stream);
}

}  // namespace md
