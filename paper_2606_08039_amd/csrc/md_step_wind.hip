// md_step_wind.hip -- instantiation of the persistent step kernel
// (md_step_kernel.h) with wind and the nominal constants: the wind state and
// its Philox draws without the randomisation's per-drone registers.
// Compiled once per action type (MD_ACT).
#include "md_step_kernel.h"

namespace md {

template <>
hipError_t launch_step_wind<MD_ACT>(const StepArgs &a, uint32_t mask, const LaunchCfg &cfg,
                                    int n_bins, int slots, hipStream_t stream) {
    return launch_step_t<MD_ACT, 1>(a, mask, cfg, n_bins, slots, stream);
}

}  // namespace md
