// md_step_dr.hip -- instantiation of the persistent step kernel
// (md_step_kernel.h) with domain randomisation (per-drone constants, motor
// bias and lag, action and sensor latency, sensor noise and bias), with or
// without wind.
// Compiled once per action type (MD_ACT).
#include "md_step_kernel.h"

namespace md {

template <>
hipError_t launch_step_dr<MD_ACT>(const StepArgs &a, uint32_t mask, const LaunchCfg &cfg,
                                  int n_bins, int slots, hipStream_t stream) {
    return launch_step_t<MD_ACT, 2>(a, mask, cfg, n_bins, slots, stream);
}

}  // namespace md
