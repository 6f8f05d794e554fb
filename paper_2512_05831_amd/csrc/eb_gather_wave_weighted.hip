// The wave gather with per-sample weights, instantiated apart from the
// unweighted one so the parts build in parallel.
#include "eb_gather_wave.h"

namespace eb_gather {

KernelFn pick_wave_weighted_kernel(bool i32, int dtype, int R, int C, bool stream)
{
    return i32 ? pick_wave_kernel<int32_t, true>(dtype, R, C, stream) : pick_wave_kernel<int64_t, true>(dtype, R, C, stream);
}

} // namespace eb_gather
