// The wave gather without weights; the weighted one is built in parallel from
// eb_gather_wave_weighted.hip.
#include "eb_gather_wave.h"

namespace eb_gather {

KernelFn pick_wave_kernel(bool weighted, bool i32, int dtype, int R, int C, bool stream)
{
    if (weighted) return pick_wave_weighted_kernel(i32, dtype, R, C, stream);
    return i32 ? pick_wave_kernel<int32_t, false>(dtype, R, C, stream) : pick_wave_kernel<int64_t, false>(dtype, R, C, stream);
}

} // namespace eb_gather
