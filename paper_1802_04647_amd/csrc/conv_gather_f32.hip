// The gather kernels (conv_gather.hpp) in float and their launch.
#include "conv_gather_launch.hpp"

namespace dmlnn {

hipError_t launch_gather_f32(bool bwd, const GatherPlan &p, gather::FwdArgs a, hipStream_t s)
{
    return bwd ? gather::launch<float, true>(p, a, s) : gather::launch<float, false>(p, a, s);
}

hipError_t launch_gather_wgrad_f32(const GatherPlan &p, gather::WgArgs a, hipStream_t s)
{
    return gather::launch_wgrad<float>(p, a, s);
}

}  // namespace dmlnn
