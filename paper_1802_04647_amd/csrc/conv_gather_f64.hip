// The gather kernels (conv_gather.hpp) in double and their launch.
#include "conv_gather_launch.hpp"

namespace dmlnn {

hipError_t launch_gather_f64(bool bwd, const GatherPlan &p, gather::FwdArgs a, hipStream_t s)
{
    return bwd ? gather::launch<double, true>(p, a, s) : gather::launch<double, false>(p, a, s);
}

hipError_t launch_gather_wgrad_f64(const GatherPlan &p, gather::WgArgs a, hipStream_t s)
{
    return gather::launch_wgrad<double>(p, a, s);
}

}  // namespace dmlnn
