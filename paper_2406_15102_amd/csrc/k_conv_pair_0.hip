#include "conv_pair_impl.hpp"

namespace hlq {

hipError_t launch_conv_pair_0(const ConvDxPlan &p, bool f32, const GemmDev &gb, bool partial, bool b_first, hipStream_t st)
{
    return f32 ? launch_conv_pair_k<true, 0>(p, gb, partial, b_first, st) : launch_conv_pair_k<false, 0>(p, gb, partial, b_first, st);
}

}  // namespace hlq
