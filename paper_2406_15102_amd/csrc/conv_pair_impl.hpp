// The image gradient of a convolution (conv_dx_body.hpp) and its weight gradient's product (128 x 128 tiles of
// gemm_body.hpp) in one launch, for the reasons given in gemm_pair_impl.hpp: neither fills the chip alone.
// A workgroup runs the body of whichever its index falls in; the one with the longer tiles goes first, padded
// to a multiple of 8 workgroups so that the other's keep their XCDs.
// One translation unit per kind of the weight gradient's operands (k_conv_pair_*.hip); k_conv_dx.hip plans and dispatches.
#pragma once
#include "conv_dx_plan.hpp"
#include "gemm_body.hpp"

namespace hlq {

template <bool F32, int KB, bool TAIL, int OUTB>
__global__ __launch_bounds__(256, 2) void k_conv_pair(ConvDx ga, GemmDev gb, int n0, int n0_pad, int b_first)
{
    const int b = static_cast<int>(blockIdx.x);
    const bool in_first = b < n0_pad;
    if (in_first && b >= n0) return;                    // padding
    const int idx = in_first ? b : b - n0_pad;
    if (in_first != (b_first != 0)) conv_dx_any<F32>(ga, idx);
    else gemm_tile<KB, 2, 2, 8, TAIL, OUTB>(gb, idx);
}

template <bool F32, int KB, bool TAIL, int OUTB>
static hipError_t launch_conv_pair_t(const ConvDxPlan &p, const GemmDev &gb, bool b_first, hipStream_t st)
{
    const size_t lds_bytes = p.lds > gemm_lds_bytes(2, 2, 8) ? p.lds : gemm_lds_bytes(2, 2, 8);
    static bool attr_set = false;     // idempotent; racing callers set the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_conv_pair<F32, KB, TAIL, OUTB>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kConvDxMaxLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int nB = gb.tiles_m * gb.tiles_n * gb.splits;
    const int n0 = b_first ? nB : p.blocks, n1 = b_first ? p.blocks : nB;
    const int n0_pad = (n0 + 7) & ~7;
    hipLaunchKernelGGL((k_conv_pair<F32, KB, TAIL, OUTB>), dim3(n0_pad + n1), dim3(256), lds_bytes, st, p.g, gb,
                       n0, n0_pad, b_first ? 1 : 0);
    return hipGetLastError();
}

// the weight gradient writes what the image gradient writes (F32), or its split-k partials
template <bool F32, int KB>
static hipError_t launch_conv_pair_k(const ConvDxPlan &p, const GemmDev &gb, bool partial, bool b_first, hipStream_t st)
{
    const bool tail = gb.Kb % 128 != 0;
    if (partial)
        return tail ? launch_conv_pair_t<F32, KB, true, 3>(p, gb, b_first, st) : launch_conv_pair_t<F32, KB, false, 3>(p, gb, b_first, st);
    return tail ? launch_conv_pair_t<F32, KB, true, F32 ? 1 : 0>(p, gb, b_first, st)
                : launch_conv_pair_t<F32, KB, false, F32 ? 1 : 0>(p, gb, b_first, st);
}

}  // namespace hlq
