// The image gradient of a convolution (conv_dx_body.hpp): as a launch of its own, and the plan of the launch that
// carries the weight gradient's product beside it (conv_pair_impl.hpp).
#include "conv_dx_plan.hpp"

namespace hlq {

hipError_t launch_conv_pair_0(const ConvDxPlan &p, bool f32, const GemmDev &gb, bool partial, bool b_first, hipStream_t st);
hipError_t launch_conv_pair_1(const ConvDxPlan &p, bool f32, const GemmDev &gb, bool partial, bool b_first, hipStream_t st);

template <bool F32>
__global__ __launch_bounds__(256, 2) void k_conv_dx(ConvDx g)
{
    conv_dx_any<F32>(g, static_cast<int>(blockIdx.x));
}

template <bool F32>
static hipError_t launch_conv_dx_t(const ConvDxPlan &p, hipStream_t st)
{
    static bool attr_set = false;     // idempotent; racing callers set the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_conv_dx<F32>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kConvDxMaxLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    hipLaunchKernelGGL((k_conv_dx<F32>), dim3(p.blocks), dim3(256), p.lds, st, p.g);
    return hipGetLastError();
}

bool conv_dx_ok(int O, const ConvShape &s, bool is_f32)
{
    const int64_t lim = int64_t(1) << 31;
    const int64_t Kb = O, I = static_cast<int64_t>(s.kh) * s.kw * s.C;
    const int64_t pixels = static_cast<int64_t>(s.Nb) * s.H * s.W;
    return s.C % 4 == 0 && Kb % 16 == 0 && s.kh * static_cast<int64_t>(s.kw) <= kConvMaxTaps &&
           static_cast<int64_t>(s.sh) * s.sw <= 64 && s.N * Kb < lim && I * Kb < lim && s.N * 4 < lim && pixels < lim &&
           (pixels / 128 + 64) * ((s.C + 63) / 64) < (int64_t(1) << 29) &&
           s.H + 2 * static_cast<int64_t>(s.ph) + static_cast<int64_t>(s.kh) * s.dh < (int64_t(1) << 29) &&
           s.W + 2 * static_cast<int64_t>(s.pw) + static_cast<int64_t>(s.kw) * s.dw < (int64_t(1) << 29) && conv_dx_wanted(s, O, is_f32);
}

hipError_t launch_conv_dx(const GemmArgs &a, const ConvShape &s, hipStream_t st)
{
    if (!conv_dx_ok(a.K, s, a.c_is_f32)) return hipErrorInvalidValue;
    const ConvDxPlan p = conv_dx_plan(a, s);
    return a.c_is_f32 ? launch_conv_dx_t<true>(p, st) : launch_conv_dx_t<false>(p, st);
}

bool conv_pair_available() { return gemm_plan_forced_tile() != 256; }

// Plan of the launch: the k split of the weight gradient's product and which of the two goes first.  Where the image
// gradient leaves room for the other's tiles beside it -- two workgroups a compute unit, 512 -- all of them are resident
// at once: as many splits as fit, of eight steps or more, behind it (whole passes: 12544 pixels x 256
// channels, 36 tiles, 500 workgroups at 3 splits 47.2 us, 536 at 4 56.0; 16 x 14 x 14 x 64, 4 x 4 with stride 2, over 64, eight
// steps: not split and no reduction 14.3, 2 splits 16.7).  Larger layers by the model of gemm_plan.hpp, with the image
// gradient's tiles as the first product.
// Neither looks at how long the weight gradient's tiles are beside a small image gradient that fills the chip (whole pass of
// 40 x 56 x 56 x 24, 5 x 5, over 384, fp32: 490 blocks leave its 15 tiles of 980 steps whole, 754 us; 16 splits 332): a choice
// that conv_pair_time prices a sixth lower takes their place.  Over 470 layers, every split in either order measured, that
// takes the mean distance to the best one from 3.7 to 2.2 %, 54 layers by more than 2 % faster, none slower; the lowest price
// throughout 1.0 %, with 18 layers slower, by up to 16 %.
hipError_t launch_conv_pair(const GemmArgs &a, const ConvShape &s, int kindB, const GemmArgs &b, hipStream_t st)
{
    if (!conv_dx_ok(a.K, s, a.c_is_f32) || a.c_is_f32 != b.c_is_f32) return hipErrorInvalidValue;
    const ConvDxPlan p = conv_dx_plan(a, s);
    const bool can_split = b.ws != nullptr && (reinterpret_cast<uintptr_t>(b.ws) & 15) == 0;
    const size_t ws_bytes = can_split ? b.ws_bytes : 0;
    const int nkB = (row_bytes(kindB, b.K) + 127) / 128;
    const double mnB = static_cast<double>(b.M) * b.N;
    const int tilesB = ((b.M + 127) / 128) * ((b.N + 127) / 128);
    int S = 1;
    bool b_first = false;
    if (p.blocks + tilesB <= 512) {
        S = (512 - p.blocks) / tilesB;
        if (S > nkB / 8) S = nkB / 8;
        if (S > 16) S = 16;
        if (S > ws_bytes / (mnB * 4.0)) S = static_cast<int>(ws_bytes / (mnB * 4.0));
        if (S < 1) S = 1;
    } else {
        const double tA = 4.0 + conv_dx_tile_us(p.g.form, s, a.K);
        double best = 1e30;
        for (int c : kSplitChoices) {
            if (c > 1 && (c > nkB || c * mnB * 4.0 > static_cast<double>(ws_bytes))) break;
            const double nB = static_cast<double>(tilesB) * c, tB = __builtin_ceil(static_cast<double>(nkB) / c) * kStepSmallShared + kFixedSmall;
            const double tab = pair_makespan(p.blocks, tA, 512, nB, tB, 512), tba = pair_makespan(nB, tB, 512, p.blocks, tA, 512);
            const double t = (tba < tab ? tba : tab) + (c > 1 ? 2.0 * c * mnB * 4.0 / 8.0e6 + 3.0 : 0.0);
            if (t < best) {
                best = t;
                S = c;
                b_first = tba < tab;
            }
        }
    }
    const auto price = [&](int c, bool first) {         // with the partials out and back and a launch more
        return conv_pair_time(p, static_cast<double>(tilesB) * c, __builtin_ceil(static_cast<double>(nkB) / c), first) +
               (c > 1 ? 2.35 + c * mnB * 4.0e-6 * 0.58 : 0.0);
    };
    double least = price(S, b_first) / 1.2;
    for (int c : kSplitChoices) {
        if (c > 1 && (c > nkB || c * mnB * 4.0 > static_cast<double>(ws_bytes))) break;
        for (const bool first : {false, true}) {
            if (const double t = price(c, first); t < least) {
                least = t;
                S = c;
                b_first = first;
            }
        }
    }
    if (const int f = gemm_plan_forced_splits(nkB, mnB, ws_bytes, can_split)) S = f;
    const GemmDev gb = gemm_dev(kindB, b, 128, 128, S);
    const hipError_t e = (kindB == 1 ? launch_conv_pair_1 : launch_conv_pair_0)(p, a.c_is_f32, gb, S > 1, b_first, st);
    if (e != hipSuccess || S == 1) return e;
    return launch_splitk_reduce(kindB == 1 ? 1 : 0, b, S, st);
}

}  // namespace hlq
