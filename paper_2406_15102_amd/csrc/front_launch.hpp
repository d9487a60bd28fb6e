// What k_front.hip calls of the units that hold its kernels (front_impl.hpp).
#pragma once
#include "hlq_device.hpp"
#include "hlq_kernels.hpp"

namespace hlq {

FrontMix front_mix_of(int n1, int n3);
FrontMix front_mix(const FrontRows &jr, const FrontHla &jx, int more);

// launch_front, launch_front_one and launch_front_q for one element type and block size
template <typename Tin, int B> struct FrontLaunch {
    static hipError_t first(const FrontRows &jr, const FrontHla &jx, const FrontFill &jf, const FrontHla &jg, const FrontAbsmax &jw,
                            const FrontRecode &jk, const FrontConv &jc, int basis, int codes, hipStream_t st);
    static hipError_t one(const FrontRows &jr, const FrontHla &jx, const FrontHla &jg, const FrontColsQ &jq, const FrontConv &jc, int basis,
                          int codes, hipStream_t st);
    static hipError_t integer(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq, const FrontRows &jr,
                              const FrontUnpack &ju, const FrontRecode &jk, const FrontConv &jc, int basis, int codes, hipStream_t st);
};

}  // namespace hlq
