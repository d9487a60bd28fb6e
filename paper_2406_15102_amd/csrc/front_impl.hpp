// The kernels of k_front.hip and what launches them, for one element type and block size: each k_front_<B>_<type>.hip
// instantiates FrontLaunch below (its kernels compile for minutes).
#pragma once
#include "front_launch.hpp"
#include "hla_body.hpp"
#include "quant_cols_body.hpp"
#include "quant_rows_body.hpp"

namespace hlq {

// workgroup `blk` of K1
template <typename Tin, int B, int CODES>
__device__ __forceinline__ void front_rows_body(const FrontRows &jr, int blk)
{
    const Tin *G = static_cast<const Tin *>(jr.G);
    if constexpr (CODES == kCodesF6)
        quant_rows_f6_body<Tin, B, 256>(G, jr.N, jr.O, jr.T, jr.k0, jr.k1, jr.qmax, reinterpret_cast<uint8_t *>(jr.Gq), jr.sG, blk);
    else
        quant_rows_body<Tin, B, 256, CODES == kCodesNibbles>(G, jr.N, jr.O, jr.T, jr.k0, jr.k1, jr.qmax, jr.Gq, jr.sG, nullptr, blk);
}

// Workgroup b of the n1 + n3 that two kinds of job share, handed out in turns (FrontMix): k1 >= 0, the index
// among the first kind, or k3 >= 0, among the second; both < 0 past the end, with b counted from there.
__device__ __forceinline__ void front_turns(const FrontMix &jm, int &b, int n1, int n3, int &k1, int &k3)
{
    const int per = jm.gran * (jm.q + 1);
    k1 = k3 = -1;
    if (b < jm.cyc * per) {
        const int turn = b / per, pos = b % per;
        if (pos < jm.gran * jm.q) k1 = turn * jm.gran * jm.q + pos;
        else k3 = turn * jm.gran + pos - jm.gran * jm.q;
        return;
    }
    b -= jm.cyc * per;
    const int k1_left = n1 - jm.cyc * jm.gran * jm.q, k3_left = n3 - jm.cyc * jm.gran;
    if (b < k1_left) k1 = jm.cyc * jm.gran * jm.q + b;
    else if (b - k1_left < k3_left) k3 = jm.cyc * jm.gran + b - k1_left;
    else b -= k1_left + k3_left;
}

// what comes behind the jobs of the first launch: the zeroing, then the weight codes that were handed over, brought into
// the f6 layout
template <int CODES>
__device__ __forceinline__ void front_fill_or_recode(const FrontFill &jf, const FrontRecode &jk, int b)
{
    const int fill = (jf.n + 255) >> 8;
    if (b < fill) {
        const int i = b * 256 + threadIdx.x;
        if (i < jf.n) jf.p[i] = 0u;
    } else if constexpr (CODES == kCodesF6) {
        f6_recode_body(jk, b - fill);
    }
}

// The widening of a 4-bit store: a thread per 32 bytes out, those behind the end of a row zeros.
__device__ __forceinline__ void front_unpack_body(const FrontUnpack &ju, int b)
{
    const int64_t i = static_cast<int64_t>(b) * 256 + threadIdx.x;
    if (i >= ju.n) return;
    uint4 *out = static_cast<uint4 *>(ju.out);
    const uint32_t row = static_cast<uint32_t>(i) / static_cast<uint32_t>(ju.row_out), p = static_cast<uint32_t>(i) - row * static_cast<uint32_t>(ju.row_out);
    if (p < static_cast<uint32_t>(ju.row_in)) {
        unpack_nibbles16(static_cast<const uint4 *>(ju.in) + static_cast<int64_t>(row) * ju.row_in + p, out + 2 * i);
    } else {
        out[2 * i] = make_uint4(0, 0, 0, 0);
        out[2 * i + 1] = make_uint4(0, 0, 0, 0);
    }
}

// CONV: X is a channels-last image and K3 reads its column matrix through ConvRows.  A kernel of
// its own: the extra address arithmetic would cost the matrix variant registers, and with them a
// wavefront of occupancy at B = 32.
template <typename Tin, int B, int CODES, int BASIS, bool CONV>
__global__ __launch_bounds__(256) void k_front_a(FrontRows jr, FrontHla jx, FrontFill jf, FrontConv jc, FrontShare js,
                                                 FrontMix jm, FrontHla jy, FrontRecode jk)
{
    int b = blockIdx.x;
    if (!CONV && js.on) {
        // K1 and K3 read the same tensor: both readers of a group of 128 rows on one XCD, one after the other
        if (b < js.blocks) {
            const int per = js.nk1 + js.gx;
            const int xcd = b & 7, q = b >> 3;
            const int unit = (q / (js.pair * per)) * 8 + xcd;
            const int u = q % (js.pair * per);
            const int grp = unit * js.pair + u / per, v = u % per;
            if (unit >= js.units) return;
            if (v < js.nk1) {
                const int blk = grp * js.nk1 + v;
                if (blk < jr.blocks)
                    front_rows_body<Tin, B, CODES>(jr, blk);
            } else {
                hla_body<Tin, B, BASIS, 2, true>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, v - js.nk1, grp);
            }
            return;
        }
        front_fill_or_recode<CODES>(jf, jk, b - js.blocks);
        return;
    }
    if (!CONV && jm.gran) {
        int k1, k3;
        front_turns(jm, b, jr.blocks, jx.nb + jy.nb, k1, k3);
        if (k1 >= 0) {
            front_rows_body<Tin, B, CODES>(jr, k1);
        } else if (k3 >= 0 && k3 < jx.nb) {
            int bx, by;
            hla_job_map(k3, jx.gx, jx.grp, bx, by);
            hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, bx, by);
        } else if (k3 >= 0) {
            int bx, by;
            hla_job_map(k3 - jx.nb, jy.gx, jy.grp, bx, by);
            hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jy.T), jy.N, jy.D, jy.r, jy.Kp, jy.out, nullptr, bx, by);
        } else {
            front_fill_or_recode<CODES>(jf, jk, b);
        }
        return;
    }
    if (b < jr.blocks) {
        front_rows_body<Tin, B, CODES>(jr, b);
        return;
    }
    b -= jr.blocks;
    if (b < jx.nb) {
        int bx, by;
        hla_job_map(b, jx.gx, jx.grp, bx, by);
        if (CONV)
            hla_body_src<B, BASIS, ConvRows<Tin>, 1, true>(ConvRows<Tin>{static_cast<const Tin *>(jx.T), jc.g}, jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, bx, by);
        else
            hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, bx, by);
        return;
    }
    b -= jx.nb;
    if (b < jy.nb) {
        int bx, by;
        hla_job_map(b, jy.gx, jy.grp, bx, by);
        hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jy.T), jy.N, jy.D, jy.r, jy.Kp, jy.out, nullptr, bx, by);
        return;
    }
    front_fill_or_recode<CODES>(jf, jk, b - jy.nb);
}

// The whole front in one launch, for weights of few rows: a workgroup per strip of columns runs both
// passes of K1T (cols_full_body), so neither a zeroing launch before it nor a launch for pass 2 is needed.
// (three wavefronts per SIMD asked for below B = 64, which the other jobs had before the strip quantiser
// joined them: left alone, the register allocator spends all 256 registers on it)
template <typename Tin, int B, int CODES, int BASIS, bool CONV>
__global__ __launch_bounds__(256, B == 64 ? 2 : 3) void k_front_one(FrontRows jr, FrontHla jx, FrontHla jg, FrontColsQ jq, FrontConv jc,
                                                                    FrontMix jm)
{
    int b = blockIdx.x;
    if (b < jq.gx) {       // first: these workgroups pass over their strip twice
        cols_full_body<Tin, B, CODES>(static_cast<const Tin *>(jq.W), jq.O, jq.I, jq.k0, jq.k1, jq.qmax, jq.WqT, jq.sW, b, jq.gy);
        return;
    }
    b -= jq.gx;
    if (jm.gran) {
        // the row quantiser's workgroups and the projections' in turns: b becomes an index in the ranges below
        int k1, k3;
        front_turns(jm, b, jr.blocks, jx.nb + jg.nb, k1, k3);
        if (k1 < 0 && k3 < 0) return;
        b = k1 >= 0 ? k1 : jr.blocks + k3;
    }
    if (b < jr.blocks) {
        front_rows_body<Tin, B, CODES>(jr, b);
        return;
    }
    b -= jr.blocks;
    if (b < jx.nb) {
        int bx, by;
        hla_job_map(b, jx.gx, jx.grp, bx, by);
        if (CONV)
            hla_body_src<B, BASIS, ConvRows<Tin>, 1, true>(ConvRows<Tin>{static_cast<const Tin *>(jx.T), jc.g}, jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, bx, by);
        else
            hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.Kp, jx.out, nullptr, bx, by);
        return;
    }
    b -= jx.nb;
    int bx, by;
    hla_job_map(b, jg.gx, jg.grp, bx, by);
    hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jg.T), jg.N, jg.D, jg.r, jg.Kp, jg.out, nullptr, bx, by);
}

template <typename Tin, int B, int BASIS>
__global__ __launch_bounds__(256) void k_front_b(FrontHla jg, FrontAbsmax jw)
{
    int b = blockIdx.x;
    if (b < jg.nb) {
        int bx, by;
        hla_job_map(b, jg.gx, jg.grp, bx, by);
        hla_body<Tin, B, BASIS, 1, true>(static_cast<const Tin *>(jg.T), jg.N, jg.D, jg.r, jg.Kp, jg.out, nullptr, bx, by);
        return;
    }
    b -= jg.nb;
    cols_absmax_body<Tin, B>(static_cast<const Tin *>(jw.W), jw.O, jw.I, jw.amax, b % jw.gx, b / jw.gx);
}

// integer g_w list, pass 1 of everything: maxima of the kept coefficients of G and of X, of H^T W
// With jr (the row quantiser of G, which waits for nothing) riding along, in turns: its arithmetic beside three
// passes that only read.
template <typename Tin, int B, int BASIS, int CODES, bool CONV>
__global__ __launch_bounds__(256) void k_front_q1(FrontHlaQ jg, FrontHlaQ jx, FrontAbsmax jw, FrontRows jr, FrontMix jm,
                                                  FrontUnpack ju, FrontConv jc, FrontRecode jk)
{
    int b = blockIdx.x;
    if (jr.blocks > 0) {
        int k1 = -1, k3 = -1;
        if (jm.gran) {
            // (the widening of a 4-bit store stays behind the turns: counted among the readers it would thin out the
            // quantiser's share of them.  Whole pass from the store with it counted / as a launch of its own / behind, us:
            // fp32 57728 x 1192 x 2688 711.7 / 688.9 / 685.7, 4096 x 768 x 3072 48.9 / 50.9 / 47.9, 512 x 8320 x 1920
            // 48.6 / 51.7 / 48.5)
            const int n3 = jg.gx * jg.gy + jx.gx * jx.gy + jw.gx * jw.gy;
            front_turns(jm, b, jr.blocks, n3, k1, k3);
            if (k1 < 0) b = k3 >= 0 ? k3 : n3 + b;
        } else if (b < jr.blocks) {
            k1 = b;
        } else {
            b -= jr.blocks;
        }
        if (k1 >= 0) {
            front_rows_body<Tin, B, CODES>(jr, k1);
            return;
        }
    }
    if (b < jg.gx * jg.gy) {
        hla_absmax_body<Tin, B, BASIS>(static_cast<const Tin *>(jg.T), jg.N, jg.D, jg.r, jg.amax, b % jg.gx, b / jg.gx, jg.table != 0);
        return;
    }
    b -= jg.gx * jg.gy;
    if (b < jx.gx * jx.gy) {
        if (CONV)
            hla_absmax_body_src<B, BASIS>(ConvRows<Tin>{static_cast<const Tin *>(jx.T), jc.g}, jx.N, jx.D, jx.r, jx.amax, b % jx.gx,
                                          b / jx.gx, jx.table != 0);
        else
            hla_absmax_body<Tin, B, BASIS>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.amax, b % jx.gx, b / jx.gx, jx.table != 0);
        return;
    }
    b -= jx.gx * jx.gy;
    if (b < jw.gx * jw.gy) {
        cols_absmax_body<Tin, B>(static_cast<const Tin *>(jw.W), jw.O, jw.I, jw.amax, b % jw.gx, b / jw.gx, jw.table != 0);
        return;
    }
    b -= jw.gx * jw.gy;
    if constexpr (CODES == kCodesF6) {
        if (b >= ju.blocks) {
            f6_recode_body(jk, b - ju.blocks);
            return;
        }
    }
    front_unpack_body(ju, b);
}

// pass 2 of everything: int8 codes of projected G and X, codes of the weight
template <typename Tin, int B, int BASIS, int CODES, bool CONV>
__global__ __launch_bounds__(256) void k_front_q2(FrontHlaQ jg, FrontHlaQ jx, FrontColsQ jq, FrontConv jc)
{
    // backwards through the jobs and through each of them (reverse_same_xcd): what the passes that took the maxima
    // read last is what the last-level cache still holds
    const int64_t bytes = (jg.T ? jg.N * jg.D : 0) + (jx.T ? jx.N * jx.D : 0) + (jq.W ? static_cast<int64_t>(jq.O) * jq.I : 0);
    int b = reverse_same_xcd(blockIdx.x, gridDim.x, bytes * static_cast<int64_t>(sizeof(Tin)));
    if (b < jg.gx * jg.gy) {
        hla_quantize_body<Tin, B, BASIS, false, false, true>(static_cast<const Tin *>(jg.T), jg.N, jg.D, jg.r, jg.amax, jg.k0, jg.k1, jg.Kp, jg.TqT,
                                         jg.sT, nullptr, b % jg.gx, b / jg.gx, jg.table);
        return;
    }
    b -= jg.gx * jg.gy;
    if (b < jx.gx * jx.gy) {
        if (CONV)
            hla_quantize_body_src<B, BASIS, false, ConvRows<Tin>, false, true>(ConvRows<Tin>{static_cast<const Tin *>(jx.T), jc.g}, jx.N, jx.D, jx.r, jx.amax,
                                                   jx.k0, jx.k1, jx.Kp, jx.TqT, jx.sT, nullptr, b % jx.gx, b / jx.gx, jx.table);
        else
            hla_quantize_body<Tin, B, BASIS, false, false, true>(static_cast<const Tin *>(jx.T), jx.N, jx.D, jx.r, jx.amax, jx.k0, jx.k1, jx.Kp, jx.TqT,
                                             jx.sT, nullptr, b % jx.gx, b / jx.gx, jx.table);
        return;
    }
    b -= jx.gx * jx.gy;
    if constexpr (CODES == kCodesF6)
        cols_quantize_f6_body<Tin, B>(static_cast<const Tin *>(jq.W), jq.O, jq.I, jq.amax, jq.k0, jq.k1, jq.qmax,
                                      reinterpret_cast<uint8_t *>(jq.WqT), jq.sW, b % jq.gx, b / jq.gx, jq.table);
    else
        cols_quantize_body<Tin, B, CODES == kCodesNibbles>(static_cast<const Tin *>(jq.W), jq.O, jq.I, jq.amax, jq.k0, jq.k1, jq.qmax,
                                                           jq.WqT, jq.sW, nullptr, b % jq.gx, b / jq.gx, jq.table);
}

template <typename Tin, int B, int BASIS, int CODES, bool CONV>
static hipError_t launch_front_q_t(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq,
                                   const FrontRows &jr, const FrontUnpack &ju, const FrontRecode &jk, const FrontConv &jc, hipStream_t st)
{
    const int n3 = jg.gx * jg.gy + jx.gx * jx.gy + jw.gx * jw.gy;
    const int n1 = n3 + jr.blocks + ju.blocks + jk.blocks;
    const FrontMix jm = jr.blocks > 0 ? front_mix_of(jr.blocks, n3) : FrontMix{0, 0, 0};
    if (n1 > 0) hipLaunchKernelGGL((k_front_q1<Tin, B, BASIS, CODES, CONV>), dim3(n1), dim3(256), 0, st, jg, jx, jw, jr, jm, ju, jc, jk);
    const int n2 = jg.gx * jg.gy + jx.gx * jx.gy + jq.gx * jq.gy;
    if (n2 > 0) hipLaunchKernelGGL((k_front_q2<Tin, B, BASIS, CODES, CONV>), dim3(n2), dim3(256), 0, st, jg, jx, jq, jc);
    return hipGetLastError();
}

template <typename Tin, int B, int BASIS>
static hipError_t launch_front_q_p(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq,
                                   const FrontRows &jr, const FrontUnpack &ju, const FrontRecode &jk, const FrontConv &jc, int codes, hipStream_t st)
{
#define HLQ_FRONT_Q(CV)                                                                                                    \
    return codes == kCodesF6 ? launch_front_q_t<Tin, B, BASIS, kCodesF6, CV>(jg, jx, jw, jq, jr, ju, jk, jc, st)               \
                             : (codes == kCodesNibbles ? launch_front_q_t<Tin, B, BASIS, kCodesNibbles, CV>(jg, jx, jw, jq, jr, ju, jk, jc, st) \
                                                       : launch_front_q_t<Tin, B, BASIS, kCodesBytes, CV>(jg, jx, jw, jq, jr, ju, jk, jc, st))
    if (jc.on) HLQ_FRONT_Q(true);
    HLQ_FRONT_Q(false);
#undef HLQ_FRONT_Q
}

// launch LAUNCH(codes, CONV) for the codes asked for
#define HLQ_FRONT_CODES(LAUNCH, CONV)                         \
    if (codes == kCodesF6) LAUNCH(kCodesF6, CONV);            \
    else if (codes == kCodesNibbles) LAUNCH(kCodesNibbles, CONV); \
    else LAUNCH(kCodesBytes, CONV);

template <typename Tin, int B, int BASIS>
static hipError_t launch_front_t(const FrontRows &jr, const FrontHla &jx, const FrontFill &jf, const FrontHla &jg,
                                 const FrontAbsmax &jw, const FrontRecode &jk, const FrontConv &jc, int codes, hipStream_t st)
{
    const FrontShare js = jc.on ? FrontShare{} : front_share(jr, jx, B, sizeof(Tin) == 4);
    // Unless that is switched off, the first launch takes both projections (the second is left with the pass
    // over W, if there is one) and hands out its workgroups in turns: the row quantiser's arithmetic then has
    // all the memory-bound work there is to run beside.
    const FrontHla none = front_hla(nullptr, 0, 0, B, 1, 0, nullptr);
    const bool both = front_mix_enabled() && !jc.on && !js.on && jg.T;
    const FrontMix jm = (jc.on || js.on) ? FrontMix{0, 0, 0} : front_mix(jr, jx, both ? jg.nb : 0);
    const FrontHla &jy = both ? jg : none;        // second projection of the first launch
    const FrontHla &jb = both ? none : jg;        // projection of the second launch
    const int na = (js.on ? js.blocks : jr.blocks + jx.nb + jy.nb) + (jf.n + 255) / 256 + jk.blocks;
    if (na > 0) {
#define HLQ_FRONT_A(P, CV) hipLaunchKernelGGL((k_front_a<Tin, B, P, BASIS, CV>), dim3(na), dim3(256), 0, st, jr, jx, jf, jc, js, jm, jy, jk)
        if (jc.on) {
            HLQ_FRONT_CODES(HLQ_FRONT_A, true)
        } else {
            HLQ_FRONT_CODES(HLQ_FRONT_A, false)
        }
#undef HLQ_FRONT_A
    }
    const int nb = jb.nb + jw.gx * jw.gy;
    if (nb > 0) hipLaunchKernelGGL((k_front_b<Tin, B, BASIS>), dim3(nb), dim3(256), 0, st, jb, jw);
    return hipGetLastError();
}

template <typename Tin, int B, int BASIS>
static hipError_t launch_front_one_t(const FrontRows &jr, const FrontHla &jx, const FrontHla &jg, const FrontColsQ &jq,
                                     const FrontConv &jc, int codes, hipStream_t st)
{
    const int n = jq.gx + jr.blocks + jx.nb + jg.nb;
    if (n == 0) return hipSuccess;
    // (layers whose quantiser has fewer than a thousand workgroups lose a little by it: 29.3 -> 30.0 us at 12544 x 896 x 224)
    const FrontMix jm = (jr.G && jr.blocks >= 1024) ? front_mix_of(jr.blocks, jx.nb + jg.nb) : FrontMix{0, 0, 0};
#define HLQ_FRONT_ONE(P, CV) hipLaunchKernelGGL((k_front_one<Tin, B, P, BASIS, CV>), dim3(n), dim3(256), 0, st, jr, jx, jg, jq, jc, jm)
    if (jc.on) {
        HLQ_FRONT_CODES(HLQ_FRONT_ONE, true)
    } else {
        HLQ_FRONT_CODES(HLQ_FRONT_ONE, false)
    }
#undef HLQ_FRONT_ONE
    return hipGetLastError();
}

template <typename Tin, int B>
hipError_t FrontLaunch<Tin, B>::first(const FrontRows &jr, const FrontHla &jx, const FrontFill &jf, const FrontHla &jg, const FrontAbsmax &jw,
                                      const FrontRecode &jk, const FrontConv &jc, int basis, int codes, hipStream_t st)
{
    return basis ? launch_front_t<Tin, B, 1>(jr, jx, jf, jg, jw, jk, jc, codes, st) : launch_front_t<Tin, B, 0>(jr, jx, jf, jg, jw, jk, jc, codes, st);
}

template <typename Tin, int B>
hipError_t FrontLaunch<Tin, B>::one(const FrontRows &jr, const FrontHla &jx, const FrontHla &jg, const FrontColsQ &jq, const FrontConv &jc,
                                    int basis, int codes, hipStream_t st)
{
    return basis ? launch_front_one_t<Tin, B, 1>(jr, jx, jg, jq, jc, codes, st) : launch_front_one_t<Tin, B, 0>(jr, jx, jg, jq, jc, codes, st);
}

template <typename Tin, int B>
hipError_t FrontLaunch<Tin, B>::integer(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq, const FrontRows &jr,
                                        const FrontUnpack &ju, const FrontRecode &jk, const FrontConv &jc, int basis, int codes, hipStream_t st)
{
    return basis ? launch_front_q_p<Tin, B, 1>(jg, jx, jw, jq, jr, ju, jk, jc, codes, st)
                 : launch_front_q_p<Tin, B, 0>(jg, jx, jw, jq, jr, ju, jk, jc, codes, st);
}

}  // namespace hlq
