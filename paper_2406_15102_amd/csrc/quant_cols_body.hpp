// Device pieces of K1T (see k_quant_cols.hip) that other kernels reuse: the row-block loader and
// pass 1, the column maxima of the transformed weight.
#pragma once
#include "hlq_device.hpp"
#include "hlq_kernels.hpp"

namespace hlq {

template <typename Tin, int B, int CPL>
__device__ __forceinline__ void load_row_block(const Tin *base, int64_t pitch, float *v)
{
#pragma unroll
    for (int j = 0; j < B; ++j) Loader<Tin, CPL>::load(base + j * pitch, v + j * CPL);
}

// pass 1: a row block per group of B lanes (256 / B groups); the groups' maxima meet in LDS and are merged
// into one maximum per column with an atomic on the bit patterns (non-negative floats order like
// their bit patterns), so the maxima must have been zeroed by an earlier launch -- or, with `table`,
// each row of workgroups leaves its own and pass 2 folds them (kAmaxTableRows).
template <typename Tin, int B>
__device__ __forceinline__ void cols_absmax_body(const Tin *__restrict__ W, int O, int I, uint32_t *__restrict__ amax_bits,
                                                 int bx, int by, bool table = false)
{
    constexpr int CPL = 128 / B, L = B, NB = 256 / B;     // lanes side by side, row blocks
    __shared__ float s_max[NB][L * CPL];
    const int tid = threadIdx.x, grp = tid / L, sub = tid % L;
    const int col0 = (bx * L + sub) * CPL;
    const int o0 = (by * NB + grp) * B;
    float cmax[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) cmax[c] = 0.0f;

    if (col0 < I && o0 < O) {
        float v[B * CPL];
        load_row_block<Tin, B, CPL>(W + static_cast<int64_t>(o0) * I + col0, I, v);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            fwht_regs<B, CPL>(v + c);
#pragma unroll
            for (int j = 0; j < B; ++j) cmax[c] = fmaxf(cmax[c], fabsf(v[j * CPL + c]));
        }
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) s_max[grp][sub * CPL + c] = cmax[c];
    __syncthreads();
    for (int idx = tid; idx < L * CPL; idx += 256) {
        float m = s_max[0][idx];
#pragma unroll
        for (int g = 1; g < NB; ++g) m = fmaxf(m, s_max[g][idx]);
        const int col = bx * L * CPL + idx;
        if (table) {   // a row of the table per `by`
            if (col < I) amax_bits[static_cast<int64_t>(by) * I + col] = __float_as_uint(m);
        } else if (col < I && m > 0.0f) {
            atomicMax(amax_bits + col, __float_as_uint(m));
        }
    }
}

// One row block (B rows from o0) of CPL columns (a lane's share) from col0: transform again, quantise against the
// reciprocal scales `inv` of those columns, write the codes transposed.
// PACKED: the codes are written two to a byte (4-bit codes only), O/2 bytes per row of WqT.
template <typename Tin, int B, bool PACKED, bool MANT, int CPL = 128 / B>
__device__ __forceinline__ void cols_quantize_block(const Tin *__restrict__ W, int O, int I, const float *inv, uint32_t k0,
                                                    uint32_t k1, int8_t *__restrict__ WqT, float *__restrict__ coeffT,
                                                    int col0, int o0)
{
    float v[B * CPL];
    load_row_block<Tin, B, CPL>(W + static_cast<int64_t>(o0) * I + col0, I, v);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        fwht_regs<B, CPL>(v + c);
        const int64_t orow = static_cast<int64_t>(col0 + c) * O + o0;
        const uint32_t cnt = static_cast<uint32_t>(col0 + c) * static_cast<uint32_t>(O >> 2) +
                             static_cast<uint32_t>(o0 >> 2);
#pragma unroll
        for (int d4 = 0; d4 < B / 16; ++d4) {
            int q[16];
            quant_codes<MANT, 4>(v + d4 * 16 * CPL + c, CPL, inv[c], cnt + d4 * 4, k0, k1, q);
            if (PACKED)
                *reinterpret_cast<uint2 *>(WqT + orow / 2 + d4 * 8) = make_uint2(pack_nibbles8(q), pack_nibbles8(q + 8));
            else
                *reinterpret_cast<uint4 *>(WqT + orow + d4 * 16) =
                    make_uint4(pack_bytes4(q), pack_bytes4(q + 4), pack_bytes4(q + 8), pack_bytes4(q + 12));
        }
        if (coeffT) {
#pragma unroll
            for (int j = 0; j < B; j += 4)
                *reinterpret_cast<float4 *>(coeffT + orow + j) =
                    make_float4(v[j * CPL + c], v[(j + 1) * CPL + c], v[(j + 2) * CPL + c], v[(j + 3) * CPL + c]);
        }
    }
}

// pass 2: a row block per group of B lanes against the column maxima that pass 1 merged.
template <typename Tin, int B, bool PACKED, bool MANT = false>
__device__ __forceinline__ void cols_quantize_body(const Tin *__restrict__ W, int O, int I,
                                                   const uint32_t *__restrict__ amax_bits, uint32_t k0, uint32_t k1,
                                                   float qmax, int8_t *__restrict__ WqT, float *__restrict__ sW,
                                                   float *__restrict__ coeffT, int bx, int by, int table = 0)
{
    constexpr int CPL = 128 / B;
    constexpr int L = B, NB = 256 / B;
    const int tid = threadIdx.x;
    const int col0 = (bx * L + tid % L) * CPL;
    const int o0 = (by * NB + tid / L) * B;
    float inv[CPL], a[CPL];
    fold_column_maxima<CPL>(amax_bits, I, table, bx, tid % L, a);
    if (col0 >= I || o0 >= O) return;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        inv[c] = absmax_to_inv(a[c], qmax);
        if (o0 == 0) sW[col0 + c] = absmax_to_scale(a[c], qmax);
    }
    cols_quantize_block<Tin, B, PACKED, MANT>(W, O, I, inv, k0, k1, WqT, coeffT, col0, o0);
}

// ---- the same with the codes in the f6 layout (hlq_device.hpp): rows of f6_row_bytes(O), zeros behind their end ----
// A lane's rows are whole groups of 32 (two Hadamard blocks at B = 16), so that a column's codes are packed within it;
// the columns a lane owns make up for it, and the reads stay runs of 256 bytes.
template <int B> struct ColsF6 {
    static constexpr int RB = B < 32 ? 32 : B, CPL = 128 / RB;
};

// RB rows from o0 of CPL columns from col0; at B = 16 the second block may lie beyond O, and its codes are 0
template <typename Tin, int B, bool MANT, int CPL = ColsF6<B>::CPL>
__device__ __forceinline__ void cols_quantize_block_f6(const Tin *__restrict__ W, int O, int I, const float *inv, uint32_t k0,
                                                       uint32_t k1, uint8_t *__restrict__ WqT, int col0, int o0)
{
    constexpr int RB = ColsF6<B>::RB;
    float v[RB * CPL];
    const Tin *w = W + static_cast<int64_t>(o0) * I + col0;
    load_row_block<Tin, B, CPL>(w, I, v);
    if (B < RB) {
        if (o0 + B < O) {
            load_row_block<Tin, B, CPL>(w + static_cast<int64_t>(B) * I, I, v + (RB - B) * CPL);
        } else {
#pragma unroll
            for (int e = B * CPL; e < RB * CPL; ++e) v[e] = 0.0f;
        }
    }
    const int64_t pitch = f6_row_bytes(O);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        fwht_regs<B, CPL>(v + c);
        if (B < RB) fwht_regs<B, CPL>(v + (RB - B) * CPL + c);
        const uint32_t cnt = static_cast<uint32_t>(col0 + c) * static_cast<uint32_t>(O >> 2) + static_cast<uint32_t>(o0 >> 2);
#pragma unroll
        for (int h = 0; h < RB; h += 32) {
            float f[32];
            quant_floats<MANT, 4>(v + h * CPL + c, CPL, inv[c], cnt + h / 4, k0, k1, f);
            quant_floats<MANT, 4>(v + (h + 16) * CPL + c, CPL, inv[c], cnt + h / 4 + 4, k0, k1, f + 16);
            *reinterpret_cast<uint4 *>(WqT + (col0 + c) * pitch + ((o0 + h) >> 1)) = f6_pack32(f);
        }
    }
}

// the rows past O that make a row of codes whole
template <int B, int CPL>
__device__ __forceinline__ void cols_clear_f6(uint8_t *__restrict__ WqT, int O, int col0, int o0)
{
#pragma unroll
    for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int h = 0; h < ColsF6<B>::RB; h += 32)
            *reinterpret_cast<uint4 *>(WqT + static_cast<int64_t>(col0 + c) * f6_row_bytes(O) + ((o0 + h) >> 1)) = make_uint4(0, 0, 0, 0);
}

// pass 2 of a workgroup: 128 columns, 256 rows -- 128 bytes of every output row, the padding among them
template <typename Tin, int B, bool MANT = false>
__device__ __forceinline__ void cols_quantize_f6_body(const Tin *__restrict__ W, int O, int I,
                                                      const uint32_t *__restrict__ amax_bits, uint32_t k0, uint32_t k1,
                                                      float qmax, uint8_t *__restrict__ WqT, float *__restrict__ sW, int bx,
                                                      int by, int table = 0)
{
    constexpr int RB = ColsF6<B>::RB, CPL = ColsF6<B>::CPL, L = RB, NB = 256 / RB;
    const int tid = threadIdx.x;
    const int col0 = (bx * L + tid % L) * CPL;
    const int o0 = (by * NB + tid / L) * RB;
    float inv[CPL], a[CPL];
    fold_column_maxima<CPL>(amax_bits, I, table, bx, tid % L, a);
    if (col0 >= I) return;
    if (o0 >= O) {
        cols_clear_f6<B, CPL>(WqT, O, col0, o0);
        return;
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        inv[c] = absmax_to_inv(a[c], qmax);
        if (o0 == 0) sW[col0 + c] = absmax_to_scale(a[c], qmax);
    }
    cols_quantize_block_f6<Tin, B, MANT>(W, O, I, inv, k0, k1, WqT, col0, o0);
}

// Weight codes that were kept, as hlq_quantize_w stores them, into the f6 layout: a thread per 32 codes.
__device__ __forceinline__ void f6_recode_body(const FrontRecode &jk, int blk)
{
    const int groups = f6_row_bytes(jk.O) / 16;
    const int64_t i = static_cast<int64_t>(blk) * 256 + threadIdx.x;
    if (i >= static_cast<int64_t>(jk.rows) * groups) return;
    const int row = static_cast<int>(i / groups), gi = static_cast<int>(i - static_cast<int64_t>(row) * groups);
    uint4 o = make_uint4(0, 0, 0, 0);
    if (gi * 32 < jk.O) {
        float f[32];
        if (jk.nibbles) {      // O % 32 == 0
            const uint4 x = *reinterpret_cast<const uint4 *>(static_cast<const uint8_t *>(jk.in) + static_cast<int64_t>(row) * (jk.O / 2) + gi * 16);
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 32; ++e) f[e] = static_cast<float>(static_cast<int>(w[e / 8] << (28 - 4 * (e % 8))) >> 28);
        } else {
            const uint8_t *p = static_cast<const uint8_t *>(jk.in) + static_cast<int64_t>(row) * jk.O + gi * 32;
            const uint4 x = *reinterpret_cast<const uint4 *>(p);
            const uint4 y = gi * 32 + 16 < jk.O ? *reinterpret_cast<const uint4 *>(p + 16) : make_uint4(0, 0, 0, 0);
            const uint32_t w[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int e = 0; e < 32; ++e) f[e] = static_cast<float>(static_cast<int>(w[e / 4] << (24 - 8 * (e % 4))) >> 24);
        }
        o = f6_pack32(f);
    }
    *reinterpret_cast<uint4 *>(jk.out + i * 16) = o;
}

// Both passes by one workgroup, for a small weight: the workgroup owns a strip of LG * CW columns
// over all of O (LG = 1 << lg lanes side by side: 16, 8 or 4; CW columns a lane, fewer than the
// 128/B of the two-pass kernels so that a lane's chain of loads, transform and quantisation is
// short: this job's latency is what the launch around it can end on), its 256 / LG groups of lanes
// take a row block each per round, the maxima meet in LDS, and the second pass finds the rows in
// the cache.  No other workgroup is waited for, so this can ride in a launch with anything.
template <int B> struct ColsFull {
    static constexpr int CW = B == 16 ? 4 : 2;      // columns a lane: 64 (B = 16, 32) or 128 values
};

// CODES: kCodesBytes, kCodesNibbles, kCodesF6
template <typename Tin, int B, int CODES>
__device__ __forceinline__ void cols_full_body(const Tin *__restrict__ W, int O, int I, uint32_t k0, uint32_t k1, float qmax,
                                               int8_t *__restrict__ WqT, float *__restrict__ sW, int bx, int lg)
{
    constexpr bool F6 = CODES == kCodesF6;
    constexpr int CW = ColsFull<B>::CW;
    __shared__ float s_strip[256 * CW];       // [group][lane of the group][column of the lane]
    const int tid = threadIdx.x, grp = tid >> lg, sub = tid & ((1 << lg) - 1), groups = 256 >> lg;
    const int col0 = ((bx << lg) + sub) * CW;
    const int nrb = O / B;
    float cmax[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) cmax[c] = 0.0f;
    if (col0 < I) {
#pragma nounroll
        for (int rb = grp; rb < nrb; rb += groups) {
            float v[B * CW];
            load_row_block<Tin, B, CW>(W + static_cast<int64_t>(rb) * B * I + col0, I, v);
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                fwht_regs<B, CW>(v + c);
#pragma unroll
                for (int j = 0; j < B; ++j) cmax[c] = fmaxf(cmax[c], fabsf(v[j * CW + c]));
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CW; ++c) s_strip[tid * CW + c] = cmax[c];
    __syncthreads();
    if (col0 >= I) return;
    // a few groups at a time: all of them in flight would cost CW registers each
#pragma unroll 4
    for (int g = 0; g < groups; ++g) {
#pragma unroll
        for (int c = 0; c < CW; ++c) cmax[c] = fmaxf(cmax[c], s_strip[((g << lg) + sub) * CW + c]);
    }
    float inv[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        inv[c] = absmax_to_inv(cmax[c], qmax);
        if (grp == 0) sW[col0 + c] = absmax_to_scale(cmax[c], qmax);
    }
    if constexpr (F6) {
        // Two columns of a group of rows at a time, for the same short chain (at B = 16 a lane's four are two units).  The rows past O
        // are cleared in a loop of their own: as the other side of a test in this one they had the compiler keep every row's address
        // over it, 111 registers spilled at B = 64 (k_front_one; none now).  Whole passes at B = 64, that form -> this: 4096 x 1024
        // x 1024 46.2 -> 31.2 us, 2048 x 512 x 512 in fp32 29.6 -> 19.8, 12608 x 768 x 768 60.0 -> 49.4.
        constexpr int RB = ColsF6<B>::RB, UNITS = CW / 2;
        const int nrb6 = (O + RB - 1) / RB;
#pragma nounroll
        for (int i = grp; i < nrb6 * UNITS; i += groups) {
            const int o0 = i / UNITS * RB, second = UNITS == 2 ? i & 1 : 0;
            const float inv2[2] = {second ? inv[CW - 2] : inv[0], second ? inv[CW - 1] : inv[1]};
            cols_quantize_block_f6<Tin, B, false, 2>(W, O, I, inv2, k0, k1, reinterpret_cast<uint8_t *>(WqT), col0 + 2 * second, o0);
        }
#pragma nounroll
        for (int i = nrb6 + grp; i < f6_row_bytes(O) * 2 / RB; i += groups)
            cols_clear_f6<B, CW>(reinterpret_cast<uint8_t *>(WqT), O, col0, i * RB);
    } else {
#pragma nounroll
        for (int rb = grp; rb < nrb; rb += groups)
            cols_quantize_block<Tin, B, CODES == kCodesNibbles, false, CW>(W, O, I, inv, k0, k1, WqT, nullptr, col0, rb * B);
    }
}

}  // namespace hlq
