// Device body of K1 (see k_quant_rows.hip), callable from any kernel whose workgroup `bx` of BLOCK
// threads is to process the rows bx * (BLOCK / T) ... of G, and the host-side choice of T.
#pragma once
#include "hlq_device.hpp"
#include "hlq_kernels.hpp"

namespace hlq {

constexpr int K1_MAXC = 8;  // chunks of 8 elements per lane

// PACKED: the codes are written two to a byte (4-bit codes only), O/2 bytes per row.
template <typename Tin, int B, int BLOCK, bool PACKED, bool MANT = false>
__device__ __forceinline__ void quant_rows_body(const Tin *__restrict__ G, int64_t N, int O, int T, uint32_t k0,
                                                uint32_t k1, float qmax, int8_t *__restrict__ Gq,
                                                float *__restrict__ sG, float *__restrict__ coeff, int bx)
{
    __shared__ float s_red[BLOCK / 64];
    const int tid = threadIdx.x;
    const int rows_per_block = BLOCK / T;
    const int g = tid % T;                       // lane index within the row's group
    const int64_t row = static_cast<int64_t>(bx) * rows_per_block + tid / T;
    const bool row_ok = row < N;
    const int nch = O >> 3;                      // 8-element chunks per row

    float v[K1_MAXC][8];
    const Tin *grow = G + (row_ok ? row : 0) * static_cast<int64_t>(O);

#pragma unroll
    for (int m = 0; m < K1_MAXC; ++m) {
        const int ci = g + m * T;
        if (ci < nch) Loader<Tin, 8>::load(grow + static_cast<int64_t>(ci) * 8, v[m]);
    }

    // Cross-lane stages leave the lane with value sign * (coefficient): see butterfly_lanes_signed8.
    const float sg1 = (tid & 1) ? -1.0f : 1.0f;
    const float sg2 = (tid & 2) ? -1.0f : 1.0f;
    const float sg4 = (tid & 4) ? -1.0f : 1.0f;
    const float sign = sg1 * (B >= 32 ? sg2 : 1.0f) * (B >= 64 ? sg4 : 1.0f);

    float amax = 0.0f;
#pragma unroll
    for (int m = 0; m < K1_MAXC; ++m) {
        const int ci = g + m * T;
        // whole Hadamard blocks are either inside or outside the row: the lanes of one block
        // (aligned groups of B/8 lanes) take this branch together
        if (ci < nch) {
            fwht_regs<8, 1>(v[m]);
            butterfly_lanes_signed8<1>(v[m], sg1);
            if (B >= 32) butterfly_lanes_signed8<2>(v[m], sg2);
            if (B >= 64) butterfly_lanes_signed8<4>(v[m], sg4);
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(v[m][e]));
        }
    }

    // absmax over the row's lanes
    if (T <= 64) {
        for (int off = 1; off < T; off *= 2) amax = fmaxf(amax, __shfl_xor(amax, off));
    } else {
        for (int off = 1; off < 64; off *= 2) amax = fmaxf(amax, __shfl_xor(amax, off));
        if ((tid & 63) == 0) s_red[tid >> 6] = amax;
        __syncthreads();
        amax = s_red[0];
#pragma unroll
        for (int w = 1; w < BLOCK / 64; ++w) amax = fmaxf(amax, s_red[w]);
    }

    if (!row_ok) return;
    const float inv = absmax_to_inv(amax, qmax) * sign;   // exact: undoes the sign the lane exchange left
    if (g == 0) sG[row] = absmax_to_scale(amax, qmax);

    const uint32_t cbase = static_cast<uint32_t>(row) * static_cast<uint32_t>(O >> 2);
    int8_t *qrow = Gq + row * static_cast<int64_t>(PACKED ? O / 2 : O);
#pragma unroll
    for (int m = 0; m < K1_MAXC; ++m) {
        const int ci = g + m * T;
        if (ci < nch) {
            int q[8];
            quant_codes<MANT, 2>(v[m], 1, inv, cbase + 2u * ci, k0, k1, q);
            if (PACKED) *reinterpret_cast<uint32_t *>(qrow + static_cast<int64_t>(ci) * 4) = pack_nibbles8(q);
            else *reinterpret_cast<uint2 *>(qrow + static_cast<int64_t>(ci) * 8) = make_uint2(pack_bytes4(q), pack_bytes4(q + 4));
            if (coeff) {
                float4 *c = reinterpret_cast<float4 *>(coeff + row * static_cast<int64_t>(O) + static_cast<int64_t>(ci) * 8);
                c[0] = make_float4(sign * v[m][0], sign * v[m][1], sign * v[m][2], sign * v[m][3]);
                c[1] = make_float4(sign * v[m][4], sign * v[m][5], sign * v[m][6], sign * v[m][7]);
            }
        }
    }
}

// K1 with the codes in the f6 layout (hlq_device.hpp): rows of f6_row_bytes(O), 16 bytes for 32 codes, zeros behind the
// row's end.  A lane owns up to kF6Rounds groups of 32 consecutive elements, g + m T, so that a group's codes are
// packed without leaving the lane; the butterflies of B = 16 and 32 stay in it too, and at B = 64 one stage, stride 32,
// pairs it with its neighbour.  (A lane's loads are then 64 bytes apart, and an instruction takes a quarter of
// four times as many lines; the next three find them in the L1.)
constexpr int kF6Rounds = 3;

template <typename Tin, int B, int BLOCK, bool MANT = false>
__device__ __forceinline__ void quant_rows_f6_body(const Tin *__restrict__ G, int64_t N, int O, int T, uint32_t k0, uint32_t k1,
                                                   float qmax, uint8_t *__restrict__ Gq, float *__restrict__ sG, int bx)
{
    __shared__ float s_red[BLOCK / 64];
    const int tid = threadIdx.x;
    const int64_t row = static_cast<int64_t>(bx) * (BLOCK / T) + tid / T;
    const bool row_ok = row < N;
    // lane of the row; where a row takes the whole workgroup, whose last round is mostly empty, the wavefront that
    // starts it changes from row to row, as the groups of one round do not fill the SIMDs evenly
    const int g = T < BLOCK ? tid % T : (tid + 64 * static_cast<int>(row & (BLOCK / 64 - 1))) % BLOCK;
    const int ng = (O + 31) >> 5;                     // groups of a row; O % 16 == 0: the last may be half of one

    float v[kF6Rounds][32];
    const Tin *grow = G + (row_ok ? row : 0) * static_cast<int64_t>(O);
#pragma unroll
    for (int m = 0; m < kF6Rounds; ++m) {
        const int gi = g + m * T;
        if (gi < ng) {
            const Tin *p = grow + static_cast<int64_t>(gi) * 32;
            Loader<Tin, 8>::load(p, v[m]);
            Loader<Tin, 8>::load(p + 8, v[m] + 8);
            if (B > 16 || gi * 32 + 16 < O) {
                Loader<Tin, 8>::load(p + 16, v[m] + 16);
                Loader<Tin, 8>::load(p + 24, v[m] + 24);
            } else {
#pragma unroll
                for (int e = 16; e < 32; ++e) v[m][e] = 0.0f;
            }
        }
    }

    const float sign = (B == 64 && (tid & 1)) ? -1.0f : 1.0f;
    float amax = 0.0f;
#pragma unroll
    for (int m = 0; m < kF6Rounds; ++m) {
        if (g + m * T < ng) {      // at B = 64 a row's groups come in pairs: both lanes of one or neither
            fwht_regs<(B < 32 ? B : 32), 1>(v[m]);
            if (B == 16) fwht_regs<16, 1>(v[m] + 16);
            if (B == 64) {
#pragma unroll
                for (int e = 0; e < 32; e += 8) butterfly_lanes_signed8<1>(v[m] + e, sign);
            }
#pragma unroll
            for (int e = 0; e < 32; ++e) amax = fmaxf(amax, fabsf(v[m][e]));
        }
    }
    if (T <= 64) {
        for (int off = 1; off < T; off *= 2) amax = fmaxf(amax, __shfl_xor(amax, off));
    } else {
        for (int off = 1; off < 64; off *= 2) amax = fmaxf(amax, __shfl_xor(amax, off));
        if ((tid & 63) == 0) s_red[tid >> 6] = amax;
        __syncthreads();
        amax = s_red[0];
#pragma unroll
        for (int w = 1; w < BLOCK / 64; ++w) amax = fmaxf(amax, s_red[w]);
    }
    if (!row_ok) return;
    const float inv = absmax_to_inv(amax, qmax) * sign;   // exact: undoes the sign the lane exchange left
    if (g == 0) sG[row] = absmax_to_scale(amax, qmax);

    const uint32_t cbase = static_cast<uint32_t>(row) * static_cast<uint32_t>(O >> 2);
    const int row_bytes = f6_row_bytes(O);
    uint8_t *qrow = Gq + row * static_cast<int64_t>(row_bytes);
#pragma unroll
    for (int m = 0; m < kF6Rounds; ++m) {
        const int gi = g + m * T;
        if (gi < ng) {
            float f[32];
            quant_floats<MANT, 4>(v[m], 1, inv, cbase + 8u * gi, k0, k1, f);
            quant_floats<MANT, 4>(v[m] + 16, 1, inv, cbase + 8u * gi + 4u, k0, k1, f + 16);
            *reinterpret_cast<uint4 *>(qrow + static_cast<int64_t>(gi) * 16) = f6_pack32(f);
        } else if (gi * 16 < row_bytes) {
            *reinterpret_cast<uint4 *>(qrow + static_cast<int64_t>(gi) * 16) = make_uint4(0, 0, 0, 0);
        }
    }
}

// Lanes per row of the f6 variant, or 0 if the row needs 1024 threads: the split with the fewest lanes idle in its last
// round, rows of whole wavefronts' lanes first.
inline int quant_rows_f6_lanes(int O)
{
    const int ng = f6_row_bytes(O) / 16;
    if (ng > kF6Rounds * 64) return ng <= kF6Rounds * 256 ? 256 : 0;
    int best = 64, waste = 1 << 30;
    for (int T = 64; T >= 4; T /= 2) {
        const int rounds = (ng + T - 1) / T;
        if (rounds > kF6Rounds) break;
        if (rounds * T - ng < waste) {
            waste = rounds * T - ng;
            best = T;
        }
    }
    return best;
}

// Lanes per row for the 256-thread variant, or 0 if the row needs the 1024-thread one.
inline int quant_rows_lanes(int O, int B)
{
    const int nch = O / 8;
    if (nch <= K1_MAXC * 64) {
        int T = 8;
        while (T * K1_MAXC < nch || T < B / 8) T *= 2;   // fewest lanes that cover the row (<= 64)
        // prefer ~4 chunks per lane when the row is long enough to keep more loads in flight
        while (T < 64 && nch / T > 4) T *= 2;
        return T;
    }
    return nch <= K1_MAXC * 256 ? 256 : 0;
}

}  // namespace hlq
