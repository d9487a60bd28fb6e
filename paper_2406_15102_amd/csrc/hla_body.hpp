// Device body of K3 (see k_hla.hip): workgroup (bx, by) of 256 threads projects token blocks
// 4 by .. 4 by + 3 of the 64 * (128 / B) features starting at bx * 64 * (128 / B).
//
// Where the rows come from is a template argument: DenseRows reads a row-major [N, D] tensor;
// ConvRows reads the column matrix of a channels-last image without it ever being stored
// (arXiv 2406.15102, Sec. 3.1: the spatial positions of a convolution are the sequence) -- a lane's
// 128 / B adjacent columns are channels of one filter tap, fixed for the lane, and the B consecutive
// rows are consecutive output positions, stepped from one division per block.
#pragma once
#include "hlq_device.hpp"
#include "hlq_kernels.hpp"

namespace hlq {

template <typename Tin> struct DenseRows {
    using elem = Tin;
    static constexpr bool image = false;
    const Tin *T;
    int64_t D;
    template <int B, int CPL> __device__ __forceinline__ void load_block(int64_t row0, int col0, float *v) const
    {
#pragma unroll
        for (int j = 0; j < B; ++j) Loader<Tin, CPL>::load(T + (row0 + j) * D + col0, v + j * CPL);
    }
};

// CPL consecutive elements at a byte offset of a buffer resource, widened to fp32; out of its range: zeros
template <typename T, int CPL> __device__ __forceinline__ void load_buffer(__amdgpu_buffer_rsrc_t rs, uint32_t ofs, float *v)
{
    constexpr int BYTES = CPL * sizeof(T), STEP = BYTES < 16 ? BYTES : 16;
    static_assert(STEP == 4 || STEP == 8 || STEP == 16, "whole dwords");
#pragma unroll
    for (int b = 0; b < BYTES; b += STEP) {
        uint32_t w[STEP / 4];
        if constexpr (STEP == 16) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, ofs + b, 0, 0);
            w[0] = q[0], w[1] = q[1], w[2] = q[2], w[3] = q[3];
        } else if constexpr (STEP == 8) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b64(rs, ofs + b, 0, 0);
            w[0] = q[0], w[1] = q[1];
        } else {
            w[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, ofs + b, 0, 0);
        }
#pragma unroll
        for (int d = 0; d < STEP / 4; ++d) {
            if constexpr (sizeof(T) == 4) {
                v[b / 4 + d] = __builtin_bit_cast(float, w[d]);
            } else {
                v[b / 2 + 2 * d] = bf16_lo(w[d]);
                v[b / 2 + 2 * d + 1] = bf16_hi(w[d]);
            }
        }
    }
}

// needs C % CPL == 0 (a lane's columns stay inside one tap) and N < 2^31
template <typename Tin> struct ConvRows {
    using elem = Tin;
    static constexpr bool image = true;
    const Tin *X;
    ConvShape g;
    template <int B, int CPL> __device__ __forceinline__ void load_block(int64_t row0, int col0, float *v) const
    {
        const int tap = col0 / g.C, c = col0 - tap * g.C;
        const int ky = tap / g.kw, kx = tap - ky * g.kw;
        const int dy = ky * g.dh - g.ph, dx = kx * g.dw - g.pw;
        const uint32_t t = static_cast<uint32_t>(row0);
        const uint32_t t2 = t / static_cast<uint32_t>(g.Wo), n0 = t2 / static_cast<uint32_t>(g.Ho);
        int wo = static_cast<int>(t - t2 * g.Wo), ho = static_cast<int>(t2 - n0 * g.Ho);
        if (B >= 32 && !g.far) {
            // Everything a wavefront reads lies within 2^31 bytes of its first image: byte offsets from there in 32
            // bits, stepped from one position to the next, and a tap outside the image is an offset out of the
            // resource's range, which loads zeros.  An address serves 128 / B channels: at B = 64 that is two, and the
            // products and selects below were what the projection spent its time on (65536 x 1728, bf16: 146 -> 60
            // us; B = 32 59.7 -> 49.7).  At B = 16, eight channels an address, they are hidden under the loads, and the
            // stepped offsets, each waiting for the one before, measure 7 % behind (65536 x 1224: 34.8 -> 37.2).
            const uint32_t first = __builtin_amdgcn_readfirstlane(n0);   // the lanes' positions ascend
            const uint32_t cb = g.C * sizeof(Tin), rb = cb * g.W;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<Tin *>(X + static_cast<int64_t>(first) * g.H * g.W * g.C), 0, 0x7FFFFFFF, 0x00020000);
            int hi = ho * g.sh + dy, wi = wo * g.sw + dx;
            const int hend = g.Ho * g.sh + dy, wend = g.Wo * g.sw + dx;
            // steps: to the next position, from the end of a row of positions to the next one, and to the next image
            // (modulo 2^32: an offset is only used where it is one into the image)
            const uint32_t next = g.sw * cb, row = g.sh * rb - g.Wo * next, image = g.H * rb - g.Ho * g.sh * rb;
            uint32_t o = ((n0 - first) * g.H + hi) * rb + wi * cb + c * static_cast<uint32_t>(sizeof(Tin));
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const bool ok = static_cast<uint32_t>(hi) < static_cast<uint32_t>(g.H) && static_cast<uint32_t>(wi) < static_cast<uint32_t>(g.W);
                load_buffer<Tin, CPL>(rs, ok ? o : 0x80000000u, v + j * CPL);
                wi += g.sw;
                o += next;
                if (wi == wend) {
                    wi = dx;
                    hi += g.sh;
                    o += row;
                    if (hi == hend) {
                        hi = dy;
                        o += image;
                    }
                }
            }
            return;
        }
        int64_t n = n0;
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int hi = ho * g.sh + dy, wi = wo * g.sw + dx;
            // a tap outside the image loads the nearest pixel instead (always a valid address, so the
            // B loads carry no branch and stay in flight together) and is zeroed afterwards
            const bool ok = hi >= 0 && hi < g.H && wi >= 0 && wi < g.W;
            const int hc = min(max(hi, 0), g.H - 1), wc = min(max(wi, 0), g.W - 1);
            Loader<Tin, CPL>::load(X + ((n * g.H + hc) * g.W + wc) * g.C + c, v + j * CPL);
#pragma unroll
            for (int k = 0; k < CPL; ++k) v[j * CPL + k] = ok ? v[j * CPL + k] : 0.0f;
            if (++wo == g.Wo) {
                wo = 0;
                if (++ho == g.Ho) {
                    ho = 0;
                    ++n;
                }
            }
        }
    }
};

// Workgroup l of a K3 job -> (column strip bx, group of 256/B token blocks by): grp consecutive by of
// one strip on one XCD (l mod 8), one after the other.  by may come out past the last group: the
// bodies return for those.
__device__ __forceinline__ void hla_job_map(int l, int gx, int grp, int &bx, int &by)
{
    const int t = l >> 3, u = (l & 7) + 8 * (t / grp);
    bx = u % gx;
    by = grp * (u / gx) + t % grp;
}

// values Kc .. Kp - 1 of CPL rows := 0 (either a multiple of 16 bytes, a row less than 128 bytes in all)
template <int CPL, typename T> __device__ __forceinline__ void clear_row_ends(T *row, int64_t Kc, int64_t Kp)
{
    constexpr int PIECE = 16 / sizeof(T);
    if (Kc == Kp) return;
#pragma nounroll
    for (int c = 0; c < CPL; ++c, row += Kp)
#pragma nounroll
        for (int64_t k = Kc; k < Kp; k += PIECE) *reinterpret_cast<uint4 *>(row + k) = make_uint4(0, 0, 0, 0);
}

// The same by the lanes of a column's last token block, behind their coefficients.  At B = 32 in fp32, and for bf16 projections of
// a bf16 image, a lane's columns and its block are worked out again from its index, hidden from the compiler for that: kept over the
// transform they were three registers too many (k_front_one<float, 32, ...> spilled 8, on the sequency basis 60; 0 and 20 so;
// the one of bf16 images 6, 0 so: 9408 x 2304 over 256 40.4 -> 40.0 us, 50176 x 576 over 64 36.6 -> 36.2).  Only there: a
// convolution of 65536 x 864 over 256 in fp32 at B = 16 takes 126.0 us and 132.9 that way, on as many wavefronts, one of
// 50176 x 576 over 64 in bf16 at B = 32 beside the integer list 65.0 and 66.5.
template <int B, typename Src, int L, int NB, int CPL, typename T>
__device__ __forceinline__ void clear_ends_of_last_block(T *out, int64_t nblk, int r, int64_t Kp, int bx, int by, int col0, int64_t blk)
{
    if constexpr (B == 32 && (sizeof(typename Src::elem) == 4 || (Src::image && sizeof(T) == 2))) {
        if (nblk * r == Kp) return;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        if (static_cast<int64_t>(by) * NB + tid / L == nblk - 1)
            clear_row_ends<CPL>(out + static_cast<int64_t>((bx * L + tid % L) * CPL) * Kp, nblk * r, Kp);
    } else {
        if (blk == nblk - 1) clear_row_ends<CPL>(out + static_cast<int64_t>(col0) * Kp, nblk * r, Kp);
    }
}

// LM: lanes side by side as a multiple of hla_lanes(B) -- 1 for the stand-alone shape (B lanes x 256/B token
// blocks), 2 for the workgroups that share their rows of G with K1 through one XCD's L2
// (2 B lanes = 256 columns x 128/B token blocks = 128 rows).
// PAD: rows of ThatT are Kp values apart, those behind the N / B * r coefficients zeros (pad_row; not with coeffT).
// The lanes of a column's last token block clear them once its coefficients are stored, not workgroups of their own in
// front of the loads: that test alone made the projections of an image (ConvRows), whose rows mostly need no padding, wait:
// whole pass of a 3 x 3 convolution of 12544 x 256 over 256 46.6 -> 46.1 us (45.9 by code that has no padding at all), 640 x 26624
// x 288 at B = 32 64.7 -> 63.5 (63.5).
template <int B, int BASIS, typename Src, int LM = 1, bool PAD = false>
__device__ __forceinline__ void hla_body_src(const Src &src, int64_t N, int D, int r, int64_t Kp, bf16_t *__restrict__ ThatT,
                                             float *__restrict__ coeffT, int bx, int by)
{
    constexpr int CPL = 128 / B;
    constexpr int L = hla_lanes(B) * LM, NB = 256 / L;
    static_assert(NB >= 1 && L * NB == 256, "a K3 workgroup is 256 lanes");
    const int tid = threadIdx.x;
    const int col0 = (bx * L + tid % L) * CPL;
    const int64_t nblk = N / B;
    const int64_t pitch = PAD ? Kp : nblk * r;
    const int64_t blk = static_cast<int64_t>(by) * NB + tid / L;
    if (col0 >= D || blk >= nblk) return;

    float v[B * CPL];
    src.template load_block<B, CPL>(blk * B, col0, v);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        fwht_regs<B, CPL>(v + c);
        const int64_t o = static_cast<int64_t>(col0 + c) * pitch + blk * r;
        if (r >= 8) {
#pragma unroll
            for (int k = 0; k < B; k += 8) {
                if (k < r) {
                    uint4 p;
                    p.x = pack_bf16(v[kept_row<B, BASIS>(k + 0) * CPL + c], v[kept_row<B, BASIS>(k + 1) * CPL + c]);
                    p.y = pack_bf16(v[kept_row<B, BASIS>(k + 2) * CPL + c], v[kept_row<B, BASIS>(k + 3) * CPL + c]);
                    p.z = pack_bf16(v[kept_row<B, BASIS>(k + 4) * CPL + c], v[kept_row<B, BASIS>(k + 5) * CPL + c]);
                    p.w = pack_bf16(v[kept_row<B, BASIS>(k + 6) * CPL + c], v[kept_row<B, BASIS>(k + 7) * CPL + c]);
                    *reinterpret_cast<uint4 *>(ThatT + o + k) = p;
                }
            }
        } else if (r == 4) {
            uint2 p;
            p.x = pack_bf16(v[kept_row<B, BASIS>(0) * CPL + c], v[kept_row<B, BASIS>(1) * CPL + c]);
            p.y = pack_bf16(v[kept_row<B, BASIS>(2) * CPL + c], v[kept_row<B, BASIS>(3) * CPL + c]);
            *reinterpret_cast<uint2 *>(ThatT + o) = p;
        } else if (r == 2) {
            *reinterpret_cast<uint32_t *>(ThatT + o) = pack_bf16(v[kept_row<B, BASIS>(0) * CPL + c], v[kept_row<B, BASIS>(1) * CPL + c]);
        } else {
            ThatT[o] = static_cast<bf16_t>(pack_bf16(v[c], 0.0f) & 0xFFFFu);
        }
        if (coeffT) {
#pragma unroll
            for (int k = 0; k < B; ++k)
                if (k < r) coeffT[o + k] = v[kept_row<B, BASIS>(k) * CPL + c];
        }
    }
    if constexpr (PAD) clear_ends_of_last_block<B, Src, L, NB, CPL>(ThatT, nblk, r, Kp, bx, by, col0, blk);
}

template <typename Tin, int B, int BASIS, int LM = 1, bool PAD = false>
__device__ __forceinline__ void hla_body(const Tin *__restrict__ T, int64_t N, int D, int r, int64_t Kp, bf16_t *__restrict__ ThatT,
                                         float *__restrict__ coeffT, int bx, int by)
{
    hla_body_src<B, BASIS, DenseRows<Tin>, LM, PAD>(DenseRows<Tin>{T, D}, N, D, r, Kp, ThatT, coeffT, bx, by);
}

template <int NW> struct Words { static constexpr int value = NW; };

// ---- integer g_w list: pass 1 (column maxima of the kept coefficients) and pass 2 (int8 codes) ----
template <int B, int BASIS, typename Src>
__device__ __forceinline__ void hla_absmax_body_src(const Src &src, int64_t N, int D, int r,
                                                    uint32_t *__restrict__ amax_bits, int bx, int by, bool table = false)
{
    constexpr int CPL = 128 / B, L = hla_lanes(B), NB = hla_blocks(B);
    __shared__ float s_max[NB][L * CPL];
    const int tid = threadIdx.x, grp = tid / L, sub = tid % L;
    const int col0 = (bx * L + sub) * CPL;
    const int64_t nblk = N / B;
    const int64_t blk = static_cast<int64_t>(by) * NB + grp;
    float cmax[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) cmax[c] = 0.0f;
    if (col0 < D && blk < nblk) {
        float v[B * CPL];
        src.template load_block<B, CPL>(blk * B, col0, v);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            fwht_regs<B, CPL>(v + c);
#pragma unroll
            for (int k = 0; k < B; ++k)
                if (k < r) cmax[c] = fmaxf(cmax[c], fabsf(v[kept_row<B, BASIS>(k) * CPL + c]));
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
            if (col < D) amax_bits[static_cast<int64_t>(by) * D + col] = __float_as_uint(m);
        } else if (col < D && m > 0.0f) {
            atomicMax(amax_bits + col, __float_as_uint(m));
        }
    }
}

template <typename Tin, int B, int BASIS>
__device__ __forceinline__ void hla_absmax_body(const Tin *__restrict__ T, int64_t N, int D, int r,
                                                uint32_t *__restrict__ amax_bits, int bx, int by, bool table = false)
{
    hla_absmax_body_src<B, BASIS>(DenseRows<Tin>{T, D}, N, D, r, amax_bits, bx, by, table);
}

// P4: codes in [-7, 7] stored two to a byte (TqT then has Kc/2 bytes per feature; needs r % 8 == 0) -- the
// 4-bit form in which the compressed activation is kept between the passes (Sec. 6.1) -- instead of
// codes in [-127, 127], one int8 each.  Same stream, same counters, same maxima either way.  PAD, Kp: as in hla_body_src.
template <int B, int BASIS, bool MANT, typename Src, bool P4 = false, bool PAD = false>
__device__ __forceinline__ void hla_quantize_body_src(const Src &src, int64_t N, int D, int r,
                                                      const uint32_t *__restrict__ amax_bits, uint32_t k0, uint32_t k1,
                                                      int64_t Kp, int8_t *__restrict__ TqT, float *__restrict__ sT,
                                                      float *__restrict__ coeffT, int bx, int by, int table = 0)
{
    constexpr int CPL = 128 / B, L = hla_lanes(B), NB = hla_blocks(B);
    const int tid = threadIdx.x;
    const int col0 = (bx * L + tid % L) * CPL;
    const int64_t nblk = N / B;
    const int64_t Kc = nblk * r;
    const int64_t blk = static_cast<int64_t>(by) * NB + tid / L;
    float amax[CPL];
    fold_column_maxima<CPL>(amax_bits, D, table, bx, tid % L, amax);
    const int64_t pitch = PAD ? Kp : Kc;
    static_assert(!PAD || !P4, "4-bit codes are stored without padding");
    if (col0 >= D || blk >= nblk) return;

    float v[B * CPL];
    src.template load_block<B, CPL>(blk * B, col0, v);
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        fwht_regs<B, CPL>(v + c);
        constexpr float QMAX = P4 ? 7.0f : 127.0f;
        const float a = amax[c];
        const float inv = absmax_to_inv(a, QMAX);
        if (blk == 0) sT[col0 + c] = absmax_to_scale(a, QMAX);
        const int64_t o = static_cast<int64_t>(col0 + c) * pitch + blk * r;          // r % 4 == 0
        const uint32_t cnt = static_cast<uint32_t>(col0 + c) * static_cast<uint32_t>(Kc >> 2) +
                             static_cast<uint32_t>((blk * r) >> 2);
        // the kept coefficients in order, a group of random words at a time
        auto codes = [&](auto nw, int k) {
            constexpr int NW = decltype(nw)::value;
            float x[4 * NW];
#pragma unroll
            for (int e = 0; e < 4 * NW; ++e) x[e] = v[kept_row<B, BASIS>(k + e) * CPL + c];
            int q[4 * NW];
            quant_codes<MANT, NW>(x, 1, inv, cnt + (k >> 2), k0, k1, q);
            if constexpr (P4) {
#pragma unroll
                for (int d = 0; d < NW / 2; ++d) *reinterpret_cast<uint32_t *>(TqT + ((o + k) >> 1) + 4 * d) = pack_nibbles8(q + 8 * d);
            } else {
#pragma unroll
                for (int d = 0; d < NW; ++d) *reinterpret_cast<uint32_t *>(TqT + o + k + 4 * d) = pack_bytes4(q + 4 * d);
            }
            if (coeffT) {
#pragma unroll
                for (int e = 0; e < 4 * NW; e += 4)
                    *reinterpret_cast<float4 *>(coeffT + o + k + e) = make_float4(x[e], x[e + 1], x[e + 2], x[e + 3]);
            }
        };
        if (r >= 16) {
#pragma unroll
            for (int k = 0; k < B; k += 16)
                if (k < r) codes(Words<4>{}, k);
        } else if (r == 8) {
            codes(Words<2>{}, 0);
        } else if constexpr (!P4) {
            codes(Words<1>{}, 0);      // r == 4
        }
    }
    if constexpr (PAD) clear_ends_of_last_block<B, Src, L, NB, CPL>(TqT, nblk, r, Kp, bx, by, col0, blk);
}

template <typename Tin, int B, int BASIS, bool MANT = false, bool P4 = false, bool PAD = false>
__device__ __forceinline__ void hla_quantize_body(const Tin *__restrict__ T, int64_t N, int D, int r,
                                                  const uint32_t *__restrict__ amax_bits, uint32_t k0, uint32_t k1,
                                                  int64_t Kp, int8_t *__restrict__ TqT, float *__restrict__ sT,
                                                  float *__restrict__ coeffT, int bx, int by, int table = 0)
{
    hla_quantize_body_src<B, BASIS, MANT, DenseRows<Tin>, P4, PAD>(DenseRows<Tin>{T, D}, N, D, r, amax_bits, k0, k1, Kp, TqT, sT, coeffT,
                                                             bx, by, table);
}

}  // namespace hlq
