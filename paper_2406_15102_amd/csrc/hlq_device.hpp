// Device-side building blocks shared by the gfx950 kernels: element loads, the in-register
// fast Walsh-Hadamard transform, the stochastic-rounding random stream and the 4-bit quantiser.
//
// Numerical contract (arXiv 2406.15102, Sec. 3.2 / 5.1 / 6.1, as fixed by this library):
//   * H is the +-1 natural-order Walsh-Hadamard matrix; a coefficient is the sum of its B signed
//     terms added pairwise in index order.  A radix-2 butterfly network with strides 1, 2, 4, ...
//     (ascending) evaluates exactly that expression tree, so the stage order below is fixed.
//   * code = floor(fma(x, qmax/absmax, (byte + 0.5)/256)) (always inside [-qmax, qmax]; qmax = 7
//     or 127), byte taken from word
//     number row*(K/4) + pos/4 of a keyed counter stream, byte pos%4 of that word.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hlq {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// Two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    v2f p = {lo, hi};
    v2bf q = __builtin_convertvector(p, v2bf);
    return __builtin_bit_cast(uint32_t, q);
}

// ---- element loads: NE consecutive elements widened to fp32 --------------------------------
template <typename T, int NE> struct Loader;

template <> struct Loader<bf16_t, 8> {
    static __device__ __forceinline__ void load(const bf16_t *p, float *v)
    {
        uint4 w = *reinterpret_cast<const uint4 *>(p);
        v[0] = bf16_lo(w.x); v[1] = bf16_hi(w.x); v[2] = bf16_lo(w.y); v[3] = bf16_hi(w.y);
        v[4] = bf16_lo(w.z); v[5] = bf16_hi(w.z); v[6] = bf16_lo(w.w); v[7] = bf16_hi(w.w);
    }
};
template <> struct Loader<bf16_t, 4> {
    static __device__ __forceinline__ void load(const bf16_t *p, float *v)
    {
        uint2 w = *reinterpret_cast<const uint2 *>(p);
        v[0] = bf16_lo(w.x); v[1] = bf16_hi(w.x); v[2] = bf16_lo(w.y); v[3] = bf16_hi(w.y);
    }
};
template <> struct Loader<bf16_t, 2> {
    static __device__ __forceinline__ void load(const bf16_t *p, float *v)
    {
        uint32_t w = *reinterpret_cast<const uint32_t *>(p);
        v[0] = bf16_lo(w); v[1] = bf16_hi(w);
    }
};
template <> struct Loader<float, 8> {
    static __device__ __forceinline__ void load(const float *p, float *v)
    {
        float4 a = *reinterpret_cast<const float4 *>(p);
        float4 b = *reinterpret_cast<const float4 *>(p + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
};
template <> struct Loader<float, 4> {
    static __device__ __forceinline__ void load(const float *p, float *v)
    {
        float4 a = *reinterpret_cast<const float4 *>(p);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    }
};
template <> struct Loader<float, 2> {
    static __device__ __forceinline__ void load(const float *p, float *v)
    {
        float2 a = *reinterpret_cast<const float2 *>(p);
        v[0] = a.x; v[1] = a.y;
    }
};

// Workgroup `lin` of `total`, counted from the other end but on the same XCD (workgroups go to the eight XCDs
// round-robin, index mod 8): the second pass over a tensor walks it backwards, so that it starts on what the
// first pass read last -- what the last-level cache still holds of a tensor larger than it -- and a workgroup
// still finds in its own XCD's L2 what its counterpart of the first pass left there.
// Only for tensors of more than half that cache (`bytes`): a smaller one is found there whole, and in order it
// measured a little better (4096 x 4096 activation, int8 store: 16.6 us against 17.5 backwards).
constexpr int64_t kReverseSecondPassBytes = int64_t(128) << 20;
__device__ __forceinline__ int reverse_same_xcd(int lin, int total, int64_t bytes)
{
    const int n8 = total & ~7;
    return (bytes > kReverseSecondPassBytes && lin < n8) ? (n8 - 8 - (lin & ~7)) + (lin & 7) : lin;
}

// ---- in-register FWHT over v[0..n), element stride `es` in the array, strides ascending -----
template <int NPT, int ES>
__device__ __forceinline__ void fwht_regs(float *v)
{
#pragma unroll
    for (int h = 1; h < NPT; h *= 2) {
#pragma unroll
        for (int base = 0; base < NPT; base += 2 * h) {
#pragma unroll
            for (int k = base; k < base + h; ++k) {
                float a = v[k * ES], b = v[(k + h) * ES];
                v[k * ES] = a + b;
                v[(k + h) * ES] = a - b;
            }
        }
    }
}

// One butterfly stage between lanes l and l^MASK (MASK in {1, 2, 4}) in ONE instruction where the
// exchange is a DPP quad permute: x <- partner * sigma + x with sigma = +1 in the lane whose MASK
// bit is clear and -1 in the other.  The product is exact, so the single rounding is that of the
// add/subtract of the butterfly.  The lower lane gets a + b; the upper lane gets b - a, i.e. the
// NEGATIVE of the butterfly's difference a - b... with a = lower lane's value: upper holds
// x_upper - x_lower = -(a - b).  Callers carry that sign per lane (it is the same for both lanes of
// every later exchange, because they differ in a higher lane bit only) and fold it into whatever
// consumes the value.  The s_nop covers the VALU-write -> DPP-read hazard, which the compiler
// cannot see inside an asm statement; the eight values of a chunk go together so that one covers them all.
// Every one of them is written before sigma is read for the last time, hence early-clobber operands.
#define HLQ_DPP8(PERM)                                                                                        \
    asm("s_nop 1\n\t"                                                                                         \
        "v_fmac_f32_dpp %0, %0, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %1, %1, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %2, %2, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %3, %3, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %4, %4, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %5, %5, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %6, %6, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"            \
        "v_fmac_f32_dpp %7, %7, %8 quad_perm:" PERM " row_mask:0xf bank_mask:0xf bound_ctrl:1"                \
        : "+&v"(x[0]), "+&v"(x[1]), "+&v"(x[2]), "+&v"(x[3]), "+&v"(x[4]), "+&v"(x[5]), "+&v"(x[6]), "+&v"(x[7]) \
        : "v"(sigma))
template <int MASK>
__device__ __forceinline__ void butterfly_lanes_signed8(float *x, float sigma)
{
    if constexpr (MASK == 1) {
        HLQ_DPP8("[1,0,3,2]");
    } else if constexpr (MASK == 2) {
        HLQ_DPP8("[2,3,0,1]");
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, x[e]), 0x101F));  // lane ^ 4
            x[e] = __builtin_fmaf(p, sigma, x[e]);
        }
    }
}
#undef HLQ_DPP8

// Row of the natural-order Hadamard matrix kept as coefficient k of the low-rank projection.
// BASIS 0: row k.  BASIS 1: the row with k sign changes (sequency order), which is the
// bit-reversed Gray code of k.  Constant-folds when k is a compile-time constant.
template <int B, int BASIS>
__host__ __device__ constexpr int kept_row(int k)
{
    if (BASIS == 0) return k;
    const int g = k ^ (k >> 1);
    int n = 0;
    for (int lo = 1, hi = B >> 1; lo < B; lo <<= 1, hi >>= 1)
        if (g & lo) n |= hi;
    return n;
}

// ---- random stream ---------------------------------------------------------------------------
// Word `counter` of the stream keyed by (k0, k1): a keyed xorshift-multiply bijection of the
// counter (multipliers of the public-domain "lowbias32" integer hash):
//   x = counter ^ k0;  x ^= x >> 16;  x *= M1;  x ^= x >> 15;  x ^= k1;  x *= M2;  x ^= x >> 16
constexpr uint32_t kMix1 = 0x7FEB352Du, kMix2 = 0x846CA68Bu;
__device__ __forceinline__ uint32_t rand_finish(uint32_t x, uint32_t k1)
{
    x ^= x >> 15;
    x ^= k1;
    x *= kMix2;
    return x ^ (x >> 16);
}

// Words counter .. counter + NW - 1 (counter a multiple of NW = 1, 2 or 4).  The words of an aligned group differ
// only in the low bits of the counter, which reach the first multiplication unmixed: with x the first word's
// factor, word i's is x ^ i = x + (+-1 for bit 0 of i) + (+-2 for bit 1), the signs set by those bits of x.  So one
// product serves the group, the others are one addition of +-M1, +-2 M1 each: a 32-bit multiplication issues
// at a quarter of the rate of anything else here, and there are two of them to four codes otherwise.
template <int NW>
__device__ __forceinline__ void rand_words(uint32_t counter, uint32_t k0, uint32_t k1, uint32_t *w)
{
    static_assert(NW == 1 || NW == 2 || NW == 4, "aligned groups of one, two or four words");
    uint32_t x = counter ^ k0;
    x ^= x >> 16;
    const uint32_t p = x * kMix1;
    w[0] = rand_finish(p, k1);
    if constexpr (NW >= 2) {
        const uint32_t s0 = 0u - (x & 1u);
        const uint32_t d0 = (s0 & (0u - kMix1)) | (~s0 & kMix1);
        w[1] = rand_finish(p + d0, k1);
        if constexpr (NW == 4) {
            const uint32_t s1 = 0u - ((x >> 1) & 1u);
            const uint32_t p2 = p + ((s1 & (0u - 2u * kMix1)) | (~s1 & (2u * kMix1)));
            w[2] = rand_finish(p2, k1);
            w[3] = rand_finish(p2 + d0, k1);
        }
    }
}

// floor(t) as an integer in one instruction (v_cvt_flr_i32_f32).
__device__ __forceinline__ int floor_to_int(float t)
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(t));
    return r;
}

// Four codes floor(fma(x, inv, u)), u = (byte + 0.5) / 256 for the four bytes of a random word.
// u has nine significant bits, so it is exact in fp16 and the four are built two to an instruction: a byte
// permutation puts each byte b under the exponent of 1024 (0x6400 + b = 1024 + b), and one packed fp16 fma
// makes (1024 + b) / 256 - (4 - 1/512).  The fma that adds u reads it as fp16 (v_fma_mix_f32: exact
// operands, one fp32 rounding), the same value as with u in fp32 -- two instructions a code fewer than
// converting each byte and scaling it were four of every fourteen.
// No clamp is needed: |x| <= absmax and inv = RN(qmax / absmax) give |x*inv| <= qmax (1 + 2^-24),
// and u lies in [2^-9, 1 - 2^-9], so the rounded sum stays inside (-qmax, qmax + 1) and its floor
// inside [-qmax, qmax] (a zero row has inv = 0 and floor(u) = 0).  Inf/NaN inputs are outside the
// contract.
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v2h round_bits_pair(uint32_t w, uint32_t sel)
{
    const v2h b = __builtin_bit_cast(v2h, __builtin_amdgcn_perm(0x64646464u, w, sel));
    const v2h scale = {static_cast<_Float16>(0.00390625f), static_cast<_Float16>(0.00390625f)};
    const v2h shift = {static_cast<_Float16>(-3.998046875f), static_cast<_Float16>(-3.998046875f)};
    return __builtin_elementwise_fma(b, scale, shift);
}
__device__ __forceinline__ void quant_codes4(const float *x, int es, float inv, uint32_t w, int *q)
{
    const v2h u01 = round_bits_pair(w, 0x04010400u), u23 = round_bits_pair(w, 0x04030402u);
    q[0] = floor_to_int(__builtin_fmaf(x[0], inv, static_cast<float>(u01[0])));
    q[1] = floor_to_int(__builtin_fmaf(x[es], inv, static_cast<float>(u01[1])));
    q[2] = floor_to_int(__builtin_fmaf(x[2 * es], inv, static_cast<float>(u23[0])));
    q[3] = floor_to_int(__builtin_fmaf(x[3 * es], inv, static_cast<float>(u23[1])));
}

// The paper's pseudo-stochastic rounding (Sec. 6.1): the low 11 bits of the value's own binary32
// pattern replace the random number, u = (m + 0.5) / 2048 (exact, one fma).  A sign flip of the
// value (see butterfly_lanes_signed8) leaves those bits alone.
__device__ __forceinline__ int quant_code_mantissa(float x, float inv)
{
    const float m = static_cast<float>(__float_as_uint(x) & 0x7FFu);
    const float u = __builtin_fmaf(m, 0.00048828125f, 0.000244140625f);
    return floor_to_int(__builtin_fmaf(x, inv, u));
}

// Codes of NW * 4 values x[0], x[es], x[2 es], ...: rounding by words counter .. of the stream keyed by k0, k1
// (counter a multiple of NW), or, with MANT, by the values' own low mantissa bits.
template <bool MANT, int NW>
__device__ __forceinline__ void quant_codes(const float *x, int es, float inv, uint32_t counter, uint32_t k0, uint32_t k1, int *q)
{
    if constexpr (MANT) {
#pragma unroll
        for (int e = 0; e < 4 * NW; ++e) q[e] = quant_code_mantissa(x[e * es], inv);
    } else {
        uint32_t w[NW];
        rand_words<NW>(counter, k0, k1, w);
#pragma unroll
        for (int d = 0; d < NW; ++d) quant_codes4(x + 4 * d * es, es, inv, w[d], q + 4 * d);
    }
}

// The same codes as floats (whole numbers), for the conversion to 6-bit floats.
__device__ __forceinline__ void quant_floats4(const float *x, int es, float inv, uint32_t w, float *f)
{
    const v2h u01 = round_bits_pair(w, 0x04010400u), u23 = round_bits_pair(w, 0x04030402u);
    f[0] = __builtin_floorf(__builtin_fmaf(x[0], inv, static_cast<float>(u01[0])));
    f[1] = __builtin_floorf(__builtin_fmaf(x[es], inv, static_cast<float>(u01[1])));
    f[2] = __builtin_floorf(__builtin_fmaf(x[2 * es], inv, static_cast<float>(u23[0])));
    f[3] = __builtin_floorf(__builtin_fmaf(x[3 * es], inv, static_cast<float>(u23[1])));
}
template <bool MANT, int NW>
__device__ __forceinline__ void quant_floats(const float *x, int es, float inv, uint32_t counter, uint32_t k0, uint32_t k1, float *f)
{
    if constexpr (MANT) {
#pragma unroll
        for (int e = 0; e < 4 * NW; ++e) {
            const float m = static_cast<float>(__float_as_uint(x[e * es]) & 0x7FFu);
            f[e] = __builtin_floorf(__builtin_fmaf(x[e * es], inv, __builtin_fmaf(m, 0.00048828125f, 0.000244140625f)));
        }
    } else {
        uint32_t w[NW];
        rand_words<NW>(counter, k0, k1, w);
#pragma unroll
        for (int d = 0; d < NW; ++d) quant_floats4(x + 4 * d * es, es, inv, w[d], f + 4 * d);
    }
}

// Four codes as the bytes of a dword, little-endian two's complement (as the int8 MFMA reads them).
__device__ __forceinline__ uint32_t pack_bytes4(const int *q)
{
    // v_perm_b32: selector bytes 0-3 pick bytes of the second operand, 4-7 of the first, 0x0c = zero
    const uint32_t lo = __builtin_amdgcn_perm(static_cast<uint32_t>(q[1]), static_cast<uint32_t>(q[0]), 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(static_cast<uint32_t>(q[3]), static_cast<uint32_t>(q[2]), 0x04000c0cu);
    return lo | hi;
}

// Eight codes as the nibbles of a dword, two's complement, code 2b in the low nibble of byte b and code 2b+1 in the
// high one: each code's low four bits enter at the top of the word and push the earlier ones down, one instruction a
// code (v_alignbit_b32: the low word of {code, word} >> 4).  Bits above the low four never reach a neighbour, so it holds
// for codes outside [-7, 7] too: a row or column whose largest value is below 7 / FLT_MAX (2.06e-38) has an infinite
// reciprocal and saturated codes.
__device__ __forceinline__ uint32_t pack_nibbles8(const int *q)
{
    uint32_t r = static_cast<uint32_t>(q[0]) << 28;
#pragma unroll
    for (int e = 1; e < 8; ++e) r = __builtin_amdgcn_alignbit(static_cast<uint32_t>(q[e]), r, 4);
    return r;
}

// ---- codes for the 6-bit matrix instructions ("f6") -------------------------------------------
// The matrix cores multiply 6-bit floats (e2m3) at twice the rate of bytes.  A code in [-7, 7] divided by 8 is a
// subnormal one: sign in bit 5, |code| in bits 0-2, bits 3 and 4 clear.  So four bits of every six carry anything, and 16
// codes, three dwords of fields, travel in two: the dwords' fields cover the bits F0, F1 and F2 (bit 3 and 4 of a
// field never set), the complements of F0 and F1 are disjoint and fill F2, so the third dword hides in the bits that the
// first two do not use.  It goes in xored with what they have there, which makes getting it out one instruction of three
// operands (v_bitop3_b32): d0 = a & F0, d1 = b & F1, d2 = (a ^ b) & F2 -- three instructions for 16 codes, half of what
// two's complement nibbles take to become bytes (Mma16<2>: 6 for 16).
constexpr uint32_t f6_field_bits(int dword)
{
    uint32_t m = 0;
    for (int b = 0; b < 32; ++b) {
        const int f = (32 * dword + b) % 6;
        if (f != 3 && f != 4) m |= 1u << b;
    }
    return m;
}
constexpr uint32_t F6M0 = f6_field_bits(0), F6M1 = f6_field_bits(1), F6M2 = f6_field_bits(2);
static_assert((~F6M0 & ~F6M1) == 0 && (~F6M0 | ~F6M1) == F6M2, "the third dword fits where the first two have no field bits");

// 32 codes as floats (integers in [-7, 7]) -> 16 bytes.  The conversion takes its two halves in turns, so a row's codes
// lie in the order 0, 16, 1, 17, ...: every row of both operands of a product is packed by this function.
// Codes that are none (a reciprocal scale that is infinite, sums that are not numbers) set one of the bits 3 and 4; they
// are then taken as the low four bits, two's complement, of what the conversion to an integer gives, as pack_nibbles8
// takes them (0 and -1 where the scale's reciprocal is infinite).  The layout has no place for -8, which no quantiser here
// makes: handed over as a weight's code, which hlq.h excludes, it comes out as 0.
typedef float v16f_t __attribute__((ext_vector_type(16)));
typedef unsigned int v6u_t __attribute__((ext_vector_type(6)));
__device__ __forceinline__ v6u_t f6_convert(const float *f)
{
    v16f_t lo, hi;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        lo[e] = f[e];
        hi[e] = f[16 + e];
    }
    return __builtin_bit_cast(v6u_t, __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(lo, hi, 8.0f));
}
__device__ __forceinline__ uint4 f6_pack32(float *f)
{
    v6u_t d = f6_convert(f);
    const uint32_t stray = (d[0] & ~F6M0) | (d[1] & ~F6M1) | (d[2] & ~F6M2) | (d[3] & ~F6M0) | (d[4] & ~F6M1) | (d[5] & ~F6M2);
    if (stray != 0) {
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const int q = floor_to_int(f[e]);
            f[e] = static_cast<float>(static_cast<int>(static_cast<uint32_t>(q) << 28) >> 28);
        }
        d = f6_convert(f);
    }
    const uint32_t x0 = d[1] ^ d[2], x1 = d[0] ^ d[2], x2 = d[4] ^ d[5], x3 = d[3] ^ d[5];
    return make_uint4((d[0] & F6M0) | (x0 & ~F6M0), (d[1] & F6M1) | (x1 & ~F6M1), (d[3] & F6M0) | (x2 & ~F6M0),
                      (d[4] & F6M1) | (x3 & ~F6M1));
}

// Maxima of a lane's CPL columns (bit patterns of non-negative floats): one row of D of them, or `table` rows to be
// folded, which the 256 threads of the workgroup do together for its 128 columns.  Every thread calls it; `sub` is the
// lane's place among those that cover the 128 columns.
template <int CPL>
__device__ __forceinline__ void fold_column_maxima(const uint32_t *__restrict__ bits, int D, int table, int bx, int sub, float *a)
{
    const float *m = reinterpret_cast<const float *>(bits);
    if (table <= 1) {
        if (bx * 128 + sub * CPL < D) Loader<float, CPL>::load(m + bx * 128 + sub * CPL, a);
        return;
    }
    __shared__ float s_fold[2][128];
    const int c = threadIdx.x & 127, half = threadIdx.x >> 7, col = bx * 128 + c;
    float f = 0.0f;
    if (col < D)
        for (int t = half; t < table; t += 2) f = fmaxf(f, m[static_cast<int64_t>(t) * D + col]);
    s_fold[half][c] = f;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CPL; ++k) a[k] = fmaxf(s_fold[0][sub * CPL + k], s_fold[1][sub * CPL + k]);
}

// 4-bit codes two to a byte -> one int8 each: a lane turns 16 bytes into 32 (see k_unpack_nibbles)
__device__ __forceinline__ void unpack_nibbles16(const uint4 *__restrict__ in, uint4 *__restrict__ out)
{
    const uint4 x = *in;
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    uint32_t o[8];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t lo = w[d] & 0x0F0F0F0Fu, hi = (w[d] >> 4) & 0x0F0F0F0Fu;
        // bytes (lo0, hi0, lo1, hi1) and (lo2, hi2, lo3, hi3): v_perm selectors 0-3 = second operand, 4-7 = first
        uint32_t a = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
        uint32_t b = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
        // sign-extend every byte's nibble: a set bit 3 fills the upper half of its byte
        a |= ((a >> 3) & 0x01010101u) * 0xF0u;
        b |= ((b >> 3) & 0x01010101u) * 0xF0u;
        o[2 * d] = a;
        o[2 * d + 1] = b;
    }
    out[0] = make_uint4(o[0], o[1], o[2], o[3]);
    out[1] = make_uint4(o[4], o[5], o[6], o[7]);
}

// qmax = 7 for 4-bit codes, 127 for 8-bit codes (int8 warm-up phase, integer g_w path).
__device__ __forceinline__ float absmax_to_inv(float a, float qmax) { return a > 0.0f ? qmax / a : 0.0f; }
__device__ __forceinline__ float absmax_to_scale(float a, float qmax) { return a / qmax; }

}  // namespace hlq
