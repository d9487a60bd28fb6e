// Device body of K2 / K4 for 256 x 256 (or 192 x 256) tiles and rows of whole 128-byte steps, and for 128 x 128
// tiles and any rows, with the operands
// streamed from global memory straight into LDS and multiplied by 16 x 16 MFMAs (arXiv 2406.15102,
// Sec. 6.1: stages 5-6 of the g_x list, stage 5 of the g_w list; the same products, tile, LDS layout
// and bits as gemm_body.hpp).
//
// In gemm_body.hpp an operand chunk travels global -> registers -> LDS.  The ds_write that moves it
// on reads 1 KB of registers per wavefront and holds up the MFMA stream, and the round trip through
// the register file costs power -- which on this chip, power-limited on matrix work, is clock.
// `buffer_load ... lds` delivers the chunks into LDS without touching the register file.  What it
// takes to make that pay (measured on MI355X with the rocprofv3 counters SQ_VMEM_TA_ADDR_FIFO_FULL,
// SQ_INST_LEVEL_VMEM, GRBM_GUI_ACTIVE):
//   * a load instruction of a wavefront fetches whole 128-byte lines (8 rows x 128 B) -- with 64-byte
//     steps every line is asked for twice and a load takes 1.7 x as long to land;
//   * loads go out singly between the MFMAs, never in a burst from all four wavefronts (the address
//     queues of the memory pipeline fill up and the wavefront stalls at issue);
//   * LDS is a ring of five units (2 AHEAD + 1), 32 KB each for a 256-tile -- all 160 KB.  Step kt keeps its A rows in unit 2 kt mod 5 and
//     its Bm rows in the next one, so while step kt is multiplied step kt + 1 is complete or landing
//     in two more units and the fifth takes the A rows of step kt + 2 already: a load has between
//     0.75 and 1.5 steps to land, about what the register-staged pipeline gives it.
// One barrier per step, before its last sub-step: by then every wavefront has waited for its own
// loads of step kt + 1, and nobody reads step kt from LDS any more (the fragments of the last
// sub-step are in registers), which frees that step's two units for the Bm rows of step kt + 2 and,
// one step later, the A rows of step kt + 3.
//
// MFMA shape: 16 x 16 x 32 (bf16) / 16 x 16 x 64 (int8), 8 x 8 accumulators of four registers per
// wavefront.  A register-resident probe sustains 5-10 % more on these shapes than on the 32 x 32 ones
// at the chip's power limit, and this loop built around them measured 8 % (long reductions) to 4 %
// faster than the same loop on 32 x 32 MFMAs, with the same bits.  Both operands of an MFMA are read as
// 16 rows x 64 B (lane -> row lane % 16, 16-byte chunk lane / 16), one ds_read_b128 each; packed 4-bit
// codes are read as 16 rows x 32 B (8 bytes a lane) and widened to one such operand in registers.
//
// A second tile shape, 192 rows x 256 columns (6 x 8 accumulators per wavefront, three quarters of the
// work), serves the last rows of a product whose 256-row tiles would leave most compute units idle in
// their last round: 11008 x 4096 is 688 tiles of 256 x 256, 2.69 rounds on 256 compute units; with the
// last 2816 rows in 192-row tiles it is 512 + 240 tiles, two rounds and one of three-quarter tiles.
//
// A third, 128 x 128 (4 x 4 accumulators per wavefront, ring units of 16 KB: 80 KB, two workgroups to a compute unit),
// serves the pairs of products whose 256-tiles would not fill the chip.  A step reads 64 KB of fragments, 512 cycles of
// LDS, for 8 x 8 x 2 MFMAs a tile, 512 cycles of every SIMD, and takes 32 KB in, so LDS bounds it, and what it saves over
// the register-staged body is that 32 KB passing through registers: 32 MFMAs a step and wavefront hide fewer cycles
// than 128, hence the second workgroup.  The launch of both products, register-staged -> this, whole passes on changing
// inputs: 4096 x 2048 x 5632 in fp32 92.1 -> 84.1 us; products called alone: 8192 x 2048 x 2048 72.4 -> 69.1, 4096 x 1024 x
// 4096 29.4 -> 26.6, 2048 x 2048 x 2048 21.3 -> 20.0; gemm_dl128_ok says where it is taken.
// Beside 256-tiles of the other product, whose LDS leaves it a compute unit to itself, its ring is nine units (AHEAD = 4): a load
// has 2.75 to 3.5 steps to land instead of 0.75 to 1.5, which one wavefront a SIMD and 32 MFMAs a step do not cover.  Whole passes
// with that pair of tiles, register-staged -> this: 9200 x 1160 x 3120 117.6 -> 113.2 us, 12608 x 768 x 3072 104.4 -> 102.6.
// 4-bit codes in the f6 layout (KIND 3; hlq_device.hpp says how it widens) are 6-bit floats to the matrix cores, 128 of k
// to an MFMA of the cycles that 64 bytes take.  Registers alone sustain 5.9 POP/s on such floats (hlq_mfma_probe, kind 3) and 4.5 on
// the bytes that nibbles widen to (kind 9), at the power limit in either case.  A step is that of bytes: 16 rows x 64 B
// and one ds_read_b128 a fragment, where nibbles are read 8 bytes a lane with two-way conflicts.  The product alone,
// nibbles -> f6: 4096 x 4096 x 11008 112.5 -> 80.8 us (4.6 POP/s), 8192 x 28672 x 8192 1168 -> 828.  The launch of both products
// at 4096 x 4096 x 11008: MFMAs busy 61 % of its cycles at 1.96 GHz (nibbles 68 % at 2.10; profiles/hlq_c4_products_f6_pmc.txt), so
// it is power here too, and an MFMA's share of the widening (1.5 instructions) and of LDS reads weighs double beside half the MFMAs.
// RAGGED (128 x 128 only): the last step of a row need not be whole.  It is multiplied behind the loop, chunks past
// the end of a row cleared in registers, so the loop of whole steps carries one subtraction a load for it.
#pragma once
#include "gemm_common.hpp"

namespace hlq {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr size_t kGemmDlLdsBytes = 5u * 256u * 128u;   // the ring; the epilogue's slabs reuse its start
constexpr size_t kGemmDl128LdsBytes = 5u * 128u * 128u;   // of a 128 x 128 tile: two to a compute unit
constexpr int kGemmDlDeep = 4;                            // steps ahead of a 128 x 128 tile that has its compute unit to itself
constexpr size_t kGemmDl128DeepLdsBytes = (2u * kGemmDlDeep + 1u) * 128u * 128u;

// 16 x 16 MFMAs.  The MFMA's A operand is fed from Bm and its B operand from A, which leaves a lane with
// C[m][n .. n + 3], m = 16 i + lane % 16, n = 16 j + 4 (lane / 16), of accumulator (i, j).
// Written out as instructions with the accumulator tied to the destination: through the builtins the
// compiler is free to give an MFMA of this size a destination other than its addend, and with all 256
// accumulator registers in use it then moves dozens of accumulators around at the top of every k step.
// What the compiler's hazard handling no longer sees is kept apart by construction: an accumulator is
// touched by one MFMA in 16 or more, operands written by vector instructions (the widened codes) are written a
// sub-step before they are multiplied (behind s_nops where no sub-step lies between), and the epilogue waits out the last MFMAs before it reads.
template <int KIND> struct Mma16;
template <> struct Mma16<0> {
    typedef v4i acc_t;
    static __device__ __forceinline__ acc_t zero() { return acc_t{0, 0, 0, 0}; }
    static __device__ __forceinline__ void mma(const u32x4 &x, const u32x4 &y, acc_t &c)
    {
        asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
    }
};
template <> struct Mma16<1> {
    typedef v4f_t acc_t;
    static __device__ __forceinline__ acc_t zero() { return acc_t{0.0f, 0.0f, 0.0f, 0.0f}; }
    static __device__ __forceinline__ void mma(const u32x4 &x, const u32x4 &y, acc_t &c)
    {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
    }
};
// packed 4-bit codes: 8 bytes (16 codes) widen to one int8 operand, the even codes in its low half and the
// odd ones in its high half, each moved to the high nibble of its byte (16 x the code, sign included: see
// Mma<2>).  Both operands of a product widen the same way, so which code meets which lane does not matter.
template <> struct Mma16<2> : Mma16<0> {
    // part 0: the odd codes (2 instructions), parts 1, 2: one dword of the even codes each (2 instructions)
    static __device__ __forceinline__ void expand_part(const u32x2 &x, u32x4 &o, int part)
    {
        if (part == 0) {
            o[2] = x[0] & 0xF0F0F0F0u;
            o[3] = x[1] & 0xF0F0F0F0u;
        } else {
            o[part - 1] = (x[part - 1] << 4) & 0xF0F0F0F0u;
        }
    }
};

// 4-bit codes in the f6 layout (hlq_device.hpp): 16 bytes (32 codes) widen to one operand of six registers
template <> struct Mma16<3> {
    typedef v4f_t acc_t;
    static __device__ __forceinline__ acc_t zero() { return acc_t{0.0f, 0.0f, 0.0f, 0.0f}; }
    static __device__ __forceinline__ void mma(const u32x6 &x, const u32x6 &y, acc_t &c)
    {
        asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0 cbsz:2 blgp:2" : "+a"(c) : "v"(x), "v"(y));
    }
    // dword `part` (0-5) of the operand, one instruction
    static __device__ __forceinline__ void expand_part(const u32x4 &x, u32x6 &o, int part)
    {
        const uint32_t a = x[part < 3 ? 0 : 2], b = x[part < 3 ? 1 : 3];
        if (part % 3 == 0) o[part] = a & F6M0;
        else if (part % 3 == 1) o[part] = b & F6M1;
        else o[part] = (a ^ b) & F6M2;
    }
};

// raw 32-bit accumulators of the 16 x 16 layout (parity export, split-k partials): direct 16-byte stores
template <int KIND, int NBM, int NB, bool GUARD>
__device__ __forceinline__ void store_raw16(typename Mma16<KIND>::acc_t (&acc)[NBM][NB], int32_t *out, int M, int N, int wm0,
                                            int wn0, int lane)
{
    const int fr = lane & 15, fq = lane >> 4;
#pragma unroll
    for (int i = 0; i < NBM; ++i) {
        const int m = wm0 + i * 16 + fr;
        int32_t *row = out + static_cast<int64_t>(m) * N + wn0 + fq * 4;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (!GUARD || ((m < M) & (wn0 + j * 16 + fq * 4 < N))) {
                const auto e0 = acc[i][j][0], e1 = acc[i][j][1], e2 = acc[i][j][2], e3 = acc[i][j][3];
                v4i raw = {Mma<KIND>::raw(e0), Mma<KIND>::raw(e1), Mma<KIND>::raw(e2), Mma<KIND>::raw(e3)};
                *reinterpret_cast<v4i *>(row + j * 16) = raw;
            }
        }
    }
}

// C = alpha * sA[m] * sB[n] * acc for the 16 x 16 layout, the arithmetic of store_scaled value for value;
// staged per 16-row group through LDS so that global stores are 16-byte, row-contiguous pieces.
template <int KIND, int NBM, int NB, bool F32, bool GUARD>
__device__ __forceinline__ void store_scaled16(typename Mma16<KIND>::acc_t (&acc)[NBM][NB], void *Cout, int M, int N,
                                               const float *sA, const float *sB, float alpha, int wm0, int wn0, int lane,
                                               char *slab)
{
    constexpr int PITCH = 16 * NB * (F32 ? 4 : 2) + 16;
    constexpr int EPL = F32 ? 4 : 8;       // elements per 16-byte piece
    constexpr int LPR = 16 * NB / EPL;         // lanes per row
    constexpr int RPI = 64 / LPR;          // rows per store instruction
    const int fr = lane & 15, fq = lane >> 4;
    f32x4 cs[NB];
    if (KIND == 1) {
        // unused
    } else if (sB) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            int n = wn0 + j * 16 + fq * 4;
            if (GUARD) n = n < N ? n : 0;
            cs[j] = *reinterpret_cast<const f32x4 *>(sB + n) * alpha;
        }
    } else {
#pragma unroll
        for (int j = 0; j < NB; ++j) cs[j] = f32x4{alpha, alpha, alpha, alpha};
    }
    float sa[NBM];
#pragma unroll
    for (int i = 0; i < NBM; ++i) {
        int m = wm0 + i * 16 + fr;
        if (GUARD) m = m < M ? m : 0;
        sa[i] = sA ? sA[m] : 1.0f;
    }
    const int rr0 = lane / LPR, cc = (lane % LPR) * EPL;
    char *wr = slab + fr * PITCH + fq * 4 * (F32 ? 4 : 2);
    const char *rd = slab + rr0 * PITCH + cc * (F32 ? 4 : 2);
#pragma unroll
    for (int i = 0; i < NBM; ++i) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (KIND == 1) o[e] = Mma<KIND>::to_float(acc[i][j][e]) * alpha;   // no scales on the bf16 product
                else o[e] = Mma<KIND>::to_float(acc[i][j][e]) * (sa[i] * cs[j][e]);
            }
            if (F32) {
                *reinterpret_cast<f32x4 *>(wr + (j * 16) * 4) = o;
            } else {
                u32x2 p = {pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
                *reinterpret_cast<u32x2 *>(wr + (j * 16) * 2) = p;
            }
        }
        lds_wave_fence();
        u32x4 v[16 / RPI];
#pragma unroll
        for (int p = 0; p < 16 / RPI; ++p) v[p] = *reinterpret_cast<const u32x4 *>(rd + p * RPI * PITCH);
        const int mbase = wm0 + i * 16 + rr0;
        char *dst = static_cast<char *>(Cout) + (static_cast<int64_t>(mbase) * N + wn0 + cc) * (F32 ? 4 : 2);
        const int64_t step = static_cast<int64_t>(RPI) * N * (F32 ? 4 : 2);
#pragma unroll
        for (int p = 0; p < 16 / RPI; ++p) {
            if (!GUARD) {
                *reinterpret_cast<u32x4 *>(dst + p * step) = v[p];
            } else {
                // one guard a store, row and column in one test: see -amdgpu-remove-redundant-endcf in build.py
                const int m = mbase + p * RPI, n = wn0 + cc;
                if (F32 || (N & 7) == 0) {
                    if ((m < M) & (n < N)) *reinterpret_cast<u32x4 *>(dst + p * step) = v[p];
                } else {   // bf16 rows that are only 8-byte aligned: two halves, the last may be missing
                    const u32x2 lo = {v[p][0], v[p][1]}, hi = {v[p][2], v[p][3]};
                    if ((m < M) & (n < N)) *reinterpret_cast<u32x2 *>(dst + p * step) = lo;
                    if ((m < M) & (n + 4 < N)) *reinterpret_cast<u32x2 *>(dst + p * step + 8) = hi;
                }
            }
        }
        lds_wave_fence();
    }
}

// OUT as in gemm_tile; `bid`: index of the workgroup among those of this product.
// Requires tiles of 32 NBM rows x 32 NB columns, NBM = 8 or 6 with NB = 8, or both 4 (g.tiles_m, g.tiles_n counted
// in such tiles; the 192-row tile is not written for packed codes), at least one whole step a workgroup, and
// g.Kb % 128 == 0 unless RAGGED (then g.Kb % 16 == 0, and at least two whole steps).  The dispatch hands over reductions of two steps and
// more (gemm_dl_ok, gemm_dl128_pays), but f6 codes any: with one step the prologue and the loop load it again where later ones would be,
// and what they read of it is never multiplied.  Such layers are no slower for it than through registers, where one step skips the
// pipeline (whole passes, nibbles / bytes there -> this: 50176 x 256 over 192 46.2 -> 42.5 us, over 240 52.0 -> 45.1, over 256 49.7 -> 44.7;
// 12544 x 1152 over 224 37.9 -> 37.0, over 256 38.6 -> 38.5; 3136 x 512 over 256 19.7 -> 16.8).
template <int KIND, int NBM, int OUT, int NB = 8, bool RAGGED = false, int AHEAD = 2>
__device__ __forceinline__ void gemm_tile_dl(const GemmDev &g, const int bid)
{
    constexpr int BT = 32 * NB, BTM = 32 * NBM, GROUP = 4;
    constexpr bool PACKED = KIND == 2, F6 = KIND == 3;
    static_assert(!F6 || (!RAGGED && NBM == NB), "f6 rows are whole steps, in square tiles");
    static_assert((NB == 8 && (NBM == 8 || (NBM == 6 && !PACKED)) && !RAGGED) || (NB == 4 && NBM == 4),
                  "tiles of 256 x 256, of 192 x 256 for byte and bf16 operands, or of 128 x 128");
    constexpr int NS = PACKED ? 4 : 2;            // sub-steps per step: 32 B of packed codes, 64 B otherwise
    constexpr int SLOTS = NBM * NB;               // MFMAs of a sub-step, one per accumulator
    constexpr int NR = NBM + NB;                  // fragments of a sub-step
    constexpr uint32_t UNIT = BT * 128u;          // one operand's rows of one step: 32 or 16 KB
    static_assert(AHEAD == 2 || (NB == 4 && !RAGGED), "a longer ring: 128 x 128 tiles of whole steps");
    constexpr int UNITS = 2 * AHEAD + 1;
    constexpr uint32_t RING = UNITS * UNIT;
    extern __shared__ u32x4 lds[];
    char *const ldsb = reinterpret_cast<char *>(lds);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1;

    // ---- workgroup id -> tile, XCD-aware (as in gemm_tile) ----
    int tm, tn;
    {
        const int nb = g.tiles_m * g.tiles_n;
        const int pid = bid % nb;                  // bid / nb is the k split
        const int xcd = pid & 7, idx = pid >> 3;
        const int per = nb >> 3, rem = nb & 7;
        const int logical = xcd * per + (xcd < rem ? xcd : rem) + idx;
        const int width = GROUP * g.tiles_n;
        const int group = logical / width;
        const int first_m = group * GROUP;
        const int gsz = (g.tiles_m - first_m) < GROUP ? (g.tiles_m - first_m) : GROUP;
        const int within = logical - group * width;
        tm = first_m + within % gsz;
        tn = within / gsz;
    }
    const int m0 = tm * BTM, n0 = tn * BT;

    // ---- loads: instruction j of this wavefront fills rows 8 (4 j + wave) .. + 7 of an operand ----
    // (NBM instructions for the A rows, NB for the Bm rows)
    // 1 KB of LDS in lane order: lane -> row lane / 8 of the block, position lane % 8 of the row, which
    // in the swizzled layout (lds_chunk<8>) holds chunk position ^ (row & 7) ^ (row >> 3 & 1) of that
    // row.  Rows past the end of an operand are redirected to the tile's first row (never stored).
    const char *baseA = g.A + static_cast<int64_t>(m0) * g.Kb;
    const char *baseB = g.Bm + static_cast<int64_t>(n0) * g.Kb;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(baseA), 0, 0x7FFFFFFF, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(baseB), 0, 0x7FFFFFFF, 0x00020000);
    uint32_t offa[NBM], offb[NB];
    {
        const int rb = lane >> 3, slot = lane & 7;
        const uint32_t c16 = static_cast<uint32_t>(slot ^ rb ^ (wave & 1)) * 16u;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int row = 8 * (4 * j + wave) + rb;
            if (j < NBM) offa[j < NBM ? j : 0] = static_cast<uint32_t>(m0 + row < g.M ? row : 0) * static_cast<uint32_t>(g.Kb) + c16;
            offb[j] = static_cast<uint32_t>(n0 + row < g.N ? row : 0) * static_cast<uint32_t>(g.Kb) + c16;
        }
    }
    const int nk_all = RAGGED ? (g.Kb + 127) / 128 : g.Kb / 128;
    const int split = bid / (g.tiles_m * g.tiles_n);
    const int kbeg = static_cast<int>(static_cast<int64_t>(nk_all) * split / g.splits);
    // RAGGED: bytes of a last step that is not whole, where this workgroup multiplies it (0: it does not).  The lanes
    // whose chunk lies beyond them load the row's chunk 0 of that step instead; its products are masked out.
    const int rag = RAGGED && split + 1 == g.splits ? g.Kb % 128 : 0;
    const int nk = static_cast<int>(static_cast<int64_t>(nk_all) * (split + 1) / g.splits) - kbeg - (rag ? 1 : 0);   // whole steps
    const int last = nk - (rag ? 0 : 1);
    uint32_t back = 0;
    if (RAGGED) {
        const uint32_t c16 = static_cast<uint32_t>((lane & 7) ^ (lane >> 3) ^ (wave & 1)) * 16u;
        back = rag && c16 >= static_cast<uint32_t>(rag) ? c16 : 0u;
    }

    // instruction J of operand OP (0 = A, 1 = Bm) of step KT into ring unit UNIT_.  Past the end, steps are
    // clamped to the last one: loaded again into a free unit, never multiplied.
#define HLQD_LOAD_ONE(KT, OP, J, UNIT_)                                                                       \
    {                                                                                                         \
        const int kt_ = (KT) < last ? (KT) : last;                                                           \
        const int kuni = (kbeg + kt_) * 128;      /* wave-uniform: lives in an SGPR */                        \
        const uint32_t dst = static_cast<uint32_t>(UNIT_) * UNIT + static_cast<uint32_t>(wave) * 1024u + (J) * 4096u; \
        const uint32_t back_ = RAGGED && kt_ == nk ? back : 0u;                                               \
        if ((OP) == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void_t *)(ldsb + dst), 16, offa[J] - back_, kuni, 0, 0); \
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void_t *)(ldsb + dst), 16, offb[J] - back_, kuni, 0, 0); \
    }

    // ---- fragment reads: one per-lane register per (operand, sub-step), holding the ring position ----
    // lane -> row lane % 16 of a 16-row block; bytes 16 (lane / 16) .. + 15 of the sub-step's 64 B, or, for
    // packed codes, bytes 8 (lane / 16) .. + 7 of its 32 B.  Block i of an operand is 2 KB further.
    const int fr = lane & 15, fq = lane >> 4;
    uint32_t rdA[NS], rdB[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int chunk = PACKED ? 2 * s + (fq >> 1) : 4 * s + fq;
        const uint32_t half = PACKED ? static_cast<uint32_t>(fq & 1) * 8u : 0u;
        rdA[s] = lds_chunk<8>(wave_m * (16 * NBM) + fr, chunk) * 16u + half;
        rdB[s] = UNIT + lds_chunk<8>(wave_n * (16 * NB) + fr, chunk) * 16u + half;
    }
    // the reads of a step are done: the read position of sub-step S2 (A or Bm) moves on two units, mod the ring
#define HLQD_NEXT_UNIT(S2, OP)                                                                                \
    {                                                                                                         \
        uint32_t &r_ = (OP) == 0 ? rdA[S2] : rdB[S2];                                                         \
        const uint32_t a_ = r_ + 2u * UNIT;                                                                   \
        r_ = a_ < a_ - RING ? a_ : a_ - RING;   /* unsigned: a_ - RING wraps when a_ < RING */                \
    }
    // MFMA operands, double-buffered by sub-step: fb[.][j] the Bm blocks, fa[.][i] the A blocks.  For packed
    // codes they hold the widened operands, and pk the 8-byte pieces between their read and their widening.
    u32x4 fa[2][NBM], fb[2][NB];
    u32x2 pk[NR];
    // f6: the widened operands, and the 16-byte pieces before.  At 8 x 8 accumulators a row of A is widened over itself,
    // behind its eight MFMAs: registers for the Bm blocks twice and the A blocks once.
    constexpr int FA = NB == 8 ? 1 : 2;
    u32x6 wa[FA][NBM], wb[2][NB];
    u32x4 pw[NR];
    // fragment Q of sub-step S (0-7: Bm blocks -- the first row of MFMAs takes them all --, 8-15: A blocks)
#define HLQD_READ_ONE(BUF, S, Q)                                                                              \
    {                                                                                                         \
        if constexpr (F6) {                                                                                   \
            if ((Q) < NB) pw[Q] = *reinterpret_cast<const u32x4 *>(ldsb + rdB[S] + (Q) * 2048u);              \
            else pw[Q] = *reinterpret_cast<const u32x4 *>(ldsb + rdA[S] + ((Q) - NB) * 2048u);                \
        } else if constexpr (PACKED) {                                                                        \
            if ((Q) < NB) pk[Q] = *reinterpret_cast<const u32x2 *>(ldsb + rdB[S] + (Q) * 2048u);              \
            else pk[Q] = *reinterpret_cast<const u32x2 *>(ldsb + rdA[S] + ((Q) - NB) * 2048u);                \
        } else {                                                                                              \
            if ((Q) < NB) fb[BUF][Q] = *reinterpret_cast<const u32x4 *>(ldsb + rdB[S] + (Q) * 2048u);         \
            else fa[BUF][(Q) - NB] = *reinterpret_cast<const u32x4 *>(ldsb + rdA[S] + ((Q) - NB) * 2048u);    \
        }                                                                                                     \
    }
    // packed codes: part P (0-2) of the widening of fragment Q into the operands of buffer BUF
#define HLQD_EXPAND(BUF, Q, P)                                                                                \
    {                                                                                                         \
        if ((Q) < NB) Mma16<2>::expand_part(pk[Q], fb[BUF][Q], P);                                            \
        else Mma16<2>::expand_part(pk[Q], fa[BUF][(Q) - NB], P);                                              \
    }

    // f6: dword P (0-5) of fragment Q widened into buffer BUF
#define HLQD_WIDEN(BUF, Q, P)                                                                                 \
    {                                                                                                         \
        if ((Q) < NB) Mma16<3>::expand_part(pw[Q], wb[BUF][(Q) < NB ? (Q) : 0], P);                           \
        else Mma16<3>::expand_part(pw[Q], wa[FA == 2 ? (BUF) : 0][(Q) < NB ? 0 : (Q) - NB], P);               \
    }

    typename Mma16<KIND>::acc_t acc[NBM][NB];
#pragma unroll
    for (int i = 0; i < NBM; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = Mma16<KIND>::zero();

    // prologue: AHEAD steps in flight (steps 0 and 1 in units 0, 1 and 2, 3), wait for step 0
#pragma unroll
    for (int a = 0; a < AHEAD; ++a) {
#pragma unroll
        for (int j = 0; j < NBM; ++j) HLQD_LOAD_ONE(a, 0, j, 2 * a)
#pragma unroll
        for (int j = 0; j < NB; ++j) HLQD_LOAD_ONE(a, 1, j, 2 * a + 1)
    }
    asm volatile("" ::: "memory");
    constexpr int AFTER = (AHEAD - 1) * NR;
    __builtin_amdgcn_s_waitcnt(0x0070 | (AFTER & 15) | ((AFTER >> 4) << 14));   // vmcnt(AFTER): step 0 has landed
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < NR; ++q) HLQD_READ_ONE(0, 0, q)
    if constexpr (F6) {
#pragma unroll
        for (int q = 0; q < NR; ++q)
#pragma unroll
            for (int p = 0; p < 6; ++p) HLQD_WIDEN(0, q, p)
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            asm volatile("" ::"v"(wb[0][q]));       // as below
            asm volatile("" ::"v"(wa[0][q]));
        }
        asm volatile("s_nop 1");
    }
    if constexpr (PACKED) {
#pragma unroll
        for (int q = 0; q < NR; ++q)
#pragma unroll
            for (int p = 0; p < 3; ++p) HLQD_EXPAND(0, q, p)
        // an MFMA may not read a register within two instructions of the vector instruction that wrote it;
        // inside the loop a sub-step lies between the two, here nothing does
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            asm volatile("" ::"v"(fb[0][q]));   // computed before this point ...
            asm volatile("" ::"v"(fa[0][q]));
        }
        asm volatile("s_nop 1");                // ... and two instructions ahead of the first MFMA
    }

    // Step kt reads units u = 2 kt mod UNITS (A) and u + 1 (Bm); step kt + 1 sits in the next two units.  (Below, for AHEAD = 2.)
    // Every sub-step is SLOTS = NBM NB MFMAs -- accumulator (q / NB, q % NB) in slot q -- and reads the NR = NBM + NB
    // fragments of the next sub-step in its even slots, from the first on (packed codes: see below).  The loop is written
    // slot by slot, what is to issue around one MFMA, with a scheduling fence after each slot, so the issue
    // order is the source order.
    //   all but the last sub-step   the A rows of step kt + 2 go into the one free unit, u + 4, evenly spread
    //   last but one                the read positions move on (128 x 128: each in the sub-step that has read from
    //                               it last); its barrier: every wavefront's loads of step kt + 1 have landed (all
    //                               but the NBM youngest have) and nobody reads step kt from LDS any more
    //   last                        fragments of step kt + 1's first sub-step; the Bm rows of step kt + 2
    //                               go into unit u, one load every fourth slot from the first on
    int u = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const int ua = u == 0 ? UNITS - 1 : u - 1;   // (2 kt + 2 AHEAD) mod UNITS
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int cur = s & 1;
            const int ns = s < NS - 1 ? s + 1 : 0;       // the sub-step whose fragments are read now
            if constexpr (F6 && NB == 8) {
                // 64 slots, a slot's share beside its MFMA one and a half of the 96 widening instructions and a quarter of a
                // read.  Bm block j: read in slot 6 j, widened one dword a slot from 6 j + 10 on.  A block j: read in slot
                // 5 j + 3, widened over the block it replaces in the six slots 8 j + 10 .. 8 j + 15, two behind that
                // block's last MFMA -- for j = 7 in the next sub-step's slots 2-7, ahead of its own MFMAs in 56-63.
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) {
                    if (q % 6 == 0 && q < 48) HLQD_READ_ONE(cur ^ 1, ns, q / 6)
                    if (q % 5 == 3 && q < 40) HLQD_READ_ONE(cur ^ 1, ns, NB + q / 5)
                    if (q >= 2 && q < 8) HLQD_WIDEN(0, NB + 7, q - 2)
                    if (q >= 8 && (q & 7) >= 2) HLQD_WIDEN(0, NB + (q >> 3) - 1, (q & 7) - 2)
                    if (q >= 10 && q < 58) HLQD_WIDEN(cur ^ 1, (q - 10) / 6, (q - 10) % 6)
                    if (s == 0 && (q & 7) == 1) HLQD_LOAD_ONE(kt + AHEAD, 0, q >> 3, ua)
                    if (s == 1 && q < 32 && (q & 3) == 1) HLQD_LOAD_ONE(kt + AHEAD, 1, q >> 2, u)
                    if (s == 0 && q >= 58 && q < 62) HLQD_NEXT_UNIT((q - 58) >> 1, q & 1)
                    Mma16<KIND>::mma(wb[cur][q & 7], wa[0][q >> 3], acc[q >> 3][q & 7]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if constexpr (F6) {
                // 16 slots: the 8 fragments in slots 0-3, the 48 dwords of their widening four a slot from slot 4 on (the
                // wavefront of the other workgroup on the SIMD issues beside them)
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) {
                    if (q < 4) {
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q)
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q + 1)
                    }
                    if ((q & 3) == 1) HLQD_LOAD_ONE(kt + AHEAD, s, q >> 2, s == 0 ? ua : u)
                    if (q == 3 || q == 7) HLQD_NEXT_UNIT(s, q == 7)
                    if (q >= 4) {
#pragma unroll
                        for (int e = 4 * (q - 4); e < 4 * (q - 4) + 4; ++e) HLQD_WIDEN(cur ^ 1, e / 6, e % 6)
                    }
                    Mma16<KIND>::mma(wb[cur][q & 3], wa[FA == 2 ? cur : 0][q >> 2], acc[q >> 2][q & 3]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if constexpr (!PACKED) {
                constexpr int APER = SLOTS * (NS - 1) / NBM;   // slots between two loads of A rows
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) {
                    if (q < 2 * NR && !(q & 1)) HLQD_READ_ONE(cur ^ 1, ns, q >> 1)
                    if (s < NS - 1 && (s * SLOTS + q) % APER == APER - 3) HLQD_LOAD_ONE(kt + AHEAD, 0, (s * SLOTS + q) / APER, ua)
                    if (s == NS - 1 && q < 4 * NB && (q & 3) == 1) HLQD_LOAD_ONE(kt + AHEAD, 1, q >> 2, u)
                    if constexpr (NB == 8) {
                        if (s == NS - 2 && q >= 4 * NB && q < 4 * NB + 2 * NS) HLQD_NEXT_UNIT((q - 4 * NB) >> 1, q & 1)
                    } else {
                        // 16 slots: each position in the sub-step behind the one that read from it
                        if (q == 3 || q == 7) HLQD_NEXT_UNIT(s, q == 7)
                    }
                    Mma16<KIND>::mma(fb[cur][q % NB], fa[cur][q / NB], acc[q / NB][q % NB]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if constexpr (NB == 4) {
                // packed codes, 16 slots: the 8 fragments in slots 0-3, the 24 parts of their widening in slots 6-15
                // (three instructions a MFMA; the wavefront of the other workgroup on the SIMD issues beside them)
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) {
                    if (q < 4) {
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q)
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q + 1)
                    }
                    if (s == 0 && (q == 4 || q == 11)) HLQD_LOAD_ONE(kt + AHEAD, 0, q == 11, ua)
                    if ((s == 1 || s == 2) && q == 4) HLQD_LOAD_ONE(kt + AHEAD, 0, s + 1, ua)
                    if (s == 3 && (q & 3) == 1) HLQD_LOAD_ONE(kt + AHEAD, 1, q >> 2, u)
                    if (s < 3 && (q == 5 || q == 12)) HLQD_NEXT_UNIT(ns, q == 12)
                    if (s == 0 && (q == 13 || q == 14)) HLQD_NEXT_UNIT(0, q == 14)
                    if (q >= 6) {
                        const int e0 = q < 10 ? 3 * (q - 6) : 12 + 2 * (q - 10), ne = q < 10 ? 3 : 2;
#pragma unroll
                        for (int e = e0; e < e0 + ne; ++e) HLQD_EXPAND(cur ^ 1, e / 3, e % 3)
                    }
                    Mma16<KIND>::mma(fb[cur][q % NB], fa[cur][q / NB], acc[q / NB][q % NB]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // packed codes: a slot has room for the MFMA and 12 more cycles of issue -- two fragment reads,
                // or one part of a widening (two instructions), or a load.  Slots 0-7 read the 16 fragments,
                // slots 12, 18, ..., 54 are kept for the loads (three of the A rows in sub-steps 0 and 1, two in
                // sub-step 2, the eight of the Bm rows in sub-step 3; read positions move on in those that stay
                // free: the one just used, and in sub-step 0 also the one that sub-step 3 will use), and the 48
                // parts of the widening take the other slots from 8 on.
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) {
                    const bool lslot = q >= 12 && q <= 54 && (q - 12) % 6 == 0;
                    const int li = (q - 12) / 6;                       // which of the eight load slots
                    if (q < NB) {
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q)
                        HLQD_READ_ONE(cur ^ 1, ns, 2 * q + 1)
                    }
                    if (lslot) {
                        if (s < 2 && li % 3 == 1) HLQD_LOAD_ONE(kt + AHEAD, 0, 3 * s + li / 3, ua)
                        if (s == 2 && (li == 1 || li == 4)) HLQD_LOAD_ONE(kt + AHEAD, 0, 6 + li / 3, ua)
                        if (s == 3) HLQD_LOAD_ONE(kt + AHEAD, 1, li, u)
                        if (s < 3 && (li == 3 || li == 6)) HLQD_NEXT_UNIT(ns, li == 6)
                        if (s == 0 && (li == 0 || li == 2)) HLQD_NEXT_UNIT(0, li == 2)
                    }
                    if (q >= 8 && !lslot) {
                        const int e = q - 8 - (q > 12 ? (q < 54 ? (q - 12 + 5) / 6 : 8) : 0);   // rank among the widening slots
                        HLQD_EXPAND(cur ^ 1, e / 3, e % 3)
                    }
                    Mma16<KIND>::mma(fb[cur][q % NB], fa[cur][q / NB], acc[q / NB][q % NB]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (s == NS - 2) {
                asm volatile("" ::: "memory");   // no memory access of the program may cross the barrier
                // vmcnt: all but the A rows of step kt + AHEAD and what is between (step kt + 2 up to it); lgkmcnt(0)
                constexpr int YOUNG = (AHEAD - 2) * NR + NBM;
                __builtin_amdgcn_s_waitcnt(0x0070 | (YOUNG & 15) | ((YOUNG >> 4) << 14));
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        u = u + 2 >= UNITS ? u + 2 - UNITS : u + 2;
    }
    if constexpr (RAGGED) {
        // the sub-steps of the ragged step, with what lies past the end of a row cleared in either operand (not in one
        // alone: infinities).  It landed before the last barrier, and its first fragments have been read.
        constexpr int SUB = 128 / NS;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (s * SUB < rag) {
                if (s > 0) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) HLQD_READ_ONE(0, s, q)
                    if constexpr (PACKED) {
#pragma unroll
                        for (int q = 0; q < NR; ++q)
#pragma unroll
                            for (int p = 0; p < 3; ++p) HLQD_EXPAND(0, q, p)
                    }
                }
                const bool in = s * SUB + fq * (SUB / 4) < rag;
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    u32x4 &x = q < NB ? fb[0][q < NB ? q : 0] : fa[0][q < NB ? 0 : q - NB];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] = in ? x[e] : 0u;
                }
#pragma unroll
                for (int q = 0; q < NR; ++q) {
                    u32x4 &x = q < NB ? fb[0][q < NB ? q : 0] : fa[0][q < NB ? 0 : q - NB];
                    asm volatile("s_nop 1" : "+v"(x));      // computed two instructions ahead of the MFMAs
                }
#pragma unroll
                for (int q = 0; q < SLOTS; ++q) Mma16<KIND>::mma(fb[0][q % NB], fa[0][q / NB], acc[q / NB][q % NB]);
                asm volatile("s_nop 15");                   // and read by them before they are written again
            }
        }
    }
#undef HLQD_LOAD_ONE
#undef HLQD_READ_ONE
#undef HLQD_NEXT_UNIT
#undef HLQD_EXPAND
#undef HLQD_WIDEN

    // ---- epilogue ----
    // the last MFMAs have written their accumulators (the compiler does not know that the statements
    // above are MFMAs and would not keep the reads below far enough from them by itself)
    asm volatile("s_nop 15\n\ts_nop 15");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // every load has landed: LDS is free for staging C
    __syncthreads();
    const int wm0 = m0 + wave_m * (16 * NBM), wn0 = n0 + wave_n * (16 * NB);
    char *slab = ldsb + wave * (16 * (128 * 4 + 16));   // wavefront-private, one 16-row group
    const bool interior = (m0 + BTM <= g.M) && (n0 + BT <= g.N) && ((g.N & 7) == 0);
    if (OUT == 2) {
        if (interior) store_raw16<KIND, NBM, NB, false>(acc, g.acc, g.M, g.N, wm0, wn0, lane);
        else store_raw16<KIND, NBM, NB, true>(acc, g.acc, g.M, g.N, wm0, wn0, lane);
    } else if (OUT == 3) {
        int32_t *part = g.partial + static_cast<int64_t>(split) * g.M * g.N;
        if (interior) store_raw16<KIND, NBM, NB, false>(acc, part, g.M, g.N, wm0, wn0, lane);
        else store_raw16<KIND, NBM, NB, true>(acc, part, g.M, g.N, wm0, wn0, lane);
    } else {
        if (interior) store_scaled16<KIND, NBM, NB, OUT == 1, false>(acc, g.C, g.M, g.N, g.sA, g.sB, g.alpha, wm0, wn0, lane, slab);
        else store_scaled16<KIND, NBM, NB, OUT == 1, true>(acc, g.C, g.M, g.N, g.sA, g.sB, g.alpha, wm0, wn0, lane, slab);
    }
}

}  // namespace hlq
