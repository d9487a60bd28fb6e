// Device body of the image gradient of a convolution (arXiv 2406.15102, Sec. 3.1 and stages 5-6 of the g_x list in
// Sec. 6.1): the product of the codes, its dequantisation and the fold onto the image in one pass, so that
// the column gradient [N, kh*kw*C] is never stored.
//   dX[pixel, c] = sum over the taps whose output position n read this pixel of
//                  1/B * sG[n] * sW[tap, c] * sum_o Gq[n, o] Wq[(tap, c), o]
// The scales differ from tap to tap, so each tap's integer sum is exact in the matrix cores and is scaled and added in fp32,
// taps in ascending (ky, kx) order.  Every entry is first rounded to the type the column gradient would be held in, so
// that the image gradient is, bit for bit, the fold of that tensor.
//
// What it replaces, the product with its column gradient and then the fold, was bound by that tensor: 160 MB written
// and read for an image of 18 MB at 65536 x 1224 over 32 out-features, 70 + 32 us of a pass of 144 (87 now); 12544 x
// 2304 over 256, both products and the fold 33.4 + 11.5 us of a pass of 63.8, now 26.9 of 45.1.
//
// Tile: WM x WN wavefronts of 16 FM pixels x 16 FN channels, 16 x 16 MFMAs.  Rows of codes go straight into LDS, RB bytes
// of each at a time (an item: one tap, or RB bytes of its reduction), two items ahead of the one that is
// multiplied (one, of the largest).  Fragments loaded straight into registers were slower (12544 pixels x 256 channels
// over 256 33 us against 23, the sum without the rounding in both): four adjacent lanes of an MFMA operand are
// four different rows, so that each load is 64 requests of 16 bytes.
// Codes are one int8 each here: 4-bit codes two to a byte would be widened by twelve vector instructions per 128 codes of
// a row, on top of the five and a half per value and tap in bf16 (four in fp32) that conversion, the two scales, the
// rounding and the sum are.  What bounds the kernel is the chain of a tile's items, each a barrier, LDS reads, MFMAs and, at the
// end of a tap, those sums one after the other, with two workgroups a compute unit at most to fill the gaps: at 12544 pixels x 256 channels over
// 256 codes (392 tiles of 18 items, about 0.7 us each where two share a unit) vector instructions issue for 34 % of the launch,
// LDS is active for 20 %, the MFMAs for 12 %, and a wavefront waits 38 % of its time.
// A stride splits the pixels into sh * sw classes (their coordinates mod the stride) that are met by different
// taps; a tile belongs to one class, so no MFMA is spent on a tap that its pixels do not have.
#pragma once
#include "gemm_dl_body.hpp"

namespace hlq {

struct ConvDx {
    const char *Gq;        // [N, Kb] codes, one int8 each, of the output gradient
    const float *sG;       // [N]
    const char *Wq;        // [kh*kw*C, Kb] codes of the weight
    const float *sW;       // [kh*kw*C]
    void *dX;              // [Nb, H, W, C]
    float alpha;           // 1/B
    ConvShape s;
    int Kb;                // codes per row, a multiple of 16
    int stepy, stepx;      // distance between the taps of one class
    int tiles_px;          // pixel tiles per class
    int tiles_c;           // channel tiles
    int form;              // the tile's shape, see conv_dx_any
};

typedef long i64x1;
template <int I> struct Const { static constexpr int value = I; };

// The MFMA operands in one fragment of 16 rows x RB bytes: RB / 4 bytes per lane (lane -> row lane % 16).
template <int RB> struct ConvMma;
template <> struct ConvMma<32> {
    typedef u32x2 op_t;
    static __device__ __forceinline__ v4i mma(const op_t &a, const op_t &b, v4i c)
    {
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(i64x1, a), __builtin_bit_cast(i64x1, b), c, 0, 0, 0);
    }
};
template <> struct ConvMma<64> {
    typedef u32x4 op_t;
    static __device__ __forceinline__ v4i mma(const op_t &a, const op_t &b, v4i c)
    {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, a), __builtin_bit_cast(v4i, b), c, 0, 0, 0);
    }
};

// LDS of a tile: stages of (rows of G, rows of W, a scale per pixel), then the column scales of every tap.
// Three stages, loads two items ahead; two of the largest, whose item takes as long as a load.
constexpr int conv_dx_bm(int form) { return form == 1 ? 256 : (form == 3 ? 64 : 128); }
constexpr int conv_dx_bn(int form) { return form == 0 ? 128 : 64; }
constexpr int conv_dx_stages(int RB) { return RB == 128 ? 2 : 3; }
constexpr int conv_dx_rb(int form, int Kb) { return Kb > 64 && form != 1 ? 128 : (Kb > 32 ? 64 : 32); }
constexpr int kConvMaxTaps = 64, kConvDxMaxLds = 160 * 1024;
constexpr size_t conv_dx_lds(int form, int Kb, int taps)
{
    const int RB = conv_dx_rb(form, Kb);
    return static_cast<size_t>(conv_dx_stages(RB)) * (conv_dx_bm(form) * (RB + 4) + conv_dx_bn(form) * RB) +
           static_cast<size_t>(taps) * conv_dx_bn(form) * 4;
}

// One value of the image gradient that came out as no number, `v`: taken again by the definition where a tap that the pixel
// does not have is in a column whose scale is not finite, else as it is.  `g`: the kernel's first argument, read from where
// the launch put it, so that what only this needs is not in registers through the kernel's loop.  (Infinite gradients or weights throughout: 164 and 595 us
// at 12544 pixels x 256 channels over 256, 50 with finite ones; all NaN sums taken again 4000.)
typedef const __attribute__((address_space(4))) ConvDx ConvDxArg;
template <bool F32>
__device__ __forceinline__ float conv_dx_again(const ConvDxArg &g, int n, int h, int w, int c, float v)
{
    const auto &s = g.s;
    const int taps = s.kh * s.kw;
    auto position = [&](int tap) {                                  // the output position that read this pixel, or -1
        const int ky = tap / s.kw, kx = tap - ky * s.kw;
        const int hn = h + s.ph - ky * s.dh, ho = hn / s.sh, wn = w + s.pw - kx * s.dw, wo = wn / s.sw;
        const bool met = hn >= 0 && ho * s.sh == hn && ho < s.Ho && wn >= 0 && wo * s.sw == wn && wo < s.Wo;
        return met ? (static_cast<int64_t>(n) * s.Ho + ho) * s.Wo + wo : int64_t(-1);
    };
    bool due = false;
    for (int tap = 0; tap < taps; ++tap)                            // (scales are not negative)
        due = due || (position(tap) < 0 && __float_as_uint(g.sW[static_cast<int64_t>(tap) * s.C + c]) >= 0x7F800000u);
    if (!due) return v;
    v = 0.0f;
    for (int tap = 0; tap < taps && v == v; ++tap) {
        const int64_t row = position(tap), col = static_cast<int64_t>(tap) * s.C + c;
        if (row < 0) continue;
        const int *a = reinterpret_cast<const int *>(g.Gq + row * g.Kb), *b = reinterpret_cast<const int *>(g.Wq + col * g.Kb);
        int acc = 0;
        for (int k = 0; k < g.Kb / 4; ++k) acc = __builtin_amdgcn_sdot4(a[k], b[k], acc, false);
        float o = static_cast<float>(acc) * (g.sG[row] * (g.sW[col] * g.alpha));
        if (!F32) o = bf16_lo(pack_bf16(o, 0.0f));
        v += o;
    }
    return v;
}

// `bid` of tiles_c * tiles_px * sh * sw workgroups
template <int RB, int WM, int WN, int FM, int FN, bool F32>
__device__ __forceinline__ void conv_dx_tile(const ConvDx &g, int bid)
{
    constexpr int BM = WM * 16 * FM, BN = WN * 16 * FN;
    static_assert(WM * WN == 4, "four wavefronts");
    constexpr int HALF = RB == 128 ? 64 : RB, NH = RB / HALF;   // bytes of a row that one MFMA takes
    typedef ConvMma<HALF> Mm;
    typedef typename Mm::op_t op_t;
    constexpr int NST = conv_dx_stages(RB);
    constexpr int RPI = 1024 / RB;                       // rows one load instruction of a wavefront fetches
    constexpr int NA = BM / RPI, NB = BN / RPI;          // load instructions per item
    constexpr int PA = NA >= 4 ? NA / 4 : 1, PB = NB >= 4 ? NB / 4 : 1;   // ... of one wavefront (fewer than four: some twice)
    static_assert(NA >= 1 && NB >= 1 && (NA < 4 || NA % 4 == 0) && (NB < 4 || NB % 4 == 0), "whole load instructions");
    constexpr int NLOAD = PA + PB + 1;
    constexpr uint32_t STAGE = BM * (RB + 4) + BN * RB, WOFS = BM * RB, SOFS = (BM + BN) * RB;
    extern __shared__ u32x4 lds[];
    char *const ldsb = reinterpret_cast<char *>(lds);
    float *const cols = reinterpret_cast<float *>(ldsb + NST * STAGE);
    const ConvShape &s = g.s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave / WN, wave_n = wave % WN;
    const int l16 = lane & 15, g4 = lane >> 4;

    // ---- workgroup -> (class, pixel tile, channel tile): consecutive ones, which share rows of codes, on one XCD ----
    int hs, ws, tile, c0;
    {
        const int classes = s.sh * s.sw, nb = g.tiles_c * g.tiles_px * classes;
        const int xcd = bid & 7, per = nb >> 3, rem = nb & 7;
        const int logical = xcd * per + (xcd < rem ? xcd : rem) + (bid >> 3);
        const int px = logical / g.tiles_c;
        c0 = (logical - px * g.tiles_c) * BN;
        const int cls = px / g.tiles_px;
        tile = px - cls * g.tiles_px;
        hs = cls / s.sw;
        ws = cls - hs * s.sw;
    }
    const int Hc = hs < s.H ? (s.H - hs + s.sh - 1) / s.sh : 0, Wc = ws < s.W ? (s.W - ws + s.sw - 1) / s.sw : 0;
    const int Mc = s.Nb * Hc * Wc;                  // pixels of this class (below 2^31: conv_dx_ok)
    const int m0 = tile * BM;
    if (m0 >= Mc) return;                           // the classes differ in size; the whole workgroup leaves
    struct Pixel { int n, h, w; };                  // image, coordinates within the class
    auto pixel = [&](int q) {
        const uint32_t t = static_cast<uint32_t>(q) / static_cast<uint32_t>(Wc), n = t / static_cast<uint32_t>(Hc);
        return Pixel{static_cast<int>(n), static_cast<int>(t - n * Hc), static_cast<int>(q - t * Wc)};
    };

    // the taps of this class: ky = kyf, kyf + stepy, ... with ky * dh = hs + ph (mod sh), kx alike
    int kyf = 0, kxf = 0;
    while (kyf < g.stepy && (hs + s.ph - kyf * s.dh) % s.sh != 0) ++kyf;
    while (kxf < g.stepx && (ws + s.pw - kxf * s.dw) % s.sw != 0) ++kxf;
    const int nky = (kyf < g.stepy && kyf < s.kh) ? (s.kh - kyf + g.stepy - 1) / g.stepy : 0;
    const int nkx = (kxf < g.stepx && kxf < s.kw) ? (s.kw - kxf + g.stepx - 1) / g.stepx : 0;
    const int nch = (g.Kb + RB - 1) / RB;
    const int items = nky * nkx * nch;

    // ---- loads: a lane fetches 16 bytes of row lane / (RB / 16) of its instruction's rows.  Rows of 64 and 128
    // bytes are kept with their pieces exchanged (piece p of row r in place p ^ swz(r)), so that the 16 lanes of a
    // fragment read that share a piece fall on all banks.  Tails of rows, pixels past the end and taps that a pixel does not have
    // come as zeros, codes and scale: bit 31 puts the offset out of the resource's range (sizes are below 2^31: conv_dx_ok).
    constexpr int PPR = RB / 16;                    // pieces per row
    auto swz = [](int row) { return RB == 128 ? (row & 7) ^ ((row >> 3) & 1) : (RB == 64 ? (row >> 2) & 3 : 0); };
    const int taps = s.kh * s.kw;
    const int lrow = lane / PPR;
    const __amdgpu_buffer_rsrc_t rsG = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(g.Gq), 0,
                                                                       static_cast<int>(s.N * g.Kb), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsS = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.sG), 0, static_cast<int>(s.N * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(g.Wq), 0, taps * s.C * g.Kb, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsC = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g.sW), 0, taps * s.C * 4, 0x00020000);
    for (int i = wave; i < taps * (BN / 64); i += 4) {     // column scales of 64 channels of a tap at a time
        const int c = c0 + i % (BN / 64) * 64 + lane;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsC, (lds_void_t *)(cols + i * 64), 4, c < s.C ? c * 4u : 0x80000000u, i / (BN / 64) * s.C * 4, 0, 0);
    }
    int hq[PA + 1], wq[PA + 1];
    uint32_t offg[PA + 1], offw[PB];                // [PA]: the scales
    int pieceg[PA], piecew[PB];
#pragma unroll
    for (int i = 0; i <= PA; ++i) {
        const int r = i < PA ? ((wave + 4 * i) % NA) * RPI + lrow : (wave * 64) % BM + lane;
        const int piece = (lane % PPR) ^ swz(((wave + 4 * i) % NA) * RPI + lrow);
        const int q = m0 + r;
        const Pixel p = pixel(q < Mc ? q : 0);
        hq[i] = q < Mc ? p.h : -(1 << 30);          // no tap meets a pixel past the end
        wq[i] = p.w;
        const uint32_t n = static_cast<uint32_t>((p.n * s.Ho + p.h) * s.Wo + p.w);
        offg[i] = i < PA ? n * static_cast<uint32_t>(g.Kb) + piece * 16u : n * 4u;
        if (i < PA) pieceg[i] = piece * 16;
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        const int c = c0 + ((wave + 4 * i) % NB) * RPI + lrow;
        piecew[i] = ((lane % PPR) ^ swz(((wave + 4 * i) % NB) * RPI + lrow)) * 16;
        offw[i] = static_cast<uint32_t>(c < s.C ? c : s.C - 1) * static_cast<uint32_t>(g.Kb) + piecew[i];
    }

    // An item is RB bytes of every row, of one tap.  (dy, dx): from a pixel's coordinates in its
    // class to the output position the tap pairs it with; the divisions below are exact.
    struct Item { int ky, kx, ch, dy, dx; };
    const int step_dy = g.stepy * s.dh / s.sh, step_dx = g.stepx * s.dw / s.sw;
    const int dx0 = (ws + s.pw - kxf * s.dw) / s.sw;
    auto advance = [&](const Item &it) {
        Item n = it;
        ++n.ch;
        if (n.ch == nch) {
            n.ch = 0;
            n.kx += g.stepx;
            n.dx -= step_dx;
            if (n.kx >= s.kw) {
                n.kx = kxf;
                n.dx = dx0;
                n.ky += g.stepy;
                n.dy -= step_dy;
            }
        }
        return n.ky >= s.kh ? it : n;               // past the last one: it again, loaded and not used
    };
    auto load = [&](const Item &it, uint32_t stage) {
        const int dn = it.dy * s.Wo + it.dx, kb = it.ch * RB, dg = dn * g.Kb + kb;
        const int left = g.Kb - kb;                 // bytes of a row from here on; pieces past them come as zeros
        const int uniw = (it.ky * s.kw + it.kx) * s.C * g.Kb + kb;
        char *const st = ldsb + stage;
#pragma unroll
        for (int i = 0; i <= PA; ++i) {
            const bool ok = static_cast<uint32_t>(hq[i] + it.dy) < static_cast<uint32_t>(s.Ho) &&
                            static_cast<uint32_t>(wq[i] + it.dx) < static_cast<uint32_t>(s.Wo);
            if (i < PA)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsG, (lds_void_t *)(st + ((wave + 4 * i) % NA) * 1024), 16,
                                                         ok && pieceg[i < PA ? i : 0] < left ? offg[i] + dg : 0x80000000u, 0, 0, 0);
            else
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsS, (lds_void_t *)(st + SOFS + (wave * 64) % BM * 4), 4,
                                                         ok ? offg[i] + dn * 4 : 0x80000000u, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < PB; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, (lds_void_t *)(st + WOFS + ((wave + 4 * i) % NB) * 1024), 16,
                                                     piecew[i] < left ? offw[i] : 0x80000000u, uniw, 0, 0);
    };

    // ---- fragments: block i of an operand (16 rows) is 16 RB bytes further ----
    uint32_t rd[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h)
        rd[h] = static_cast<uint32_t>(l16) * RB + (RB >= 64 ? static_cast<uint32_t>((4 * h + g4) ^ swz(l16)) * 16u : static_cast<uint32_t>(g4) * 8u);
    const uint32_t ofsG = wave_m * (16 * FM * RB), ofsW = WOFS + wave_n * (16 * FN * RB);
    const int nj = min(FN, (s.C - c0 - wave_n * (16 * FN) + 15) / 16);      // blocks of 16 channels that exist
    v4i acc[FM][FN];
    f32x4 sum[FM][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j) sum[f][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto products = [&](uint32_t stage, auto firstc) {   // firstc: 1 = the tap's sums start here
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            op_t og[FM], ow[FN];
#pragma unroll
            for (int f = 0; f < FM; ++f) og[f] = *reinterpret_cast<const op_t *>(ldsb + (stage + ofsG + f * (16 * RB) + rd[h]));
#pragma unroll
            for (int j = 0; j < FN; ++j) ow[j] = *reinterpret_cast<const op_t *>(ldsb + (stage + ofsW + j * (16 * RB) + rd[h]));
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int f = 0; f < FM; ++f) acc[f][j] = Mm::mma(ow[j], og[f], decltype(firstc)::value && h == 0 ? v4i{0, 0, 0, 0} : acc[f][j]);
        }
    };
    if (items > 0) {
        Item cur{kyf, kxf, 0, (hs + s.ph - kyf * s.dh) / s.sh, dx0};
        Item nxt = advance(cur), mid = nxt;             // the item after this one, and the one to load
        load(cur, 0);
        if (NST == 3) {
            load(nxt, STAGE);
            nxt = advance(nxt);
        }
        uint32_t stage = 0;
        for (int i = 0; i < items; ++i) {
            // this item has landed (with three stages, all but the youngest NLOAD loads have), and nobody reads the
            // stage before it any more
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0x0070 | (NST == 3 ? NLOAD : 0));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            load(nxt, stage == 0 ? (NST - 1) * STAGE : stage - STAGE);
            const Item loaded = nxt;
            nxt = advance(nxt);
            if (cur.ch == 0) products(stage, Const<1>{});
            else products(stage, Const<0>{});
            if (cur.ch == nch - 1) {                     // the tap's integer sums are complete
                const float *cw = cols + (cur.ky * s.kw + cur.kx) * BN + wave_n * (16 * FN) + g4 * 4;
                const float *cg = reinterpret_cast<const float *>(ldsb + stage + SOFS) + wave_m * (16 * FM) + l16;
                float sg[FM];
#pragma unroll
                for (int f = 0; f < FM; ++f) sg[f] = cg[f * 16];
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    if (j >= nj) break;
                    const f32x4 cs = *reinterpret_cast<const f32x4 *>(cw + j * 16) * g.alpha;
#pragma unroll
                    for (int f = 0; f < FM; ++f) {
                        f32x4 o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = static_cast<float>(acc[f][j][e]) * (sg[f] * cs[e]);
                        if (!F32) {                      // an entry of the column gradient, in the type it is held in
                            const uint32_t p = pack_bf16(o[0], o[1]), q = pack_bf16(o[2], o[3]);
                            o = f32x4{bf16_lo(p), bf16_hi(p), bf16_lo(q), bf16_hi(q)};
                        }
                        sum[f][j] += o;
                    }
                }
            }
            cur = NST == 3 ? mid : loaded;
            mid = loaded;
            stage = stage == (NST - 1) * STAGE ? 0 : stage + STAGE;
        }
    }
    // the loads of the items past the last one land before this workgroup's LDS is given to another
    __builtin_amdgcn_s_waitcnt(0x0070);

    // A tap that a pixel does not have has codes and scale 0 and added 0, unless the column's scale is not finite:
    // 0 * inf.  Sums that are not numbers are looked at again, behind the stores (`nans` is not one if any of them is not).
    // Half an instruction a value here: 70 layers within 1 % of the sums unchecked.  The taps left out in the loop, by a
    // second copy of the additions for tiles with such a scale, cost all tiles 2 to 17 % (56 x 56 x 32 over 32, 7 x 7: 115 ->
    // 135 us), scalar registers spilled in the loop.
    float nans = 0.0f;

    // ---- a lane holds four consecutive channels of one pixel per fragment pair ----
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int q = m0 + (wave_m * FM + f) * 16 + l16;
        if (q >= Mc) continue;
        const Pixel p = pixel(q);
        const int64_t row = (static_cast<int64_t>(p.n * s.H + p.h * s.sh + hs) * s.W + p.w * s.sw + ws) * s.C;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int c = c0 + wave_n * (16 * FN) + j * 16 + g4 * 4;
            if (c >= s.C) continue;                 // C is a multiple of 4: conv_dx_ok
            const f32x4 v = sum[f][j];
            nans = fmaf(v[2], v[3], fmaf(v[0], v[1], nans));
            if (F32) {
                *reinterpret_cast<f32x4 *>(static_cast<float *>(g.dX) + row + c) = v;
            } else {
                const u32x2 p = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                *reinterpret_cast<u32x2 *>(static_cast<bf16_t *>(g.dX) + row + c) = p;
            }
        }
    }
    if (nans == nans) return;
    ConvDxArg *arg = (ConvDxArg *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(arg));
    uint64_t again = 0;
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) again |= static_cast<uint64_t>(sum[f][j][e] != sum[f][j][e]) << ((f * FN + j) * 4 + e);
    for (; again != 0; again &= again - 1) {
        const int i = __ffsll(static_cast<unsigned long long>(again)) - 1, f = i / (4 * FN), j = i / 4 % FN;
        const int q = m0 + (wave_m * FM + f) * 16 + l16, c = c0 + wave_n * (16 * FN) + j * 16 + g4 * 4 + i % 4;
        if (q >= Mc || c >= s.C) continue;
        const Pixel p = pixel(q);
        const int h = p.h * s.sh + hs, w = p.w * s.sw + ws;
        const int64_t at = (static_cast<int64_t>(p.n * s.H + h) * s.W + w) * s.C + c;
        const float v = conv_dx_again<F32>(*arg, p.n, h, w, c, __builtin_nanf(""));
        if (v != v) continue;
        if (F32) static_cast<float *>(g.dX)[at] = v;
        else static_cast<bf16_t *>(g.dX)[at] = static_cast<bf16_t>(pack_bf16(v, 0.0f) & 0xFFFFu);
    }
}

// the forms of the body that a launch chooses from: the tile's shape, and the bytes of a row per item
template <bool F32>
__device__ __forceinline__ void conv_dx_any(const ConvDx &g, int bid)
{
    const int rb = conv_dx_rb(g.form, g.Kb);
    if (g.form == 0) {              // 128 pixels x 128 channels
        if (rb == 128) conv_dx_tile<128, 2, 2, 4, 4, F32>(g, bid);
        else if (rb == 64) conv_dx_tile<64, 2, 2, 4, 4, F32>(g, bid);
        else conv_dx_tile<32, 2, 2, 4, 4, F32>(g, bid);
    } else if (g.form == 1) {       // 256 x 64
        if (rb == 64) conv_dx_tile<64, 4, 1, 4, 4, F32>(g, bid);
        else conv_dx_tile<32, 4, 1, 4, 4, F32>(g, bid);
    } else if (g.form == 3) {       // 64 x 64
        if (rb == 128) conv_dx_tile<128, 2, 2, 2, 2, F32>(g, bid);
        else if (rb == 64) conv_dx_tile<64, 2, 2, 2, 2, F32>(g, bid);
        else conv_dx_tile<32, 2, 2, 2, 2, F32>(g, bid);
    } else {                        // 128 x 64
        if (rb == 128) conv_dx_tile<128, 4, 1, 2, 4, F32>(g, bid);
        else if (rb == 64) conv_dx_tile<64, 4, 1, 2, 4, F32>(g, bid);
        else conv_dx_tile<32, 4, 1, 2, 4, F32>(g, bid);
    }
}

}  // namespace hlq
