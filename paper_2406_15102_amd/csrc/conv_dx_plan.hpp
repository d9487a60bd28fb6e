// Host-side planning of the image gradient of a convolution (conv_dx_body.hpp), shared by its launchers.
#pragma once
#include "conv_dx_body.hpp"
#include "gemm_plan.hpp"

namespace hlq {

struct ConvDxPlan {
    ConvDx g;
    int blocks;
    size_t lds;
};

// whether a compute unit's LDS holds one tile only (128 x 128 with more than 30 taps over more than 64 codes, or more than 61)
static inline bool conv_dx_alone(int form, int O, int taps) { return conv_dx_lds(form, O, taps) > kConvDxMaxLds / 2; }

static inline int conv_gcd(int a, int b)
{
    while (b) {
        const int t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// Tile of a layer: 128 pixels x 128 channels where the channels fill it, else 256 x 64; 128 x 64 where fewer than a
// workgroup a compute unit would come of that, 64 x 64 where 128 x 64 fills little more than half of the chip
// (whole passes of 3 x 3 layers, us, 256 x 64 or 128 x 128 / 128 x 64 / 64 x 64 pixels x channels: 12544 pixels x 256 channels over
// 256 codes 53.2 / 46.9 / 55.2, 200704 x 64 over 64 118.8 / 120.5 / 135.3, 3136 x 512 over 512 51.8 / 45.2 / 52.6, 12544 x 48
// over 448 61.1 / 43.0 / 42.6, 4096 x 128 over 128 28.7 / 27.3 / 23.0).
static inline void conv_dx_shape(const ConvShape &s, int &form, int &tiles_px, int &tiles_c, int &blocks)
{
    const int64_t most = static_cast<int64_t>(s.Nb) * ((s.H + s.sh - 1) / s.sh) * ((s.W + s.sw - 1) / s.sw);   // pixels of a class
    const int classes = s.sh * s.sw, c64 = (s.C + 63) / 64;
    form = c64 % 2 == 0 ? 0 : 1;
    if ((most + 255) / 256 * c64 * classes < 256) form = (most + 127) / 128 * c64 * classes < 160 ? 3 : 2;
    const int bm = conv_dx_bm(form);
    tiles_c = form == 0 ? c64 / 2 : c64;
    tiles_px = static_cast<int>((most + bm - 1) / bm);
    blocks = tiles_px * tiles_c * classes;
}

// Time of a tile, us, two to a compute unit: an item (RB codes of every row, of one tap) by shape and RB, from the
// measurements of conv_dx_wanted.
static inline double conv_dx_tile_us(int form, const ConvShape &s, int O)
{
    static const double item[4][3] = {{0.6, 0.75, 1.1}, {0.55, 0.6, 0.6}, {0.4, 0.5, 0.75}, {0.25, 0.3, 0.5}};
    const int rb = conv_dx_rb(form, O);
    return static_cast<double>(s.kh) * s.kw / (s.sh * s.sw) * ((O + rb - 1) / rb) * item[form][rb / 64];
}

// Whether the image gradient is taken straight from the codes: not where the column gradient is small beside the
// chain of taps and codes that one tile goes through.  The alternative writes the column gradient at about 2.3 TB/s and
// reads it at about 5 (65536 x 1224: 70 and 32 us), in a launch of its own more.  Whole passes of both gradients, us, column
// gradient -> straight (images x height x width x channels, kernel, over codes): 64 x 56 x 56 x 64, 3 x 3, over 64 247 -> 119;
// 64 x 28 x 28 x 128, 3 x 3, over 128 97 -> 69; 64 x 14 x 14 x 256, 3 x 3, over 256 57.1 -> 46.3; 128 x 16 x 16 x 512, 3 x 3, over 512
// 395 -> 272; 32 x 28 x 28 x 128, 5 x 5, over 128 127 -> 72; 32 x 56 x 56 x 32, 7 x 7, over 32 335 -> 118; fp32 64 x 28 x 28 x
// 128, 7 x 7, over 128 755 -> 383; 64 x 32 x 32 x 256, 8 x 8 with stride 2, over 128 508 -> 332; kept on the column gradient by this rule:
// 8 x 20 x 20 x 64, 7 x 7, over 512 48 -> 115; 4 x 32 x 32 x 128, 7 x 7, over 704 100 -> 185; 80 x 64 x 64 x 16, 7 x 7 with stride 2, over
// 736 290 -> 653.
// Tiles that fill a compute unit's LDS go one to a unit, each in 0.82 of the time (64 x 14 x 14 x 384, 8 x 8, over 96: 294 of them,
// 1.7 times the column gradient's time; 120 layers of 6 x 6 to 8 x 8 taps come to 0.3 % from the faster of the two in the
// mean, 2.7 % counted as two; the plan of launch_conv_pair counts two there as well, 0.5 % behind one in the mean and up to 8 % ahead).
// Of 233 layers that it takes (2 x 2 to 8 x 8 taps, whole passes of both gradients; 0.72 of the column gradient's time in the
// geometric mean) three are more than a tenth slower: 32 x 14 x 14 x 512 over 512 68 -> 77 us, whose weight gradient finds no room beside
// 392 tiles (the image gradient alone 54 -> 47); 112 x 16 x 16 x 56, 4 x 4, over 160 46 -> 56; 128 x 20 x 20 x 112, 7 x 7 with stride 2, over
// 512 183 -> 209.  No constants of this form were found that leave those out and lose none of the others.
// A 1 x 1 kernel with a stride has fewer taps than classes of pixels: most workgroups would write zeros only
// (50176 x 128 over 256, stride 2, 25.9 -> 28.6).
static inline bool conv_dx_wanted(const ConvShape &s, int O, bool is_f32)
{
    if (s.kh * s.kw < s.sh * s.sw) return false;
    int form, tiles_px, tiles_c, blocks;
    conv_dx_shape(s, form, tiles_px, tiles_c, blocks);
    const double mb = static_cast<double>(s.N) * s.kh * s.kw * s.C * (is_f32 ? 4e-6 : 2e-6);
    const double columns = 10.0 + (s.sh * s.sw > 1 ? 1.0 : 0.0) + mb / 2.3 + mb / 5.0;
    const bool alone = conv_dx_alone(form, O, s.kh * s.kw);
    const double rounds = alone ? __builtin_ceil(blocks / 256.0) * (blocks <= 256 ? 0.62 : 0.82)
                                : __builtin_ceil(blocks / 512.0) * (blocks <= 256 && form != 3 ? 0.75 : 1.0);
    return 9.3 + rounds * conv_dx_tile_us(form, s, O) < columns;
}

static inline ConvDxPlan conv_dx_plan(const GemmArgs &a, const ConvShape &s)
{
    ConvDxPlan p;
    p.g.Gq = static_cast<const char *>(a.A);
    p.g.sG = a.sA;
    p.g.Wq = static_cast<const char *>(a.Bm);
    p.g.sW = a.sB;
    p.g.dX = a.C;
    p.g.alpha = a.alpha;
    p.g.s = s;
    p.g.Kb = a.K;
    p.g.stepy = s.sh / conv_gcd(s.sh, s.dh);
    p.g.stepx = s.sw / conv_gcd(s.sw, s.dw);
    conv_dx_shape(s, p.g.form, p.g.tiles_px, p.g.tiles_c, p.blocks);
    p.lds = conv_dx_lds(p.g.form, p.g.Kb, s.kh * s.kw);
    return p;
}

// Time of the launch that carries both products, us: the image gradient's blocks and nb tiles of the weight gradient of
// `steps` k steps each.  Fitted to whole passes of 470 layers at every split in either order, on changing inputs: a
// tile of the image gradient takes 3.95, `item` for RB codes of a tap, and `tap` for the sums of a tap; one of the
// weight gradient 2.45 and 0.45 a step; where they have a compute unit to themselves, 0.86 and 0.68 of that.
static inline double conv_pair_time(const ConvDxPlan &p, double nb, double steps, bool b_first)
{
    static const double item[4][3] = {{0.60, 0.65, 0.68}, {0.82, 0.40, 0.40}, {0.28, 0.40, 0.36}, {0.28, 0.12, 0.19}};
    static const double tap[4] = {0.48, 0.48, 0.24, 0.12};
    constexpr double kFixedA = 3.95, kFixedB = 2.45, kStepB = 0.45, kAloneA = 0.86, kAloneB = 0.68;
    const ConvShape &s = p.g.s;
    const int form = p.g.form, rb = conv_dx_rb(form, p.g.Kb);
    const double taps = static_cast<double>(s.kh) * s.kw / (s.sh * s.sw);
    const double a = taps * (((p.g.Kb + rb - 1) / rb) * item[form][rb / 64] + tap[form]), b = steps * kStepB;
    const double ta = kFixedA + a, tb = kFixedB + b, all = p.blocks + nb;
    if (all <= 256) return __builtin_fmax(kFixedA + a * kAloneA, kFixedB + b * kAloneB);
    if (all <= 512) return ta < tb ? ta + (tb - ta) * kAloneB : tb + (ta - tb) * kAloneA;    // all resident
    return b_first ? pair_makespan(nb, tb, 512, p.blocks, ta, 512) : pair_makespan(p.blocks, ta, 512, nb, tb, 512);
}

}  // namespace hlq
