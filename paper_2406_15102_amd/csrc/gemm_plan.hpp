// Host-side planning shared by the launchers of the matrix products (k_gemm.hip, k_gemm_pair.hip).
#pragma once
#include "gemm_common.hpp"

namespace hlq {

// bytes per operand row: int8 codes, bf16 values, nibble-packed codes, codes in the f6 layout (whole 128-byte steps)
static inline int row_bytes(int kind, int K)
{
    return kind == 0 ? K : (kind == 1 ? 2 * K : (kind == 2 ? K / 2 : f6_row_bytes(K)));
}

// Plan: tile size and number of k splits, from a small cost model (microseconds) fitted to
// measurements on MI355X: a 256-tile step (128 B of k) costs ~1.6 us and a tile ~12 us of fixed
// prologue/epilogue, one workgroup per compute unit; a 128-tile step ~0.5 us alone on its compute
// unit and ~0.95 us when two share it, ~6 us fixed; the split-K partials cost their HBM round trip
// plus a launch.  A step of the packed product carries twice the MFMAs of a byte-operand step.
constexpr double P4_STEP_SCALE = 1.8;
constexpr double F6_STEP_SCALE = 1.0;    // a step of f6 codes: as many MFMA cycles as one of bytes
// cost of a step of operand kind `kind` in steps of bytes
static inline double step_scale(int kind) { return kind == 2 ? P4_STEP_SCALE : (kind == 3 ? F6_STEP_SCALE : 1.0); }
struct GemmPlan {
    bool big;
    int splits;
};
// `nk` = k steps of the product (128 B of k per operand row); `scale` = cost of such a step relative
// to the byte-operand kernels.
GemmPlan plan_gemm(int M, int N, int nk, double scale, size_t ws_bytes, bool allow_split);
GemmPlan plan_for(int kind, int M, int N, int K, size_t ws_bytes, bool allow_split);

// measurement overrides of the plans (hlq_set_option): tile = 0 (the model decides), 128 or 256 for every
// product; splits = 0 (the model decides) or the k split of a single product / of the g_w product of a
// pair, cut down to what the reduction and the scratch allow.  A negative argument leaves that setting.
void gemm_plan_force(int tile, int splits);
int gemm_plan_forced_tile();
int gemm_plan_forced_splits(int nk, double mn, size_t ws_bytes, bool allow_split);

// whether a 256-tiled product with rows of Kb bytes, its k split `splits` ways, takes the kernel that
// loads its operands straight into LDS (gemm_dl_body.hpp)
bool gemm_dl_ok(int Kb, int splits);
void gemm_dl_enable(bool on);
// the same for two products on 128-tiles in one launch; scale_a: cost of a step of `a` in steps of `b`
bool gemm_dl128_ok(const GemmDev &a, double scale_a, const GemmDev &b);
bool gemm_dl128_pays(int steps_a, double scale_a, double tiles_a, int steps_b, double tiles_b);   // whole steps a workgroup, workgroups

// Rows at the end of a product of M x N in 256 x 256 tiles that are better served by 192-row tiles
// (gemm_dl_body.hpp), 0 = none: when `before` tiles of the same launch are dispatched ahead of it and its
// last round on `slots` compute units would be partly empty, the row tiles that reach into that round --
// and as many more as it takes for the rest to fit the full rounds -- are cut into 192-row tiles if those
// then fit one round: the last round shrinks to three quarters.  Switched off by gemm_tail_enable(false).
void gemm_tail_enable(bool on);
bool gemm_tail_enabled();
static inline int gemm_tail_rows(int M, int N, int before, int slots = 256)
{
    if (!gemm_tail_enabled()) return 0;
    const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
    const int64_t total = static_cast<int64_t>(before) + static_cast<int64_t>(tiles_m) * tiles_n;
    const int rem = static_cast<int>(total % slots);
    if (rem == 0 || total < slots) return 0;               // whole rounds, or less than one
    const int64_t cap = total - rem;                          // what the full rounds hold
    const int rt = (rem + tiles_n - 1) / tiles_n;             // row tiles that reach into the last round
    if (rt > tiles_m) return 0;
    const int main_rows = (tiles_m - rt) * 256;
    const int tail_rows = M - main_rows;
    const int64_t main_tiles = static_cast<int64_t>(tiles_m - rt) * tiles_n;
    const int64_t tail_tiles = static_cast<int64_t>((tail_rows + 191) / 192) * tiles_n;
    if (before + main_tiles + tail_tiles > cap + slots) return 0;   // the 192-row tiles would start another round
    return tail_rows;
}

// kernel argument block of one product tiled BM x BN, k split `splits` ways
static inline GemmDev gemm_dev(int kind, const GemmArgs &a, int BM, int BN, int splits)
{
    GemmDev g;
    g.A = static_cast<const char *>(a.A);
    g.Bm = static_cast<const char *>(a.Bm);
    g.M = a.M;
    g.N = a.N;
    g.Kb = row_bytes(kind, a.K);
    g.sA = a.sA;
    g.sB = a.sB;
    g.alpha = a.alpha;
    g.C = a.C;
    g.c_is_f32 = a.c_is_f32 ? 1 : 0;
    g.acc = a.acc;
    g.tiles_m = (a.M + BM - 1) / BM;
    g.tiles_n = (a.N + BN - 1) / BN;
    g.splits = splits;
    g.partial = static_cast<int32_t *>(a.ws);
    return g;
}

// the last `tail_rows` rows of the product `g` (tiled 256 x 256, no k split, output C) as a product of
// its own in tiles of 192 x 256; `g` is cut back to the rows before them
static inline GemmDev gemm_dev_cut_tail(GemmDev &g, int tail_rows)
{
    GemmDev t = g;
    const int main_rows = g.M - tail_rows;
    const int64_t esz = g.c_is_f32 ? 4 : 2;
    t.A = g.A + static_cast<int64_t>(main_rows) * g.Kb;
    t.M = tail_rows;
    t.sA = g.sA ? g.sA + main_rows : nullptr;
    t.C = static_cast<char *>(g.C) + static_cast<int64_t>(main_rows) * g.N * esz;
    t.tiles_m = (tail_rows + 191) / 192;
    g.M = main_rows;
    g.tiles_m = main_rows / 256;
    return t;
}

// ---- model of a launch that carries two products (k_gemm_pair.hip says how it is fitted), microseconds ----
constexpr double kStepBig = 1.3, kStepSmallAlone = 0.6, kStepSmallShared = 0.9;
constexpr double kFixedBig = 16.0, kFixedSmall = 6.5;
// one product's tiles: a step, and what a tile costs beside its steps
struct TileCost {
    double step, fixed;
};
// 256-tiles, 128-tiles beside 256-tiles of the other product (a compute unit each), 128-tiles of both products that have one
// each, and that share one in twos
struct TileCosts {
    TileCost big, beside, alone, shared;
};
constexpr TileCosts kTileCosts = {{kStepBig, kFixedBig}, {kStepSmallAlone, kFixedSmall}, {kStepSmallAlone, kFixedSmall}, {kStepSmallShared, kFixedSmall}};
// The same where the g_x product is on codes in the f6 layout: its tiles, and the g_w product's with operands straight into LDS or
// through registers.  Fitted to every plan of 653 layers of 2 to 800 GFLOP (whole passes, either dispatch order): the plan
// taken was 1.2 % from the best one in the mean, 2.0 % with the constants above, and 12608 x 768 x 3072 took 102.6 us where those
// picked one of 114.9 (one session).  Over the 861 other layers of profiles/pair_plans_f6.txt it is 1.3 %.  All of these fitted anew to those
// come to 1.0 % of them, but the next box's best plans are others by as much, and 13 layers lose more than 2 %: left as they are.
constexpr TileCosts kTileCostsF6 = {{1.35, 16.4}, {0.58, 6.8}, {0.58, 7.3}, {1.02, 4.0}};
constexpr TileCosts kTileCostsDirect = {{1.2, 17.0}, {0.55, 5.3}, {0.58, 4.7}, {1.0, 4.2}}, kTileCostsStaged = {{2.0, 17.3}, {0.77, 3.6}, {0.72, 3.6}, {1.32, 4.1}};
// 128-tiles of both products in many rounds fetch each operand twice as often as 256-tiles, which the costs above, fitted to layers of
// more tokens, do not have: wide layers of few tokens went to them and lost to the nibbles' 256-tiles.  So much more for launches of at
// least four rounds whose g_w tiles have 7 to 16 steps; of 861 layers whose every plan was timed (profiles/pair_plans_f6.txt) 13 are
// faster by more than 2 %, none slower.  Whole passes, before -> this, with nibbles: 1024 x 28672 x 8192 723 -> 653 us, 697; 1024 x 8192 x 28672
// 654 -> 613, 641; 1024 x 8192 x 8192 214 -> 194, 207; 2048 x 11008 x 4096 227 -> 220, 228.
constexpr double kManyRoundsMore = 1.06, kManyRounds = 4.0;
constexpr int kManyRoundsSteps[2] = {7, 16};
constexpr double kPartialUs = 1.0e-6, kReduceUs = 3.0;     // a k split: of each partial value, and of the reduction's launch
constexpr double kPartialUsF6 = 1.54e-6, kReduceUsF6 = 4.5;
constexpr double kOneStepSaves = 2.0;    // a tile of one step skips the pipeline (gemm_body.hpp)
constexpr int kSplitChoices[] = {1, 2, 3, 4, 6, 8, 12, 16};

struct TileClass {
    double step, fixed;
    int slots;   // tiles in flight on the chip
};
inline TileClass tile_class(const TileCosts &c, bool big, bool mixed, double n)
{
    const bool share = !big && !mixed && n > 256.0;
    const TileCost &t = big ? c.big : (mixed ? c.beside : (share ? c.shared : c.alone));
    return {t.step, t.fixed, share ? 512 : 256};
}

// nA tiles of tA on mA slots, then nB tiles of tB on mB slots (the same silicon, possibly cut finer)
inline double pair_makespan(double nA, double tA, int mA, double nB, double tB, int mB)
{
    const double qA = __builtin_floor(nA / mA), rA = nA - qA * mA;
    const double T1 = qA * tA, T2 = rA > 0 ? T1 + tA : T1;
    const double g2 = __builtin_round(rA / mA * mB), g1 = mB - g2;      // slots free at T2 / at T1
    // candidate finishing times: T1 + k tB and T2 + k tB; the first with enough capacity
    double best = 1e30;
    for (int grp = 0; grp < 2; ++grp) {
        const double base = grp ? T2 : T1;
        const double gs = grp ? g2 : g1;
        if (gs <= 0) continue;
        // smallest k with g1 floor((T - T1)/tB) + g2 floor((T - T2)/tB) >= nB at T = base + k tB
        double lo = grp ? 0 : 1, hi = __builtin_ceil(nB / gs) + 1;
        while (lo < hi) {
            const double k = __builtin_floor((lo + hi) / 2), T = base + k * tB;
            const double c1 = g1 * __builtin_fmax(0.0, __builtin_floor((T - T1) / tB + 1e-9));
            const double c2 = g2 * __builtin_fmax(0.0, __builtin_floor((T - T2) / tB + 1e-9));
            if (c1 + c2 >= nB) hi = k; else lo = k + 1;
        }
        const double T = base + lo * tB;
        if (T < best) best = T;
    }
    return best > T2 ? best : T2;
}

// dynamic LDS of a workgroup: two operand stages, or the four epilogue slabs if those are larger
constexpr size_t gemm_lds_bytes(int WM, int WN, int KCH)
{
    const size_t main_bytes = 2u * (64 * WM + 64 * WN) * KCH * 16u;
    const size_t epi_bytes = 4u * (32u * (32u * WN * 4u + 16u));
    return main_bytes > epi_bytes ? main_bytes : epi_bytes;
}

}  // namespace hlq
