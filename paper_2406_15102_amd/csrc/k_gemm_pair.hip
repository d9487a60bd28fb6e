// K2 | K4 in one launch: the plan and the dispatch over the operand kinds.  The kernels live in
// gemm_pair_impl.hpp, instantiated by k_gemm_pair_KK.hip for KK = (kind of the g_x product, kind of
// the g_w product): 31 the default lists (4-bit codes in the f6 layout, bf16 projections), 30 with the integer
// g_w list, 21 / 20 the same with codes two to a byte (rows that f6 would mostly pad, weight codes handed over beside few
// tokens, the stage entry point), 01 / 00 with one int8 per g_x code (8-bit warm-up, unpacked storage).
#include "gemm_plan.hpp"

namespace hlq {

hipError_t launch_pair_21(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);
hipError_t launch_pair_31(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);
hipError_t launch_pair_30(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);
hipError_t launch_pair_20(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);
hipError_t launch_pair_01(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);
hipError_t launch_pair_00(const GemmDev &ga, const GemmDev &gb, const GemmDev &gbt, bool bigA, bool f32, bool bigB, int outB,
                          bool b_first, hipStream_t st);

// Plan of the pair: tile size of either product and the k split of the g_w product, by a model of
// how the launch unfolds (microseconds; constants fitted to a sweep of every plan, either dispatch
// order, over thirteen layer shapes on MI355X).  A tile of nk steps (128 B of k) takes nk * step + fixed.  A 256-tile owns a
// compute unit.  128-tiles share one in twos only if both products use them (the launch has one LDS
// size, the larger) and there are more of them than compute units; they step faster alone.
// Workgroups are dispatched in index order, one product's tiles then the other's (both orders are
// priced), each to the first free slot: after the first product's full rounds, the slots of its last, partial round free up one
// tile later than the rest, and the other product's tiles -- all equal -- finish at the first instant
// by which enough of them fit.
struct PairPlan {
    bool bigA, bigB;
    int splitsB;
    bool b_first;    // the g_w product's tiles are dispatched first
};


static PairPlan plan_pair(const GemmArgs &a, int kindA, const GemmArgs &b, int kindB, size_t ws_bytes)
{
    const bool f6 = kindA == 3;
    const TileCosts &costsA = f6 ? kTileCostsF6 : kTileCosts;
    const double saves = f6 ? 0.0 : kOneStepSaves;
    const double partial = f6 ? kPartialUsF6 : kPartialUs, reduce = f6 ? kReduceUsF6 : kReduceUs;
    const int nkA = (row_bytes(kindA, a.K) + 127) / 128, nkB = (row_bytes(kindB, b.K) + 127) / 128;
    const double scaleA = step_scale(kindA), scaleB = step_scale(kindB);
    const double mnB = static_cast<double>(b.M) * b.N;
    PairPlan best{true, true, 1, false};
    double best_t = 1e30;
    for (int bigA = 1; bigA >= 0; --bigA) {
        for (int bigB = 1; bigB >= 0; --bigB) {
            const bool mixed = bigA != bigB;
            const int ta = bigA ? 256 : 128, tb = bigB ? 256 : 128;
            const double nA = static_cast<double>((a.M + ta - 1) / ta) * ((a.N + ta - 1) / ta);
            const double nB1 = static_cast<double>((b.M + tb - 1) / tb) * ((b.N + tb - 1) / tb);
            const TileClass ca = tile_class(costsA, bigA != 0, mixed, nA);
            const double tA = nkA * scaleA * ca.step + ca.fixed - (nkA == 1 ? saves : 0.0);
            for (int S : kSplitChoices) {
                if (S > 1 && (S > nkB || S * mnB * 4.0 > static_cast<double>(ws_bytes))) break;
                // by sizes alone: rows of a store, which may end inside a step, are split like the padded ones (same sums)
                const bool direct = bigA || bigB ? nkB / S >= 4 : gemm_dl128_pays(nkA, scaleA, nA, nkB / S, nB1 * S);
                const TileClass cb = tile_class(f6 ? (direct ? kTileCostsDirect : kTileCostsStaged) : kTileCosts, bigB != 0, mixed, nB1 * S);
                const double stepsB = __builtin_ceil(static_cast<double>(nkB) / S);
                const double tB = stepsB * scaleB * cb.step + cb.fixed - (stepsB == 1.0 ? saves : 0.0);
                const double extra = S > 1 ? partial * S * mnB + reduce : 0.0;     // partials out and back, one more launch
                // no shorter than its longest tile, nor (but for rounding) than its work spread over the chip: most plans need
                // no look at how they unfold
                const double least = __builtin_fmax(__builtin_fmax(tA, tB), 0.99 * (nA * tA / ca.slots + nB1 * S * tB / cb.slots));
                if (least + extra >= best_t) continue;
                // either product may go first: usually the one with the longer tiles, which must not start late
                const double tab = pair_makespan(nA, tA, ca.slots, nB1 * S, tB, cb.slots);
                const double tba = pair_makespan(nB1 * S, tB, cb.slots, nA, tA, ca.slots);
                const bool b_first = tba < tab;
                const bool many = f6 && !bigA && !bigB && nA + nB1 * S >= kManyRounds * 512.0 && stepsB >= kManyRoundsSteps[0] && stepsB <= kManyRoundsSteps[1];
                const double t = (b_first ? tba : tab) * (many ? kManyRoundsMore : 1.0) + extra;
                if (t < best_t) {
                    best_t = t;
                    best = PairPlan{bigA != 0, bigB != 0, S, b_first};
                }
            }
        }
    }
    if (const int t = gemm_plan_forced_tile()) best.bigA = best.bigB = t == 256;
    if (const int S = gemm_plan_forced_splits(nkB, mnB, ws_bytes, ws_bytes > 0)) best.splitsB = S;
    return best;
}

// split-k scratch the pair's plan asks for when it may have up to `cap` bytes
size_t gemm_pair_ws_bytes(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, size_t cap)
{
    const PairPlan p = plan_pair(a, kindA, b, kindB, cap);
    return p.splitsB > 1 ? static_cast<size_t>(p.splitsB) * b.M * b.N * 4 : 0;
}

void gemm_pair_describe(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, size_t ws_bytes, int plan[5])
{
    const PairPlan p = plan_pair(a, kindA, b, kindB, ws_bytes);
    plan[0] = p.bigA ? 256 : 128;
    plan[1] = p.bigB ? 256 : 128;
    plan[2] = p.splitsB;
    plan[3] = p.b_first ? 1 : 0;
    plan[4] = (p.bigA && p.bigB && p.splitsB == 1 && gemm_stream_wanted(kindA, a, kindB, &b)) ? 1 : 0;
}

bool gemm_pair_available(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b)
{
    // the grid of the launch (128-tiles of both products, the second split 16 ways) must fit 31 bits with room
    const int64_t blocks = static_cast<int64_t>((a.M + 127) / 128) * ((a.N + 127) / 128) +
                           16 * static_cast<int64_t>((b.M + 127) / 128) * ((b.N + 127) / 128);
    return (kindA == 3 || kindA == 2 || kindA == 0) && (kindB == 1 || kindB == 0) && a.C && b.C && !a.acc && !b.acc &&
           a.c_is_f32 == b.c_is_f32 && blocks < (int64_t(1) << 30);
}

hipError_t launch_gemm_pair(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, hipStream_t st, SplitReduce *defer)
{
    if (defer) defer->blocks = 0;
    if (!gemm_pair_available(kindA, a, kindB, b)) return hipErrorInvalidValue;
    const bool can_split = b.ws != nullptr && (reinterpret_cast<uintptr_t>(b.ws) & 15) == 0;
    const PairPlan p = plan_pair(a, kindA, b, kindB, can_split ? b.ws_bytes : 0);
    if (p.bigA && p.bigB && p.splitsB == 1 && gemm_stream_wanted(kindA, a, kindB, &b))
        return launch_gemm_stream(kindA, a, kindB, &b, st);
    const GemmDev ga = gemm_dev(kindA, a, p.bigA ? 256 : 128, p.bigA ? 256 : 128, 1);
    GemmDev gb = gemm_dev(kindB, b, p.bigB ? 256 : 128, p.bigB ? 256 : 128, p.splitsB);
    const int outB = p.splitsB > 1 ? 3 : (b.c_is_f32 ? 1 : 0);
    // the g_w product's last rows in 192-row tiles when it closes the launch on 256-tiles that load straight
    // into LDS and its last round would be partly empty (gemm_plan.hpp)
    GemmDev gbt = gb;
    gbt.tiles_m = 0;
    if (p.bigA && p.bigB && p.splitsB == 1 && !p.b_first && kindB != 2 && gemm_dl_ok(gb.Kb, 1)) {
        const int tail_rows = gemm_tail_rows(b.M, b.N, ga.tiles_m * ga.tiles_n);
        if (tail_rows > 0) gbt = gemm_dev_cut_tail(gb, tail_rows);
    }
    hipError_t e;
    if (kindA == 3)
        e = kindB == 1 ? launch_pair_31(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st)
                       : launch_pair_30(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st);
    else if (kindA == 2)
        e = kindB == 1 ? launch_pair_21(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st)
                       : launch_pair_20(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st);
    else
        e = kindB == 1 ? launch_pair_01(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st)
                       : launch_pair_00(ga, gb, gbt, p.bigA, a.c_is_f32, p.bigB, outB, p.b_first, st);
    if (e != hipSuccess || p.splitsB == 1) return e;
    if (defer) {
        *defer = splitk_reduce_job_of(kindB == 1 ? 1 : 0, b, p.splitsB);
        return hipSuccess;
    }
    return launch_splitk_reduce(kindB == 1 ? 1 : 0, b, p.splitsB, st);
}

}  // namespace hlq
