// The transforms of one backward pass, launched together.  Stages 1-2 of the g_x list (K1 on G),
// stages 1 and 3 of the g_w list (K3 on X and on G) and the first pass of stages 3-4 of the g_x
// list (column maxima of H^T W) do not depend on one another (arXiv 2406.15102, Sec. 6.1), and each
// costs a few tens of microseconds, of which four to five are the fixed price of a launch that
// waits for its predecessor to drain.  Two launches carry them instead of six:
//   front A   K1(G)  |  K3(G)  |  K3(X)  |  zeroing of the column maxima    (workgroups of the quantiser and of
//                                                                           the projections in turns)
//   front B   column maxima of H^T W                                        (needs the zeroing)
// (with HLQ_OPT_FRONT_INTERLEAVE off, each job keeps its own index range and K3(X) rides in front B; a
// convolution has K3 of the image, read as its column matrix, in front A and K3(G) in front B)
// or ONE, when the weight has few row blocks (k_front_one below): the maxima stay per row block.
// and two or three launches carry the integer g_w list, whose projections are quantised in two passes too:
//   front A   zeroing of the maxima where they are merged by atomics (kAmaxTableRows, kAmaxTableReads)
//   front Q1  K1(G)  |  maxima of projected G  |  of projected X  |  of H^T W  |  widening of a 4-bit store
//   front Q2  int8 codes of projected G  |  of projected X  |  codes of the weight
// A workgroup looks up its job from its index (jobs occupy consecutive index ranges, a job may be
// empty) and runs the same device body as the stand-alone kernel of that stage.
// Here: what the jobs look like and which unit launches them; the kernels are in front_impl.hpp, compiled for an element
// type and a block size at a time (k_front_<B>_<type>.hip).
#include "front_launch.hpp"
#include "quant_cols_body.hpp"
#include "quant_rows_body.hpp"

#include <atomic>

namespace hlq {

FrontUnpack front_unpack(const void *in, void *out, int64_t rows, int64_t Kc, int64_t Kp)
{
    FrontUnpack j{in, out, in ? rows * (Kp / 32) : 0, static_cast<int>(Kc / 32), static_cast<int>(Kp / 32), 0};
    j.blocks = static_cast<int>((j.n + 255) / 256);
    return j;
}

FrontRecode front_recode(const void *in, int rows, int O, bool nibbles, void *out)
{
    FrontRecode j{in, static_cast<uint8_t *>(out), in ? rows : 0, O, nibbles ? 1 : 0, 0};
    j.blocks = static_cast<int>((static_cast<int64_t>(j.rows) * (f6_row_bytes(O) / 16) + 255) / 256);
    return j;
}

__global__ __launch_bounds__(256) void k_f6_recode(FrontRecode jk) { f6_recode_body(jk, blockIdx.x); }

hipError_t launch_f6_recode(const FrontRecode &jk, hipStream_t st)
{
    if (jk.blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_f6_recode, dim3(jk.blocks), dim3(256), 0, st, jk);
    return hipGetLastError();
}

FrontHlaQ front_hlaq(const void *T, int64_t N, int D, int B, int r, uint32_t *amax, int table, uint32_t k0, uint32_t k1,
                     int64_t Kp, int8_t *TqT, float *sT)
{
    FrontHlaQ j{T, N, D, r, amax, k0, k1, Kp, TqT, sT, 0, 0, table};
    if (!T) return j;
    j.gx = hla_grid_x(D, B);
    j.gy = hla_grid_y(N, B);
    return j;
}

FrontColsQ front_colsq(const void *W, int O, int I, int B, const uint32_t *amax, int table, uint32_t k0, uint32_t k1,
                       float qmax, int8_t *WqT, float *sW)
{
    FrontColsQ j{W, O, I, amax, k0, k1, qmax, WqT, sW, 0, 0, table};
    if (!W) return j;
    j.gx = cols_grid_x(I, B);
    j.gy = cols_grid_y(O, B);
    return j;
}

// CALL of the unit for the element type and block size at hand
#define HLQ_FRONT_UNIT(BB, CALL)                                                    \
    case BB: return is_f32 ? FrontLaunch<float, BB>::CALL : FrontLaunch<bf16_t, BB>::CALL;
#define HLQ_FRONT_UNITS(CALL)                                                       \
    switch (B) {                                                                    \
        HLQ_FRONT_UNIT(16, CALL)                                                    \
        HLQ_FRONT_UNIT(32, CALL)                                                    \
        HLQ_FRONT_UNIT(64, CALL)                                                    \
    }                                                                               \
    return hipErrorInvalidValue

hipError_t launch_front_q(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq,
                          const FrontRows &jr, const FrontUnpack &ju, const FrontRecode &jk, const ConvShape *conv, int B, int basis, bool is_f32,
                          int codes, hipStream_t st)
{
    FrontConv jc{};
    if (conv && jx.T) {
        if (!hla_conv_ok(*conv, B)) return hipErrorInvalidValue;
        jc.g = *conv;
        jc.on = 1;
    }
    HLQ_FRONT_UNITS(integer(jg, jx, jw, jq, jr, ju, jk, jc, basis, codes, st));
}

bool front_fusable(int O, int B)
{
    const int T = quant_rows_lanes(O, B);
    return T > 0;   // rows that need the 1024-thread K1 keep their own launch
}

FrontRows front_rows(const void *G, int64_t N, int O, int B, int codes, uint32_t k0, uint32_t k1, float qmax, int8_t *Gq, float *sG)
{
    FrontRows j{G, N, O, 0, k0, k1, qmax, Gq, sG, 0};
    if (!G) return j;
    j.T = codes == kCodesF6 ? quant_rows_f6_lanes(O) : quant_rows_lanes(O, B);
    const int rows_per_block = 256 / j.T;     // T == 256: one row per workgroup
    j.blocks = static_cast<int>((N + rows_per_block - 1) / rows_per_block);
    return j;
}

FrontHla front_hla(const void *T, int64_t N, int D, int B, int r, int64_t Kp, uint16_t *out)
{
    FrontHla j{T, N, D, r, Kp, out, 0, 0, 1, 0};
    if (!T) return j;
    j.gx = hla_grid_x(D, B);
    j.gy = hla_grid_y(N, B);
    j.grp = hla_job_grp(B, r);
    j.nb = hla_job_blocks(j.gx, j.gy, j.grp);
    return j;
}

FrontAbsmax front_absmax(const void *W, int O, int I, int B, uint32_t *amax, int table)
{
    FrontAbsmax j{W, O, I, amax, 0, 0, table};
    if (!W) return j;
    j.gx = cols_grid_x(I, B);
    j.gy = cols_grid_y(O, B);
    return j;
}

bool cols_full_ok(int O, int I, int B, bool is_f32)
{
    return O / B <= kColsFullMaxRowBlocks && static_cast<int64_t>(O) * I * (is_f32 ? 4 : 2) <= kColsFullMaxBytes;
}

FrontColsQ front_cols_full(const void *W, int O, int I, int B, uint32_t k0, uint32_t k1, float qmax, int8_t *WqT, float *sW)
{
    FrontColsQ j{W, O, I, nullptr, k0, k1, qmax, WqT, sW, 0, 0, 0};
    if (!W) return j;
    // as many groups of lanes as there are row blocks, so that a pass is one round where it can be: 16, 32 or
    // 64; beyond 64 row blocks there are several rounds anyway and the longer runs of 32 groups measure better
    const int nrb = O / B;
    const int lg = nrb <= 16 ? 4 : (nrb <= 32 ? 3 : (nrb <= 64 ? 2 : 3));
    const int strip = (B == 16 ? ColsFull<16>::CW : (B == 32 ? ColsFull<32>::CW : ColsFull<64>::CW)) << lg;
    j.gx = (I + strip - 1) / strip;
    j.gy = lg;
    return j;
}

namespace {
// Off by default.  Measured at 4096 x 4096 x 11008 (rocprofv3, 212 launches each way): with the shared
// read the launch fetches 98.5 MB instead of 180.6 MB from beyond the L2s -- G comes in once -- and
// takes 51.5 us instead of 53.0, the whole pass the same either way: the launch is bound by the
// quantiser's arithmetic and by latency, not by those bytes (its second read of G is served by the
// last-level cache).  A first form with groups of 64 rows and narrower K3 workgroups, whose write
// runs were shorter, took 62.4 us.
std::atomic<int> g_share_enabled{0};
}
void front_share_enable(bool on) { g_share_enabled.store(on ? 1 : 0); }

namespace {
// On by default.  Whole pass at 4096 x 4096 x 11008, alternating runs on one card: 371.9 us with each job in its
// own range, 364-367 with turns of 8 to 128 workgroups of the projection (32 the best by a microsecond);
// 8192 x 28672 x 8192 and the small layers do not move.
std::atomic<int> g_mix_enabled{1};
constexpr int kMixGran = 32;     // a multiple of 8: hla_job_map counts on index mod 8 being the XCD
}
void front_mix_enable(bool on) { g_mix_enabled.store(on ? 1 : 0); }
bool front_mix_enabled() { return g_mix_enabled.load() != 0; }

// turns for n1 workgroups of the quantiser and n3 of the projections; gran == 0 if either has too few
FrontMix front_mix_of(int n1, int n3)
{
    FrontMix m{0, 0, 0};
    if (!g_mix_enabled.load() || n1 < kMixGran || n3 < kMixGran) return m;
    m.gran = kMixGran;
    m.q = (n1 + n3 / 2) / n3;     // workgroups of the quantiser per workgroup of the projections
    if (m.q < 1) m.q = 1;
    const int c1 = n1 / (m.gran * m.q), c3 = n3 / m.gran;
    m.cyc = c1 < c3 ? c1 : c3;
    if (m.cyc == 0) m.gran = 0;
    return m;
}

FrontMix front_mix(const FrontRows &jr, const FrontHla &jx, int more)
{
    if (!jr.G || !jx.T) return FrontMix{0, 0, 0};
    return front_mix_of(jr.blocks, jx.nb + more);
}

FrontShare front_share(const FrontRows &jr, const FrontHla &jx, int B, bool is_f32)
{
    FrontShare s{};
    if (!g_share_enabled.load() || !jr.G || jr.G != jx.T || jr.N != jx.N || jr.O != jx.D) return s;
    constexpr int RG = 128;                             // rows of a group: 128 / B token blocks of K3
    const int rows_per_k1 = 256 / jr.T;                 // T = 256: one row per workgroup
    if (RG % rows_per_k1 != 0) return s;
    // Only where it pays: a group's rows (and what is written for them) must sit in one XCD's L2
    // together (4 MB), and the tensor must be large enough for its second read to cost real time.
    const int64_t row_bytes = static_cast<int64_t>(jr.O) * (is_f32 ? 4 : 2);
    if (row_bytes * RG > (int64_t(3) << 20) || row_bytes * jr.N < (int64_t(16) << 20)) return s;
    const int64_t groups = (jr.N + RG - 1) / RG;
    int pair = B / (2 * jx.r);                          // K3 writes 256 r / B bytes per column and group
    if (pair < 1) pair = 1;
    if (pair > 8) pair = 8;
    const int64_t units = (groups + pair - 1) / pair;
    s.nk1 = RG / rows_per_k1;
    s.gx = (jr.O + 255) / 256;
    s.pair = pair;
    const int64_t blocks = 8 * ((units + 7) / 8) * pair * (s.nk1 + s.gx);
    if (blocks >= (int64_t(1) << 30)) return FrontShare{};
    s.units = static_cast<int>(units);
    s.blocks = static_cast<int>(blocks);
    s.on = 1;
    return s;
}

hipError_t launch_front_one(const FrontRows &jr, const FrontHla &jx, const FrontHla &jg, const FrontColsQ &jq,
                            const ConvShape *conv, int B, int basis, bool is_f32, int codes, hipStream_t st)
{
    FrontConv jc{};
    if (conv) {
        if (!hla_conv_ok(*conv, B)) return hipErrorInvalidValue;
        jc.g = *conv;
        jc.on = 1;
    }
    if (jq.W && (jq.O / B > kColsFullMaxRowBlocks || jq.gy < 2 || jq.gy > 4)) return hipErrorInvalidValue;
    HLQ_FRONT_UNITS(one(jr, jx, jg, jq, jc, basis, codes, st));
}

hipError_t launch_front(const FrontRows &jr, const FrontHla &jx, const FrontFill &jf, const FrontHla &jg,
                        const FrontAbsmax &jw, const FrontRecode &jk, const ConvShape *conv, int B, int basis, bool is_f32, int codes,
                        hipStream_t st)
{
    FrontConv jc{};
    if (conv) {
        if (!hla_conv_ok(*conv, B)) return hipErrorInvalidValue;
        jc.g = *conv;
        jc.on = 1;
    }
    HLQ_FRONT_UNITS(first(jr, jx, jf, jg, jw, jk, jc, basis, codes, st));
}

}  // namespace hlq
