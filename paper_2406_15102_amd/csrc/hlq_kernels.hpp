// Host-side launchers of the gfx950 kernels.  Every launcher only enqueues work on `st`; shapes
// have been validated by the caller (hlq_api.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace hlq {

// How the codes of the g_x list are stored: one int8 each; 4-bit codes two to a byte, two's complement (O/2 bytes a
// row); or 4-bit codes in the f6 layout (hlq_device.hpp), f6_row_bytes(O) a row.
constexpr int kCodesBytes = 0, kCodesNibbles = 1, kCodesF6 = 2;
// bytes of a row of K codes in the f6 layout: two to a byte, zeros up to whole steps of 128 bytes
__host__ __device__ constexpr int f6_row_bytes(int K) { return (K + 255) / 256 * 128; }
// Rows of G are written and read with their padding, and layers of few out-features wait for memory: with half of each
// row padding (44416 x 176 over 128) a pass took 31.2 us against 30.5 with nibbles.  (Rows that pass fit the scratch of one
// int8 a code.)
inline bool f6_rows_ok(int K) { return 2 * K >= 3 * f6_row_bytes(K); }
// Weight codes that are handed over, nibbles or bytes, are read and written once more to come into that layout, which the g_x product
// pays back with its tokens, the sooner the fewer tiles it has beside long reductions: d_out of 1.5 d_in on is told apart.  Passes for both
// gradients with the codes as they come / in the layout, us: 256 x 4096 x 11008 72 / 56, 256 x 3936 x 17280 121 / 94, 256 x 8192 x 14336 158 / 125,
// above 2^27 codes 512 x 8192 x 28672 324 / 366 and 1024 tokens 452 / 447; the others 512 x 28672 x 8192 273 / 341, 1024 tokens 444 / 452,
// 1536 tokens 623 / 608, 256 x 16384 x 8192 118 / 132, 1024 x 16384 x 8192 256 / 258, 1536 tokens 360 / 345.  Beside the integer g_w list, whose
// int8 product is the shorter one, from 2048 on: 1536 x 28672 x 8192 544 / 592, 2048 tokens 646 / 634.  Calls for dX alone: 256 x 4096 x 11008 31.4 / 34,
// 512 tokens 43.7 / 43.7, 512 x 3936 x 17280 57 / 54; 512 x 28672 x 8192 88 / 114, 768 tokens 170 / 160, 768 x 8192 x 8192 60 / 55; above 2^27
// codes and long 768 x 8192 x 28672 162 / 175, 1024 tokens 228 / 195.  Up to 2^25 codes the layout is ahead or even throughout (256 x
// 4096 x 4096 34 / 27, dX alone 27.7 / 19.2).
inline bool f6_recode_pays(int64_t N, int64_t d_in, int64_t d_out, bool dx_alone, bool gw_int8)
{
    const int64_t codes = d_in * d_out;
    if (codes <= (int64_t(1) << 25)) return true;
    if (2 * d_out < 3 * d_in) return dx_alone ? N >= 768 : (N >= 2048 || (N > 1024 && !gw_int8));
    if (codes > (int64_t(1) << 27)) return N >= 1024;
    return !dx_alone || N >= 512;
}

// Rows of the projections that the whole path makes and multiplies itself, in elements of `esz` bytes: zeros up to whole
// 128-byte steps of the dW product, so that none is ragged and operands can be loaded straight into LDS.  (The rows of a
// store that is handed over have no padding.)  Not rows of at most four steps, which are multiplied through registers anyway.
// Whole pass, ragged rows -> padded: 9200 x 1160 x 3120 126.9 -> 117.7 us, 12608 x 768 x 3072 117.0 -> 113.9, 12608 x 768 x 2304
// in 8 bits 104.6 -> 99.6.
inline int64_t pad_row(int64_t Kc, int esz) { return Kc * esz <= 512 ? Kc : (Kc * esz + 127) / 128 * 128 / esz; }

// K1: rows of G -> codes + per-row scales (and optionally, not with kCodesF6, the fp32 coefficients).
// `mant`: round by the low 11 mantissa bits of each value instead of the seeded stream (k0, k1 unused).
hipError_t launch_quant_rows(const void *G, int64_t N, int O, int B, bool is_f32, uint32_t k0, uint32_t k1,
                             float qmax, int codes, bool mant, int8_t *Gq, float *sG, float *coeff, hipStream_t st);

// K1T: W [O, I] -> WqT [I, O] codes + per-in-feature scales.  `ws` holds the partial column
// maxima and the reciprocal scales: quant_cols_ws_bytes(O, I) bytes.
size_t quant_cols_ws_bytes(int64_t O, int64_t I);
hipError_t launch_quant_cols(const void *W, int O, int I, int B, bool is_f32, uint32_t k0, uint32_t k1,
                             float qmax, int codes, bool mant, int8_t *WqT, float *sW, float *coeffT, void *ws,
                             hipStream_t st);

// The same scratch as a file-scope device array inside the library (k_quant_cols.hip), for callers that
// cannot allocate: room for the column maxima of a weight with up to kQuantColsStaticMaxI in-features
// (256 KiB per GPU).  Returns the array's address on the current device (asked for once per device).
constexpr int kQuantColsStaticMaxI = 65536;
hipError_t quant_cols_static_scratch(void **ptr);

// Shape of a workgroup of K1T's two passes, as for K3: B lanes side by side (runs of 256 B of a row
// of bf16) times 256/B row blocks, whose codes are neighbours in a row of the transposed output
// (runs of 256 bytes, 128 packed).
inline int cols_grid_x(int I, int B) { return (I + 127) / 128; }
inline int cols_grid_y(int O, int B) { return (O + 255) / 256; }       // 256/B row blocks of B rows

// K1T split in its two passes, for callers that run pass 1 elsewhere (the fused front launches):
// pass 2 alone, reading the column maxima pass 1 left in `ws`.
hipError_t launch_quant_cols_pass2(const void *W, int O, int I, int B, bool is_f32, uint32_t k0, uint32_t k1,
                                   float qmax, int codes, bool mant, int8_t *WqT, float *sW, float *coeffT,
                                   const void *ws, hipStream_t st);
// The weights that one workgroup per strip of columns quantises completely, both passes, inside the
// one-launch front (launch_front_one below): at most 256 row blocks (O / B; 64 groups of four lanes
// take one each per round, so four rounds a pass) and small enough for the second pass to find
// them in the cache.  Measured: a gain up to these sizes, none at 13-20 MB, a loss beyond.
constexpr int kColsFullMaxRowBlocks = 256;
constexpr int64_t kColsFullMaxBytes = 8 << 20;
bool cols_full_ok(int O, int I, int B, bool is_f32);

// Geometry of a convolution over channels-last tensors.  N = Nb * Ho * Wo rows of the column matrix.
// far: the images that the positions of a wavefront (at most 64 in a row, and the block they begin in) fall into
// take 2^31 bytes of fp32 or more, and are not addressed in 32 bits from the first of them.
struct ConvShape {
    int Nb, H, W, C, kh, kw, sh, sw, ph, pw, dh, dw, Ho, Wo;
    int64_t N;
    int far;
};
inline bool conv_far(const ConvShape &s)
{
    const int64_t image = static_cast<int64_t>(s.H) * s.W;           // below 2^62
    const int64_t images = 128 / (static_cast<int64_t>(s.Ho) * s.Wo) + 2;
    return image >= (int64_t(1) << 31) || image * s.C >= (int64_t(1) << 31) / 4 / images ||
           // the taps next to an image, too: offsets are stepped through them
           (static_cast<int64_t>(s.H) + 2 * static_cast<int64_t>(s.ph) + static_cast<int64_t>(s.kh) * s.dh) *
                   (static_cast<int64_t>(s.W) + 2 * static_cast<int64_t>(s.pw) + static_cast<int64_t>(s.kw) * s.dw) >= (int64_t(1) << 31);
}

// The independent transforms of one backward pass in two launches (k_front.hip).  A job with a
// null tensor is empty.
struct FrontRows {   // K1 on G, 256-thread variant
    const void *G;
    int64_t N;
    int O, T;
    uint32_t k0, k1;
    float qmax;
    int8_t *Gq;
    float *sG;
    int blocks;
};
struct FrontHla {    // K3 on one tensor
    const void *T;
    int64_t N;
    int D, r;
    int64_t Kp;      // values from one row of `out` to the next (pad_row)
    uint16_t *out;
    int gx, gy;      // column strips of 128, groups of 256/B token blocks
    int grp, nb;     // hla_job_map's grouping and the workgroups it needs (>= gx * gy)
};
// Shape of a K3 workgroup: B lanes side by side (each CPL = 128/B columns: 256 B of a row of bf16
// whatever B) times 256/B token blocks, so that both the reads (runs of 256 B) and the writes
// (r coefficients of 256/B consecutive token blocks: 512 r/B bytes of an output row) come in long
// runs.  Measured at B = 16 on cold inputs against 64 lanes x 4 token blocks (1 KB reads, 8 r byte
// writes), us: X of 65536 x 576: 54.8 -> 25.1, G of 4096 x 11008: 41.7 -> 34.2, G of 12608 x 3072:
// 36.5 -> 27.5.  (16 lanes at B = 64 would read runs of 64 B: the whole pass 424 -> 451 us.)
constexpr int hla_lanes(int B) { return B; }
constexpr int hla_blocks(int B) { return 256 / B; }
inline int hla_grid_x(int D, int B) { return (D + 127) / 128; }      // B lanes x 128/B columns = 128 columns
inline int hla_grid_y(int64_t N, int B) { return static_cast<int>((N / B + hla_blocks(B) - 1) / hla_blocks(B)); }
// Order of the workgroups of a K3 job.  A workgroup writes 512 r/B bytes of each of its output rows
// and the workgroup of the next `by` the bytes after them; workgroups go round-robin to the eight
// XCDs (index mod 8), each with its own L2.  Where that is less than a 128-byte line, hla_job_map
// (hla_body.hpp) keeps the `grp` consecutive `by` that complete a line on one XCD, back to back, so
// that their pieces meet in that L2 and leave it as whole lines.
inline int hla_job_grp(int B, int r)
{
    const int bytes = 512 * r / B;
    return bytes >= 128 ? 1 : (bytes >= 64 ? 2 : (bytes >= 32 ? 4 : 8));
}
inline int hla_job_blocks(int gx, int gy, int grp)
{
    const int units = gx * ((gy + grp - 1) / grp);
    return 8 * grp * ((units + 7) / 8);
}
// K1(G) and K3(G) of one launch sharing ONE read of G from memory: rows of G go through in groups of
// 128; the workgroups of a group -- its K1 rows, then its K3 strips of 256 columns -- sit next to one
// another in the index sequence of ONE XCD (index mod 8), so that whichever of the two readers of a row
// comes second finds it in that XCD's L2.  `pair` consecutive groups (the ones whose K3 output pieces
// complete a 128-byte line) go to the same XCD back to back.  on == 0: the jobs keep their own ranges.
struct FrontShare {
    int on;
    int nk1;      // K1 workgroups per group of 128 rows
    int gx;       // K3 workgroups per group (strips of 256 columns)
    int pair;     // groups per unit handed to an XCD
    int units;    // units in all
    int blocks;   // workgroups of the two jobs together: 8 * ceil(units / 8) * pair * (nk1 + gx)
};
// The two jobs of the first launch in turns along the index sequence: `gran * q` workgroups of the row
// quantiser, then `gran` of the projection, `cyc` times over, then what is left of either.  The quantiser is
// bound by its arithmetic and the projection by memory: side by side on a compute unit they take less than
// one after the other.  gran == 0: each job keeps its own range of indices.
struct FrontMix {
    int gran, q, cyc;
};
struct FrontConv {   // on: the K3(X) job of front A reads the column matrix of an image (jx.T = the image)
    ConvShape g;
    int on;
};
struct FrontFill {   // n words at p := 0
    uint32_t *p;
    int n;
};
struct FrontAbsmax { // pass 1 of K1T
    const void *W;
    int O, I;
    uint32_t *amax;
    int gx, gy;
    int table;       // see kAmaxTableRows; 0: one maximum per column, merged by atomics
};
struct FrontHlaQ {   // K3 + int8 quantisation of one tensor: pass 1 (amax) and pass 2 (codes) read the same fields
    const void *T;
    int64_t N;
    int D, r;
    uint32_t *amax;
    uint32_t k0, k1;
    int64_t Kp;      // codes from one row of TqT to the next (pad_row)
    int8_t *TqT;
    float *sT;
    int gx, gy;
    int table;       // see kAmaxTableRows; 0: one maximum per column, merged by atomics
};
struct FrontUnpack { // 4-bit codes two to a byte -> one int8 each; n pieces of 32 codes out, row_out a row, the first row_in of them from `in`
    const void *in;
    void *out;
    int64_t n;       // below 2^31
    int row_in, row_out;
    int blocks;
};
struct FrontRecode { // weight codes [rows][O], one int8 each or two to a byte -> the f6 layout; 256 groups of 32 codes a workgroup
    const void *in;
    uint8_t *out;
    int rows, O, nibbles, blocks;
};
struct FrontColsQ {  // pass 2 of K1T
    const void *W;
    int O, I;
    const uint32_t *amax;
    uint32_t k0, k1;
    float qmax;
    int8_t *WqT;
    float *sW;
    int gx, gy;
    int table;       // see kAmaxTableRows; 0: one maximum per column, merged by atomics.  front_cols_full: unused
};
// Column maxima of the integer g_w list.  A workgroup of a pass 1 covers 256 rows.  Where a tensor has at most
// kAmaxTableRows of them, each leaves its maxima in a row of its own of a table, [groups of 256 rows][columns],
// and pass 2 folds the rows: nothing has to be zeroed, and when every tensor of the call is of that kind the
// launch that zeroes, about 2 us, is not there.  Otherwise one row merged by atomics.
// Every workgroup of a pass 2 folds the whole table of its columns, rows * rows * columns reads over a tensor.  Their sum
// over the call decides (whole pass, atomics -> tables, one binary, us): up to 1.4 M reads tables are ahead or
// even (512 x 1024 x 1024 22.9 -> 20.8, 4096 x 1024 x 1024 37.2 -> 34.3, 2048 x 4096 x 11008 with weight codes 162.6 -> 162.0),
// to 2.25 M it goes either way by 1 % (3072 x 4096 x 4096 120.0 -> 118.6, fp32 4096 x 3072 x 3072 127.5 -> 129.2), beyond tables
// are behind (4096 x 8192 x 1024 with codes, 2.4 M, 99.7 -> 101.1; 4096 x 4096 x 4096, 3.1 M, 136.1 -> 137.5; 4096 x 11008 x 3072,
// 5.2 M, 264.0 -> 271.1).  With tables of more than 16 rows, 4096: 8192 x 768 x 3072 82.1 -> 87.6, 16384 x 4096 x 4096 with codes
// 438 -> 471.
constexpr int kAmaxTableRows = 16;
constexpr int64_t kAmaxTableReads = 2250000;
inline int amax_table_rows(int64_t rows) { return rows <= 256 * kAmaxTableRows ? static_cast<int>((rows + 255) / 256) : 0; }
inline int64_t amax_table_reads(int64_t rows, int64_t cols)
{
    const int64_t t = amax_table_rows(rows);
    return t * t * cols;
}
inline size_t amax_table_bytes(int64_t rows, int64_t cols)
{
    const int t = amax_table_rows(rows);
    // (a single row has a place anyway)
    return t > 1 && amax_table_reads(rows, cols) <= kAmaxTableReads ? static_cast<size_t>(t) * static_cast<size_t>(cols) * 4 : 0;
}
FrontHlaQ front_hlaq(const void *T, int64_t N, int D, int B, int r, uint32_t *amax, int table, uint32_t k0, uint32_t k1,
                     int64_t Kp, int8_t *TqT, float *sT);
FrontColsQ front_colsq(const void *W, int O, int I, int B, const uint32_t *amax, int table, uint32_t k0, uint32_t k1,
                       float qmax, int8_t *WqT, float *sW);
FrontUnpack front_unpack(const void *in, void *out, int64_t rows, int64_t Kc, int64_t Kp);   // in == NULL: empty
FrontRecode front_recode(const void *in, int rows, int O, bool nibbles, void *out);   // in == NULL: empty
hipError_t launch_f6_recode(const FrontRecode &jk, hipStream_t st);
// The integer g_w list in two launches: every pass 1 (maxima of projected G, projected X, transformed W),
// then every pass 2; where maxima are merged by atomics, a launch of launch_front zeroes them first.  `jr`, if it
// is not empty, is K1(G) riding in the first of them, its workgroups in turns with the passes 1; `ju`, if it is not
// empty, widens a 4-bit store beside them, and `jk` brings weight codes into the f6 layout (codes == kCodesF6).  conv: NULL, or the geometry whose column matrix jx.T (an image) stands for.
hipError_t launch_front_q(const FrontHlaQ &jg, const FrontHlaQ &jx, const FrontAbsmax &jw, const FrontColsQ &jq,
                          const FrontRows &jr, const FrontUnpack &ju, const FrontRecode &jk, const ConvShape *conv, int B, int basis, bool is_f32,
                          int codes, hipStream_t st);
bool front_fusable(int O, int B);
FrontRows front_rows(const void *G, int64_t N, int O, int B, int codes, uint32_t k0, uint32_t k1, float qmax, int8_t *Gq, float *sG);
FrontHla front_hla(const void *T, int64_t N, int D, int B, int r, int64_t Kp, uint16_t *out);
FrontAbsmax front_absmax(const void *W, int O, int I, int B, uint32_t *amax, int table = 0);
// all of K1T for a weight that passes cols_full_ok: one workgroup per strip of columns (gy carries the
// strip's width as a shift)
FrontColsQ front_cols_full(const void *W, int O, int I, int B, uint32_t k0, uint32_t k1, float qmax, int8_t *WqT, float *sW);
// K1(G) | K3(X) | K3(G) | all of K1T in ONE launch (jq from front_cols_full, or without a weight):
// nothing has to be zeroed beforehand and no launch for pass 2 follows.
hipError_t launch_front_one(const FrontRows &jr, const FrontHla &jx, const FrontHla &jg, const FrontColsQ &jq,
                            const ConvShape *conv, int B, int basis, bool is_f32, int codes, hipStream_t st);
// conv: NULL, or the geometry whose column matrix jx.T (an image) stands for; needs hla_conv_ok.
hipError_t launch_front(const FrontRows &jr, const FrontHla &jx, const FrontFill &jf, const FrontHla &jg,
                        const FrontAbsmax &jw, const FrontRecode &jk, const ConvShape *conv, int B, int basis, bool is_f32, int codes,
                        hipStream_t st);
// whether launch_front lets K1 (jr) and its first K3 job (jx) share the read of their tensor; switch for A/B
FrontShare front_share(const FrontRows &jr, const FrontHla &jx, int B, bool is_f32);
void front_share_enable(bool on);
void front_mix_enable(bool on);
bool front_mix_enabled();

// K3: token-axis Hadamard low-rank projection, T [N, D] -> ThatT [D, N/B*r] bf16.
// basis: which r rows of the order-B matrix are kept, 0 = rows 0..r-1, 1 = the r of lowest sequency.
hipError_t launch_hla(const void *T, int64_t N, int D, int B, int r, int basis, bool is_f32, uint16_t *ThatT,
                      float *coeffT, hipStream_t st);

// K3q: token-axis projection followed by int8 quantisation with one scale per feature (stages
// 1-2 / 3-4 of the g_w list): T [N, D] -> TqT [D, N/B*r] int8 + sT [D].  `ws` holds D words of
// column maxima: hla_quant_ws_bytes(D) bytes.  Needs r % 4 == 0.
size_t hla_quant_ws_bytes(int64_t D);
// p4: codes in [-7, 7] stored two to a byte (TqT [D, N/B*r/2] bytes; needs r % 8 == 0; seeded rounding only)
hipError_t launch_hla_quant(const void *T, int64_t N, int D, int B, int r, int basis, bool is_f32, uint32_t k0,
                            uint32_t k1, bool mant, int8_t *TqT, float *sT, float *coeffT, void *ws, hipStream_t st,
                            bool p4 = false);
// 4-bit codes two to a byte -> one int8 each; bytes_in a multiple of 16, both pointers 16-byte aligned
hipError_t launch_unpack_nibbles(const void *in, int8_t *out, int64_t bytes_in, hipStream_t st);

// K2 / K4: C = alpha * sA (x) sB * (A . Bm^T).  kind 0: int8 operands, int32 accumulate;
// kind 1: bf16 operands, fp32 accumulate; kind 2: 4-bit codes two to a byte; kind 3: 4-bit codes in the f6
// layout.  K in elements.
struct GemmArgs {
    const void *A;
    const void *Bm;
    int M, N, K;
    const float *sA;
    const float *sB;
    float alpha;
    void *C;          // bf16 or fp32 [M, N], may be null
    bool c_is_f32;
    int32_t *acc;     // raw int32 accumulators (int8 kind only), may be null
    void *ws;         // device scratch for split-K partial sums, may be null (then k is never split)
    size_t ws_bytes;
};
hipError_t launch_gemm_nt(int kind, const GemmArgs &a, hipStream_t st);
hipError_t launch_splitk_reduce(int kind, const GemmArgs &a, int splits, hipStream_t st);
// The same reduction as a job description, for a later launch of the caller's that carries it
// beside its own work (the fold of a convolution): `blocks` workgroups of 256 threads, 0 = none.
struct SplitReduce {
    const int32_t *partial;
    int splits, M, N;
    const float *sA, *sB;
    float alpha;
    void *C;
    int kind, c_is_f32;
    int blocks;
};
SplitReduce splitk_reduce_job_of(int kind, const GemmArgs &a, int splits);
// K2 | K4 in one launch (k_gemm_pair.hip): product `a` of kind 2 and product `b` of kind 1, both
// with a scaled output of the same dtype.  Only b's k may be split (b.ws).  gemm_pair_available
// says whether the combination is built; the results are those of two launch_gemm_nt calls up to
// the summation order of b's k splits.
bool gemm_pair_available(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b);
// defer: if not null and b's k is split, the reduction is not launched but described there (blocks > 0).
hipError_t launch_gemm_pair(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, hipStream_t st,
                            SplitReduce *defer = nullptr);
// The products as ONE persistent launch (k_gemm_stream.hip): a workgroup per compute unit walks a
// fixed list of 256 x 256 tiles of `a`, then of `b` (NULL: one product only), loading across tile
// boundaries.  Same bits as launch_gemm_nt without a k split.  gemm_stream_wanted: the shapes allow it
// (bf16 output, whole k steps, at least four tiles per compute unit in all) and it has not been
// switched off; callers ask it after their plan has chosen 256-tiles and no k split.
bool gemm_stream_wanted(int kindA, const GemmArgs &a, int kindB, const GemmArgs *b);
hipError_t launch_gemm_stream(int kindA, const GemmArgs &a, int kindB, const GemmArgs *b, hipStream_t st);
void gemm_stream_enable(bool on);
bool gemm_stream_enabled();
void gemm_dl_enable(bool on);   // operands of 256-tiles straight into LDS where the shape allows (default on)
void gemm_tail_enable(bool on);   // 192-row tiles for the last rows of a product whose last round would be partly empty (default on)
void gemm_plan_force(int tile, int splits);   // measurement overrides of the plans, see gemm_plan.hpp
// What launch_gemm_pair would do with these shapes and this much split-k scratch, without doing it:
// plan[0], plan[1] = tile edge (256 or 128) of a's and b's product, plan[2] = k splits of b,
// plan[3] = 1 if b's tiles are dispatched first, plan[4] = 1 if the persistent form takes the launch.
void gemm_pair_describe(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, size_t ws_bytes, int plan[5]);
// split-k scratch (b.ws) that the pair's plan would use if it may have up to `cap` bytes; only the
// shapes and kinds of a and b are read
size_t gemm_pair_ws_bytes(int kindA, const GemmArgs &a, int kindB, const GemmArgs &b, size_t cap);
// Scratch that lets launch_gemm_nt split k whenever that is the faster plan for this shape
// (few output tiles, long reduction); 0 if the plan does not split.
size_t gemm_ws_bytes(int kind, int M, int N, int K);

// Convolution glue (k_conv.hip), channels-last tensors.
// x [Nb, H, W, C] -> cols [N, kh*kw*C], columns ordered (ky, kx, c), zero padding
hipError_t launch_im2col(const void *X, const ConvShape &g, bool is_f32, void *cols, hipStream_t st);
// cols [N, kh*kw*C] -> dx [Nb, H, W, C]: each pixel sums the entries copied from it (fp32, fixed order)
// red: NULL, or a split-K reduction (independent of the fold) that the first red->blocks workgroups run
hipError_t launch_col2im(const void *cols, const ConvShape &g, bool is_f32, void *dx, hipStream_t st,
                         const SplitReduce *red = nullptr);

// Image gradient of a convolution, product and fold in one (conv_dx_body.hpp), the bits of the two passes it replaces:
// `a` is the g_x product of the column matrix as launch_gemm_nt takes it for kind 0 (A = codes of G, Bm = codes of the
// weight, K = out-features), a.C the image gradient [Nb, H, W, C].  launch_conv_pair: with the weight gradient's
// product `b` in the same launch on 128 x 128 tiles (conv_pair_available: no other tile is asked for), its k split by
// the plan (b.ws) and reduced behind it.
bool conv_dx_ok(int O, const ConvShape &s, bool is_f32);   // the shape is taken that way
hipError_t launch_conv_dx(const GemmArgs &a, const ConvShape &s, hipStream_t st);
bool conv_pair_available();
hipError_t launch_conv_pair(const GemmArgs &a, const ConvShape &s, int kindB, const GemmArgs &b, hipStream_t st);

// K3 / K3q on the column matrix of X [Nb, H, W, C] without storing it: same outputs as launch_hla /
// launch_hla_quant on launch_im2col's result, D = kh*kw*C.  Needs hla_conv_ok (C a multiple of the
// 128 / B features a lane owns).
bool hla_conv_ok(const ConvShape &g, int B);
hipError_t launch_hla_conv(const void *X, const ConvShape &g, int B, int r, int basis, bool is_f32, uint16_t *ThatT,
                           float *coeffT, hipStream_t st);
hipError_t launch_hla_quant_conv(const void *X, const ConvShape &g, int B, int r, int basis, bool is_f32, uint32_t k0,
                                 uint32_t k1, bool mant, int8_t *TqT, float *sT, float *coeffT, void *ws, hipStream_t st);

// Diagnostic: `blocks` workgroups of 4 wavefronts each run `iters` x 8 independent 32x32 MFMAs
// (kind 0: i8, K = 32; kind 1: bf16, K = 16) from registers.
hipError_t launch_mfma_probe(int kind, int blocks, int iters, float *sink, hipStream_t st);

}  // namespace hlq
