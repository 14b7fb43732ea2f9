// Host side of the C ABI: argument validation, the choice of kernel, tile shape
// and K split, and the launches.  No arithmetic of the matrix product happens
// here; everything numeric runs in the device kernels.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "../../include/prism_gemm.h"
#include "grid.hpp"
#include "launch.hpp"

namespace {

using prism::GemmParams;

constexpr int kComputeUnits = 256;
constexpr int kPersistentMaxSteps = 16;  // longest K loop (in K steps) the persistent kernel is chosen for
constexpr int kSkinnyRows = 64;          // rows of C up to which the kernel for few rows is chosen
constexpr int64_t kSkinnyMaxWorkgroups = 1 << 21;  // of 1024 threads: what one launch takes; tiles of 128 columns beyond
constexpr int kMaxSplit = 64;
constexpr int kVeryLongK = 512;              // K steps from which few 256x256 tiles with many slices beat small tiles
constexpr int kMinSliceStepsStaged = 8;      // shortest K loop (in K steps) a slice of the staged kernel gets
constexpr int64_t kIntMax = 2147483647;
constexpr int64_t kMaxTiles = kIntMax / 64;  // output tiles of all problems of a call

struct Problem {
    GemmParams p;
    prism_gemm_plan_t plan;
    int ab_dtype;
    int pipe_config;  // index into kPipeConfigs when plan.kernel is 2 or 3
    int dealt_rows;   // rows of C per workgroup of the kernel that deals K steps to waves (0: another kernel)
    bool odd_rows;    // of that kernel: operand rows that start in the middle of 32-bit words
    int total_units;  // (tile, unit) pairs the persistent kernel walks
};

bool valid_dtype_ab(int v) { return v == PRISM_DTYPE_BF16 || v == PRISM_DTYPE_F16 || v == PRISM_DTYPE_F32; }
bool valid_dtype_c(int v) { return v == PRISM_DTYPE_BF16 || v == PRISM_DTYPE_F16 || v == PRISM_DTYPE_F32; }
bool valid_layout(int v) { return v == PRISM_ROW_MAJOR || v == PRISM_COL_MAJOR; }
bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Elements spanned by a rows x cols matrix with leading dimension ld.
int64_t span(int layout, int64_t rows, int64_t cols, int64_t ld)
{
    if (rows == 0 || cols == 0) return 0;
    return layout == PRISM_ROW_MAJOR ? (rows - 1) * ld + cols : (cols - 1) * ld + rows;
}

bool overlaps(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes)
{
    if (!a || !b || a_bytes <= 0 || b_bytes <= 0) return false;
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + static_cast<uintptr_t>(b_bytes) && b0 < a0 + static_cast<uintptr_t>(a_bytes);
}

// Hooks for tests and experiments, read from the environment once (at the first call that
// needs them, or again on prism_reread_environment) and kept:
//   PRISM_GEMM_CONFIG=0|1      pins the pipeline's tile (0: 256x256, 1: 128x128) and keeps few rows on tiles
//   PRISM_PERSISTENT=0|1       never / whenever possible use the persistent kernel
//   PRISM_LOG=1                one line per launch on stderr: problem, kernel, tile, split
struct Hooks {
    int pipe_config = -1;  // -1: the library decides
    int persistent = -1;   // -1: the library decides, 0: never, 1: whenever possible
    bool log = false;
};
Hooks g_hooks;
bool g_hooks_loaded = false;
std::mutex g_hooks_mutex;

void load_hooks_locked()
{
    Hooks h;
    if (const char* e = std::getenv("PRISM_GEMM_CONFIG"); e && *e) {
        const int v = std::atoi(e);
        if (v == 0 || v == 1) h.pipe_config = v;  // (others name nothing)
    }
    if (const char* e = std::getenv("PRISM_PERSISTENT"); e && (e[0] == '0' || e[0] == '1')) h.persistent = e[0] - '0';
    if (const char* e = std::getenv("PRISM_LOG"); e && e[0] == '1') h.log = true;
    g_hooks = h;
    g_hooks_loaded = true;
}

Hooks hooks()
{
    std::lock_guard<std::mutex> lock(g_hooks_mutex);
    if (!g_hooks_loaded) load_hooks_locked();
    return g_hooks;
}

// ---- K split: the library's own choice of slices for `units` output tiles (of all problems).
// A split costs a round trip of fp32 partial sums and a second kernel: it pays only for
// a long K loop, and every slice must keep a K loop of its own.  Small tiles run two
// workgroups per compute unit, so they are split until there are about twice as many
// workgroups as compute units (measured: 512x512x16384 23 us with 16 slices, 28 with
// 8 or 32).  short_steps: 16-bit operands on the pipeline (a K step of fp32 operands holds four
// times the matrix instructions).
int64_t slices_wanted(int64_t units, int64_t ksteps, bool small_tiles, bool short_steps)
{
    const int64_t slots = small_tiles ? 2 * kComputeUnits : kComputeUnits;
    const int64_t min_slice = !short_steps ? kMinSliceStepsStaged : (small_tiles ? 16 : 32);
    const int64_t min_k = !short_steps ? 4 * kMinSliceStepsStaged : 64;
    if (units * 2 > slots || ksteps < min_k) return 1;
    int64_t want = slots / units;
    if (want > ksteps / min_slice) want = ksteps / min_slice;
    if (small_tiles && want > 32) want = 32;
    if (want > kMaxSplit) want = kMaxSplit;
    return want < 1 ? 1 : want;
}
struct Slices {
    int64_t count, steps;  // slices, none of them empty, and K steps of each but the last
};
Slices slices_of(int64_t want, int64_t ksteps)
{
    const int64_t steps = ceil_div(ksteps, want < ksteps ? want : ksteps);
    return Slices{ceil_div(ksteps, steps), steps};
}

// ---- 256x256 or 128x128 tiles where an operand is not contiguous along K: whichever the measured
// times of a K step and of a round of workgroups predict to be faster.  (Microseconds.  Large tiles,
// one workgroup per compute unit: 1.07 per K step, 15.6 per round for the first loads and the
// epilogue, 5.1 of them hidden in the first; small ones: 1.05 per K step with two workgroups per
// compute unit, 0.42 where each has one to itself, and 5 per round; the reduction by the megabyte of
// partial sums.)  The rounds of small tiles with loops of fewer than twelve steps run into each
// other, and large ones must then be 15 % faster, otherwise 5 %; from kVeryLongK steps on small
// tiles take a tenth longer than predicted.  Measured over 3400 products of 17 to 4096 rows and columns and 1 to 1024
// K steps in 1 to 64 problems: 9 are more than 3 % slower than with small tiles (at most 17 %), and
// 21 more than 5 % slower than with the better choice.  Taking large tiles for 128 of them or for any very
// long K was up to three times slower: 256 x 256 x 65536 has 32 slices of one large tile, 128 of small ones.
bool large_k_row_tiles(int64_t M, int64_t N, int64_t batch, int64_t ksteps, int64_t requested_split)
{
    // (more small tiles than a launch can take: the large ones may still do)
    if (ceil_div(M, 128) * ceil_div(N, 128) > kMaxTiles / batch) return true;
    const int64_t large = ceil_div(M, 256) * ceil_div(N, 256) * batch, small = ceil_div(M, 128) * ceil_div(N, 128) * batch;
    const Slices ls = slices_of(requested_split ? requested_split : slices_wanted(large, ksteps, false, true), ksteps);
    const Slices ss = slices_of(requested_split ? requested_split : slices_wanted(small, ksteps, true, true), ksteps);
    const double slab_mb = 4e-6 * static_cast<double>(M) * static_cast<double>(N) * static_cast<double>(batch);
    const double round_l = 1.07 * static_cast<double>(ls.steps) + 15.6;
    double t_large = static_cast<double>(ceil_div(large * ls.count, kComputeUnits)) * round_l - 5.1;
    if (ls.count > 1) t_large += 0.83 * slab_mb * static_cast<double>(ls.count);
    const bool alone = small * ss.count <= kComputeUnits;
    const double round_s = (alone ? 0.42 : 1.05) * static_cast<double>(ss.steps) + 5.0;
    const double pairs = static_cast<double>(small * ss.count) / (2 * kComputeUnits);
    const double rounds_s = alone || pairs <= 1.0 ? 1.0 : ksteps < 12 ? pairs : std::ceil(pairs);
    double t_small = rounds_s * round_s - 0.7;
    if (ss.count > 1) t_small += 4.0 + 0.44 * slab_mb * static_cast<double>(ss.count);
    return t_large < (ksteps >= kVeryLongK ? 1.05 : ksteps >= 12 ? 0.95 : 0.85) * t_small;
}

// ---- few rows: the kernel without tiles, or tiles with a split?  Both are predicted from times measured
// on 2864 products of 1 to 64 rows, 1 to 16384 columns and K from 8 to 65536 in 1 to 128 problems
// (16-bit and fp32, rows on chunks, words and single elements; the predictions are mostly within
// 8 to 21 %).  By the predictions 69 of them are more than 5 % slower than with the other
// kernel.  By size alone, with no look at alignment and rounds, 124 were more than 3 % slower than
// tiles, up to five times: a long way for few workgroups (54 x 52 x 59410: 148 us, with tiles and 31 slices
// 32; 64 x 512 x 16384: 27.7 and 19.6) and workgroups in many rounds (125 problems of 56 x 584 x 59:
// 34.9 and 17.3).  Where no split can be made the tiles' way is as long: two workgroups of 1024 K steps
// for 16 x 512 x 65536, against 32 of the other kernel.
struct FewRowsTimes {
    double first, round;      // us: a call of one round of workgroups, and each further round
    double unit_bytes_ns;     // bytes a compute unit takes in per ns
    double bytes_us;          // MB per us from memory
};
struct TileTimes {
    double first, round;      // us: a call of one round of workgroups, and each further round
    double step, pair_step;   // us of a K step, at one and at two workgroups per compute unit (256x256: always one)
    double reduce, reduce_mb; // us of a reduction, and per MB of partial sums
    double bytes_us;
};
// 16-bit elements in rows that start on whole 4-byte words, 16-bit ones in others, fp32
constexpr FewRowsTimes kFewRows[3] = {{4.1, 1.9, 114, 5.0}, {4.5, 3.4, 42, 3.2}, {4.1, 2.4, 65, 4.7}};
constexpr TileTimes kStagedTiles[3] = {{4.9, 4.3, 0.65, 1.02, 6.2, 2.0, 5.0}, {5.1, 3.8, 0.98, 1.88, 10.4, 0.7, 3.3}, {4.7, 3.0, 2.12, 4.0, 6.0, 1.4, 1.95}};
constexpr TileTimes kPipeTiles[3] = {{4.3, 14.0, 0.33, 0.55, 4.1, 1.33, 5.0}, {}, {4.2, 2.9, 1.74, 3.5, 5.9, 0.46, 2.1}};  // (whole words always)
constexpr double kFewRowsMargin = 2.0;  // us by which tiles must be ahead: what a prediction of short calls is worth
constexpr TileTimes kLargePipeTiles = {7.7, 7.1, 1.05, 1.05, 0.8, 5.0, 3.55};

// `bytes`: operands, once each, and C
double few_rows_us(const FewRowsTimes& t, int64_t rows, int64_t columns, int waves, int64_t workgroups, int64_t ksteps, double bytes)
{
    // workgroups of a compute unit at a time: four waves per SIMD, and their steps in LDS
    const int64_t lds = waves * (rows + columns) * 128, fit = (160 << 10) / lds;
    const int64_t resident = fit < 1 ? 1 : fit < 16 / waves ? fit : 16 / waves;
    const double unit_bytes = static_cast<double>(ceil_div(workgroups, kComputeUnits) * (rows + columns)) * 128.0 * static_cast<double>(ksteps);
    // (beyond what the memory-side cache can hold from call to call, a compute unit gets 45)
    const double rate = bytes > 1.2e8 && t.unit_bytes_ns > 45.0 ? 45.0 : t.unit_bytes_ns;
    const double way = 1e-3 * unit_bytes / rate, all = 1e-6 * bytes / t.bytes_us;
    return t.first + t.round * static_cast<double>(ceil_div(workgroups, kComputeUnits * resident) - 1) + (way > all ? way : all);
}
double tiles_us(const TileTimes& t, bool large, int64_t workgroups, const Slices& slices, double slab_bytes, double bytes)
{
    const bool alone = large || workgroups <= kComputeUnits;
    const double rounds = static_cast<double>(ceil_div(workgroups, (alone ? 1 : 2) * kComputeUnits));
    double us = t.first + t.round * (rounds - 1.0) + rounds * static_cast<double>(slices.steps) * (alone ? t.step : t.pair_step);
    if (us < 1e-6 * bytes / t.bytes_us) us = 1e-6 * bytes / t.bytes_us;
    if (slices.count > 1) us += t.reduce + t.reduce_mb * 1e-6 * slab_bytes * static_cast<double>(slices.count);
    return us;
}

// ---- K steps dealt to the waves of a workgroup (dealt.hip), or tiles with a K loop of their own?  Both
// are predicted, from times measured on 3400 products of 17 to 4000 rows and columns and K from 17
// to 60000 in 1 to 200 problems (all layout pairs; 16-bit operands whose rows start on whole words, 16-bit
// ones that do not, fp32).  The predictions are mostly within 10 to 20 %, so tiles must be behind by
// kDealtMargin, more for calls of several rounds and for long rows of both operands, whose loads
// touch many pages; and operands beyond what the memory-side cache holds from call to call stay on
// tiles.  Measured over all of them, the calls take 0.69 of the time that tiles alone take (the
// best choice each time: 0.66), and 25 are more than 5 % slower (the worst 32 %).
struct DealtTimes {
    double first, round;      // us: a call of one round of workgroups, and each further round
    double step;              // us of a wave's K step
    double unit_kb_us;        // kB a compute unit takes in per us
    double k_rows;            // by how much more an operand costs that is not contiguous along K
    double mb_us, reduce, reduce_mb;  // MB per us from memory; us of a reduction, and per MB of partial sums
};
struct DealtShape {
    int rows, columns, waves, waves_m, resident;  // of a workgroup; waves side by side along m; workgroups of a compute unit
    int split_workgroups;                         // of all units together, up to which sums are split (0: never)
    DealtTimes times[3];                          // by kind of operands, as above
};
constexpr DealtShape kDealtShapes[4] = {
    {32, 32, 4, 1, 5, 2 * kComputeUnits,
     {{3.4, 2.3, 0.05, 81.3, 0.29, 4.0, 3.3, 0.05}, {3.8, 2.8, 0.01, 65.4, 0.27, 3.4, 4.8, 0.01}, {3.9, 3.1, 0.01, 52.5, 0.02, 4.0, 4.2, 0.01}}},
    {32, 32, 8, 1, 2, 2 * kComputeUnits,
     {{3.0, 1.8, 0.59, 90.7, 0.36, 4.1, 3.4, 0.16}, {3.3, 2.0, 0.82, 68.0, 0.27, 5.3, 5.3, 0.01}, {3.8, 2.6, 0.27, 60.1, 0.04, 3.1, 4.3, 0.12}}},
    {64, 64, 8, 1, 1, 0,
     {{4.6, 3.6, 0.09, 83.4, 0.09, 3.4, 3.2, 0.24}, {5.0, 4.1, 0.49, 66.9, 0.10, 3.0, 4.6, 0.07}, {5.6, 4.6, 0.04, 33.6, 0.01, 3.5, 4.5, 0.39}}},
    {128, 64, 8, 2, 1, kComputeUnits,
     {{5.1, 4.3, 0.01, 92.6, 0.08, 2.9, 2.6, 0.26}, {5.7, 4.9, 0.01, 71.0, 0.05, 2.7, 3.6, 0.17}, {5.5, 4.6, 1.67, 34.1, 0.01, 2.0, 4.3, 0.34}}},
};
constexpr double kDealtMargin = 1.15, kDealtRoundMargin = 0.1, kDealtLongRowMargin = 0.1;
constexpr double kDealtMaxMb = 100.0;
constexpr int kDealtLongRow = 48;       // K steps
constexpr int kDealtMinSliceSteps = 8;
double dealt_us(const DealtShape& shape, const DealtTimes& t, int64_t workgroups, const Slices& slices, int k_row_operands, double slab_mb, double mb)
{
    const double rounds = static_cast<double>(ceil_div(workgroups, kComputeUnits * shape.resident));
    const double kb = 0.128 * static_cast<double>((shape.rows + shape.columns * shape.waves_m) * slices.steps);
    const double way = static_cast<double>(ceil_div(workgroups, kComputeUnits)) * kb / t.unit_kb_us * (1.0 + t.k_rows * k_row_operands);
    const double waits = rounds * static_cast<double>(ceil_div(slices.steps, shape.waves / shape.waves_m)) * t.step;
    const double partial = slices.count > 1 ? slab_mb * static_cast<double>(slices.count) : 0.0;
    double us = t.first + t.round * (rounds - 1.0) + (way > waits ? way : waits);
    if (us < 2.0 + mb / t.mb_us) us = 2.0 + mb / t.mb_us;
    return slices.count > 1 ? us + t.reduce + t.reduce_mb * partial : us;
}
// How far the rounding errors of a sum add up, in additions one after the other: the matrix instructions
// of one wave's steps, then the sums of its waves, then those of the slices.  A call's must not be longer than the
// tiles' would be (1620 x 122 x 3120 fp32, thirteen steps a wave against slices of eight: 3.6e-7
// off the exact product against 3.1e-7).
int64_t sum_length(int64_t steps, int64_t waves, int64_t slices, int esize)
{
    return ceil_div(steps, waves) * (esize == 4 ? 8 : 2) + (steps < waves ? steps : waves) + slices;
}
// The tiles' side of it: staged kernel by kind, pipeline with 128x128 tiles of 16-bit operands contiguous along
// K, of others, of fp32, and with 256x256 tiles.  (As tiles_us, fitted to these products.)
constexpr TileTimes kTilesStaged[3] = {{6.3, 5.0, 0.54, 1.16, 3.9, 0.39, 2.9}, {6.4, 4.6, 0.73, 1.40, 4.6, 0.37, 2.4}, {6.1, 7.2, 1.88, 3.85, 5.7, 0.34, 2.4}};
constexpr TileTimes kTilesPipe = {4.6, 3.0, 0.54, 0.68, 1.6, 0.45, 2.8}, kTilesKRows = {4.5, 3.8, 0.55, 0.79, 1.6, 0.41, 3.3};
constexpr TileTimes kTilesPipeF32 = {5.4, 6.6, 1.78, 3.77, 3.0, 0.26, 2.2}, kTilesLarge = {7.2, 7.4, 1.03, 1.03, 0.0, 1.37, 2.3};
double loop_tiles_us(const TileTimes& t, bool large, int64_t workgroups, const Slices& slices, double slab_mb, double mb)
{
    const int64_t per_unit = ceil_div(workgroups, kComputeUnits);
    const double steps = static_cast<double>(slices.steps);
    double us = large ? t.first + static_cast<double>(per_unit) * steps * t.step + t.round * static_cast<double>(per_unit - 1)
                      : t.first + t.round * static_cast<double>(ceil_div(per_unit, 2) - 1) +
                            steps * (static_cast<double>(per_unit / 2) * t.pair_step + static_cast<double>(per_unit % 2) * t.step);
    if (us < 2.0 + mb / t.bytes_us) us = 2.0 + mb / t.bytes_us;
    return slices.count > 1 ? us + t.reduce + t.reduce_mb * slab_mb * static_cast<double>(slices.count) : us;
}

// Validates everything, normalises to a row-major C and chooses the launch.
prism_status_t make_problem(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K,
                            const void* A, int64_t lda, int64_t strideA, const void* B, int64_t ldb,
                            int64_t strideB, const void* C, int64_t ldc, int64_t strideC, int64_t batch,
                            bool need_pointers, Problem* out, bool allow_few_rows = true, bool allow_dealt = true)
{
    if (!d || !out) return PRISM_ERR_INVALID_ARG;
    if (!valid_dtype_ab(d->ab_dtype) || !valid_dtype_c(d->c_dtype) || !valid_layout(d->layout_a) ||
        !valid_layout(d->layout_b) || !valid_layout(d->layout_c))
        return PRISM_ERR_UNSUPPORTED;
    if (d->ab_dtype == PRISM_DTYPE_F32 && d->c_dtype != PRISM_DTYPE_F32) return PRISM_ERR_UNSUPPORTED;
    if (d->reserved != 0) return PRISM_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0 || batch < 0 || d->split_k < 0) return PRISM_ERR_INVALID_ARG;
    if (M > kIntMax || N > kIntMax || K > kIntMax - 64 || batch > kIntMax) return PRISM_ERR_INVALID_ARG;
    if (lda < 1 || ldb < 1 || ldc < 1) return PRISM_ERR_INVALID_ARG;
    if (lda < (d->layout_a == PRISM_ROW_MAJOR ? K : M)) return PRISM_ERR_INVALID_ARG;
    if (ldb < (d->layout_b == PRISM_ROW_MAJOR ? N : K)) return PRISM_ERR_INVALID_ARG;
    if (ldc < (d->layout_c == PRISM_ROW_MAJOR ? N : M)) return PRISM_ERR_INVALID_ARG;
    if (!(d->alpha == d->alpha) || !(d->beta == d->beta)) return PRISM_ERR_INVALID_ARG;  // NaN scales

    std::memset(out, 0, sizeof(*out));
    const Hooks hk = hooks();
    prism_gemm_plan_t& plan = out->plan;
    plan.split_k = 1;
    const bool empty = M == 0 || N == 0 || batch == 0;
    if (empty) return PRISM_OK;  // plan.kernel == 0: nothing to do

    const int64_t c_span = span(d->layout_c, M, N, ldc);
    const int64_t a_span = span(d->layout_a, M, K, lda), b_span = span(d->layout_b, K, N, ldb);
    const int c_esize = d->c_dtype == PRISM_DTYPE_F32 ? 4 : 2;
    const int ab_esize = d->ab_dtype == PRISM_DTYPE_F32 ? 4 : 2;
    const int epc = 16 / ab_esize;  // operand elements per 16-byte chunk
    if (need_pointers) {
        if (!C || (K > 0 && (!A || !B))) return PRISM_ERR_INVALID_ARG;
    }
    if (batch > 1) {
        const int64_t sc = strideC < 0 ? -strideC : strideC;
        if (sc < c_span) return PRISM_ERR_INVALID_ARG;  // C matrices of the batch would overlap
    }
    if (batch == 1 || (strideA >= 0 && strideB >= 0 && strideC >= 0)) {
        // C must not share memory with A or B (checked over the whole batch extent)
        const int64_t nb = batch - 1;
        const int64_t c_bytes = (nb * strideC + c_span) * c_esize;
        if (overlaps(C, c_bytes, A, (nb * strideA + a_span) * ab_esize) ||
            overlaps(C, c_bytes, B, (nb * strideB + b_span) * ab_esize))
            return PRISM_ERR_INVALID_ARG;
    }

    // ---- normalise: a column-major C is the row-major C^T = B^T A^T
    GemmParams& p = out->p;
    int64_t a_sm = d->layout_a == PRISM_ROW_MAJOR ? lda : 1, a_sk = d->layout_a == PRISM_ROW_MAJOR ? 1 : lda;
    int64_t b_sk = d->layout_b == PRISM_ROW_MAJOR ? ldb : 1, b_sn = d->layout_b == PRISM_ROW_MAJOR ? 1 : ldb;
    if (d->layout_c == PRISM_COL_MAJOR) {
        plan.swapped = 1;
        p.A = static_cast<const char*>(B); p.a_sm = b_sn; p.a_sk = b_sk; p.batch_a = strideB;
        p.B = static_cast<const char*>(A); p.b_sn = a_sm; p.b_sk = a_sk; p.batch_b = strideA;
        p.M = static_cast<int>(N); p.N = static_cast<int>(M);
        p.bias_along_m = 1;
    } else {
        p.A = static_cast<const char*>(A); p.a_sm = a_sm; p.a_sk = a_sk; p.batch_a = strideA;
        p.B = static_cast<const char*>(B); p.b_sn = b_sn; p.b_sk = b_sk; p.batch_b = strideB;
        p.M = static_cast<int>(M); p.N = static_cast<int>(N);
        p.bias_along_m = 0;
    }
    p.K = static_cast<int>(K);
    p.C = static_cast<char*>(const_cast<void*>(C));
    p.ldc = ldc;
    p.batch_c = strideC;
    p.batch = static_cast<int>(batch);
    p.bias = d->bias;
    p.alpha = d->alpha;
    p.beta = d->beta;
    p.c_dtype = d->c_dtype;
    out->ab_dtype = d->ab_dtype;

    // ---- alignment facts
    const bool a_kfast = p.a_sk == 1, b_kfast = p.b_sk == 1;
    // K-contiguous with 16-byte aligned rows
    const bool a_vec = a_kfast && aligned(p.A, 16) && p.a_sm % epc == 0 && (p.batch == 1 || p.batch_a % epc == 0);
    const bool b_vec = b_kfast && aligned(p.B, 16) && p.b_sn % epc == 0 && (p.batch == 1 || p.batch_b % epc == 0);

    if (K == 0) {  // C <- bias + beta*C: only the epilogue kernel runs
        plan.kernel = 0;
        p.split_k = 0;
        p.tiles_m = p.tiles_n = 0;
        return PRISM_OK;
    }

    // ---- kernel and tile shape
    const int64_t step_k = 128 / ab_esize;  // a K step is 128 bytes of every operand row
    const int64_t ksteps = ceil_div(K, step_k);
    const bool pitch_ok = p.a_sm < (int64_t{1} << 21) && p.b_sn < (int64_t{1} << 21) && p.a_sk < (int64_t{1} << 21) &&
                          p.b_sk < (int64_t{1} << 21);
    // An operand contiguous along m (column-major A) or n (row-major B): whole, aligned 16-byte
    // chunks of every k-row
    const bool a_along_m = p.a_sm == 1 && p.a_sk != 1 && aligned(p.A, 16) && p.a_sk % epc == 0 && p.M % epc == 0 &&
                           (p.batch == 1 || p.batch_a % epc == 0);
    const bool b_along_n = p.b_sn == 1 && p.b_sk != 1 && aligned(p.B, 16) && p.b_sk % epc == 0 && p.N % epc == 0 &&
                           (p.batch == 1 || p.batch_b % epc == 0);
    const bool pipe_ok = (a_vec || a_along_m) && (b_vec || b_along_n) && K % step_k == 0 && pitch_ok;
    // ---- few rows: no tile loop and no split, see skinny.hip.  Both operands K-contiguous, K at
    // least a chunk; chosen over tiles further down.  Not for more than 32 rows where 128x128 tiles give
    // half of the compute units a workgroup, because every 16 or 32 columns read all rows of A again
    // (64 x 16384 x 4096: 39.2 us with tiles, 41.3 without; 128 problems of 64 x 512 x 512: 24.4 and 38.6).
    // Two blocks of columns where that still gives every compute unit a workgroup, and where the last round of
    // workgroups is not much emptier than with one (16 x 8400 x 4096, 263 workgroups or 525: 20.8 -> 15.8 us;
    // 5 x 8223 x 10880 49.2 -> 40.5, 4 x 18000 x 4096 35.3 -> 29.1).  More than 16 rows pay for one block with half as
    // many loads again: only where B is what counts (30 x 9000 x 4096 21.4 -> 19.8, but 28 x 8500 x 1280 8.9 -> 10.8).
    const int64_t skinny_m = p.M <= 16 ? 16 : p.M <= 32 ? 32 : 64;
    const auto last_round = [](int64_t workgroups) {
        return static_cast<double>(workgroups) / static_cast<double>(ceil_div(workgroups, kComputeUnits) * kComputeUnits);
    };
    const int64_t one_block = ceil_div(p.N, 16) * batch, two_blocks = ceil_div(p.N, 32) * batch;
    const double b_bytes = static_cast<double>(ab_esize) * static_cast<double>(p.N) * static_cast<double>(K) * static_cast<double>(p.batch_b == 0 ? 1 : batch);
    const bool uneven = last_round(one_block) > 1.15 * last_round(two_blocks) && (p.M <= 16 || b_bytes > 4.8e7) &&
                        !prism::few_rows_stream_b(p.N, K, ab_esize, batch, p.batch_b);
    const int64_t skinny_n = two_blocks >= kComputeUnits && !uneven ? 32 : 16;
    const int64_t skinny_workgroups = ceil_div(p.N, skinny_n) * batch;
    // as many waves as have K steps of their own, sixteen only where workgroups are few
    // (and up to one per compute unit where that leaves four to eight whole steps to a wave, all of them on their way at
    // once: 16 x 4096 x 4096 8.6 -> 8.2 us, 8 x 2500 x 8192 11.1 -> 10.6; but 16 x 4096 x 2048 5.6 -> 6.2,
    // 5 x 4000 x 16384 28.4 -> 29.1, 60 x 4096 x 4096 11.6 -> 12.2, and 7 x 3967 x 4801, whose rest comes last, 10.6 -> 12.0)
    const bool four_to_eight = ksteps >= 64 && ksteps <= 128 && K % step_k == 0 && skinny_m <= 32 && skinny_n == 16 && skinny_workgroups <= kComputeUnits;
    const int skinny_waves = ksteps >= 32 && (skinny_workgroups <= kComputeUnits / 2 || four_to_eight) ? 16 : ksteps >= 8 ? 8 : 4;
    const bool many_tiles = p.M > 32 && pipe_ok && ceil_div(p.N, prism::kStagedTileN) * batch >= kComputeUnits / 2;
    const bool few_rows = allow_few_rows && p.M <= kSkinnyRows && a_kfast && b_kfast && K >= epc && pitch_ok && d->split_k <= 1 &&
                          hk.pipe_config < 0 && hk.persistent != 1 && skinny_workgroups <= kSkinnyMaxWorkgroups && !many_tiles;
    int tile_m = prism::kStagedTileM, tile_n = prism::kStagedTileN, waves = prism::kStagedWaves;
    plan.kernel = 1;
    if (pipe_ok) {
        plan.kernel = 2;
        int cfg = hk.pipe_config;
        if (cfg < 0) {
            // Big tiles when they give at least half of the compute units a workgroup, or for a
            // very long K (the split then needs fewer slices); else small tiles, two workgroups
            // per compute unit.  Measured: 128x128 tiles win on square problems up to 2560^3
            // (2048^3: 26 against 40 us) and on 1024x1024x8192 (30 against 38 us), 256x256 tiles
            // from 3072^3 on and on 1024x1024x32768.
            // (operands that are not contiguous along K: see large_k_row_tiles)
            const int64_t big = ceil_div(p.M, 256) * ceil_div(p.N, 256) * batch;
            if (a_vec && b_vec) cfg = (big >= kComputeUnits / 2 || ksteps >= kVeryLongK) ? 0 : 1;
            else cfg = large_k_row_tiles(p.M, p.N, batch, ksteps, d->split_k) ? 0 : 1;
        }
        // an operand that is not K-contiguous is kept as k-rows in LDS, with either tile
        if (!a_vec || !b_vec) cfg = (cfg == 0 ? 9 : 2) + (!a_vec ? (!b_vec ? 2 : 1) : 0);
        // fp32 operands: 128x128 tiles in all four layout pairs
        if (ab_esize == 4) cfg = 5 + (b_vec ? 0 : 1) + (a_vec ? 0 : 2);
        out->pipe_config = cfg;
        tile_m = prism::kPipeConfigs[cfg].tile_m;
        tile_n = prism::kPipeConfigs[cfg].tile_n;
        waves = prism::kPipeConfigs[cfg].waves;
    }
    const int64_t tiles_m = ceil_div(p.M, tile_m), tiles_n = ceil_div(p.N, tile_n);
    if (tiles_m * tiles_n > kMaxTiles || tiles_m * tiles_n * batch > kMaxTiles) return PRISM_ERR_INVALID_ARG;

    // ---- K split: explicit request, or enough slices to give every compute unit a workgroup
    const int64_t units = tiles_m * tiles_n * batch;
    const size_t slab_bytes = static_cast<size_t>(batch) * p.M * p.N * sizeof(float);
    const int64_t want = d->split_k ? d->split_k : slices_wanted(units, ksteps, tile_m != 256, plan.kernel == 2 && ab_esize == 2);
    Slices slices = slices_of(want, ksteps);
    size_t ws_need = slices.count > 1 ? slab_bytes * static_cast<size_t>(slices.count) : 0;
    if (slices.count > 1 && need_pointers && (!d->workspace || d->workspace_bytes < ws_need)) {
        if (d->split_k > 1) return PRISM_ERR_WORKSPACE;
        // The library's own choice makes do with as many slices as the workspace holds.  Its size was asked
        // for without pitches and alignments, which may send the call to another kernel with other
        // wishes, and no split at all is far slower than a few slices less: 896 x 64 x 60032 at an
        // odd offset 74 us with 32 slices and 954 with one.
        const int64_t held = d->workspace ? static_cast<int64_t>(d->workspace_bytes / slab_bytes) : 0;
        slices = slices_of(held > 1 ? held : 1, ksteps);
        ws_need = slices.count > 1 ? slab_bytes * static_cast<size_t>(slices.count) : 0;
    }
    const int64_t split = slices.count, slice_steps = slices.steps;
    if (few_rows) {
        const double bytes = static_cast<double>(ab_esize) * static_cast<double>(K) *
                                 (static_cast<double>(p.M) * static_cast<double>(p.batch_a == 0 ? 1 : batch) +
                                  static_cast<double>(p.N) * static_cast<double>(p.batch_b == 0 ? 1 : batch)) +
                             static_cast<double>(slab_bytes) / 4.0 * c_esize * (p.beta != 0.0f ? 2 : 1);
        const bool words = aligned(p.A, 4) && aligned(p.B, 4) && p.a_sm % 2 == 0 && p.b_sn % 2 == 0 &&
                           (batch == 1 || (p.batch_a % 2 == 0 && p.batch_b % 2 == 0));
        const int kind = ab_esize == 4 ? 2 : words ? 0 : 1;
        const TileTimes& tiles = plan.kernel == 1 ? kStagedTiles[kind] : tile_m == 256 ? kLargePipeTiles : kPipeTiles[kind];
        // The times were taken on operands that the memory-side cache holds in part.  From memory a tile's
        // K step takes longer, most where every tile has a compute unit to itself (8 x 15702 x 2816: 36.6 us
        // with 123 tiles, 21.7 without), so tiles must be ahead by half there and by a fifth elsewhere;
        // not so for a long way of few workgroups, 1.5 MB each, measured both ways.
        const bool long_way = skinny_workgroups <= kComputeUnits && (skinny_m + skinny_n) * K * ab_esize > (3 << 19) && slices.count > 1;
        const double ahead = long_way ? 1.0 : plan.kernel == 2 && slices.count == 1 ? 1.5 : 1.2;
        if (few_rows_us(kFewRows[kind], skinny_m, skinny_n, skinny_waves, skinny_workgroups, ksteps, bytes) <=
            ahead * tiles_us(tiles, tile_m == 256, units * split, slices, static_cast<double>(slab_bytes), bytes) + kFewRowsMargin) {
            plan.kernel = 4;
            plan.tile_m = static_cast<int32_t>(skinny_m);
            plan.tile_n = static_cast<int32_t>(skinny_n);
            plan.tile_k = static_cast<int32_t>(step_k);
            plan.tiles_m = 1;
            plan.tiles_n = ceil_div(p.N, skinny_n);
            plan.workgroups = skinny_workgroups;
            plan.waves = skinny_waves;
            p.split_k = 1;
            p.k_slice = p.K;
            p.tiles_m = 1;
            p.tiles_n = static_cast<int>(plan.tiles_n);
            return PRISM_OK;
        }
    }
    // ---- few tiles for the chip, or short K loops: K steps dealt to the waves of smaller workgroups
    // (its loads are whole chunks: they lie inside a row, or, of k-rows shorter than a chunk, inside the operand,
    // those of all steps but the last towards its end, those of the last, at the end of a row, towards its start)
    auto chunks = [&](bool kfast, int64_t extent, int64_t pitch) {
        if (kfast || extent >= epc) return (kfast ? K : extent) >= epc;
        return K > step_k && (K - 1) % step_k * pitch + pitch + extent >= epc;
    };
    if (allow_dealt && chunks(a_kfast, p.M, p.a_sk) && chunks(b_kfast, p.N, p.b_sk) && pitch_ok && d->split_k <= 1 && hk.pipe_config < 0 && hk.persistent != 1) {
        const double slab_mb = 1e-6 * static_cast<double>(slab_bytes);
        const double mb = 1e-6 * ab_esize * static_cast<double>(batch) * static_cast<double>(K) * (static_cast<double>(p.M) + static_cast<double>(p.N)) +
                          slab_mb / 4.0 * c_esize * (p.beta != 0.0f ? 2 : 1);
        const bool word_pitches = (a_kfast ? p.a_sm : p.a_sk) % 2 == 0 && (b_kfast ? p.b_sn : p.b_sk) % 2 == 0 &&
                                  (batch == 1 || (p.batch_a % 2 == 0 && p.batch_b % 2 == 0));
        const bool word_bases = aligned(p.A, 4) && aligned(p.B, 4);
        const int kind = ab_esize == 4 ? 2 : word_pitches && word_bases ? 0 : 1;
        const int k_row_operands = (a_kfast ? 0 : 1) + (b_kfast ? 0 : 1);
        const TileTimes& tiles = plan.kernel == 1 ? kTilesStaged[kind] : ab_esize == 4 ? kTilesPipeF32 : tile_m == 256 ? kTilesLarge : k_row_operands ? kTilesKRows : kTilesPipe;
        double best = mb <= kDealtMaxMb ? loop_tiles_us(tiles, tile_m == 256, units * split, slices, slab_mb, mb) : 0.0;
        const double margin = kDealtMargin + (k_row_operands == 0 && ksteps >= kDealtLongRow ? kDealtLongRowMargin : 0.0);
        const int64_t tiles_length = sum_length(slices.steps, 1, slices.count, ab_esize);
        const DealtShape* chosen = nullptr;
        Slices chosen_slices{1, ksteps};
        for (const DealtShape& shape : kDealtShapes) {
            if (best <= 0.0) break;
            const int64_t own = ceil_div(p.M, shape.rows) * ceil_div(p.N, shape.columns);
            if (own > kMaxTiles / batch) continue;
            int64_t most = d->split_k ? 1 : shape.split_workgroups / (own * batch);
            if (most > ksteps / kDealtMinSliceSteps) most = ksteps / kDealtMinSliceSteps;
            if (most > kMaxSplit) most = kMaxSplit;
            if (need_pointers && most > 1) {
                const int64_t held = d->workspace ? static_cast<int64_t>(d->workspace_bytes / slab_bytes) : 0;
                if (most > held) most = held;
            }
            // whole sums, or as many slices as give every compute unit its workgroups
            for (int64_t count : {int64_t{1}, most}) {
                if (count < 1 || (count == 1 && chosen == &shape)) continue;
                const Slices some = slices_of(count, ksteps);
                if (sum_length(some.steps, shape.waves / shape.waves_m, some.count, ab_esize) > tiles_length) continue;
                const int64_t workgroups = own * batch * some.count;
                const double us = dealt_us(shape, shape.times[kind], workgroups, some, k_row_operands, slab_mb, mb);
                const double rounds = static_cast<double>(ceil_div(workgroups, kComputeUnits * shape.resident));
                const double needed = chosen ? us : us * (margin + kDealtRoundMargin * (rounds - 1.0));
                if (needed >= best) continue;
                best = us;
                chosen = &shape;
                chosen_slices = some;
            }
        }
        if (chosen) {
            // The schedule deals blocks of four tile rows, one below the other, to neighbouring workgroups: 128 rows
            // are a block of four, two or one.
            plan.tile_m = 128;
            plan.tile_n = chosen->columns;
            plan.tile_k = static_cast<int32_t>(step_k);
            plan.waves = chosen->waves;
            plan.split_k = static_cast<int32_t>(chosen_slices.count);
            plan.tiles_m = ceil_div(p.M, 128);
            plan.tiles_n = ceil_div(p.N, chosen->columns);
            p.tiles_m = static_cast<int>(ceil_div(p.M, chosen->rows));
            p.tiles_n = static_cast<int>(plan.tiles_n);
            p.split_k = static_cast<int>(chosen_slices.count);
            p.k_slice = static_cast<int>(chosen_slices.steps * step_k);
            p.partial = p.split_k > 1 ? static_cast<float*>(d->workspace) : nullptr;
            plan.workgroups = static_cast<int64_t>(p.tiles_m) * p.tiles_n * batch * p.split_k;
            plan.workspace_bytes = p.split_k > 1 ? slab_bytes * static_cast<size_t>(p.split_k) : 0;
            out->dealt_rows = chosen->rows;
            // (a row that starts in the middle of a word is read from the word before: there must be one)
            out->odd_rows = kind == 1 && word_bases && (batch == 1 || (p.batch_a >= 0 && p.batch_b >= 0));
            return PRISM_OK;
        }
    }
    p.split_k = static_cast<int>(split);
    p.k_slice = static_cast<int>(slice_steps * step_k);
    p.partial = split > 1 ? static_cast<float*>(d->workspace) : nullptr;
    p.tiles_m = static_cast<int>(tiles_m);
    p.tiles_n = static_cast<int>(tiles_n);

    plan.tile_m = tile_m; plan.tile_n = tile_n; plan.waves = waves;
    plan.tile_k = plan.kernel >= 2 ? prism::kPipeConfigs[out->pipe_config].tile_k : static_cast<int32_t>(step_k);
    plan.split_k = static_cast<int32_t>(split);
    plan.tiles_m = tiles_m; plan.tiles_n = tiles_n;
    plan.workgroups = units * split;
    // More (tile, unit) pairs than compute units, each with a short K loop: 256x256 tiles whose
    // slices all have two or more K steps go to the persistent kernel, one workgroup per
    // compute unit walking several pairs with the next pair's operands loaded under the tail of
    // the current one.  With long K loops the start of a tile is a small share of its time and
    // the hardware's own dealing of workgroups to free compute units balances better than the
    // fixed assignment of the persistent kernel (measured).
    {
        const bool never = hk.persistent == 0, always = hk.persistent == 1;
        const int64_t last_slice_steps = ksteps - (split - 1) * slice_steps;
        const bool possible = plan.kernel == 2 && out->pipe_config == 0 && slice_steps >= 2 && last_slice_steps >= 2 &&
                              slice_steps % 2 == 0 && last_slice_steps % 2 == 0;  // it walks K two steps at a time
        const bool pays = units * split > kComputeUnits && slice_steps <= kPersistentMaxSteps;
        if (possible && !never && (always || pays)) {
            plan.kernel = 3;
            out->total_units = static_cast<int>(units * split);
            if (plan.workgroups > kComputeUnits) plan.workgroups = kComputeUnits;
        }
    }
    plan.workspace_bytes = ws_need;
    if (plan.workgroups > kIntMax) return PRISM_ERR_INVALID_ARG;
    return PRISM_OK;
}

prism_status_t run(const Problem& pr, hipStream_t stream)
{
    const GemmParams& p = pr.p;
    if (p.M == 0 || p.N == 0 || p.batch == 0) return PRISM_OK;
    hipError_t e = hipSuccess;
    if (pr.dealt_rows)
        e = prism::launch_dealt(pr.ab_dtype, pr.dealt_rows, pr.plan.waves, pr.odd_rows, p, static_cast<int>(pr.plan.workgroups), stream);
    else if (pr.plan.kernel == 3)
        e = prism::launch_persistent(pr.ab_dtype, p, pr.total_units, static_cast<int>(pr.plan.workgroups), stream);
    else if (pr.plan.kernel == 2)
        e = prism::launch_pipelined(pr.pipe_config, pr.ab_dtype, p, static_cast<int>(pr.plan.workgroups), stream);
    else if (pr.plan.kernel == 1)
        e = prism::launch_staged(pr.ab_dtype, p, static_cast<int>(pr.plan.workgroups), stream);
    else if (pr.plan.kernel == 4)
        e = prism::launch_skinny(pr.ab_dtype, pr.plan.tile_m, pr.plan.tile_n, pr.plan.waves, p, static_cast<int>(pr.plan.workgroups), stream);
    if (e != hipSuccess) return PRISM_ERR_LAUNCH;
    if (hooks().log) {
        static const char* const names[] = {"none", "gemm_staged", "gemm_pipelined", "gemm_persistent", "gemm_skinny"};
        std::fprintf(stderr, "prism_gemm: M=%d N=%d K=%d batch=%d%s kernel=%s tile=%dx%dx%d waves=%d split_k=%d workgroups=%lld%s\n",
                     p.M, p.N, p.K, p.batch, pr.plan.swapped ? " (run as C^T = B^T A^T)" : "",
                     names[pr.plan.kernel >= 0 && pr.plan.kernel <= 4 ? pr.plan.kernel : 0], pr.plan.tile_m, pr.plan.tile_n,
                     pr.plan.tile_k, pr.plan.waves, pr.plan.split_k, static_cast<long long>(pr.plan.workgroups), pr.dealt_rows ? " k_steps=dealt" : "");
    }
    if (p.split_k != 1) {  // K == 0 (split_k == 0) or a real split: the reduction writes C
        e = prism::launch_reduce(p, stream);
        if (e != hipSuccess) return PRISM_ERR_LAUNCH;
    }
    return PRISM_OK;
}

}  // namespace

extern "C" {

prism_status_t prism_gemm_batched(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K,
                                  const void* A, int64_t lda, int64_t strideA, const void* B, int64_t ldb,
                                  int64_t strideB, void* C, int64_t ldc, int64_t strideC, int64_t batch,
                                  void* hip_stream)
{
    Problem pr;
    const prism_status_t s =
        make_problem(d, M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch, true, &pr);
    if (s != PRISM_OK) return s;
    return run(pr, static_cast<hipStream_t>(hip_stream));
}

prism_status_t prism_gemm_batched_stamped(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K,
                                          const void* A, int64_t lda, int64_t strideA, const void* B, int64_t ldb,
                                          int64_t strideB, void* C, int64_t ldc, int64_t strideC, int64_t batch,
                                          uint64_t* stamps, size_t stamp_bytes, void* hip_stream)
{
    Problem pr;
    const prism_status_t s =
        make_problem(d, M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch, true, &pr);
    if (s != PRISM_OK) return s;
    if (pr.plan.kernel != 2 && pr.plan.kernel != 4) return PRISM_ERR_UNSUPPORTED;  // the others leave no stamps
    if (!stamps || reinterpret_cast<uintptr_t>(stamps) % 8 != 0) return PRISM_ERR_INVALID_ARG;
    if (stamp_bytes < static_cast<size_t>(pr.plan.workgroups) * PRISM_STAMP_BYTES_PER_WORKGROUP) return PRISM_ERR_WORKSPACE;
    static_assert(PRISM_STAMP_BYTES_PER_WORKGROUP == prism::kStampWords * sizeof(uint64_t), "stamp layout");
    pr.p.stamps = stamps;
    return run(pr, static_cast<hipStream_t>(hip_stream));
}

prism_status_t prism_gemm(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K, const void* A,
                          int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc, void* hip_stream)
{
    return prism_gemm_batched(d, M, N, K, A, lda, 0, B, ldb, 0, C, ldc, 0, 1, hip_stream);
}

prism_status_t prism_gemm_plan(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K, const void* A,
                               int64_t lda, int64_t strideA, const void* B, int64_t ldb, int64_t strideB,
                               const void* C, int64_t ldc, int64_t strideC, int64_t batch,
                               prism_gemm_plan_t* plan_out)
{
    if (!plan_out) return PRISM_ERR_INVALID_ARG;
    Problem pr;
    const prism_status_t s =
        make_problem(d, M, N, K, A, lda, strideA, B, ldb, strideB, C, ldc, strideC, batch, false, &pr);
    if (s != PRISM_OK) return s;
    *plan_out = pr.plan;
    return PRISM_OK;
}

prism_status_t prism_gemm_workspace_size(const prism_gemm_desc_t* d, int64_t M, int64_t N, int64_t K,
                                         int64_t batch, size_t* bytes_out)
{
    if (!d || !bytes_out) return PRISM_ERR_INVALID_ARG;
    // Leading dimensions are not known here: packed ones are assumed, and tiles, because rows too
    // far apart keep a call off the kernel for few rows, which needs no workspace.
    const int64_t lda = d->layout_a == PRISM_ROW_MAJOR ? K : M, ldb = d->layout_b == PRISM_ROW_MAJOR ? N : K;
    const int64_t ldc = d->layout_c == PRISM_ROW_MAJOR ? N : M;
    // A call may also find another kernel the faster one than these do: enough for either.
    size_t most = 0;
    for (const bool allow_dealt : {false, true}) {
        Problem pr;
        const prism_status_t s =
            make_problem(d, M, N, K, nullptr, lda < 1 ? 1 : lda, M * K, nullptr, ldb < 1 ? 1 : ldb, K * N, nullptr,
                         ldc < 1 ? 1 : ldc, M * N, batch, false, &pr, false, allow_dealt);
        if (s != PRISM_OK) return s;
        if (pr.plan.workspace_bytes > most) most = pr.plan.workspace_bytes;
    }
    *bytes_out = most;
    return PRISM_OK;
}

prism_status_t prism_sched_map(int64_t wg, int64_t tiles_m, int64_t tiles_n, int64_t units, int64_t* tile_m,
                               int64_t* tile_n, int64_t* unit)
{
    if (!tile_m || !tile_n || !unit || tiles_m < 1 || tiles_n < 1 || units < 1) return PRISM_ERR_INVALID_ARG;
    if (tiles_m > kIntMax || tiles_n > kIntMax || units > kIntMax) return PRISM_ERR_INVALID_ARG;
    if (tiles_m * tiles_n > kIntMax || tiles_m * tiles_n * units > kIntMax) return PRISM_ERR_INVALID_ARG;
    if (wg < 0 || wg >= tiles_m * tiles_n * units) return PRISM_ERR_INVALID_ARG;
    const prism::grid::TileCoord c = prism::grid::schedule(static_cast<int>(wg), static_cast<int>(tiles_m),
                                                           static_cast<int>(tiles_n), static_cast<int>(units));
    *tile_m = c.tile_m;
    *tile_n = c.tile_n;
    *unit = c.unit;
    return PRISM_OK;
}

const char* prism_status_string(prism_status_t s)
{
    switch (s) {
    case PRISM_OK: return "PRISM_OK";
    case PRISM_ERR_INVALID_ARG: return "PRISM_ERR_INVALID_ARG";
    case PRISM_ERR_UNSUPPORTED: return "PRISM_ERR_UNSUPPORTED";
    case PRISM_ERR_WORKSPACE: return "PRISM_ERR_WORKSPACE";
    case PRISM_ERR_LAUNCH: return "PRISM_ERR_LAUNCH";
    }
    return "PRISM_ERR_UNKNOWN";
}

int prism_version(void) { return 200; }

void prism_reread_environment(void)
{
    {
        std::lock_guard<std::mutex> lock(g_hooks_mutex);
        load_hooks_locked();
    }
    prism::scan_reread_environment();
}

}  // extern "C"
