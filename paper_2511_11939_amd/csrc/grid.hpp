// Grid layer: which workgroup computes which output tile, and what happens to a
// finished accumulator tile (scale, bias, conversion, store, or a split-K
// partial).  The scheduler plays the part of the tile loop with super-tile
// ordering in the paper's persistent hgemm kernel (code appendix, scheduler of
// `my_h100_match_no_tail`); the alpha/beta epilogue is the paper's sgemm
// epilogue (section 6.1) extended by a bias vector.
#pragma once

#include "lane.hpp"
#include "stamp.hpp"

namespace prism {

enum : int { DT_BF16 = 0, DT_F16 = 1, DT_F32 = 2 };

// Problem as the kernels see it: C is row-major (a column-major C has been
// turned into the transposed problem on the host), strides are in elements.
struct GemmParams {
    const char* A;        // element (m, k) at A + esize*(m*a_sm + k*a_sk), esize 2 or 4
    const char* B;        // element (k, n) at B + esize*(n*b_sn + k*b_sk)
    char* C;              // element (m, n) at C + esize*(m*ldc + n)
    const float* bias;    // or nullptr
    float* partial;       // split-K scratch [batch][split_k][M][N] fp32, or nullptr
    int64_t a_sm, a_sk, b_sn, b_sk, ldc;
    int64_t batch_a, batch_b, batch_c;
    int M, N, K;
    int batch, split_k, k_slice;   // k_slice: K extent of one slice, whole K steps
    int tiles_m, tiles_n;
    float alpha, beta;
    int c_dtype;          // DT_*
    int bias_along_m;     // 1 when the problem was transposed on the host
    uint64_t* stamps;     // nullptr, or kStampWords uint64 per workgroup of the main kernel (measurement aid)
};

namespace grid {

constexpr int kDies = 8;        // accelerator dies (XCDs); workgroup ids are dealt round-robin
constexpr int kGroupRows = 4;   // tile rows per super-tile group

struct TileCoord {
    int tile_m, tile_n, unit;
};

// floor(x / d) for 0 <= x, 1 <= d, both below 2^30.  On the device both must be the same in
// every lane of the wave: the estimate from the reciprocal is moved to the scalar unit and
// corrected there, which replaces the compiler's general expansion (four quarter-rate
// integer multiplies per division, in front of a workgroup's first copies) by a handful of
// full-rate instructions.  The correction loops make the result exact whatever the error of
// the estimate, so host and device agree.
__host__ __device__ inline int uniform_quotient(int x, int d)
{
#if defined(__HIP_DEVICE_COMPILE__)
    int q = __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<float>(x) * __builtin_amdgcn_rcpf(static_cast<float>(d))));
    int rest = x - q * d;
    while (rest < 0) { --q; rest += d; }
    while (rest >= d) { ++q; rest -= d; }
    return __builtin_amdgcn_readfirstlane(q);  // stays on the scalar unit, and so does what is derived from it
#else
    return x / d;
#endif
}

// Position r in the locality order -> tile: groups of kGroupRows tile rows, m fastest, so that
// a contiguous run of positions is a compact block sharing few A and B panels.
__host__ __device__ inline void tile_at(int r, int tiles_m, int tiles_n, int& tile_m, int& tile_n)
{
    const int group_span = kGroupRows * tiles_n;
    const int group = uniform_quotient(r, group_span);
    const int first_m = group * kGroupRows;
    const int rows = tiles_m - first_m < kGroupRows ? tiles_m - first_m : kGroupRows;
    const int in_group = r - group * group_span;
    tile_n = uniform_quotient(in_group, rows);
    tile_m = first_m + in_group - tile_n * rows;
}

// The share of die `die` when `total` positions are dealt to the dies as contiguous runs
// (the first `total % kDies` dies take one more): first position and count.
__host__ __device__ inline void die_run(int die, int total, int& first, int& count)
{
    const int per = (total + kDies - 1) / kDies;
    int tall = total % kDies;
    if (tall == 0) tall = kDies;
    first = die < tall ? die * per : tall * per + (die - tall) * (per - 1);
    count = die < tall ? per : per - 1;
}

// Workgroup id -> (tile, unit).  Step 1 undoes the round-robin dealing so that
// the workgroups resident on one die form a contiguous run of a tile order;
// step 2 walks the tiles in groups of kGroupRows tile rows, m fastest, so that
// such a run is a compact block sharing few A and B panels in that die's L2.
// On the device `wg` must be uniform over the wave (a workgroup id is).
__host__ __device__ inline TileCoord schedule(int wg, int tiles_m, int tiles_n, int units)
{
    const int tiles = tiles_m * tiles_n;
    int first, count;
    die_run(wg % kDies, tiles * units, first, count);
    const int q = first + wg / kDies;
    TileCoord t;
    t.unit = units == 1 ? 0 : uniform_quotient(q, tiles);
    tile_at(q - t.unit * tiles, tiles_m, tiles_n, t.tile_m, t.tile_n);
    return t;
}

// ---- epilogue ------------------------------------------------------------------------
// Where a finished accumulator tile goes and what is applied on the way: C of one problem with
// the scalars and the bias of the call, or one slice's partial sums (fp32, nothing applied).
struct Target {
    char* c;             // element (0, 0)
    int64_t row_bytes;
    const float* bias;   // or nullptr
    float alpha, beta;
    int dtype;           // DT_*
    bool bias_along_m;
};
__device__ __forceinline__ Target target_of(const GemmParams& p, int batch)
{
    const int esize = p.c_dtype == DT_F32 ? 4 : 2;
    return Target{p.C + static_cast<int64_t>(batch) * p.batch_c * esize, p.ldc * esize, p.bias, p.alpha, p.beta, p.c_dtype, p.bias_along_m != 0};
}
__device__ __forceinline__ Target partial_of(const GemmParams& p, int batch, int slice)
{
    float* slab = p.partial + (static_cast<int64_t>(batch) * p.split_k + slice) * p.M * p.N;
    return Target{reinterpret_cast<char*>(slab), static_cast<int64_t>(p.N) * 4, nullptr, 1.0f, 0.0f, DT_F32, false};
}

// Four consecutive results of one row: conversions and memory accesses, at any alignment.  The
// `some` forms touch only the first `count` of them (fewer than four, at the end of a row).
template <int OUT>  // DT_BF16 / DT_F16 / DT_F32
constexpr int out_bytes() { return OUT == DT_F32 ? 4 : 2; }
template <int OUT>
__device__ __forceinline__ u32x2 pack4(f32x4 v)
{
    static_assert(OUT == DT_BF16 || OUT == DT_F16, "16-bit output types");
    // round to nearest even (as vectors: the compiler then has one conversion instruction per pair of bf16)
    if constexpr (OUT == DT_BF16) return __builtin_bit_cast(u32x2, __builtin_convertvector(v, bf16x4));
    else return __builtin_bit_cast(u32x2, __builtin_convertvector(v, f16x4));
}
template <int OUT>
__device__ __forceinline__ float decode16(uint32_t h)
{
    return OUT == DT_BF16 ? lane::from_bf16_bits(static_cast<uint16_t>(h)) : lane::from_f16_bits(static_cast<uint16_t>(h));
}
template <int OUT>
__device__ __forceinline__ f32x4 load4(const char* src)
{
    if constexpr (OUT == DT_F32) {
        return *reinterpret_cast<const f32x4_any*>(src);
    } else {
        const u32x2 w = *reinterpret_cast<const u32x2_any*>(src);
        return f32x4{decode16<OUT>(w[0] & 0xffffu), decode16<OUT>(w[0] >> 16), decode16<OUT>(w[1] & 0xffffu), decode16<OUT>(w[1] >> 16)};
    }
}
template <int OUT>
__device__ __forceinline__ f32x4 load_some(const char* src, int count)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if (q < count) {
            if constexpr (OUT == DT_F32) v[q] = reinterpret_cast<const float*>(src)[q];
            else v[q] = decode16<OUT>(reinterpret_cast<const uint16_t*>(src)[q]);
        }
    return v;
}
template <int OUT>
__device__ __forceinline__ void store4(char* dst, f32x4 v)
{
    if constexpr (OUT == DT_F32) *reinterpret_cast<f32x4_any*>(dst) = v;
    else *reinterpret_cast<u32x2_any*>(dst) = pack4<OUT>(v);
}
// The first `count` (1 .. 7) of eight 16-bit results.
__device__ __forceinline__ void store_some16(char* dst, u32x4 w, int count)
{
    if (count & 4) {
        *reinterpret_cast<u32x2_any*>(dst) = u32x2{w[0], w[1]};
        w = u32x4{w[2], w[3], 0u, 0u};
        dst += 8;
    }
    if (count & 2) {
        reinterpret_cast<uint16_t*>(dst)[0] = static_cast<uint16_t>(w[0]);
        reinterpret_cast<uint16_t*>(dst)[1] = static_cast<uint16_t>(w[0] >> 16);
        w[0] = w[1];
        dst += 4;
    }
    if (count & 1) *reinterpret_cast<uint16_t*>(dst) = static_cast<uint16_t>(w[0]);
}
template <int OUT>
__device__ __forceinline__ void store_some(char* dst, f32x4 v, int count)
{
    if constexpr (OUT == DT_F32) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (q < count) reinterpret_cast<float*>(dst)[q] = v[q];
    } else if (count > 0) {
        const u32x2 w = pack4<OUT>(v);
        store_some16(dst, u32x4{w[0], w[1], 0u, 0u}, count);
    }
}
__device__ __forceinline__ f32x4 scaled(float alpha, f32x4 v)
{
    return f32x4{alpha * v[0], alpha * v[1], alpha * v[2], alpha * v[3]};
}
__device__ __forceinline__ f32x4 scaled(float alpha, f32x4 v, f32x4 bias)
{
    return f32x4{alpha * v[0] + bias[0], alpha * v[1] + bias[1], alpha * v[2] + bias[2], alpha * v[3] + bias[3]};
}

}  // namespace grid
}  // namespace prism
