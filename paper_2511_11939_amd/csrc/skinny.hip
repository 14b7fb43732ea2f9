// Products with few rows (decoding: a handful of tokens against a weight matrix): C of up to 64
// rows, both operands contiguous along K, any sizes and alignments.
//
// Bound by B, which is read once and used for a few rows only: what matters is how many bytes of it
// are on their way at any time.  So there is no tile that waves share and no barrier in the
// loop: a workgroup takes 16 * NT columns over the whole of K, its W waves deal the K steps (128
// bytes of every row) out among themselves, and every wave loads its steps into registers, U at
// a time with the next U already under way, eight lanes to a row.  A step passes through LDS of
// the wave's own to get from that order into the matrix instruction's: loaded in the latter
// straight away, sixteen neighbouring lanes touch sixteen rows, and the vector cache answers at 14
// bytes a clock (16 x 4096 x 4096 took 12.8 us).  The rows of A come from the caches, once per
// workgroup.  The waves' sums are added in wave order, so the result does not depend on timing, and
// none go through memory: no workspace and no second launch.
// Measured: 16 x 4096 x 4096 bf16 with bias 16.4 -> 8.7 us (128x128 tiles, K split and a reduction
// before), 1 x 4096 x 4096 15.8 -> 8.0, 5 x 704 x 3264 20.9 -> 5.6, 16 x 16384 x 16384 143 -> 92 (5.8
// TB/s).  Two steps ahead and two workgroups per compute unit beat four steps and one: 8 x 16384 x
// 4096 29.6 against 34.6 us.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "grid.hpp"
#include "lane.hpp"
#include "launch.hpp"
#include "wave.hpp"
#include "workgroup.hpp"

namespace prism {
namespace {

template <typename T, int MT, int NT, int W>
struct Skinny {
    static constexpr int ES = Frag<T>::kElemBytes, EPC = lane::kChunkBytes / ES;
    static constexpr int STEP_BYTES = 128, STEP = STEP_BYTES / ES;
    // K steps loaded together (eight rows of a block in each of the two loads): what the registers of two waves per SIMD (W = 16: four) hold twice
    static constexpr int U = MT + NT <= 3 ? 2 : 1;
    static constexpr int THREADS = 64 * W;
    // waves per SIMD that the registers are meant for: four, or what LDS has room for with 64 rows
    // by two blocks of columns (two of a workgroup of eight, three of one of four)
    static constexpr int WAVES_PER_SIMD = MT + NT == 6 ? 2 : 4;
    using frag_t = typename Frag<T>::type;
    struct Steps {
        u32x4 a[U][MT][2], b[U][NT][2];
    };
};

template <typename T, int MT, int NT, int W, bool STREAM>
__global__ __launch_bounds__(64 * W, (Skinny<T, MT, NT, W>::WAVES_PER_SIMD)) void gemm_skinny(const GemmParams p)
{
    using S = Skinny<T, MT, NT, W>;
    using frag_t = typename S::frag_t;
    constexpr int ES = S::ES, U = S::U;
    const persp::Block<S::THREADS> wgp = persp::Grid::at_kernel_entry().workgroup<S::THREADS>();
    const persp::Wave wv = wgp.wave();
    using L = lane::TileLayout<64>;  // rows of 128 bytes
    constexpr int BLOCK_BYTES = lane::kBlock * L::kRowBytes, WAVE_BYTES = (MT + NT) * BLOCK_BYTES;
    static_assert(MT * NT * 64 * sizeof(f32x4) <= WAVE_BYTES, "a wave's sums take the place of its step");
    __shared__ __attribute__((aligned(1024))) char lds[W * WAVE_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stamp(p.stamps, STAMP_ENTRY);
    const int batch = p.batch == 1 ? 0 : grid::uniform_quotient(blockIdx.x, p.tiles_n);
    const int n0 = (static_cast<int>(blockIdx.x) - batch * p.tiles_n) * lane::kBlock * NT;

    // Lane l: chunk l % 8 of rows l / 8 and l / 8 + 8 of a block.
    // (rows beyond the matrix re-read its last one and are never stored)
    const int x = lane & 15, g = lane >> 4, chunk = lane & 7;
    const char* a_rows = p.A + ES * (batch * p.batch_a);
    const char* b_rows = p.B + ES * (batch * p.batch_b + n0 * p.b_sn);
    uint32_t a_off[MT][2], b_off[NT][2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int row = (lane >> 3) + 8 * r;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = lane::kBlock * i + row;
            a_off[i][r] = static_cast<uint32_t>((m < p.M ? m : p.M - 1) * static_cast<uint32_t>(p.a_sm * ES)) + chunk * lane::kChunkBytes;
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int n = lane::kBlock * j + row;
            b_off[j][r] = static_cast<uint32_t>((n0 + n < p.N ? n : p.N - 1 - n0) * static_cast<uint32_t>(p.b_sn * ES)) + chunk * lane::kChunkBytes;
        }
    }
    char* slot = lds + wave * WAVE_BYTES;
    char* put = slot + L::offset(lane >> 3, chunk);  // (rows l / 8 and l / 8 + 8 have the same swizzle)
    const char* passed = slot + wave::unknown_offset(wv);
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const u32x4 (&a)[MT][2], const u32x4 (&b)[NT][2]) __attribute__((always_inline)) {
        // (B's first fragments are read while the loads of A may still be on their way)
        frag_t fa[MT], fb[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 2; ++r) *reinterpret_cast<u32x4*>(put + j * BLOCK_BYTES + 8 * r * L::kRowBytes) = b[j][r];
        PRISM_PARANOID_WAIT();
        wave::load_fragments<T, 64, NT>(wv, fb, passed, 0, 0, lane);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 2; ++r) *reinterpret_cast<u32x4*>(put + (NT + i) * BLOCK_BYTES + 8 * r * L::kRowBytes) = a[i][r];
        PRISM_PARANOID_WAIT();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h > 0) wave::load_fragments<T, 64, NT>(wv, fb, passed, 0, h, lane);
            wave::load_fragments<T, 64, MT>(wv, fa, passed + NT * BLOCK_BYTES, 0, h, lane);
#pragma unroll
            for (int e = 0; e < wave::mfma_parts(frag_t{}); ++e)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[i][j] = wave::mfma_part(wv, fb[j], fa[i], e, acc[i][j]);
        }
        PRISM_PARANOID_WAIT();
    };

    // Whole K steps wave, wave + W, wave + 2 W ...: `mine` of them.
    const int whole = p.K / S::STEP;
    const int mine = whole > wave ? (whole - wave + W - 1) / W : 0;
    typename S::Steps set[2];
    auto load = [&](int first, typename S::Steps& to) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = first + u < mine ? first + u : mine - 1;  // (past the end: the last one again, left out below)
            const int64_t at = static_cast<int64_t>(wave + q * W) * S::STEP_BYTES;
            const wg::global_bytes b = (wg::global_bytes)wg::scalarize(b_rows + at), a = (wg::global_bytes)wg::scalarize(a_rows + at);
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    auto* src = (const __attribute__((address_space(1))) u32x4_any*)(b + b_off[j][r]);
                    to.b[u][j][r] = STREAM ? __builtin_nontemporal_load(src) : *src;
                }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int r = 0; r < 2; ++r) to.a[u][i][r] = *(const __attribute__((address_space(1))) u32x4_any*)(a + a_off[i][r]);
        }
    };
    auto use = [&](int first, const typename S::Steps& from) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (first + u < mine) multiply(from.a[u], from.b[u]);
    };
    if (mine > 0) {
        load(0, set[0]);
        stamp(p.stamps, STAMP_FIRST_FRAGMENTS);
        for (int q = 0; q < mine; q += 2 * U) {
            load(q + U, set[1]);
            __builtin_amdgcn_sched_barrier(0);
            use(q, set[0]);
            load(q + 2 * U, set[0]);
            __builtin_amdgcn_sched_barrier(0);
            use(q + U, set[1]);
        }
    } else {
        stamp(p.stamps, STAMP_FIRST_FRAGMENTS);
    }
    // The rest of K, less than a step: chunks are loaded where they lie inside their row and moved
    // into place, zeros behind (K is a chunk or more).
    if (whole * S::STEP < p.K && wave == whole % W) {
        u32x4 a[MT][2], b[NT][2];
        const int k = whole * S::STEP + chunk * S::EPC, from = k + S::EPC <= p.K ? k : p.K - S::EPC;
        const int64_t at = static_cast<int64_t>(from) * ES - chunk * lane::kChunkBytes;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i][r] = wg::chunk_moved_down(*reinterpret_cast<const u32x4_any*>(a_rows + a_off[i][r] + at), (k - from) * ES);
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j][r] = wg::chunk_moved_down(*reinterpret_cast<const u32x4_any*>(b_rows + b_off[j][r] + at), (k - from) * ES);
        }
        multiply(a, b);
    }
    stamp(p.stamps, STAMP_K_LOOP_DONE);

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) reinterpret_cast<f32x4*>(slot)[(i * NT + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    auto sum_of = [&](int w, int block) __attribute__((always_inline)) { return reinterpret_cast<const f32x4*>(lds + w * WAVE_BYTES)[block * 64 + lane]; };
    const grid::Target to = grid::target_of(p, batch);
    auto finish = [&](auto out_c) __attribute__((always_inline)) {
        constexpr int OUT = decltype(out_c)::value;
        for (int block = wave; block < MT * NT; block += W) {
            const int m = lane::kBlock * (block / NT) + x, n = n0 + lane::kBlock * (block % NT) + 4 * g, left = p.N - n;
            f32x4 sum = sum_of(0, block);
#pragma unroll
            for (int w = 1; w < W; ++w) sum += sum_of(w, block);
            if (m >= p.M || left <= 0) continue;
            f32x4 add = {0.f, 0.f, 0.f, 0.f};
            if (to.bias) {
                const char* src = reinterpret_cast<const char*>(to.bias + n);
                if (to.bias_along_m) add = f32x4{to.bias[m], to.bias[m], to.bias[m], to.bias[m]};
                else add = left >= 4 ? grid::load4<DT_F32>(src) : grid::load_some<DT_F32>(src, left);
            }
            sum = grid::scaled(to.alpha, sum, add);
            char* dst = to.c + m * to.row_bytes + static_cast<int64_t>(n) * grid::out_bytes<OUT>();
            if (to.beta != 0.0f) sum = grid::scaled(to.beta, left >= 4 ? grid::load4<OUT>(dst) : grid::load_some<OUT>(dst, left), sum);
            if (left >= 4) grid::store4<OUT>(dst, sum);
            else grid::store_some<OUT>(dst, sum, left);
        }
    };
    if (to.dtype == DT_BF16) finish(std::integral_constant<int, DT_BF16>{});
    else if (to.dtype == DT_F16) finish(std::integral_constant<int, DT_F16>{});
    else finish(std::integral_constant<int, DT_F32>{});
    if (p.stamps) {
        wg::wait_counts<0, 0>();
        stamp(p.stamps, STAMP_STORES_DONE);
    }
}

template <typename T, int MT, int NT, int W, bool STREAM = false>
void launch(const GemmParams& p, int workgroups, hipStream_t stream)
{
    hipLaunchKernelGGL((gemm_skinny<T, MT, NT, W, STREAM>), dim3(workgroups), dim3(64 * W), 0, stream, p);
}
template <typename T, int MT, int NT>
void launch_waves(int waves, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if constexpr (NT == 1)  // (two blocks of columns: only with so many workgroups that eight waves do)
        if (waves == 16) return launch<T, MT, NT, 16>(p, workgroups, stream);
    if constexpr (NT == 2)
        if (waves == 8 && few_rows_stream_b(p.N, p.K, Frag<T>::kElemBytes, p.batch, p.batch_b)) return launch<T, MT, NT, 8, true>(p, workgroups, stream);
    if (waves == 8) launch<T, MT, NT, 8>(p, workgroups, stream);
    else launch<T, MT, NT, 4>(p, workgroups, stream);
}
template <typename T>
hipError_t launch_typed(int tile_m, int tile_n, int waves, const GemmParams& p, int workgroups, hipStream_t stream)
{
    const int shape = tile_m / 16 * 10 + tile_n / 16;
    switch (shape) {
    case 11: launch_waves<T, 1, 1>(waves, p, workgroups, stream); break;
    case 12: launch_waves<T, 1, 2>(waves, p, workgroups, stream); break;
    case 21: launch_waves<T, 2, 1>(waves, p, workgroups, stream); break;
    case 22: launch_waves<T, 2, 2>(waves, p, workgroups, stream); break;
    case 41: launch_waves<T, 4, 1>(waves, p, workgroups, stream); break;
    case 42: launch_waves<T, 4, 2>(waves, p, workgroups, stream); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_skinny(int ab_dtype, int tile_m, int tile_n, int waves, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if (ab_dtype == DT_BF16) return launch_typed<bf16_t>(tile_m, tile_n, waves, p, workgroups, stream);
    if (ab_dtype == DT_F16) return launch_typed<f16_t>(tile_m, tile_n, waves, p, workgroups, stream);
    return launch_typed<f32_t>(tile_m, tile_n, waves, p, workgroups, stream);
}

}  // namespace prism
