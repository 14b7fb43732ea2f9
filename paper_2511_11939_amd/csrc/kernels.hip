// Device kernels: thin __global__ shells that place a workgroup on its tile
// (grid layer), run a workgroup main loop and hand the accumulators to the
// epilogue.  All arithmetic of the matrix product happens here on the GPU.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "grid.hpp"
#include "lane.hpp"
#include "launch.hpp"
#include "wave.hpp"
#include "workgroup.hpp"

namespace prism {

const PipeConfig kPipeConfigs[kNumPipeConfigs] = {
    {0, 256, 256, 64, 4, 2, "256x256x64_w4"},
    {1, 128, 128, 64, 4, 2, "128x128x64_w4"},
    {2, 128, 128, 64, 4, 2, "128x128x64_w4_b_along_n"},
    {3, 128, 128, 64, 4, 2, "128x128x64_w4_a_along_m"},
    {4, 128, 128, 64, 4, 2, "128x128x64_w4_a_along_m_b_along_n"},
    {5, 128, 128, 32, 4, 2, "f32_128x128x32_w4"},
    {6, 128, 128, 32, 4, 2, "f32_128x128x32_w4_b_along_n"},
    {7, 128, 128, 32, 4, 2, "f32_128x128x32_w4_a_along_m"},
    {8, 128, 128, 32, 4, 2, "f32_128x128x32_w4_a_along_m_b_along_n"},
    {9, 256, 256, 64, 4, 2, "256x256x64_w4_b_along_n"},
    {10, 256, 256, 64, 4, 2, "256x256x64_w4_a_along_m"},
    {11, 256, 256, 64, 4, 2, "256x256x64_w4_a_along_m_b_along_n"},
};

namespace {

struct Placement {
    int batch, slice, m0, n0, k_begin, k_end;
};

template <int BM, int BN>
__device__ __forceinline__ Placement place(const GemmParams& p, int wg)
{
    const grid::TileCoord c = grid::schedule(wg, p.tiles_m, p.tiles_n, p.batch * p.split_k);
    Placement q;
    q.batch = p.split_k == 1 ? c.unit : grid::uniform_quotient(c.unit, p.split_k);
    q.slice = c.unit - q.batch * p.split_k;
    q.m0 = c.tile_m * BM;
    q.n0 = c.tile_n * BN;
    q.k_begin = q.slice * p.k_slice;
    q.k_end = q.k_begin + p.k_slice < p.K ? q.k_begin + p.k_slice : p.K;
    // uniform values: held in scalar registers, so that the tile addresses derived from them
    // are computed by the scalar unit
    q.batch = __builtin_amdgcn_readfirstlane(q.batch);
    q.slice = __builtin_amdgcn_readfirstlane(q.slice);
    q.m0 = __builtin_amdgcn_readfirstlane(q.m0);
    q.n0 = __builtin_amdgcn_readfirstlane(q.n0);
    q.k_begin = __builtin_amdgcn_readfirstlane(q.k_begin);
    q.k_end = __builtin_amdgcn_readfirstlane(q.k_end);
    return q;
}

// Accumulators of one wave tile -> C or the split-K scratch.
// OWN_PATCH false: the patches reuse the operand slots; workgroup-collective, every wave
// must call it (it starts with a barrier that retires the slots).  OWN_PATCH true: `patch`
// is this wave's private patch outside the slots; no barrier.
//
// Three forms: plain (the whole wave tile inside C, nothing read back, the bias, if any, along
// the columns and held in registers), inside (the same with beta or a bias per row) and edge (every access
// bounded; the pieces that lie wholly in their row still move as vectors).  None asks for an
// alignment: rows of odd length, where every access used to be a single element, cost what
// aligned ones do up to the cache lines they straddle.  Measured: 1999 x 2001 x 1003 bf16 24.2 ->
// 21.7 us, 128 x 791 x 128 fp32 with beta 28.4 -> 17.8 us; with a row-major B, whose tile no longer
// drains fp32 values through LDS, 8192 x 4096 x 4096 bf16 255 -> 232 us; 4096 x 4096 x 8192 with fp32
// C and beta = 1 300 -> 278 us.
template <typename TileT, int MT, int NT, bool OWN_PATCH = false, bool PAIRED = false>
__device__ __forceinline__ void epilogue(persp::Workgroup wgp, const GemmParams& p, const Placement& q, const TileT& acc,
                                         int m_wave, int n_wave, char* lds, int wave, int lane)
{
    const persp::Wave wv = wgp.wave();
    const grid::Target to = p.split_k > 1 ? grid::partial_of(p, q.batch, q.slice) : grid::target_of(p, q.batch);
    const bool inside = m_wave + lane::kBlock * MT <= p.M && n_wave + lane::kBlock * NT <= p.N;
    char* patch = lds;
    if constexpr (!OWN_PATCH) {
        wg::sync(wgp);  // every wave has finished with the operand slots: they become patches
        patch = lds + wave * wg::rows_patch_bytes(NT);
    }
    if (m_wave >= p.M || n_wave >= p.N) return;
    const int64_t row_bytes = to.row_bytes;
    const int m_lane = m_wave + (lane & 15), n_lane = n_wave + lane::acc_first_col<PAIRED>(0, lane);
    auto column = [](int j) { return lane::acc_first_col<PAIRED>(j, 0); };  // of block column j, beyond n_lane
    auto nothing = [](int) {};

    auto plain = [&](auto out_c, auto bias_c) {
        constexpr int OUT = decltype(out_c)::value, ES = grid::out_bytes<OUT>();
        constexpr bool BIAS = decltype(bias_c)::value;
        f32x4 bias[BIAS ? NT : 1];
        if constexpr (BIAS) {
#pragma unroll
            for (int j = 0; j < NT; ++j) bias[j] = *reinterpret_cast<const f32x4_any*>(to.bias + n_lane + column(j));
        }
        auto value = [&](int j, f32x4 v) {
            if constexpr (BIAS) return grid::scaled(to.alpha, v, bias[j]);
            else return grid::scaled(to.alpha, v);
        };
        if constexpr (OUT == DT_F32) {
            char* lane_base = to.c + m_lane * row_bytes + static_cast<int64_t>(n_lane) * ES;
            wg::drain_direct<MT, NT>(wv, acc, nothing, [&](int i, int j, f32x4 v) {
                grid::store4<OUT>(lane_base + lane::kBlock * i * row_bytes + column(j) * ES, value(j, v));
            });
        } else {
            // streaming stores: C is not read again by this kernel
            char* wave_base = to.c + m_wave * row_bytes + static_cast<int64_t>(n_wave) * ES;
            wg::drain_rows<PAIRED, MT, NT>(
                wv, acc, patch, lane, nothing, [&](int, int j, f32x4 v) { return grid::pack4<OUT>(value(j, v)); },
                [&](int r_uniform, int r_lane, int byte_in_row, u32x4 piece) {
                    __builtin_nontemporal_store(piece, reinterpret_cast<u32x4_any*>(wave_base + (r_uniform + r_lane) * row_bytes + byte_in_row));
                });
        }
    };

    auto general = [&](auto out_c, auto inside_c) {
        constexpr int OUT = decltype(out_c)::value, ES = grid::out_bytes<OUT>();
        constexpr bool INSIDE = decltype(inside_c)::value;
        // Of an edge tile most blocks are wholly inside C or wholly outside, which is the same for
        // the whole wave; only the others are bounded lane by lane.
        auto left = [&](int j) { return p.N - (n_lane + column(j)); };  // columns of C from the lane's first one on
        auto has_row = [&](int i) { return INSIDE || m_lane + lane::kBlock * i < p.M; };
        auto any_row = [&](int i) { return INSIDE || m_wave + lane::kBlock * i < p.M; };
        auto all_rows = [&](int i) { return INSIDE || m_wave + lane::kBlock * (i + 1) <= p.M; };
        constexpr int SPAN = PAIRED ? 32 : lane::kBlock;  // columns that a block (a pair of blocks) covers
        auto any_column = [&](int j) { return INSIDE || n_wave + column(j) < p.N; };
        auto all_columns = [&](int j) { return INSIDE || n_wave + (PAIRED ? column(j & ~1) : column(j)) + SPAN <= p.N; };
        auto load_left = [&](auto type_c, const char* src, int j) __attribute__((always_inline)) {
            constexpr int TYPE = decltype(type_c)::value;
            if (all_columns(j)) return grid::load4<TYPE>(src);
            if (!any_column(j)) return f32x4{0.f, 0.f, 0.f, 0.f};
            return left(j) >= 4 ? grid::load4<TYPE>(src) : grid::load_some<TYPE>(src, left(j));
        };
        // Beside the next tile's fragments, which the persistent kernel holds meanwhile
        // (OWN_PATCH), there are no registers to fetch anything ahead.
        constexpr int AHEAD = OWN_PATCH ? 0 : 1;
        const bool bias_n = to.bias && !to.bias_along_m;
        auto fetch_bias = [&](int j) __attribute__((always_inline)) {
            return load_left(std::integral_constant<int, DT_F32>{}, reinterpret_cast<const char*>(to.bias + n_lane + column(j)), j);
        };
        f32x4 bias[AHEAD ? NT : 1];
        if constexpr (AHEAD) {
#pragma unroll
            for (int j = 0; j < NT; ++j) bias[j] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (bias_n) {
#pragma unroll
                for (int j = 0; j < NT; ++j) bias[j] = fetch_bias(j);
            }
        }
        char* lane_base = to.c + m_lane * row_bytes + static_cast<int64_t>(n_lane) * ES;
        // What C holds is fetched one block row ahead, so that its way from memory is covered by
        // the stores of the row before.
        f32x4 old[1 + AHEAD][NT];
        float bias_m[1 + AHEAD] = {};
        auto fetch = [&](int i) __attribute__((always_inline)) {
            if (to.beta != 0.0f && has_row(i)) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    old[i & AHEAD][j] = load_left(out_c, lane_base + lane::kBlock * i * row_bytes + column(j) * ES, j);
            }
            if (to.bias && to.bias_along_m && has_row(i)) bias_m[i & AHEAD] = to.bias[m_lane + lane::kBlock * i];
        };
        auto row = [&](int i) __attribute__((always_inline)) {
            if (i == 0 || !AHEAD) fetch(i);
            if (AHEAD && i + 1 < MT) fetch(i + 1);
        };
        auto value = [&](int i, int j, f32x4 v) __attribute__((always_inline)) {
            f32x4 add = {0.f, 0.f, 0.f, 0.f};
            if constexpr (AHEAD) add = bias[j];
            else if (bias_n) add = fetch_bias(j);
            const float bm = bias_m[i & AHEAD];
            if (to.bias_along_m) add = f32x4{bm, bm, bm, bm};
            f32x4 r = grid::scaled(to.alpha, v, add);
            if (to.beta != 0.0f) r = grid::scaled(to.beta, old[i & AHEAD][j], r);
            return r;
        };
        if constexpr (OUT == DT_F32) {
            wg::drain_direct<MT, NT>(wv, acc, row, [&](int i, int j, f32x4 v) {
                if (!any_row(i) || !any_column(j)) return;
                char* dst = lane_base + lane::kBlock * i * row_bytes + column(j) * ES;
                v = value(i, j, v);
                if (all_rows(i) && all_columns(j)) grid::store4<OUT>(dst, v);
                else if (has_row(i)) {
                    if (left(j) >= 4) grid::store4<OUT>(dst, v);
                    else grid::store_some<OUT>(dst, v, left(j));
                }
            });
        } else {
            char* wave_base = to.c + m_wave * row_bytes + static_cast<int64_t>(n_wave) * ES;
            wg::drain_rows<PAIRED, MT, NT>(
                wv, acc, patch, lane, row, [&](int i, int j, f32x4 v) { return grid::pack4<OUT>(value(i, j, v)); },
                [&](int r_uniform, int r_lane, int byte_in_row, u32x4 piece) {
                    const int i = r_uniform / lane::kBlock;
                    if (!any_row(i)) return;
                    char* dst = wave_base + (r_uniform + r_lane) * row_bytes + byte_in_row;
                    const int count = p.N - n_wave - byte_in_row / ES;
                    if ((all_rows(i) || m_wave + r_uniform + r_lane < p.M)) {
                        if (INSIDE || count >= 8) __builtin_nontemporal_store(piece, reinterpret_cast<u32x4_any*>(dst));
                        else if (count > 0) grid::store_some16(dst, piece, count);
                    }
                });
        }
    };

    auto out_type = [&](auto&& run) {
        if (to.dtype == DT_BF16) run(std::integral_constant<int, DT_BF16>{});
        else if (to.dtype == DT_F16) run(std::integral_constant<int, DT_F16>{});
        else run(std::integral_constant<int, DT_F32>{});
    };
    out_type([&](auto out_c) {
        if (!inside) general(out_c, std::false_type{});
        else if (to.beta != 0.0f || (to.bias && to.bias_along_m)) general(out_c, std::true_type{});
        else if (to.bias) plain(out_c, std::true_type{});
        else plain(out_c, std::false_type{});
    });
}

template <typename P, int BM, int BN, int BK, int WAVES_N>
__global__ __launch_bounds__(P::THREADS) void gemm_pipelined(const GemmParams p)
{
    const persp::Workgroup wgp = persp::Grid::at_kernel_entry().workgroup();
    __shared__ __attribute__((aligned(1024))) char lds[P::LDS_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stamp(p.stamps, STAMP_ENTRY);
    const Placement q = place<BM, BN>(p, blockIdx.x);

    constexpr int ES = P::ES;
    const char* a_tile = p.A + ES * (q.batch * p.batch_a + q.m0 * p.a_sm + q.k_begin * p.a_sk);
    const char* b_tile = p.B + ES * (q.batch * p.batch_b + q.n0 * p.b_sn + q.k_begin * p.b_sk);
    const int a_rows = p.M - q.m0 < BM ? p.M - q.m0 : BM;
    const int b_rows = p.N - q.n0 < BN ? p.N - q.n0 : BN;
    // pitch of a row of an LDS tile: a row of the matrix (K-contiguous operand) or a k-row
    const uint32_t a_ld = static_cast<uint32_t>(ES * (p.a_sk == 1 ? p.a_sm : p.a_sk));
    const uint32_t b_ld = static_cast<uint32_t>(ES * (p.b_sk == 1 ? p.b_sn : p.b_sk));

    typename P::tile_t acc;
    acc.clear();
    P::run(wgp, acc, a_tile, a_ld, a_rows, b_tile, b_ld, b_rows,
           (q.k_end - q.k_begin) / P::K_PER_STEP, lds, wave, lane, p.stamps, (q.n0 / BN) & 3, (q.m0 / BM) & 3);
    stamp(p.stamps, STAMP_K_LOOP_DONE);

    // The epilogue's per-lane addressing is computed after the K loop: kept live across it, it
    // would not fit in registers beside the accumulators and fragments.
    int lane_now = lane;
    asm volatile("" : "+v"(lane_now));
    epilogue<typename P::tile_t, P::MT, P::NT, false, P::PAIRED_N>(wgp, p, q, acc, q.m0 + (wave / WAVES_N) * P::WTM,
                                                                   q.n0 + (wave % WAVES_N) * P::WTN, lds, wave, lane_now);
    if (p.stamps) {  // the last stamp is taken when this wave's stores have been acknowledged
        wg::wait_counts<0, 0>();
        stamp(p.stamps, STAMP_STORES_DONE);
    }
}

// Persistent form for the 256x256x64 tile: workgroup w takes tiles w, w + gridDim.x, ...
// and streams their K steps through wg::PersistentPipe.  Every unit must have an even number
// of K steps, at least two (the host guarantees it).
template <typename T>
__global__ __launch_bounds__(256) void gemm_persistent(const GemmParams p, const int total)
{
    const persp::Workgroup wgp = persp::Grid::at_kernel_entry().workgroup();
    using P = wg::PersistentPipe<T>;
    __shared__ __attribute__((aligned(1024))) char lds[P::LDS_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    auto source = [&](const Placement& q) {
        typename P::Source s;
        s.a = p.A + 2 * (q.batch * p.batch_a + q.m0 * p.a_sm + q.k_begin);
        s.b = p.B + 2 * (q.batch * p.batch_b + q.n0 * p.b_sn + q.k_begin);
        s.a_ld = static_cast<uint32_t>(2 * p.a_sm);
        s.b_ld = static_cast<uint32_t>(2 * p.b_sn);
        s.a_rows = p.M - q.m0 < P::BM ? p.M - q.m0 : P::BM;
        s.b_rows = p.N - q.n0 < P::BN ? p.N - q.n0 : P::BN;
        return s;
    };
    int tile = blockIdx.x;
    Placement cur = place<P::BM, P::BN>(p, tile), nxt = cur;
    P::run(
        wgp, lds, wave, lane, source(cur), (cur.k_end - cur.k_begin) / P::BK,
        [&](typename P::Source& s, int& ksteps) {
            if (tile + static_cast<int>(gridDim.x) >= total) return false;
            nxt = place<P::BM, P::BN>(p, tile + gridDim.x);
            s = source(nxt);
            ksteps = (nxt.k_end - nxt.k_begin) / P::BK;
            return true;
        },
        [&](typename P::tile_t& acc) {
            // The epilogue's per-lane addressing is recomputed for every tile: kept live across
            // the K loop it would not fit in registers beside the accumulators and fragments.
            int lane_now = lane;
            asm volatile("" : "+v"(lane_now));
            epilogue<typename P::tile_t, P::MT, P::NT, true, P::PAIRED_N>(wgp, p, cur, acc, cur.m0 + (wave / P::WAVES_N) * P::WTM,
                                                                          cur.n0 + (wave % P::WAVES_N) * P::WTN,
                                                                          lds + P::PATCH_BASE + wave * P::PATCH_BYTES, wave, lane_now);
        },
        [&]() {
            cur = nxt;
            tile += gridDim.x;
        });
}

template <typename S>
__global__ __launch_bounds__(256, 2) void gemm_staged(const GemmParams p)
{
    const persp::Workgroup wgp = persp::Grid::at_kernel_entry().workgroup();
    __shared__ __attribute__((aligned(1024))) char lds[S::LDS_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const Placement q = place<S::BM, S::BN>(p, blockIdx.x);

    const char* a_tile = p.A + S::ES * (q.batch * p.batch_a + q.m0 * p.a_sm);
    const char* b_tile = p.B + S::ES * (q.batch * p.batch_b + q.n0 * p.b_sn);
    const int a_rows = p.M - q.m0 < S::BM ? p.M - q.m0 : S::BM;
    const int b_rows = p.N - q.n0 < S::BN ? p.N - q.n0 : S::BN;

    typename S::tile_t acc;
    acc.clear();
    S::run(wgp, acc, a_tile, p.a_sm, p.a_sk, a_rows, p.a_sk == 1 ? p.K : p.M, b_tile, p.b_sn, p.b_sk, b_rows,
           p.b_sk == 1 ? p.K : p.N, q.k_begin, q.k_end, p.K, lds, wave, lane);

    epilogue<typename S::tile_t, S::MT, S::NT, false, S::PAIRED_N>(wgp, p, q, acc, q.m0 + (wave >> 1) * S::WTM,
                                                                   q.n0 + (wave & 1) * S::WTN, lds, wave, lane);
}

// One thread per group of four consecutive n.  Slices are added in order
// 0, 1, ..., split_k-1 so the result does not depend on scheduling.
// Partial sums that the caches hold are bound by the latency of their loads, so four slices are
// asked for before the first is added (4 slices of 16 x 4096: the call 16.4 -> 15.2 us; 19 of
// 640 x 192: 51.8 -> 49.0).  More than that are bound by memory, where a wave that asks for
// several slices, megabytes apart, at a time is slower (16 slices of 1024 x 1024: 84.6 us one by
// one, 85.7 with four, 86.4 with eight ahead) and where each is read once: as a stream the same call
// takes 81.9 us.
__global__ __launch_bounds__(256) void splitk_reduce(const GemmParams p)
{
    constexpr int kAhead = 4;
    constexpr int64_t kCached = int64_t{16} << 20;
    const uint32_t groups_n = (p.N + 3) / 4;
    const int64_t slab = static_cast<int64_t>(p.M) * p.N;
    const int64_t total = static_cast<int64_t>(p.batch) * p.M * groups_n;
    const bool ahead = p.batch * p.split_k * slab * 4 <= kCached;
    for (int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; idx < total;
         idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int g, m, b;
        if (total <= INT32_MAX) {  // a 64-bit division costs as much as the additions of a short sum
            const uint32_t i = static_cast<uint32_t>(idx), bm = i / groups_n;
            g = static_cast<int>(i - bm * groups_n);
            b = static_cast<int>(p.batch == 1 ? 0u : bm / static_cast<uint32_t>(p.M));
            m = static_cast<int>(bm - static_cast<uint32_t>(b) * static_cast<uint32_t>(p.M));
        } else {
            const int64_t bm = idx / groups_n;
            g = static_cast<int>(idx - bm * groups_n);
            b = static_cast<int>(bm / p.M);
            m = static_cast<int>(bm - static_cast<int64_t>(b) * p.M);
        }
        const int n0 = 4 * g, left = p.N - n0;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        const char* src = reinterpret_cast<const char*>(p.partial + static_cast<int64_t>(b) * p.split_k * slab + static_cast<int64_t>(m) * p.N + n0);
        if (left >= 4 && !ahead) {
            for (int s = 0; s < p.split_k; ++s, src += 4 * slab) sum += __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(src));
        } else if (left >= 4) {
            int s = 0;
            for (; s + kAhead <= p.split_k; s += kAhead, src += 4 * kAhead * slab) {
                f32x4 part[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) part[u] = grid::load4<DT_F32>(src + 4 * u * slab);
#pragma unroll
                for (int u = 0; u < kAhead; ++u) sum += part[u];
            }
            if (s < p.split_k) {  // the rest, those beyond the last slice read again and left out
                f32x4 part[kAhead - 1];
#pragma unroll
                for (int u = 0; u < kAhead - 1; ++u) part[u] = grid::load4<DT_F32>(src + 4 * (s + u < p.split_k ? u : p.split_k - 1 - s) * slab);
#pragma unroll
                for (int u = 0; u < kAhead - 1; ++u)
                    if (s + u < p.split_k) sum += part[u];
            }
        } else {
            for (int s = 0; s < p.split_k; ++s, src += 4 * slab) sum += grid::load_some<DT_F32>(src, left);
        }
        const grid::Target to = grid::target_of(p, b);
        f32x4 add = {0.f, 0.f, 0.f, 0.f};
        if (to.bias && to.bias_along_m) add = f32x4{to.bias[m], to.bias[m], to.bias[m], to.bias[m]};
        else if (to.bias && left >= 4) add = grid::load4<DT_F32>(reinterpret_cast<const char*>(to.bias + n0));
        else if (to.bias) add = grid::load_some<DT_F32>(reinterpret_cast<const char*>(to.bias + n0), left);
        sum = grid::scaled(to.alpha, sum, add);
        auto finish = [&](auto out_c) {
            constexpr int OUT = decltype(out_c)::value;
            char* dst = to.c + m * to.row_bytes + static_cast<int64_t>(n0) * grid::out_bytes<OUT>();
            if (to.beta != 0.0f) sum = grid::scaled(to.beta, left >= 4 ? grid::load4<OUT>(dst) : grid::load_some<OUT>(dst, left), sum);
            if (left >= 4) grid::store4<OUT>(dst, sum);
            else grid::store_some<OUT>(dst, sum, left);
        };
        if (to.dtype == DT_BF16) finish(std::integral_constant<int, DT_BF16>{});
        else if (to.dtype == DT_F16) finish(std::integral_constant<int, DT_F16>{});
        else finish(std::integral_constant<int, DT_F32>{});
    }
}

template <typename P, int BM, int BN, int BK, int WAVES_N>
hipError_t launch_pipe(const GemmParams& p, int workgroups, hipStream_t stream)
{
    hipLaunchKernelGGL((gemm_pipelined<P, BM, BN, BK, WAVES_N>), dim3(workgroups), dim3(P::THREADS), 0, stream, p);
    return hipGetLastError();
}

// Operands that the memory-side cache (256 MB) does not hold from call to call, beside C and what else the program
// touches: their lines are asked for ahead of the copies (Pipeline's AHEAD).  Measured with inputs that change from
// call to call: 16384 x 4096 x 4096 (168 MB) 378 -> 367 us, 16384 x 10240 x 2048 (109 MB) 484 -> 480,
// 2048 x 4096 x 16384 (201 MB) 229 -> 210, 1024 x 1024 x 32768 (134 MB) 82 -> 74, row-major B 8192 x 4096 x 8192
// (201 MB) 375 -> 370; but 4096 x 4096 x 4096 (67 MB) 89.3 -> 90.6, row-major B 8192 x 4096 x 4096 (101 MB) 187 ->
// 189.  With both operands as k-rows, whose steps lie megabytes apart, earlier: 4096 x 4096 x 4096 107 -> 103,
// 4096 x 4096 x 8192 with beta 207 -> 203.
bool operands_from_memory(const GemmParams& p)
{
    const double bytes = 2.0 * p.K * (static_cast<double>(p.M) * (p.batch_a == 0 ? 1 : p.batch) + static_cast<double>(p.N) * (p.batch_b == 0 ? 1 : p.batch));
    return bytes > (p.a_sk != 1 && p.b_sk != 1 ? 6.0e7 : 1.05e8);
}

template <typename P, typename P_AHEAD>
hipError_t launch_large(const GemmParams& p, int workgroups, hipStream_t stream)
{
    return operands_from_memory(p) ? launch_pipe<P_AHEAD, 256, 256, 64, 2>(p, workgroups, stream) : launch_pipe<P, 256, 256, 64, 2>(p, workgroups, stream);
}
template <typename T, bool B_KN, bool A_MK, bool AHEAD = false>
using Large = wg::Pipeline<T, 256, 256, 64, 2, 2, 2, B_KN, A_MK, AHEAD>;

template <typename T>
hipError_t launch_pipe_config(int config, const GemmParams& p, int workgroups, hipStream_t stream)
{
    switch (config) {
    case 0: return launch_large<Large<T, false, false>, Large<T, false, false, true>>(p, workgroups, stream);
    case 1: return launch_pipe<wg::Pipeline<T, 128, 128, 64, 2, 2, 2>, 128, 128, 64, 2>(p, workgroups, stream);
    case 2: return launch_pipe<wg::Pipeline<T, 128, 128, 64, 2, 2, 2, true>, 128, 128, 64, 2>(p, workgroups, stream);
    case 3: return launch_pipe<wg::Pipeline<T, 128, 128, 64, 2, 2, 2, false, true>, 128, 128, 64, 2>(p, workgroups, stream);
    case 4: return launch_pipe<wg::Pipeline<T, 128, 128, 64, 2, 2, 2, true, true>, 128, 128, 64, 2>(p, workgroups, stream);
    case 9: return launch_large<Large<T, true, false>, Large<T, true, false, true>>(p, workgroups, stream);
    case 10: return launch_large<Large<T, false, true>, Large<T, false, true, true>>(p, workgroups, stream);
    case 11: return launch_large<Large<T, true, true>, Large<T, true, true, true>>(p, workgroups, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_pipelined(int config, int ab_dtype, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if (ab_dtype == DT_F32) {  // fp32 operands: 128x128 tiles, the four layout pairs
        switch (config) {
        case 5: return launch_pipe<wg::Pipeline<f32_t, 128, 128, 64, 2, 2, 2>, 128, 128, 64, 2>(p, workgroups, stream);
        case 6: return launch_pipe<wg::Pipeline<f32_t, 128, 128, 64, 2, 2, 2, true>, 128, 128, 64, 2>(p, workgroups, stream);
        case 7: return launch_pipe<wg::Pipeline<f32_t, 128, 128, 64, 2, 2, 2, false, true>, 128, 128, 64, 2>(p, workgroups, stream);
        case 8: return launch_pipe<wg::Pipeline<f32_t, 128, 128, 64, 2, 2, 2, true, true>, 128, 128, 64, 2>(p, workgroups, stream);
        default: return hipErrorInvalidValue;
        }
    }
    return ab_dtype == DT_BF16 ? launch_pipe_config<bf16_t>(config, p, workgroups, stream)
                               : launch_pipe_config<f16_t>(config, p, workgroups, stream);
}

hipError_t launch_persistent(int ab_dtype, const GemmParams& p, int total, int workgroups, hipStream_t stream)
{
    if (ab_dtype == DT_BF16)
        hipLaunchKernelGGL(gemm_persistent<bf16_t>, dim3(workgroups), dim3(256), 0, stream, p, total);
    else
        hipLaunchKernelGGL(gemm_persistent<f16_t>, dim3(workgroups), dim3(256), 0, stream, p, total);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_staged_typed(const GemmParams& p, int workgroups, hipStream_t stream)
{
    const dim3 grid(workgroups), block(256);
    const bool a_mk = p.a_sk != 1, b_kn = p.b_sk != 1;  // contiguous along m / n and not along k
    if (a_mk && b_kn) hipLaunchKernelGGL((gemm_staged<wg::Staged<T, 128, 128, true, true>>), grid, block, 0, stream, p);
    else if (a_mk) hipLaunchKernelGGL((gemm_staged<wg::Staged<T, 128, 128, true, false>>), grid, block, 0, stream, p);
    else if (b_kn) hipLaunchKernelGGL((gemm_staged<wg::Staged<T, 128, 128, false, true>>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((gemm_staged<wg::Staged<T, 128, 128, false, false>>), grid, block, 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_staged(int ab_dtype, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if (ab_dtype == DT_BF16) return launch_staged_typed<bf16_t>(p, workgroups, stream);
    if (ab_dtype == DT_F16) return launch_staged_typed<f16_t>(p, workgroups, stream);
    return launch_staged_typed<f32_t>(p, workgroups, stream);
}

hipError_t launch_reduce(const GemmParams& p, hipStream_t stream)
{
    const int64_t total = static_cast<int64_t>(p.batch) * p.M * ((p.N + 3) / 4);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 16) blocks = 256 * 16;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(splitk_reduce, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, p);
    return hipGetLastError();
}

}  // namespace prism
