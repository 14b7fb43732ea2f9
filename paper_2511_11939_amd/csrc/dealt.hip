// Products that give too few 128x128 tiles for the chip, or whose K loops are short: small workgroups
// whose waves deal the K steps (128 bytes of every row) out among themselves, any layout and alignment.
//
// What bounds such a product on tiles is the chain of its K steps: with one workgroup per compute unit
// a step takes 0.5 (direct-to-LDS copies) to 0.9 us (staged, odd rows) however little of the chip
// is in use.  Here every wave runs a fraction of the steps by itself: it loads its next step into registers while
// it computes the present one, passes the step through LDS of its own (from the order of whole rows into
// the matrix instruction's), and no barrier stands in the loop.  At the end the waves' sums are added in wave order, so
// the result does not depend on timing.  32 x 32 results per workgroup of four or eight waves fill the chip
// from a quarter of a million results on; 64 x 64 by eight waves, and 128 x 64 by eight (two halves of 64 rows,
// four waves along K each), take half the loads per result and serve larger products.  From there on the loads
// bind, 64 bytes a clock per compute unit, at a quarter and at half of the matrix rate, and tiles are
// faster: the host predicts both.  Measured (whole call, tiles before): 704 x 704 x 1856 row-major B
// 19.7 -> 9.5 us, 157 x 1353 x 384 10.0 -> 5.2, 183 x 512 x 1241 21.8 -> 5.3, 265 x 1344 x 768 fp32 58.6 -> 11.7,
// 64 x 192 x 20352 in slices 16.6 -> 9.3, 256 x 256 x 256 row-major B 5.6 -> 5.2.  Tried and
// not kept: 64 x 32 and 128 x 32 results per workgroup, 64 x 64 by four waves, and sixteen waves (best for one product
// in ten, by half a percent over all of them).
//
// Rows that start in the middle of a 32-bit word (16-bit operands, odd pitches): the vector memory unit takes
// such a 16-byte load in pieces (38 bytes a ns and compute unit against 110 for loads at whole
// words), so rows are loaded from the word that they start in, and put in place with the neighbouring
// lane's first word; the one element that no lane holds, a row's last of the step, is
// fetched by one more load for all rows (90).  997 x 991 x 1501 with odd rows 14.1 -> 11.7 us.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "grid.hpp"
#include "lane.hpp"
#include "launch.hpp"
#include "wave.hpp"
#include "workgroup.hpp"

namespace prism {
namespace {

// Rows of 16-bit elements may start in the middle of a 32-bit word.  The vector memory unit takes a 16-byte load from
// there in pieces: 38 bytes a ns and compute unit (60 where every other row is such a one) against 110 for loads
// at whole words.  So a chunk is loaded from the word that it starts in, and put in place, `shift`
// (0 or 2) bytes further down, with the first word of the next lane's, which holds the chunk behind
// it; the last chunk of a row lacks its last element.
__device__ __forceinline__ u32x4 chunk_in_place(u32x4 v, uint32_t shift)
{
    constexpr int kRowShl1 = 0x101;  // from the next lane of 16
    const uint32_t next = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v[0]), kRowShl1, 0xF, 0xF, true));
    return u32x4{__builtin_amdgcn_alignbyte(v[1], v[0], shift), __builtin_amdgcn_alignbyte(v[2], v[1], shift),
                 __builtin_amdgcn_alignbyte(v[3], v[2], shift), __builtin_amdgcn_alignbyte(next, v[3], shift)};
}
using u16_alias = uint16_t __attribute__((may_alias));  // (an element of what was written as chunks)

// What one wave does with one operand: 16 * BLK rows (m or n) of a K step (128 bytes of k).
// K-contiguous rows become the 128-byte rows of TileLayout, an operand contiguous along its other
// index (K_ROWS) becomes k-rows whose fragments come from the transposing reads (fp32: 4-byte reads).
// Either way a load is 1024 contiguous bytes of LDS, a lane's 16 bytes at a place of its own.
template <typename T, int BLK, bool K_ROWS, bool ODD>
struct WaveOperand {
    using L = lane::TileLayout<64>;
    static constexpr int ES = Frag<T>::kElemBytes, EPC = lane::kChunkBytes / ES, STEP = L::kRowBytes / ES;
    static constexpr int ROWS = lane::kBlock * BLK, LOADS = 2 * BLK, BYTES = 1024 * LOADS;
    static constexpr int ROW_BYTES = K_ROWS ? ROWS * ES : L::kRowBytes, PER_ROW = ROW_BYTES / lane::kChunkBytes, ROW_STEP = 64 / PER_ROW;
    static_assert(!ODD || ES == 2, "rows of 32-bit elements start on whole words");
    using frag_t = typename Frag<T>::type;

    const char* tile;  // element (first row of the tile, k 0)
    const char* words; // the 32-bit word it lies in (ODD), or the same
    int64_t pitch;     // bytes between rows, or between k-rows
    int rows;          // rows of the tile that exist, >= 1
    int row0, chunk;
    uint32_t put[2];   // where loads of even and odd number go, beyond 1024 times their number
    uint32_t off[LOADS];
    // ODD: by how many bytes this lane's rows start after a whole word; where the one element comes from and goes to
    uint32_t shift, last_off, last_put;

    static __device__ __forceinline__ int swizzle(int row)
    {
        if constexpr (!K_ROWS) return L::swizzle(row);
        else if constexpr (ES == 2) return ((row & 3) << 1) & (PER_ROW - 1);
        else return (((row >> 2) & 1) << 2) & (PER_ROW - 1);
    }
    // (rows below 2^7, pitches below 2^23 bytes)
    __device__ __forceinline__ uint32_t row_offset(int row) const { return __umul24(static_cast<uint32_t>(row), static_cast<uint32_t>(pitch)); }
    __device__ __forceinline__ void init(const char* tile_, int64_t s_row, int64_t s_k, int rows_, int lane)
    {
        tile = tile_;
        pitch = ES * (K_ROWS ? s_k : s_row);
        rows = rows_;
        row0 = lane / PER_ROW;
        chunk = lane % PER_ROW;
        const int last = (rows - 1) / EPC;
        // (words are counted from the one that the tile starts in, so that no offset is negative)
        const uint32_t into = ODD ? static_cast<uint32_t>(reinterpret_cast<uintptr_t>(tile)) & 2u : 0u;
        words = tile - into;
        shift = ODD ? (into + row_offset(row0)) & 2u : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) put[h] = row0 * ROW_BYTES + ((chunk ^ swizzle(row0 + h * ROW_STEP)) * lane::kChunkBytes);
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            const int row = row0 + r * ROW_STEP;
            if constexpr (K_ROWS) off[r] = row_offset(row) + (chunk < last ? chunk : last) * lane::kChunkBytes;
            else off[r] = row_offset(row < rows ? row : rows - 1) + chunk * lane::kChunkBytes;
            if constexpr (ODD) off[r] = (off[r] + into) & ~3u;
        }
        if constexpr (ODD && K_ROWS) {
            const int col = (rows < ROWS ? rows : ROWS) - 1;
            last_off = into + row_offset(lane) + col * ES;
            last_put = lane * ROW_BYTES + (((col / EPC) ^ swizzle(lane)) * lane::kChunkBytes) + col % EPC * ES;
        } else if constexpr (ODD) {
            const int row = lane % ROWS;
            last_off = into + row_offset(row < rows ? row : rows - 1) + L::kRowBytes - ES;
            last_put = L::offset(row, L::kChunksPerRow - 1) + lane::kChunkBytes - ES;
        }
    }
    __device__ __forceinline__ void load(u32x4 (&regs)[LOADS], uint32_t& last, int64_t k0)
    {
        const wg::global_bytes step = (wg::global_bytes)wg::scalarize(words + (K_ROWS ? k0 * pitch : k0 * ES));
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            asm volatile("" : "+v"(off[r]));
            regs[r] = *(const __attribute__((address_space(1))) u32x4_any*)(step + off[r]);
        }
        if constexpr (ODD) {
            asm volatile("" : "+v"(last_off));
            last = *(const __attribute__((address_space(1))) uint16_t*)(step + last_off);
        }
    }
    // The elements k0 .. k_end - 1 of the rows, at most a step, or a step whose last k-row ends the operand:
    // chunks are loaded from where they lie inside their row and moved into place when they are stored.
    __device__ __forceinline__ int last_from(int k0, int k_end) const
    {
        const int first = K_ROWS ? chunk * EPC : k0 + chunk * EPC, end = K_ROWS ? rows : k_end;
        return first + EPC <= end ? first : end - EPC;
    }
    __device__ __forceinline__ void load_last(u32x4 (&regs)[LOADS], int k0, int k_end) const
    {
        // (where the row has less than a chunk, the chunk that ends with it)
        const uint32_t from = lane::kChunkBytes + last_from(k0, k_end) * ES;
        const wg::global_bytes base = (wg::global_bytes)wg::scalarize(tile + (K_ROWS ? k0 * pitch : 0) - lane::kChunkBytes);
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            const int row = row0 + r * ROW_STEP, exist = K_ROWS ? k_end - k0 : rows;
            regs[r] = *(const __attribute__((address_space(1))) u32x4_any*)(base + (row_offset(row < exist ? row : exist - 1) + from));
        }
    }
    __device__ __forceinline__ void store_last(const u32x4 (&regs)[LOADS], int k0, int k_end, char* slot) const
    {
        const uint32_t down = ((K_ROWS ? 0 : k0) + chunk * EPC - last_from(k0, k_end)) * ES;
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            const bool beyond = K_ROWS && k0 + row0 + r * ROW_STEP >= k_end;
            *reinterpret_cast<u32x4*>(slot + put[r & 1] + 1024 * r) = wg::chunk_moved_down(regs[r], beyond ? lane::kChunkBytes : down);
        }
    }
    __device__ __forceinline__ void store(const u32x4 (&regs)[LOADS], uint32_t last, char* slot) const
    {
        if constexpr (ODD) {
#pragma unroll
            for (int r = 0; r < LOADS; ++r) *reinterpret_cast<u32x4*>(slot + put[r & 1] + 1024 * r) = chunk_in_place(regs[r], shift);
            *reinterpret_cast<u16_alias*>(slot + last_put) = static_cast<uint16_t>(last);
        } else {
#pragma unroll
            for (int r = 0; r < LOADS; ++r) *reinterpret_cast<u32x4*>(slot + put[r & 1] + 1024 * r) = regs[r];
        }
    }
    __device__ __forceinline__ static void fragments(persp::Wave wv, frag_t (&f)[BLK], const char* slot, int ks, int lane)
    {
        if constexpr (!K_ROWS) {
            wave::load_fragments<T, 64, BLK>(wv, f, slot, 0, ks, lane);
        } else if constexpr (ES == 2) {
            uint32_t part[4];
#pragma unroll
            for (int jl = 0; jl < 4; ++jl) part[jl] = wave::k_rows_lane_part<ROW_BYTES>(wv, jl, lane);
#pragma unroll
            for (int j = 0; j < BLK; ++j) {
                const wave::v4s lo = wave::read_k_rows_half<ROW_BYTES>(wv, slot, 0, j, ks, 0, part);
                const wave::v4s hi = wave::read_k_rows_half<ROW_BYTES>(wv, slot, 0, j, ks, 1, part);
                f[j] = __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        } else {
            const int x = lane & 15, g = lane >> 4;
#pragma unroll
            for (int j = 0; j < BLK; ++j) {
                const int n = lane::kBlock * j + x;
                const char* src = slot + (16 * ks + 4 * g) * ROW_BYTES + (((n >> 2) ^ (((g & 1) << 2) & (PER_ROW - 1))) * lane::kChunkBytes) + (n & 3) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) f[j][e] = *reinterpret_cast<const float*>(src + e * ROW_BYTES);
            }
        }
    }
};

// MT x NT blocks of 16 x 16 per wave, WM waves side by side along m, WK along K.
template <typename T, int MT, int NT, int WM, int WK, bool A_MK, bool B_KN, bool ODD>
__global__ __launch_bounds__(64 * WM * WK, (WM * WK) / 4) void gemm_dealt(const GemmParams p)
{
    constexpr int THREADS = 64 * WM * WK, BM = lane::kBlock * MT * WM, BN = lane::kBlock * NT;
    using OA = WaveOperand<T, MT, A_MK, ODD>;
    using OB = WaveOperand<T, NT, B_KN, ODD>;
    constexpr int ES = OA::ES, STEP = OA::STEP, WAVE_BYTES = OA::BYTES + OB::BYTES;
    static_assert(MT * NT * 1024 <= WAVE_BYTES, "a wave's sums take the place of its step");
    const persp::Block<THREADS> wgp = persp::Grid::at_kernel_entry().workgroup<THREADS>();
    const persp::Wave wv = wgp.wave();
    __shared__ __attribute__((aligned(1024))) char lds[WM * WK * WAVE_BYTES];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_m = wave % WM, wave_k = wave / WM;
    stamp(p.stamps, STAMP_ENTRY);

    const grid::TileCoord c = grid::schedule(blockIdx.x, p.tiles_m, p.tiles_n, p.batch * p.split_k);
    const int batch = __builtin_amdgcn_readfirstlane(p.split_k == 1 ? c.unit : grid::uniform_quotient(c.unit, p.split_k));
    const int slice = __builtin_amdgcn_readfirstlane(c.unit - batch * p.split_k);
    const int m0 = __builtin_amdgcn_readfirstlane(c.tile_m * BM), n0 = __builtin_amdgcn_readfirstlane(c.tile_n * BN);
    const int k_begin = slice * p.k_slice, k_end = k_begin + p.k_slice < p.K ? k_begin + p.k_slice : p.K;

    using frag_t = typename Frag<T>::type;
    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int m_wave = m0 + wave_m * lane::kBlock * MT;
    char* slot = lds + wave * WAVE_BYTES;
    const bool has_rows = m_wave < p.M;
    if (has_rows) {
        OA a;
        OB b;
        a.init(p.A + ES * (batch * p.batch_a + m_wave * p.a_sm), p.a_sm, p.a_sk, p.M - m_wave < OA::ROWS ? p.M - m_wave : OA::ROWS, lane);
        b.init(p.B + ES * (batch * p.batch_b + n0 * p.b_sn), p.b_sn, p.b_sk, p.N - n0 < OB::ROWS ? p.N - n0 : OB::ROWS, lane);
        const char* passed = slot + wave::unknown_offset(wv);
        auto compute = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                frag_t fa[MT], fb[NT];
                OB::fragments(wv, fb, passed, ks, lane);
                OA::fragments(wv, fa, passed + OB::BYTES, ks, lane);
#pragma unroll
                for (int e = 0; e < wave::mfma_parts(frag_t{}); ++e)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NT; ++j) acc[i][j] = wave::mfma_part(wv, fb[j], fa[i], e, acc[i][j]);
            }
            PRISM_PARANOID_WAIT();
        };
        // Steps loaded at fixed offsets: all whole ones but the last where its loads would run past the
        // end of an operand's last k-row.
        const int steps = (k_end - k_begin) / STEP;
        const bool runs_over = k_end == p.K && steps * STEP == k_end - k_begin &&
                               ((A_MK && p.M % OA::EPC != 0) || (B_KN && p.N % OB::EPC != 0));
        const int whole = steps - (runs_over ? 1 : 0);
        const int mine = whole > wave_k ? (whole - wave_k + WK - 1) / WK : 0;
        u32x4 ra[OA::LOADS], rb[OB::LOADS];
        uint32_t last_a = 0, last_b = 0;
        auto load = [&](int q) __attribute__((always_inline)) {
            const int64_t k0 = k_begin + static_cast<int64_t>(wave_k + q * WK) * STEP;
            b.load(rb, last_b, k0);
            a.load(ra, last_a, k0);
        };
        const int rest = k_begin + whole * STEP;
        const bool mine_too = rest < k_end && wave_k == whole % WK;
        auto load_rest = [&]() __attribute__((always_inline)) {
            b.load_last(rb, rest, k_end);
            a.load_last(ra, rest, k_end);
        };
        if (mine > 0) load(0);
        else if (mine_too) load_rest();
        stamp(p.stamps, STAMP_FIRST_FRAGMENTS);
        for (int q = 0; q < mine; ++q) {
            b.store(rb, last_b, slot);
            a.store(ra, last_a, slot + OB::BYTES);
            PRISM_PARANOID_WAIT();
            if (q + 1 < mine) load(q + 1);
            else if (mine_too) load_rest();
            __builtin_amdgcn_sched_barrier(0);
            compute();
        }
        if (mine_too) {
            b.store_last(rb, rest, k_end, slot);
            a.store_last(ra, rest, k_end, slot + OB::BYTES);
            PRISM_PARANOID_WAIT();
            compute();
        }
    }
    stamp(p.stamps, STAMP_K_LOOP_DONE);

    // The waves' sums: lane (x, g) holds columns 4 g .. + 3 of row x of a block.  They are kept so that
    // lanes that read a row piece by piece find its pieces on different banks.
    const int x = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) reinterpret_cast<f32x4*>(slot)[(i * NT + j) * 64 + 16 * g + (x ^ (4 * j + g))] = acc[i][j];
    __syncthreads();
    const grid::Target to = p.split_k > 1 ? grid::partial_of(p, batch, slice) : grid::target_of(p, batch);
    auto finish = [&](auto out_c) __attribute__((always_inline)) {
        constexpr int OUT = decltype(out_c)::value, QUADS = 4 * NT;
        for (int e = threadIdx.x; e < BM * QUADS; e += THREADS) {
            const int row = e / QUADS, q = e % QUADS, wm = row / (lane::kBlock * MT), i = row / lane::kBlock % MT;
            const int at = (i * NT + q / 4) * 64 + 16 * (q % 4) + ((row & 15) ^ q);
            const int m = m0 + row, n = n0 + 4 * q, left = p.N - n;
            if (m >= p.M || left <= 0) continue;
            f32x4 sum = reinterpret_cast<const f32x4*>(lds + wm * WAVE_BYTES)[at];
#pragma unroll
            for (int w = 1; w < WK; ++w) sum += reinterpret_cast<const f32x4*>(lds + (w * WM + wm) * WAVE_BYTES)[at];
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

template <typename T, int MT, int NT, int WM, int WK>
void launch_layout(bool odd_rows, const GemmParams& p, int workgroups, hipStream_t stream)
{
    const dim3 grid(workgroups), block(64 * WM * WK);
    const bool a_mk = p.a_sk != 1, b_kn = p.b_sk != 1;
    if constexpr (Frag<T>::kElemBytes == 2)
        if (odd_rows) {
            if (a_mk && b_kn) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, true, true, true>), grid, block, 0, stream, p);
            else if (a_mk) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, true, false, true>), grid, block, 0, stream, p);
            else if (b_kn) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, false, true, true>), grid, block, 0, stream, p);
            else hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, false, false, true>), grid, block, 0, stream, p);
            return;
        }
    if (a_mk && b_kn) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, true, true, false>), grid, block, 0, stream, p);
    else if (a_mk) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, true, false, false>), grid, block, 0, stream, p);
    else if (b_kn) hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, false, true, false>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((gemm_dealt<T, MT, NT, WM, WK, false, false, false>), grid, block, 0, stream, p);
}
template <typename T>
hipError_t launch_typed(int rows, int waves, bool odd_rows, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if (rows == 128) launch_layout<T, 4, 4, 2, 4>(odd_rows, p, workgroups, stream);
    else if (rows == 64) launch_layout<T, 4, 4, 1, 8>(odd_rows, p, workgroups, stream);
    else if (waves == 8) launch_layout<T, 2, 2, 1, 8>(odd_rows, p, workgroups, stream);
    else launch_layout<T, 2, 2, 1, 4>(odd_rows, p, workgroups, stream);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_dealt(int ab_dtype, int rows, int waves, bool odd_rows, const GemmParams& p, int workgroups, hipStream_t stream)
{
    if (ab_dtype == DT_BF16) return launch_typed<bf16_t>(rows, waves, odd_rows, p, workgroups, stream);
    if (ab_dtype == DT_F16) return launch_typed<f16_t>(rows, waves, odd_rows, p, workgroups, stream);
    return launch_typed<f32_t>(rows, waves, odd_rows, p, workgroups, stream);
}

}  // namespace prism
