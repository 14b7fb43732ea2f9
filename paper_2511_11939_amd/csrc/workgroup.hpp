// Workgroup layer: everything the wavefronts of one workgroup do together --
// moving operand tiles from global memory into LDS, the barriers that order
// those moves against the fragment reads, and the K loop around the wave
// tiles.  Functions take the calling wave's index inside the workgroup and the
// lane's index inside the wave; they never look at grid coordinates.
//
// The structure follows what the paper says a peak-rate matrix multiply needs
// (section 6.2): data movement pipelined under the matrix instructions with
// statically sized, individually synchronised pipeline slots.  On gfx950 the
// asynchronous copy is the direct global->LDS load and the slot hand-over is
// one workgroup barrier per K step, placed by hand where the paper's compiler
// would insert it (section 5, synchronisation at loop back-edges).
#pragma once

#include <type_traits>

#include "lane.hpp"
#include "stamp.hpp"
#include "wave.hpp"

namespace prism {
namespace wg {

// s_waitcnt immediate for gfx9-family encodings: at most `vm` vector-memory and
// `lgkm` LDS/scalar operations of this wave may still be outstanding.
constexpr int waitcnt_imm(int vm, int lgkm)
{
    return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | ((lgkm & 15) << 8);
}
template <int VM, int LGKM>
__device__ __forceinline__ void wait_counts()
{
    static_assert(VM >= 0 && VM <= 63 && LGKM >= 0 && LGKM <= 15, "counter out of range");
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(VM, LGKM));
}

__device__ __forceinline__ uint32_t lds_address(const void* p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (const __attribute__((address_space(3))) char*)p));
}

// Asynchronous 16-bytes-per-lane copy global -> LDS for one wavefront: lane l
// reads 16 bytes at (uniform_base + lane_offset) and the hardware deposits them
// at lds_addr + 16*l.  The wave's vector-memory counter tracks completion.
__device__ __forceinline__ const char* scalarize(const char* p)
{
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
}

// Workgroup barrier: only code that holds the workgroup token -- code every wave of the
// workgroup executes -- can reach it (the paper's block-level synchronisation, section 3.5).
__device__ __forceinline__ void barrier(persp::Workgroup) { __builtin_amdgcn_s_barrier(); }
// Barrier that also waits for the caller's outstanding LDS and memory operations.
__device__ __forceinline__ void sync(persp::Workgroup) { __syncthreads(); }

// Race check by construction: built with PRISM_PARANOID_BARRIERS, every phase of a main loop
// that touches LDS ends with a full workgroup barrier (all of the wave's memory operations
// waited for first).  The hand-placed waits and the one barrier per K step are meant to be
// sufficient, so the results of that build must be bit-identical to the normal one's.
#ifdef PRISM_PARANOID_BARRIERS
#define PRISM_PARANOID_SYNC(wgp) ::prism::wg::sync(wgp)
#else
#define PRISM_PARANOID_SYNC(wgp) do { } while (0)
#endif

// One wave-wide copy of 64 x 16 bytes from global memory straight into LDS: lane l's bytes
// land at lds_base + lds_offset + 16*l.  Wave-level: base and LDS address are per-wave
// values; lds_offset must be a compile-time constant at the point of use, so that a copy
// costs two instructions (the LDS address goes to M0 with one scalar add).
__device__ __forceinline__ void copy_async_16(persp::Wave, const char* uniform_base, uint32_t lane_offset,
                                              uint32_t lds_base, int lds_offset)
{
    uniform_base = scalarize(uniform_base);  // no-ops when the values already live in SGPRs
    lds_base = __builtin_amdgcn_readfirstlane(lds_base);
    asm volatile("s_add_u32 m0, %2, %3\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(lane_offset), "s"(uniform_base), "s"(lds_base), "i"(lds_offset)
                 : "memory", "scc");
}

// Asks for the 128-byte lines that hold the lanes' bytes, so that they are in the die's L2 when their copies are
// issued: one word per lane, dropped at `lds_sink` (256 bytes nobody reads).
__device__ __forceinline__ void touch_lines(persp::Wave, const char* uniform_base, uint32_t lane_offset, uint32_t lds_sink)
{
    uniform_base = scalarize(uniform_base);
    lds_sink = __builtin_amdgcn_readfirstlane(lds_sink);
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" : : "v"(lane_offset), "s"(uniform_base), "s"(lds_sink) : "memory");
}

// ---- from the accumulators to memory ---------------------------------------------------
// Every lane holds four consecutive columns of one row per block: row 16 i + lane % 16 of the
// wave tile, columns lane::acc_first_col<PAIRED>(j, lane) and on.  Two ways out:
//
// A block's values are taken from the accumulators at this place and no earlier: without it the moves of
// all blocks drift to the top of the epilogue and spill.  Tiles of 16 blocks leave it to the compiler where
// they are: asked for in the accumulation registers, they would halve the others (128 of 256 at two
// waves per SIMD), which the staged loop's steps on their way and two sets of fragments need.
template <int BLOCKS>
__device__ __forceinline__ void taken_here(f32x4& v)
{
    if constexpr (BLOCKS > 16) asm volatile("" : "+a"(v));
    else asm volatile("" : "+v"(v));
}

// drain_direct (32-bit results): the four values go straight out, 64 contiguous bytes of a row
// (PAIRED: 128 in two instructions) from the four lanes that share it.
// row(i) is called before the blocks of block row i, put(i, j, values) for each of them.
template <int MT, int NT, typename TileT, typename Row, typename Put>
__device__ __forceinline__ void drain_direct(persp::Wave, const TileT& acc, Row&& row, Put&& put)
{
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        row(i);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            f32x4 v = acc.acc[i][j];
            taken_here<MT * NT>(v);
            put(i, j, v);
        }
        __builtin_amdgcn_sched_barrier(0);  // one block row at a time keeps the register need small
    }
}

// drain_rows (16-bit results): pack(i, j, values) returns the four results of a block as 8
// bytes.  The pieces of one block row (16 rows of 32 * NT bytes) pass through the wave's LDS
// patch and come back row by row, so that store(row_uniform, row_lane, byte_in_row, piece)
// writes whole rows of the wave tile (16 consecutive lanes hold 256 contiguous bytes): a
// quarter of the LDS traffic of draining the fp32 accumulators, and full cache lines per store
// instruction.  `patch` is this wave's, rows_patch_bytes(NT) long; the padding of 16 bytes per
// row spreads both the writes (16 rows, one piece each) and the reads over all banks.
constexpr int rows_patch_bytes(int nt) { return lane::kBlock * (2 * lane::kBlock * nt + 16); }
template <bool PAIRED, int MT, int NT, typename TileT, typename Row, typename Pack, typename Store>
__device__ __forceinline__ void drain_rows(persp::Wave wv, const TileT& acc, char* patch, int lane, Row&& row, Pack&& pack, Store&& store)
{
    static_assert(NT % 2 == 0, "block columns come in pairs");
    constexpr int ROW_BYTES = 2 * lane::kBlock * NT, PITCH = ROW_BYTES + 16;
    constexpr int PIECES = ROW_BYTES / 16;        // lanes that share a row on the way out
    constexpr int ROWS_PER_ITER = 64 / PIECES, ITERS = lane::kBlock / ROWS_PER_ITER;
    char* wr = patch + (lane & 15) * PITCH + (PAIRED ? 16 : 8) * (lane >> 4);
    const int piece = lane % PIECES, sub = lane / PIECES;
    const char* rd = patch + wave::unknown_offset(wv) + sub * PITCH + 16 * piece;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        row(i);
#pragma unroll
        for (int s = 0; s < NT / 2; ++s) {
            f32x4 lo = acc.acc[i][2 * s], hi = acc.acc[i][2 * s + 1];
            taken_here<MT * NT>(lo);
            taken_here<MT * NT>(hi);
            const u32x2 a = pack(i, 2 * s, lo), b = pack(i, 2 * s + 1, hi);
            if constexpr (PAIRED) {
                *reinterpret_cast<u32x4*>(wr + 64 * s) = u32x4{a[0], a[1], b[0], b[1]};
            } else {
                *reinterpret_cast<u32x2*>(wr + 64 * s) = a;
                *reinterpret_cast<u32x2*>(wr + 64 * s + 32) = b;
            }
        }
        PRISM_PARANOID_WAIT();
        u32x4 out[ITERS];
#pragma unroll
        for (int it = 0; it < ITERS; ++it) out[it] = *reinterpret_cast<const u32x4*>(rd + it * ROWS_PER_ITER * PITCH);
        PRISM_PARANOID_WAIT();
#pragma unroll
        for (int it = 0; it < ITERS; ++it) store(lane::kBlock * i + it * ROWS_PER_ITER, sub, 16 * piece, out[it]);
        __builtin_amdgcn_sched_barrier(0);  // one block row at a time keeps the register need small
    }
}

// ------------------------------------------------------------------------------------
// Pipelined main loop: direct-to-LDS copies, STAGES slots.  An operand is K-contiguous
// (its LDS tile is BM or BN rows of BK elements) or contiguous along its other index
// (A_MK: A along m, B_KN: B along n; the LDS tile is then BK k-rows of BM or BN elements,
// copied as it lies in memory, and the fragments, which need consecutive k per lane, are
// fetched with the transposing LDS read of gfx950, two per fragment).
// ------------------------------------------------------------------------------------
template <typename T, int BM, int BN, int BK, int WAVES_M, int WAVES_N, int STAGES, bool B_KN = false, bool A_MK = false, bool AHEAD = false>
struct Pipeline {
    using L = lane::TileLayout<BK>;
    static constexpr int ES = Frag<T>::kElemBytes;
    static constexpr int K_PER_STEP = L::kRowBytes / ES;  // elements of K one step consumes (BK counts 2-byte units)
    // Every read of a k-row tile is one of four per-lane addresses kept in registers plus a
    // constant, as with the rows of a K-contiguous operand; addresses worked out per read would
    // not fit beside the 256 accumulators of the 256x256 tile (several hundred spills).
    static_assert(!B_KN || (BK == 64 && (BN == 128 || (BN == 256 && ES == 2))), "n-contiguous B: k-rows of 128 or 256 elements");
    static_assert(!A_MK || (BK == 64 && (BM == 128 || (BM == 256 && ES == 2))), "m-contiguous A: k-rows of 128 or 256 elements");
    static_assert(!(A_MK && B_KN) || BM == BN, "both operands as k-rows: square tile");
    // A K-contiguous B is dealt to the LDS rows in the paired order (lane::paired_tile_row), so
    // that the epilogue can store from the registers; the k-row form keeps the plain order.
    static constexpr bool PAIRED_N = !B_KN;
    static constexpr int NW = WAVES_M * WAVES_N;
    static constexpr int THREADS = NW * 64;
    static constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
    static constexpr int MT = WTM / lane::kBlock, NT = WTN / lane::kBlock;
    static constexpr int KSUB = BK / lane::kBlockK;
    static constexpr int A_BYTES = BM * L::kRowBytes, B_BYTES = BN * L::kRowBytes;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int SINK_BYTES = AHEAD ? NW * 256 : 0;  // where touched lines go, behind the slots
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES + SINK_BYTES;
    // LDS: the A tiles of all slots first, then the B tiles.  A lane's fragment addresses are then
    // one base per operand and sub-step plus constants below 64 KiB (block, slot), which fit the
    // offset field of the LDS read: no address arithmetic inside the K loop.
    static constexpr int a_slot(int stage) { return stage * A_BYTES; }
    static constexpr int b_slot(int stage) { return STAGES * A_BYTES + stage * B_BYTES; }
    static constexpr int COPY_ROWS = 1024 / L::kRowBytes;  // rows moved by one wave-wide copy
    static constexpr int A_COPIES = BM / COPY_ROWS / NW, B_COPIES = BN / COPY_ROWS / NW;  // per wave per K step
    static constexpr int COPIES = A_COPIES + B_COPIES;
    static_assert(BM % (COPY_ROWS * NW) == 0 && BN % (COPY_ROWS * NW) == 0, "tile rows must split over the waves");
    static_assert((NW * COPY_ROWS) % 16 == 0, "the swizzle of a lane's row must not depend on the copy index");
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile is made of pairs of 16x16 blocks");
    static_assert(LDS_BYTES <= 163840, "LDS budget of one gfx950 compute unit");
    static_assert(NW * rows_patch_bytes(NT) <= LDS_BYTES, "epilogue patches reuse the operand slots");
    static_assert(STAGES >= 2 && (STAGES - 1) * COPIES <= 63, "vmcnt range");

    using tile_t = wave::Tile<T, MT, NT>;
    using frag_t = typename Frag<T>::type;

    // a_tile / b_tile: uniform byte pointers to element (first row of the tile,
    // first k of the slice); a_ld / b_ld: row pitch in bytes; a_rows / b_rows:
    // rows of the tile that exist (>= 1; missing rows re-read the last one and
    // their results are never stored).  ksteps >= 1 steps of BK k each.
    //
    // Schedule of one K step (KSUB sub-steps of 32 k, NM = MT*NT MFMAs each):
    //   sub-steps 0 .. KSUB-2 : MFMAs of sub-step s, the fragment reads of
    //                           sub-step s+1 dealt one by one between them;
    //   sub-step KSUB-1       : wait for my copies of the next step, barrier,
    //                           then the MFMAs with the copies of step
    //                           t+STAGES (into the slot just retired) and the
    //                           fragment reads of (t+1, 0) dealt between them.
    // Every piece is pinned with a scheduling fence so the matrix pipe always
    // has the next MFMA queued while the memory instructions issue.
    __device__ __forceinline__ static void run(persp::Workgroup wgp, tile_t& acc, const char* a_tile, uint32_t a_ld, int a_rows,
                               const char* b_tile, uint32_t b_ld, int b_rows, int ksteps,
                               char* lds, int wave, int lane, uint64_t* stamps = nullptr, int a_share = 0, int b_share = 0)
    {
        const persp::Wave wv = wgp.wave();  // every wave of the workgroup runs this code
        constexpr int PARTS = wave::mfma_parts(frag_t{});  // matrix instructions per block and sub-step
        constexpr int NM = MT * NT * PARTS;                // MFMAs per sub-step
        constexpr int NR = MT + NT;                        // fragments to read per sub-step
        // -- per-lane copy offsets: wave-copy i moves row block (i*NW + wave) of COPY_ROWS rows;
        //    a lane fills one chunk position of one row with the logical chunk the swizzle wants.
        // (row pitches in bytes stay below 2^24 and rows below 2^8 -- the host refuses larger
        // pitches for this kernel -- so the full-rate 24-bit multiply gives the exact product)
        const int sub_row = lane / L::kChunksPerRow;
        const int chunk = (lane % L::kChunksPerRow) ^ L::swizzle(wave * COPY_ROWS + sub_row);
        uint32_t g_off[COPIES];
        // An operand kept as k-rows: a k-row of the tile is 128 elements and a wave-wide copy
        // moves 1024 bytes of them.  16-bit types: the 16-byte chunk c of k-row k sits at position
        // c ^ 2*(k%4), so that the four k-rows a transposing read touches fall on four different
        // 32-byte bank groups.  fp32: at position c ^ 4*((k/4)%2), so that the four k-rows of a
        // 4-byte gather (k = 4g + e for lane group g) alternate between the two halves of the
        // banks.  `cols` counts the elements of a k-row that exist (whole chunks); chunks beyond
        // them re-read the last one that exists and only feed results that are never stored.
        constexpr int KN_WIDTH = B_KN ? BN : BM;  // elements of a k-row (with both operands as k-rows BM == BN)
        constexpr int KN_ROW_BYTES = KN_WIDTH * ES, KN_CHUNKS = KN_ROW_BYTES / lane::kChunkBytes, KN_ROWS = 1024 / KN_ROW_BYTES;
        constexpr int PER_CHUNK = lane::kChunkBytes / ES;
        auto k_row_offset = [&](int i, uint32_t ld, int cols) __attribute__((always_inline)) {
            const int k_row = (i * NW + wave) * KN_ROWS + lane / KN_CHUNKS;
            const int swz = ES == 2 ? (k_row & 3) << 1 : ((k_row >> 2) & 1) << 2;
            int c = (lane % KN_CHUNKS) ^ swz;
            const int last = (cols - 1) / PER_CHUNK;
            c = c < last ? c : last;
            return __umul24(static_cast<uint32_t>(k_row), ld) + c * lane::kChunkBytes;
        };
#pragma unroll
        for (int i = 0; i < A_COPIES; ++i) {
            if constexpr (!A_MK) {
                int row = (i * NW + wave) * COPY_ROWS + sub_row;
                row = row < a_rows ? row : a_rows - 1;
                g_off[i] = __umul24(static_cast<uint32_t>(row), a_ld) + chunk * lane::kChunkBytes;
            } else {
                g_off[i] = k_row_offset(i, a_ld, a_rows);
            }
        }
#pragma unroll
        for (int i = 0; i < B_COPIES; ++i) {
            if constexpr (!B_KN) {
                int row = lane::paired_tile_row((i * NW + wave) * COPY_ROWS + sub_row);
                row = row < b_rows ? row : b_rows - 1;
                g_off[A_COPIES + i] = __umul24(static_cast<uint32_t>(row), b_ld) + chunk * lane::kChunkBytes;
            } else {
                g_off[A_COPIES + i] = k_row_offset(i, b_ld, b_rows);
            }
        }
        const uint32_t lds0 = lds_address(lds) + wave * 1024;

        // copy number c (0 .. COPIES-1) of K step `step` into slot `stage`
        auto copy = [&](int c, int step, int stage) __attribute__((always_inline)) {
            const int64_t k_bytes = static_cast<int64_t>(step) * L::kRowBytes;
            const int64_t a_bytes = A_MK ? static_cast<int64_t>(step) * K_PER_STEP * a_ld : k_bytes;
            const int64_t b_bytes = B_KN ? static_cast<int64_t>(step) * K_PER_STEP * b_ld : k_bytes;
            // (the slot's offset goes into the instruction's constant when the slot is known at compile time,
            // as in the steady loop, and into the base otherwise)
            const char* src = c < A_COPIES ? a_tile + a_bytes : b_tile + b_bytes;
            const int slot = c < A_COPIES ? a_slot(stage) : b_slot(stage);
            const int in_slot = (c < A_COPIES ? c : c - A_COPIES) * NW * 1024;
            if (__builtin_constant_p(stage)) copy_async_16(wv, src, g_off[c], lds0, slot + in_slot);
            else copy_async_16(wv, src, g_off[c], lds0 + slot, in_slot);
        };
        // AHEAD: the lines of a K step are asked for one step before its copies, so that a copy from memory has
        // two steps to arrive.  The two slots alone leave one: 4 MiB of different lines on their way in the
        // whole chip where 256 workgroups share their panels by fours, half of what memory's latency takes to
        // keep up 5 TB/s.  The workgroups of a die that share a panel share the asking: each asks for a
        // quarter of its rows of A (waves 0 and 1, every row by two lanes) and of B.  Measured with operands from
        // memory: 1024 x 1024 x 32768 in slices 82.3 -> 74.1 us, 2048 x 4096 x 16384 233.6 -> 215.5; half of the rows,
        // or two steps earlier, is no better.  Where the caches hold the operands the lines only cost power:
        // 4096 x 4096 x 4096 89.3 -> 90.6.
        uint32_t touch_off = 0;
        const char* touch_tile = wave < NW / 2 ? a_tile : b_tile;
        const uint32_t sink = lds_address(lds) + STAGES * STAGE_BYTES + wave * 256;
        int64_t touch_step = L::kRowBytes;
        if constexpr (AHEAD) {
            static_assert(BM == 256 && BN == 256 && NW == 4 && ES == 2, "a quarter of a panel's lines by two waves");
            const bool of_a = wave < 2, k_rows = of_a ? A_MK : B_KN;
            const int share = of_a ? a_share : b_share, exist = of_a ? a_rows : b_rows;
            const uint32_t ld = of_a ? a_ld : b_ld;
            if (k_rows) {  // sixteen k-rows of four lines
                const int k_row = share * 16 + (wave & 1) * 8 + (lane & 31) / 4, byte = (lane & 3) * 128;
                touch_off = __umul24(static_cast<uint32_t>(k_row), ld) + (byte < exist * ES ? byte : 0);
                touch_step = static_cast<int64_t>(K_PER_STEP) * ld;
            } else {
                const int row = share * 64 + (wave & 1) * 32 + (lane & 31);
                touch_off = __umul24(static_cast<uint32_t>(row < exist ? row : exist - 1), ld);
            }
        }
        auto touch = [&](int step) __attribute__((always_inline)) {
            touch_lines(wv, touch_tile + (step < ksteps ? step : ksteps - 1) * touch_step, touch_off, sink);
        };
        // -- prologue, first part: fill the slots.  The copies go out before the addressing of the
        //    fragment reads is worked out: that arithmetic then runs while the first bytes travel.
#pragma unroll
        for (int s = 0; s < STAGES; ++s)
            if (s < ksteps) {
#pragma unroll
                for (int c = 0; c < COPIES; ++c) copy(c, s, s);
            }
        if constexpr (AHEAD) touch(STAGES);
        __builtin_amdgcn_sched_barrier(0);

        // fp32 fragment from k-rows: element e of lane (x, g) is the value at k-row 16*ksub + 4g + e,
        // element first + x; nothing to transpose, four 4-byte reads.
        auto gather_k_rows = [&](const char* tile, int first, int ksub) __attribute__((always_inline)) {
            const int n = first + (lane & 15), g = lane >> 4;
            const char* src = tile + (16 * ksub + 4 * g) * KN_ROW_BYTES + (((n >> 2) ^ ((g & 1) << 2)) * lane::kChunkBytes) + (n & 3) * 4;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const float*>(src + e * KN_ROW_BYTES);
            return v;
        };

        const int wave_m = wave / WAVES_N, wave_n = wave % WAVES_N;
        const int a_row0 = wave_m * WTM, b_row0 = wave_n * WTN;
        // 16-bit operands kept as k-rows: fragments come from the transposing LDS read, see
        // wave::read_k_rows_half; four per-lane addresses and constants serve all reads.
        uint32_t ka_off[4], kb_off[4];
        if constexpr (ES == 2 && (A_MK || B_KN)) {
            static_assert(WTM % 64 == 0 && WTN % 64 == 0, "wave tiles start at whole groups of 64 elements");
#pragma unroll
            for (int jl = 0; jl < 4; ++jl) {
                const uint32_t part = wave::k_rows_lane_part<KN_ROW_BYTES>(wv, jl, lane);
                ka_off[jl] = a_row0 * ES + part;
                kb_off[jl] = b_slot(0) + b_row0 * ES + part;
                if constexpr (A_MK) asm volatile("" : "+v"(ka_off[jl]));
                if constexpr (B_KN) asm volatile("" : "+v"(kb_off[jl]));
            }
        }
        static_assert(WTM % 8 == 0 && WTN % 8 == 0 && lane::kBlock % 8 == 0, "row blocks start at multiples of 8 rows");
        // The lane's share of a fragment address, one per operand and sub-step: wave tile's first
        // row, the lane's row and chunk inside a block, and for B the start of the B tiles.  Every
        // read of the K loop is one of these plus a constant (block, slot) below 64 KiB.
        uint32_t fa_off[KSUB], fb_off[KSUB];
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) {
            const uint32_t part = lane::fragment_lane_part<BK>(wv.lane(), ks, lane);
            fa_off[ks] = a_row0 * L::kRowBytes + part;
            fb_off[ks] = b_slot(0) + b_row0 * L::kRowBytes + part;
            asm volatile("" : "+v"(fa_off[ks]), "+v"(fb_off[ks]));  // kept in registers, not re-derived per read
        }
        frag_t fa[2][MT], fb[2][NT];
        // read number r (0 .. NR-1) of sub-step ksub of slot `stage` into buffer `buf`;
        // order: a0, all b, remaining a -- what the first MFMAs of the next group need first
        // (the two halves of a fragment from k-rows are read in one place and brought together at
        // once: kept as two values over the slots between them they end up in registers apart)
        auto read_halves = [&](const char* st, int j, int ksub, const uint32_t (&part)[4]) __attribute__((always_inline)) {
            const wave::v4s lo = wave::read_k_rows_half<KN_ROW_BYTES>(wv, st, 0, j, ksub, 0, part);
            const wave::v4s hi = wave::read_k_rows_half<KN_ROW_BYTES>(wv, st, 0, j, ksub, 1, part);
            return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        auto read_a = [&](int x, int buf, int stage, int ksub) __attribute__((always_inline)) {
            const char* st = lds + a_slot(stage);
            if constexpr (A_MK && ES == 2) fa[buf][x] = __builtin_bit_cast(frag_t, read_halves(st, x, ksub, ka_off));
            else if constexpr (A_MK) fa[buf][x] = __builtin_bit_cast(frag_t, gather_k_rows(st, a_row0 + lane::kBlock * x, ksub));
            else fa[buf][x] = lane::load_fragment_at<T>(wv.lane(), st + lane::kBlock * x * L::kRowBytes, fa_off[ksub]);
        };
        auto read_b = [&](int x, int buf, int stage, int ksub) __attribute__((always_inline)) {
            const char* st = lds + b_slot(stage);
            if constexpr (B_KN && ES == 2) fb[buf][x] = __builtin_bit_cast(frag_t, read_halves(st - b_slot(0), x, ksub, kb_off));
            else if constexpr (B_KN) fb[buf][x] = __builtin_bit_cast(frag_t, gather_k_rows(st, b_row0 + lane::kBlock * x, ksub));
            else fb[buf][x] = lane::load_fragment_at<T>(wv.lane(), st - b_slot(0) + lane::kBlock * x * L::kRowBytes, fb_off[ksub]);
        };
        auto read = [&](int r, int buf, int stage, int ksub) __attribute__((always_inline)) {
            if (r == 0) read_a(0, buf, stage, ksub);
            else if (r <= NT) read_b(r - 1, buf, stage, ksub);
            else read_a(r - NT, buf, stage, ksub);
        };
        auto mfma = [&](int m, int buf) __attribute__((always_inline)) {
            const int e = m / (MT * NT), blk = m % (MT * NT), i = blk / NT, j = blk % NT;
            acc.acc[i][j] = wave::mfma_part(wv, fb[buf][j], fa[buf][i], e, acc.acc[i][j]);
        };

        // -- prologue, second part: wait for step 0, fetch its first fragments
        if (ksteps >= STAGES) wait_counts<(STAGES - 1) * COPIES + (AHEAD ? 1 : 0), 0>();
        else wait_counts<AHEAD ? 1 : 0, 0>();
        barrier(wgp);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < NR; ++r) read(r, 0, 0, 0);
        PRISM_PARANOID_SYNC(wgp);
        stamp(stamps, STAMP_FIRST_FRAGMENTS);

        // MFMA slots of the memory instructions of a group: reads on the even slots, copies on
        // the odd ones, so no MFMA has more than one of them in its 16-cycle shadow.
        // Read r sits on slot READ_SPACING*r, head copy c on slot 2c+1, tail copy c on slot
        // TAIL_SPACING*c+1.  The first TAILN copies of a step are issued right after the slot
        // is released, the last HEADN at the start of the following step.  (The slot of an
        // instruction is computed from the slot index, not searched for: the loops below are
        // unrolled in full, and their size before unrolling is limited.)
        // (All copies go out right after the release when a slot every fourth MFMA is enough for
        // them: with the sustained clock that is as fast on 4096^3 and 2 % faster on 8192^3.)
        constexpr int HEADN = 4 * (COPIES - 1) + 1 < NM ? 0 : COPIES / 4, TAILN = COPIES - HEADN;
        constexpr int TAIL_SPACING = 4 * (TAILN - 1) + 1 < NM ? 4 : 2;
        constexpr int READ_SPACING = 2 * NR <= NM ? 2 : 1;  // reads share slots with copies only when they must
        static_assert(NR <= NM && 2 * HEADN <= NM && TAIL_SPACING * (TAILN - 1) + 1 < NM,
                      "every memory instruction of a group needs an MFMA slot");

        // One K step t on slot `stage`.
        //   HEAD: the last HEADN copies of step t+1 are issued in sub-step 0
        //   TAIL: the first TAILN copies of step t+2 are issued after the hand-over
        //   LAST: no step follows (no hand-over)
        // Issuing most copies as early as the slot allows gives them a whole K step to land
        // (rows 16 KiB apart miss the L2 and the address translation caches far more often
        // than the MFMAs of half a step can hide); spreading them keeps every MFMA slot down
        // to one memory instruction, which is what a wave can issue in the shadow of one MFMA.
        auto k_step = [&](auto head_c, auto tail_c, auto last_c, int t, int stage, int next) __attribute__((always_inline)) {
            constexpr bool HEAD = decltype(head_c)::value;
            constexpr bool TAIL = decltype(tail_c)::value;
            constexpr bool LAST = decltype(last_c)::value;
#pragma unroll
            for (int ks = 0; ks < KSUB; ++ks) {
                const int cur = ks & 1, nxt = cur ^ 1;
                if (ks + 1 < KSUB) {
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        if (m % READ_SPACING == 0 && m / READ_SPACING < NR) read(m / READ_SPACING, nxt, stage, ks + 1);
                        if (HEAD && ks == 0 && m % 2 == 1 && m / 2 < HEADN) copy(TAILN + m / 2, t + 1, next);
                        __builtin_amdgcn_sched_barrier(0);  // memory instructions stay in front of their MFMA
                        mfma(m, cur);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else if (!LAST) {
                    // Hand-over: my copies for step t+1 have landed and my reads of this
                    // slot are done; after the barrier that holds for every wave.
                    // (lines asked for after those copies may still be on their way, see AHEAD)
                    wait_counts<AHEAD ? 1 : 0, 0>();
                    barrier(wgp);
                    asm volatile("" ::: "memory");  // keep what follows on this side of the barrier
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        if (m % READ_SPACING == 0 && m / READ_SPACING < NR) read(m / READ_SPACING, nxt, next, 0);
                        if (TAIL && m % TAIL_SPACING == 1 && m / TAIL_SPACING < TAILN) copy(m / TAIL_SPACING, t + 2, stage);
                        if (AHEAD && m == NM - 1) touch(t + 3);
                        __builtin_amdgcn_sched_barrier(0);  // memory instructions stay in front of their MFMA
                        mfma(m, cur);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int m = 0; m < NM; ++m) mfma(m, cur);
                }
                PRISM_PARANOID_SYNC(wgp);
            }
        };
        static_assert(KSUB % 2 == 0, "fragment buffers must return to slot 0 at the end of a K step");
        static_assert(STAGES == 2 && COPIES % 2 == 0, "the copy schedule below is written for two slots");

        using yes = std::integral_constant<bool, true>;
        using no = std::integral_constant<bool, false>;
        // step t's copies: the first TAILN issued after the hand-over of step t-2, the rest in
        // sub-step 0 of step t-1; steps 0 and 1 came whole from the prologue.
        int t = 0;
        if constexpr (MT * NT == 64 && (A_MK || B_KN)) {
            // The large tile with k-rows compiles without spills and without moving accumulators
            // about only as one small loop: a single step per trip, the slot toggled in the address
            // registers, no branch around a copy (past the end the copies fetch the last step
            // again into slots that nobody reads).  Measured against 128x128 tiles, which the LDS
            // reads of their smaller wave tiles bound: 8192 x 4096 x 4096 row-major B 232 -> 191 us,
            // 4096 x 4096 x 8192 column-major A, row-major B, fp32 C with beta 278 -> 209 us.
            static_assert(KSUB == 2 && HEADN == 0 && A_BYTES == 32768 && B_BYTES == 32768 && STAGES == 2, "the slot is bit 15 of an LDS address");
            auto pin_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc.acc[i][j]));
            };
            auto toggle = [&](uint32_t& address) __attribute__((always_inline)) {
                address ^= 32768u;
                asm volatile("" : "+v"(address));
            };
            pin_acc();
            for (; t < ksteps; ++t) {
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    if (m % READ_SPACING == 0 && m / READ_SPACING < NR) read(m / READ_SPACING, 1, 0, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma(m, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                PRISM_PARANOID_SYNC(wgp);
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    if constexpr (A_MK) toggle(ka_off[x]);
                    else if (x < KSUB) toggle(fa_off[x]);
                    if constexpr (B_KN) toggle(kb_off[x]);
                    else if (x < KSUB) toggle(fb_off[x]);
                }
                const int after_next = (t + 2 < ksteps ? t + 2 : ksteps - 1), stage = t & 1;
                wait_counts<AHEAD ? 1 : 0, 0>();
                barrier(wgp);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    if (m % READ_SPACING == 0 && m / READ_SPACING < NR) read(m / READ_SPACING, 0, 0, 0);
                    if (m % TAIL_SPACING == 1 && m / TAIL_SPACING < COPIES) copy(m / TAIL_SPACING, after_next, stage);
                    if (AHEAD && m == NM - 1) touch(t + 3);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma(m, 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                PRISM_PARANOID_SYNC(wgp);
            }
            pin_acc();
            wait_counts<0, 0>();  // the copies issued past the end
            __builtin_amdgcn_sched_barrier(0);
            return;
        }
        if (ksteps == 1) {
            k_step(no{}, no{}, yes{}, 0, 0, 0);
            if constexpr (AHEAD) wait_counts<0, 0>();
            __builtin_amdgcn_sched_barrier(0);
            return;
        }
        if (ksteps > 2) k_step(no{}, yes{}, no{}, 0, 0, 1);
        else k_step(no{}, no{}, no{}, 0, 0, 1);
        // steady state, two steps per trip so that the slot of a step is a compile-time constant
        // (LDS addresses fold into instruction offsets instead of being recomputed every step)
        for (t = 1; t + 3 < ksteps; t += 2) {
            k_step(yes{}, yes{}, no{}, t, 1, 0);
            k_step(yes{}, yes{}, no{}, t + 1, 0, 1);
        }
        if (t + 2 < ksteps) {  // t is odd here
            k_step(yes{}, yes{}, no{}, t, 1, 0);
            ++t;
        }
        if (t + 1 < ksteps) {  // t == ksteps - 2 >= 1: step t+1 >= 2 still needs its second half
            k_step(yes{}, no{}, no{}, t, t & 1, (t & 1) ^ 1);
            ++t;
        }
        k_step(no{}, no{}, yes{}, t, t & 1, t & 1);
        if constexpr (AHEAD) wait_counts<0, 0>();  // the lines asked for past the end
        __builtin_amdgcn_sched_barrier(0);  // nothing of the epilogue moves up into the K loop
    }
};

// ------------------------------------------------------------------------------------
// Persistent form of the pipeline: one workgroup walks a sequence of 256x256 tiles and
// treats their K steps as one stream.  The copies issued in the last two steps of a tile
// already belong to the next tile, so its first operands sit in LDS when its first MFMA
// issues, and the fixed cost of starting a tile (first loads from memory) disappears for
// every tile but the first.  This is the tile loop of the paper's persistent hgemm kernel
// (code appendix, `while(true)` over tiles) with the loads of the next tile pipelined
// under the tail of the current one.
//
// LDS: two operand slots (128 KiB) and, behind them, one epilogue patch of 4352 bytes per wave,
// 145 of the 160 KiB of a compute unit together; the patches are separate so
// that the epilogue of a tile can run while the slots already hold the next tile.
// ------------------------------------------------------------------------------------
template <typename T, int HEADN = 0>  // copies of a step left for the start of the next one (0: measured best)
struct PersistentPipe {
    using L = lane::TileLayout<64>;
    static constexpr int BM = 256, BN = 256, BK = 64, WAVES_M = 2, WAVES_N = 2, NW = 4, THREADS = 256;
    static constexpr bool PAIRED_N = true;  // B rows in the paired order, as in Pipeline
    static constexpr int WTM = 128, WTN = 128, MT = WTM / lane::kBlock, NT = WTN / lane::kBlock;
    static constexpr int KSUB = BK / lane::kBlockK, NM = MT * NT, NR = MT + NT;
    static constexpr int A_BYTES = BM * L::kRowBytes, B_BYTES = BN * L::kRowBytes, STAGE_BYTES = A_BYTES + B_BYTES;
    static constexpr int a_slot(int stage) { return stage * A_BYTES; }              // A tiles of both slots first,
    static constexpr int b_slot(int stage) { return 2 * A_BYTES + stage * B_BYTES; }  // then the B tiles (see Pipeline)
    static constexpr int PATCH_BYTES = rows_patch_bytes(NT);
    static constexpr int PATCH_BASE = 2 * STAGE_BYTES;
    static constexpr int LDS_BYTES = PATCH_BASE + NW * PATCH_BYTES;
    static constexpr int COPY_ROWS = 8, A_COPIES = BM / COPY_ROWS / NW, COPIES = 2 * A_COPIES;
    static constexpr int TAILN = COPIES - HEADN;
    static_assert(HEADN >= 0 && HEADN <= COPIES && 4 * (TAILN - 1) + 1 < MT * NT && 2 * (MT + NT) <= MT * NT,
                  "every memory instruction of a group needs an MFMA slot of its own kind");
    static_assert(LDS_BYTES <= 163840 && KSUB == 2 && BM == BN, "written for the 256x256x64 tile");

    using tile_t = wave::Tile<T, MT, NT>;
    using frag_t = typename Frag<T>::type;

    // Operand rows of one tile: a / b point at (first row of the tile, first k of the slice).
    struct Source {
        const char* a;
        const char* b;
        uint32_t a_ld, b_ld;  // row pitch in bytes
        int a_rows, b_rows;   // rows that exist (>= 1)
    };

    // Walks the tiles of one workgroup.
    //   first / first_ksteps: operands and K steps (even, >= 2) of the first tile
    //   peek(Source&, int& ksteps) -> bool: describes the tile after the current one, false if none
    //   finish(tile_t&): epilogue of the current tile (its accumulators are complete)
    //   advance(): the tile described by the last peek becomes the current one
    template <typename Peek, typename Finish, typename Advance>
    __device__ __forceinline__ static void run(persp::Workgroup wgp, char* lds, int wave, int lane, Source first, int first_ksteps,
                                               Peek&& peek, Finish&& finish, Advance&& advance)
    {
        const persp::Wave wv = wgp.wave();  // every wave of the workgroup runs this code
        tile_t acc;
        frag_t fa[2][MT], fb[2][NT];
        uint32_t g_off[COPIES];
        const uint32_t lds0 = lds_address(lds) + wave * 1024;
        const int a_row0 = (wave / WAVES_N) * WTM, b_row0 = (wave % WAVES_N) * WTN;

        // per-lane copy offsets for a tile (rows beyond the matrix re-read the last row)
        auto set_offsets = [&](const Source& s) __attribute__((always_inline)) {
            const int sub_row = lane / L::kChunksPerRow;
            const int chunk = (lane % L::kChunksPerRow) ^ L::swizzle(wave * COPY_ROWS + sub_row);
#pragma unroll
            for (int i = 0; i < A_COPIES; ++i) {
                const int row = (i * NW + wave) * COPY_ROWS + sub_row, row_b = lane::paired_tile_row(row);
                const int ra = row < s.a_rows ? row : s.a_rows - 1;
                const int rb = row_b < s.b_rows ? row_b : s.b_rows - 1;
                g_off[i] = __umul24(static_cast<uint32_t>(ra), s.a_ld) + chunk * lane::kChunkBytes;
                g_off[A_COPIES + i] = __umul24(static_cast<uint32_t>(rb), s.b_ld) + chunk * lane::kChunkBytes;
                // (kept as they are in registers: left to itself the compiler splits every offset into a
                // uniform and a per-lane part and adds them again in front of each copy of the K loop)
                asm volatile("" : "+v"(g_off[i]), "+v"(g_off[A_COPIES + i]));
            }
        };
        // copy number c of the K step whose operands start at a_src / b_src, into slot `stage`
        auto copy = [&](int c, const char* a_src, const char* b_src, int stage) __attribute__((always_inline)) {
            if (c < A_COPIES) copy_async_16(wv, a_src, g_off[c], lds0, a_slot(stage) + c * NW * 1024);
            else copy_async_16(wv, b_src, g_off[c], lds0, b_slot(stage) + (c - A_COPIES) * NW * 1024);
        };
        uint32_t fa_off[KSUB], fb_off[KSUB];  // the lane's share of a fragment address per operand and sub-step (see Pipeline)
#pragma unroll
        for (int ks = 0; ks < KSUB; ++ks) {
            const uint32_t part = lane::fragment_lane_part<BK>(wv.lane(), ks, lane);
            fa_off[ks] = a_row0 * L::kRowBytes + part;
            fb_off[ks] = b_slot(0) + b_row0 * L::kRowBytes + part;
            asm volatile("" : "+v"(fa_off[ks]), "+v"(fb_off[ks]));
        }
        auto read = [&](int r, int buf, int stage, int ksub) __attribute__((always_inline)) {
            const char* sa = lds + a_slot(stage);
            const char* sb = lds + b_slot(stage) - b_slot(0);
            if (r == 0) fa[buf][0] = lane::load_fragment_at<T>(wv.lane(), sa, fa_off[ksub]);
            else if (r <= NT) fb[buf][r - 1] = lane::load_fragment_at<T>(wv.lane(), sb + lane::kBlock * (r - 1) * L::kRowBytes, fb_off[ksub]);
            else fa[buf][r - NT] = lane::load_fragment_at<T>(wv.lane(), sa + lane::kBlock * (r - NT) * L::kRowBytes, fa_off[ksub]);
        };
        auto mfma = [&](int m, int buf) __attribute__((always_inline)) {
            const int i = m / NT, j = m % NT;
            acc.acc[i][j] = wave::mfma_block(wv, fb[buf][j], fa[buf][i], acc.acc[i][j]);
        };
        constexpr int TAIL_SPACING = 4;  // read r on slot 2r, head copy c on 2c+1, tail copy c on 4c+1

        // One K step computing from slot `stage`.  After the hand-over (wait, barrier, first
        // fragments of the next step) this slot is free, and sub-step 1 issues the first TAILN
        // copies of the step after next (from a2 / b2) into it; the remaining HEADN copies of
        // that step follow in sub-step 0 of the next step (here: from a1 / b1 into the other
        // slot).  "Next" steps past the end of a tile are the first steps of the following
        // tile, so the loop never drains; switch_now loads that tile's copy offsets between
        // the two halves.
        auto k_step = [&](auto stage_c, const char* a1, const char* b1, bool switch_now, const Source& to,
                          const char* a2, const char* b2) __attribute__((always_inline)) {
            constexpr int stage = decltype(stage_c)::value, next = stage ^ 1;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                if (m % 2 == 0 && m / 2 < NR) read(m / 2, 1, stage, 1);
                if (m % 2 == 1 && m / 2 < HEADN) copy(TAILN + m / 2, a1, b1, next);
                __builtin_amdgcn_sched_barrier(0);
                mfma(m, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            PRISM_PARANOID_SYNC(wgp);
            if (switch_now) set_offsets(to);
            wait_counts<0, 0>();
            barrier(wgp);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                if (m % 2 == 0 && m / 2 < NR) read(m / 2, 0, next, 0);
                if (m % TAIL_SPACING == 1 && m / TAIL_SPACING < TAILN) copy(m / TAIL_SPACING, a2, b2, stage);
                __builtin_amdgcn_sched_barrier(0);
                mfma(m, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            PRISM_PARANOID_SYNC(wgp);
        };
        constexpr int STEP = L::kRowBytes;  // bytes one K step advances in a row
        // Keeps every accumulator block in the accumulation registers at the edges of the K
        // loop, so that the register allocator does not rotate blocks through VGPRs inside it.
        auto pin_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc.acc[i][j]));
        };

        // -- before the first tile: step 0 whole, the first TAILN copies of step 1, the first fragments
        Source sc = first;
        int ksteps = first_ksteps;
        set_offsets(sc);
#pragma unroll
        for (int c = 0; c < COPIES; ++c) copy(c, sc.a, sc.b, 0);
#pragma unroll
        for (int c = 0; c < TAILN; ++c) copy(c, sc.a + STEP, sc.b + STEP, 1);
        wait_counts<TAILN, 0>();
        barrier(wgp);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < NR; ++r) read(r, 0, 0, 0);

        using slot0 = std::integral_constant<int, 0>;
        using slot1 = std::integral_constant<int, 1>;
        for (;;) {
            // Without a following tile the copies past the end re-read this tile's last two
            // steps (just fetched, so they come from the cache) into slots nobody reads again:
            // no branch around any copy and no traffic to memory.
            Source sn = sc;
            int next_ksteps = ksteps;
            const bool has_next = peek(sn, next_ksteps);
            if (!has_next) {
                sn.a = sc.a + static_cast<int64_t>(ksteps - 2) * L::kRowBytes;
                sn.b = sc.b + static_cast<int64_t>(ksteps - 2) * L::kRowBytes;
            }
            acc.clear();
            pin_acc();
            // Every tile has an even number of K steps, so a trip of two steps always starts on
            // slot 0 and slots are compile-time constants.  Past the end of the tile the copies
            // continue with the first two steps of the next one.
            for (int t = 0; t < ksteps; t += 2) {
                const bool last = t + 2 == ksteps;
                const char* a1 = sc.a + static_cast<int64_t>(t + 1) * STEP;
                const char* b1 = sc.b + static_cast<int64_t>(t + 1) * STEP;
                const char* a2 = last ? sn.a : sc.a + static_cast<int64_t>(t + 2) * STEP;
                const char* b2 = last ? sn.b : sc.b + static_cast<int64_t>(t + 2) * STEP;
                k_step(slot0{}, a1, b1, last, sn, a2, b2);
                k_step(slot1{}, a2, b2, false, sn, a2 + STEP, b2 + STEP);
            }
            pin_acc();
            finish(acc);
            if (!has_next) break;
            advance();
            sc = sn;
            ksteps = next_ksteps;
        }
        wait_counts<0, 0>();  // the copies issued past the end of the last tile
    }
};

// ------------------------------------------------------------------------------------
// Staged main loop: any sizes, pitches and alignments, 16-bit or fp32 operands.  The operands
// of a K step pass through registers on their way to LDS, because a direct-to-LDS copy needs
// whole aligned 16-byte chunks and a register load does not: the vector memory unit takes a
// 16-byte load from any element boundary.  A K step is 128 bytes of every operand row (64
// elements of a 16-bit type, 32 of fp32).
//
// An operand keeps the shape it has in memory: K-contiguous rows become the 128-byte rows of
// TileLayout, an operand contiguous along its other index becomes k-rows whose fragments come
// from the transposing reads (wave::read_k_rows_half; fp32: four 4-byte reads).  Either way a
// thread moves whole 16-byte chunks.
//
// What bounds it: the time from a load to its use, at one or two workgroups per compute unit, and then the
// LDS, which takes every step's 32 KiB in and gives 64 out.  So two K steps are in flight in
// registers beside the two in LDS (a load issued in step t is written to LDS in step t + 2 and used
// in step t + 3), and a step has one barrier and nothing that waits for it: reads, writes and loads stand
// between the matrix instructions as in Pipeline, with the next sub-step's fragments already in registers.
// Measured: 1999 x 2001 x 1003 bf16, odd pitches, 21.2 -> 17.0 us (reads, matrix instructions and
// writes one after the other before), 1999 x 2001 x 1004 18.2 -> 15.8, 3001 x 2003 x 1005 fp32 134 -> 122.
// Rows at odd elements loaded in whole words and moved into place, as in dealt.hip, cost more here than their
// slower loads do (18.6 us).
//
// Only the last K step can hold k beyond the matrix or read past an operand's last element.  It
// is computed first and takes the careful fetch: chunks are loaded from where they lie wholly inside their row and
// moved into place in registers, zeros behind (from a k-row shorter than a chunk the chunk is the 16
// bytes that end with it: the rows before it lie there).  All other steps are loads at a uniform base plus
// fixed per-lane offsets: rows beyond the matrix re-read its last row, and a chunk that
// straddles the end of a k-row brings elements of the next one, which only feed results that
// are never stored.
// This is the paper's sgemm structure (section 6.1: block tile staged in shared memory, then
// warp- and thread-level tiles), with the thread-level tile replaced by MFMA blocks.
// ------------------------------------------------------------------------------------
using global_bytes = const __attribute__((address_space(1))) char*;

// The 16 bytes of v moved down by `bytes` (0 .. 16 and more), zeros behind them.
__device__ __forceinline__ u32x4 chunk_moved_down(u32x4 v, uint32_t bytes)
{
    const uint32_t b = bytes & 3;
    uint32_t w0 = __builtin_amdgcn_alignbyte(v[1], v[0], b), w1 = __builtin_amdgcn_alignbyte(v[2], v[1], b);
    uint32_t w2 = __builtin_amdgcn_alignbyte(v[3], v[2], b), w3 = __builtin_amdgcn_alignbyte(0u, v[3], b);
    if (bytes & 4) { w0 = w1; w1 = w2; w2 = w3; w3 = 0u; }
    if (bytes & 8) { w0 = w2; w1 = w3; w2 = 0u; w3 = 0u; }
    return bytes < 16 ? u32x4{w0, w1, w2, w3} : u32x4{0u, 0u, 0u, 0u};
}

// One operand of the staged loop: EXT rows (m or n) of a tile, K-contiguous or (K_ROWS) as
// k-rows.  DEAL_PAIRED: the rows are dealt to LDS in the paired order (lane::paired_tile_row).
template <typename T, int EXT, bool K_ROWS, bool DEAL_PAIRED, int THREADS>
struct StagedOperand {
    using L = lane::TileLayout<64>;  // rows of 128 bytes
    static constexpr int ES = Frag<T>::kElemBytes, EPC = lane::kChunkBytes / ES;
    static constexpr int BK = L::kRowBytes / ES;
    static constexpr int CHUNKS = EXT * L::kChunksPerRow / THREADS;   // per thread
    static constexpr int ROW_BYTES = K_ROWS ? EXT * ES : L::kRowBytes, PER_ROW = ROW_BYTES / lane::kChunkBytes;
    static constexpr int ROW_STEP = THREADS / PER_ROW;                // LDS rows between a thread's chunks
    static constexpr int BYTES = EXT * L::kRowBytes;
    static_assert(ROW_STEP % 8 == 0 && EXT % ROW_STEP == 0, "the swizzle of a thread's chunks must not depend on their number");
    static_assert(!K_ROWS || !DEAL_PAIRED, "k-rows lie in LDS as in memory");

    const char* tile;   // element (first row of the tile, k 0)
    int64_t pitch;      // bytes between rows, or between k-rows
    int rows;           // rows of the tile that exist, >= 1
    bool narrow;        // the contiguous dimension is shorter than a chunk
    int row0, chunk;    // this thread's first LDS row and its chunk of every row
    uint32_t lds_off;
    uint32_t off[CHUNKS];

    __device__ __forceinline__ int tile_row(int i) const
    {
        const int r = row0 + i * ROW_STEP;
        return DEAL_PAIRED ? lane::paired_tile_row(r) : r;
    }
    // s_row / s_k: element strides, one of them 1; extent: elements of the contiguous dimension
    __device__ __forceinline__ void init(const char* tile_, int64_t s_row, int64_t s_k, int rows_, int64_t extent, int tid)
    {
        tile = tile_;
        pitch = ES * (K_ROWS ? s_k : s_row);
        rows = rows_;
        narrow = extent < EPC;
        row0 = tid / PER_ROW;
        chunk = tid % PER_ROW;
        int swz;
        if constexpr (!K_ROWS) swz = L::swizzle(row0);
        else if constexpr (ES == 2) swz = (row0 & 3) << 1;
        else swz = ((row0 >> 2) & 1) << 2;
        lds_off = row0 * ROW_BYTES + (chunk ^ swz) * lane::kChunkBytes;
        const int last = (rows - 1) / EPC;
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) {
            if constexpr (K_ROWS)
                off[i] = static_cast<uint32_t>((row0 + i * ROW_STEP) * pitch) + (chunk < last ? chunk : last) * lane::kChunkBytes;
            else {
                const int r = tile_row(i);
                off[i] = static_cast<uint32_t>((r < rows ? r : rows - 1) * pitch) + chunk * lane::kChunkBytes;
            }
        }
    }
    // can a K step inside the matrix be fetched by fixed 32-bit offsets?
    __device__ __forceinline__ bool regular() const { return pitch < (int64_t{1} << 31) / (K_ROWS ? BK : EXT) - 1024; }
    // With `k_left` >= 1 rows of the matrix after them: do the fixed 16-byte loads of a step's k-rows stay
    // inside the operand?  A k-row of a chunk or more reaches at most into the next one; a shorter
    // one's only chunk may reach over several.
    __device__ __forceinline__ bool stays_inside(int k_left) const
    {
        return !K_ROWS || !narrow || k_left * pitch + rows * ES >= lane::kChunkBytes;
    }

    __device__ __forceinline__ global_bytes step_base(int k0) const
    {
        return (global_bytes)scalarize(tile + (K_ROWS ? k0 * pitch : static_cast<int64_t>(k0) * ES));
    }
    __device__ __forceinline__ void fetch_one(int i, u32x4 (&regs)[CHUNKS], global_bytes step)
    {
        // (seen as a fresh 32-bit value, so that the load takes it as its offset register
        // beside the uniform base instead of a 64-bit sum kept per chunk)
        asm volatile("" : "+v"(off[i]));
        regs[i] = *(const __attribute__((address_space(1))) u32x4_any*)(step + off[i]);
    }
    __device__ __forceinline__ void fetch(u32x4 (&regs)[CHUNKS], int k0)
    {
        const global_bytes step = step_base(k0);
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) fetch_one(i, regs, step);
    }
    template <bool MAYBE_NARROW>
    __device__ __forceinline__ void fetch_careful(u32x4 (&regs)[CHUNKS], int k0, int k_end) const
    {
        // a chunk's first element, the end of the row it lies in, and that row
        const int first = K_ROWS ? chunk * EPC : k0 + chunk * EPC, end = K_ROWS ? rows : k_end;
        auto row = [&](int i) __attribute__((always_inline)) {
            const int r = tile_row(i);
            return tile + (K_ROWS ? (k0 + r < k_end ? k0 + r : k_end - 1) : (r < rows ? r : rows - 1)) * pitch;
        };
        if (!MAYBE_NARROW || !narrow) {
            const int from = first + EPC <= end ? first : end - EPC;
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) regs[i] = *reinterpret_cast<const u32x4_any*>(row(i) + static_cast<int64_t>(from) * ES);
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) regs[i] = chunk_moved_down(regs[i], (first - from) * ES);
        } else {
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i) {
                const char* src = row(i);
                uint32_t h[EPC];
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    const int at = first + e < end ? first + e : end - 1;
                    if constexpr (ES == 2) h[e] = *reinterpret_cast<const uint16_t*>(src + static_cast<int64_t>(at) * ES);
                    else h[e] = *reinterpret_cast<const uint32_t*>(src + static_cast<int64_t>(at) * ES);
                    if (first + e >= end) h[e] = 0u;
                }
                if constexpr (ES == 2) regs[i] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
                else regs[i] = u32x4{h[0], h[1], h[2], h[3]};
                __builtin_amdgcn_sched_barrier(0);  // a chunk at a time: few registers
            }
        }
        if constexpr (K_ROWS) {
#pragma unroll
            for (int i = 0; i < CHUNKS; ++i)
                if (k0 + tile_row(i) >= k_end) regs[i] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    __device__ __forceinline__ void commit_one(int i, const u32x4 (&regs)[CHUNKS], char* slot) const
    {
        *reinterpret_cast<u32x4*>(slot + lds_off + i * ROW_STEP * ROW_BYTES) = regs[i];
    }
    __device__ __forceinline__ void commit(const u32x4 (&regs)[CHUNKS], char* slot) const
    {
#pragma unroll
        for (int i = 0; i < CHUNKS; ++i) commit_one(i, regs, slot);
    }
};

template <typename T, int BM_, int BN_, bool A_MK, bool B_KN>
struct Staged {
    using L = lane::TileLayout<64>;
    static constexpr int ES = Frag<T>::kElemBytes;
    static constexpr int BM = BM_, BN = BN_, BK = L::kRowBytes / ES, NW = 4, THREADS = 256;
    static constexpr int WTM = BM / 2, WTN = BN / 2, MT = WTM / lane::kBlock, NT = WTN / lane::kBlock;
    static constexpr int KSUB = L::kChunksPerRow / 4;  // a fragment read covers 4 chunks of a row
    static constexpr bool PAIRED_N = !B_KN;            // as in Pipeline
    using A = StagedOperand<T, BM, A_MK, false, THREADS>;
    using B = StagedOperand<T, BN, B_KN, PAIRED_N, THREADS>;
    static constexpr int a_slot(int s) { return s * A::BYTES; }
    static constexpr int b_slot(int s) { return 2 * A::BYTES + s * B::BYTES; }
    static constexpr int LDS_BYTES = 2 * (A::BYTES + B::BYTES);
    static_assert(NW * rows_patch_bytes(NT) <= LDS_BYTES, "epilogue patches reuse the operand slots");
    static_assert(WTM % 64 == 0 && WTN % 64 == 0, "wave tiles start at whole groups of 64 elements");

    using tile_t = wave::Tile<T, MT, NT>;
    using frag_t = typename Frag<T>::type;

    // The fragment of block j (16 rows) of a sub-step, from row `first` of the tile (the first row of a wave
    // tile, a multiple of 64); `part`: the lane parts of a 16-bit operand's k-rows.
    template <int EXT, bool K_ROWS>
    __device__ __forceinline__ static frag_t read(persp::Wave wv, const char* slot, int first, int j, int ks, int lane, const uint32_t (&part)[4])
    {
        constexpr int ROW_BYTES = EXT * ES;
        if constexpr (!K_ROWS) {
            return lane::load_fragment<T, 64>(wv.lane(), slot, first + lane::kBlock * j, ks, lane);
        } else if constexpr (ES == 2) {
            const wave::v4s lo = wave::read_k_rows_half<ROW_BYTES>(wv, slot, first, j, ks, 0, part);
            const wave::v4s hi = wave::read_k_rows_half<ROW_BYTES>(wv, slot, first, j, ks, 1, part);
            return __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            const int x = lane & 15, g = lane >> 4, n = first + lane::kBlock * j + x;
            const char* src = slot + (16 * ks + 4 * g) * ROW_BYTES + (((n >> 2) ^ ((g & 1) << 2)) * lane::kChunkBytes) + (n & 3) * 4;
            frag_t f;
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = *reinterpret_cast<const float*>(src + e * ROW_BYTES);
            return f;
        }
    }

    // a_tile / b_tile: element (first row of the tile, k 0); a_extent / b_extent: elements of the
    // operand's contiguous dimension; k_end: end of the slice, a whole number of steps from
    // k_begin unless it is the end of the matrix (K).
    __device__ __forceinline__ static void run(persp::Workgroup wgp, tile_t& acc, const char* a_tile, int64_t a_sm, int64_t a_sk, int a_rows,
                               int a_extent, const char* b_tile, int64_t b_sn, int64_t b_sk, int b_rows, int b_extent,
                               int k_begin, int k_end, int K, char* lds, int wave, int lane)
    {
        const persp::Wave wv = wgp.wave();  // every wave of the workgroup runs this code
        const int tid = wave * 64 + lane;
        const int a_row0 = (wave >> 1) * WTM, b_row0 = (wave & 1) * WTN;
        A a;
        B b;
        a.init(a_tile, a_sm, a_sk, a_rows, a_extent, tid);
        b.init(b_tile, b_sn, b_sk, b_rows, b_extent, tid);
        const int steps = (k_end - k_begin + BK - 1) / BK;
        // Steps fetched by fixed offsets: all but the last, or but the last two where those loads would
        // run past the end of an operand with very short k-rows.
        const int k_left = K - (k_begin + (steps - 1) * BK);
        const int fixed = a.stays_inside(k_left) && b.stays_inside(k_left) ? steps - 1 : steps - 2;
        const bool regular = a.regular() && b.regular() && fixed > 0;

        u32x4 ra[2][A::CHUNKS], rb[2][B::CHUNKS];  // two K steps on their way
        // Step t (past the end: the last whole one again, never used, so that the loop has no
        // branch around a load and waits for exactly the loads it needs)
        auto fetch = [&](int t, int set) __attribute__((always_inline)) {
            const int k0 = k_begin + (t < fixed - 1 ? t : fixed - 1) * BK;
            a.fetch(ra[set], k0);
            b.fetch(rb[set], k0);
        };
        auto commit = [&](int set, int slot) __attribute__((always_inline)) {
            a.commit(ra[set], lds + a_slot(slot));
            b.commit(rb[set], lds + b_slot(slot));
        };
        uint32_t part_a[4] = {}, part_b[4] = {};
        if constexpr (ES == 2) {
#pragma unroll
            for (int jl = 0; jl < 4; ++jl) {
                if constexpr (A_MK) part_a[jl] = wave::k_rows_lane_part<BM * ES>(wv, jl, lane);
                if constexpr (B_KN) part_b[jl] = wave::k_rows_lane_part<BN * ES>(wv, jl, lane);
            }
        }
        constexpr int PARTS = wave::mfma_parts(frag_t{}), NM = MT * NT * PARTS, NR = MT + NT;
        frag_t fa[2][MT], fb[2][NT];
        // fragment number r of sub-step ks: a0, all b, remaining a (what the first matrix instructions need first)
        auto read_one = [&](int r, int buf, int slot, int ks) __attribute__((always_inline)) {
            if (r == 0 || r > NT) fa[buf][r == 0 ? 0 : r - NT] = read<BM, A_MK>(wv, lds + a_slot(slot), a_row0, r == 0 ? 0 : r - NT, ks, lane, part_a);
            else fb[buf][r - 1] = read<BN, B_KN>(wv, lds + b_slot(slot), b_row0, r - 1, ks, lane, part_b);
        };
        auto mfma = [&](int m, int buf) __attribute__((always_inline)) {
            const int e = m / (MT * NT), blk = m % (MT * NT), i = blk / NT, j = blk % NT;
            acc.acc[i][j] = wave::mfma_part(wv, fb[buf][j], fa[buf][i], e, acc.acc[i][j]);
        };
        auto compute = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int ks = 0; ks < KSUB; ++ks) {
#pragma unroll
                for (int r = 0; r < NR; ++r) read_one(r, ks, slot, ks);
#pragma unroll
                for (int m = 0; m < NM; ++m) mfma(m, ks);
            }
        };
        // my LDS reads and writes are done; loads into registers stay in flight across the barrier
        auto hand_over = [&]() __attribute__((always_inline)) {
            wait_counts<63, 0>();
            asm volatile("" ::: "memory");
            barrier(wgp);
            asm volatile("" ::: "memory");
            PRISM_PARANOID_SYNC(wgp);
        };

        // One step through slot 1 by the careful fetch, nothing ahead of it.
        u32x4 ca[A::CHUNKS], cb[B::CHUNKS];
        if (!regular) {
            for (int k0 = k_begin; k0 < k_end; k0 += BK) {
                a.template fetch_careful<true>(ca, k0, k_end);
                b.template fetch_careful<true>(cb, k0, k_end);
                a.commit(ca, lds + a_slot(1));
                b.commit(cb, lds + b_slot(1));
                hand_over();
                compute(1);
                hand_over();
            }
            return;
        }
        if (fixed < steps - 1) {
            a.template fetch_careful<false>(ca, k_begin + fixed * BK, k_end);
            b.template fetch_careful<false>(cb, k_begin + fixed * BK, k_end);
            a.commit(ca, lds + a_slot(1));
            b.commit(cb, lds + b_slot(1));
            hand_over();
            compute(1);
            hand_over();
        }
        // The last step goes first, through slot 1, while the first two travel.
        fetch(0, 0);
        fetch(1, 1);
        a.template fetch_careful<false>(ca, k_begin + (steps - 1) * BK, k_end);
        b.template fetch_careful<false>(cb, k_begin + (steps - 1) * BK, k_end);
        a.commit(ca, lds + a_slot(1));
        b.commit(cb, lds + b_slot(1));
        commit(0, 0);
        fetch(2, 0);
        hand_over();
        compute(1);
        hand_over();
        // Step t computes from slot t % 2.  Its first sub-step's matrix instructions have between them the reads of the
        // second's fragments and the writes of step t + 1, from its registers into the other slot
        // (everybody left that slot before the last barrier); after the barrier those of the second have
        // the reads of step t + 1's first fragments and the loads of step t + 3 into the registers so
        // freed.  Every piece is pinned in front of its matrix instruction, as in Pipeline.
        constexpr int PIECES = A::CHUNKS + B::CHUNKS, GAP = NM / (PIECES > NR ? PIECES : NR);
        static_assert(GAP >= 2 && KSUB == 2, "every memory instruction of a sub-step needs a slot of its own kind");
        auto step = [&](int t, int slot) __attribute__((always_inline)) {
            const int from = t + 3 < fixed ? t + 3 : fixed - 1;  // (as in fetch)
            const global_bytes a_src = a.step_base(k_begin + from * BK), b_src = b.step_base(k_begin + from * BK);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int piece = m / GAP;
                if (m % GAP == 0 && piece < NR) read_one(piece, 1, slot, 1);
                if (m % GAP == 1 && piece < A::CHUNKS) a.commit_one(piece, ra[slot ^ 1], lds + a_slot(slot ^ 1));
                else if (m % GAP == 1 && piece < PIECES) b.commit_one(piece - A::CHUNKS, rb[slot ^ 1], lds + b_slot(slot ^ 1));
                __builtin_amdgcn_sched_barrier(0);
                mfma(m, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            hand_over();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int piece = m / GAP;
                if (m % GAP == 0 && piece < NR) read_one(piece, 0, slot ^ 1, 0);
                if (m % GAP == 1 && piece < A::CHUNKS) a.fetch_one(piece, ra[slot ^ 1], a_src);
                else if (m % GAP == 1 && piece < PIECES) b.fetch_one(piece - A::CHUNKS, rb[slot ^ 1], b_src);
                __builtin_amdgcn_sched_barrier(0);
                mfma(m, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            PRISM_PARANOID_SYNC(wgp);
        };
#pragma unroll
        for (int r = 0; r < NR; ++r) read_one(r, 0, 0, 0);
        int t = 0;
        for (; t + 1 < fixed; t += 2) {
            step(t, 0);
            step(t + 1, 1);
        }
        if (t < fixed) compute(0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

}  // namespace wg
}  // namespace prism
