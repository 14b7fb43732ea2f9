// Host-visible launchers of the device kernels (defined in kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "grid.hpp"

namespace prism {

// Workgroup-tile configurations of the direct-to-LDS pipeline.
struct PipeConfig {
    int id;
    int tile_m, tile_n, tile_k, waves, stages;
    const char* name;
};
// 0, 1: both operands K-contiguous; 2-4: B along n, A along m, both; 5-8: fp32, same four; 9-11: 2-4 with large tiles
constexpr int kNumPipeConfigs = 12;
extern const PipeConfig kPipeConfigs[kNumPipeConfigs];

constexpr int kStagedTileM = 128, kStagedTileN = 128, kStagedWaves = 4;

// Each returns the launch error of the HIP runtime (hipSuccess when accepted).
// `workgroups` = p.tiles_m * p.tiles_n * p.batch * p.split_k.
hipError_t launch_pipelined(int config, int ab_dtype, const GemmParams& p, int workgroups, hipStream_t stream);
hipError_t launch_staged(int ab_dtype, const GemmParams& p, int workgroups, hipStream_t stream);
// 256x256x64 tile, `workgroups` persistent workgroups walking `total` (tile, unit) pairs;
// every unit must span at least two K steps of 64.
hipError_t launch_persistent(int ab_dtype, const GemmParams& p, int total, int workgroups, hipStream_t stream);
// Few rows: `workgroups` = tiles_n * batch workgroups of `waves` (4, 8 or 16) waves; tile_m (16, 32
// or 64) covers p.M, tile_n is 16 or 32.
// A B beyond the memory-side cache (256 MB) cannot be there for the next call either and is read as a
// stream: 16 x 16384 x 16384 99.6 -> 92.1 us.  Below that a stream loses what the cache would have
// kept (64 x 4096 x 4096 11.6 -> 14.1 us, 16 x 901 x 5632 7.3 -> 9.4), also when many problems share
// one B (batch_b == 0; 64 problems of 16 x 4096 x 4096: 158 us, 326 as a stream).
constexpr bool few_rows_stream_b(int64_t N, int64_t K, int esize, int64_t batch, int64_t batch_b)
{
    return static_cast<double>(N) * static_cast<double>(K) * esize * static_cast<double>(batch_b == 0 ? 1 : batch) > 268435456.0;
}
hipError_t launch_skinny(int ab_dtype, int tile_m, int tile_n, int waves, const GemmParams& p, int workgroups, hipStream_t stream);
// K steps dealt to the waves of a workgroup: `rows` of C (32, by 32 columns and 4 or 8 waves; 64 or 128, by 64 columns and 8 waves); odd_rows:
// 16-bit operands some of whose rows start in the middle of a 32-bit word, all in words of the operand.
hipError_t launch_dealt(int ab_dtype, int rows, int waves, bool odd_rows, const GemmParams& p, int workgroups, hipStream_t stream);
// Sums the split_k partial slabs in slice order and applies the epilogue; with
// p.split_k == 0 it writes C <- bias + beta*C (the K == 0 case).
hipError_t launch_reduce(const GemmParams& p, hipStream_t stream);

// The scan's own hook (PRISM_SCAN_SPIN_LIMIT), read again from the environment.
void scan_reread_environment();

}  // namespace prism
