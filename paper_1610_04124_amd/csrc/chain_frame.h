// chain_frame.h -- host-side launches of the fused chain kernels: a column is
// reduced, tabulated, solved and backtracked by one workgroup (chain.h).
#pragma once

#include <hip/hip_runtime.h>

#include "batch_kernel.h"

namespace stx::persist {

// Intermediates of a frame that its launch also leaves in memory (all or
// none): reduced pixels [ncols][H], ranges [ncols][2], prefixes
// [4][ncols][H+1] (ground, sky, 2q+1, 2).
struct ChainExports {
    int16_t* q = nullptr;
    int32_t* range = nullptr;
    float* prefix = nullptr;
};

// Floats of a column's object prefix table.
constexpr size_t chain_table_floats(int H, int D) { return (size_t)D * po_row_floats(H); }

// One frame, a workgroup per column; column c's table at po + c *
// chain_table_floats(H, D).
hipError_t launch_chain_frame(const JobDesc& job, float* po, const ChainExports& ex, int num_cu,
                              hipStream_t st);

// One frame with its tables in a workspace of ws_bytes that may hold fewer
// than its columns (bytes needed: chain_arena_bytes).
size_t chain_arena_bytes(int ncols, int H, int D, int tables);
// Whether that pays against a wave per column in the same workspace.
bool chain_arena_pays(int ncols, int H, int D, size_t ws_bytes, int num_cu);
hipError_t launch_chain_arena(const JobDesc& job, void* ws, size_t ws_bytes, int num_cu,
                              hipStream_t st);

// The tasks of a batch, pulled from *counter (zero before) by `grid`
// workgroups of `waves` waves; workgroup g's table at scratch + g * stride
// floats.  hmax: the tallest frame.
hipError_t launch_chain_batch(const JobDesc* jobs, const int2* tasks, int ntasks,
                              unsigned int* counter, float* scratch, long long stride, int hmax,
                              int grid, int waves, hipStream_t st);
// Waves of a workgroup for a launch of ntasks columns, and how many such
// workgroups stay resident on a compute unit.
int chain_batch_waves(int hmax, int ntasks, int num_cu);
int chain_batch_per_cu(int hmax, int waves);

// Lets the current device's launches of these kernels use up to lds_per_block
// bytes of LDS (once per device; repeating it is harmless).
hipError_t chain_frame_setup(int lds_per_block);

}  // namespace stx::persist
