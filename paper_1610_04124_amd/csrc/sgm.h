// sgm.h -- semi-global matching stage (census costs, four path directions)
// ahead of the stixel path: internal launch interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace stx::sgm {

// Device workspace of a matching handle, sized for max_frames frames of
// max_width x max_height: census words of both views, and either planes of path
// costs in bytes, [direction][frame][y][x][d] of the call's size, or their sums
// S [frame][y][x][d] (uint16).
struct SgmWorkspace {
    uint64_t* cl = nullptr;
    uint64_t* cr = nullptr;
    uint16_t* S = nullptr;
    uint8_t* planes = nullptr;
    size_t plane_bytes = 0;         // of all planes
    int num_cu = 0;
};

struct PathArgs {
    const uint64_t* cl;
    const uint64_t* cr;
    uint16_t* S;
    float* disp;            // [frame][y][x], written by the last pass
    int W, H, D, P1, P2;
};

// Disparities per lane of a path wave for D disparities (D <= 64 DPL).
int dpl_of(int D);

// Whether path costs fit a byte under this penalty; whether a call's lines are
// few enough that all four directions go to planes (else three); the place of
// disparity d among a pixel's bytes; and the path passes with costs in bytes
// (sgm_packed.hip).
bool packed_costs(int P2);
bool packed_four(int D, int H, int frames, int num_cu);
int packed_place(int D, int W, int d);
hipError_t launch_packed_paths(const uint64_t* cl, const uint64_t* cr, uint8_t* planes,
                               size_t plane, bool four, int W, int H, int frames, int D, int P1,
                               int P2, float* disp, hipStream_t st);

// The whole stage over `frames` frames stored back to back ([frame][H][W]
// uint8 images, [frame][H][W] float disparity out); enqueued on st.
hipError_t launch_sgm(const uint8_t* left, const uint8_t* right, int W, int H, int frames,
                      const SgmWorkspace& ws, int D, int P1, int P2, float* disp, hipStream_t st);

}  // namespace stx::sgm
