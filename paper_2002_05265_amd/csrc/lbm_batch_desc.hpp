// What the batched kernels know of an instance, and the launches of the batch's walking and resident
// passes (lbm_batch_walk_*.hip, lbm_batch_resident_*.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_cell.hpp"

namespace lbm {

template <typename R>
struct BDesc {
    int nx, ny, model, N;
    int cells, tile0;       // node count, first tile of this instance (for the current NPT)
    long long off;          // element offset of the instance inside each copy
    long long plane;        // elements per population plane of the instance
    long long foff;         // offset of the instance's initial fields
    float inv_nx;
    Ref<R> ref;             // storage reference (rho_s, U) in the arithmetic type
    Ref<double> ref_d;      // the same values in FP64 (initialisation)
    Coef<R> c;
};

__device__ __forceinline__ int row_of(int c, int nx, float inv_nx) {
    int y = (int)((float)c * inv_nx);
    if (y * nx > c) --y;
    else if ((y + 1) * nx <= c) ++y;
    return y;
}

// One wave's work in a walking pass: rows y0 .. y1 - 1 of strip `strip` of instance j (j < 0: none).
struct WalkTask {
    int j, strip, y0, y1;
};

// What a pass works on: `first` is the step it starts at, counted from *step_ctr; with `advance` 0 (timing)
// the instances' records of the copy they end in stay as they are.
struct BatchPass {
    hipStream_t stream;
    char* base;
    long long copy_elems;
    const void* desc;
    int n;
    int* blowup;
    const int* active;
    int* lastcopy;
    const long long* step_ctr;
    int first, advance;
};

// `depth` (3, 5 or, in FP64 and FP32, 7) steps of every task, 4 tasks per block.
void launch_batch_walk_f64(const BatchPass& p, int depth, const WalkTask* tasks, int ntasks);
void launch_batch_walk_f32(const BatchPass& p, int depth, const WalkTask* tasks, int ntasks);
void launch_batch_walk_f16(const BatchPass& p, int depth, const WalkTask* tasks, int ntasks);

// Nodes of the largest instance that a resident pass takes: the eight moving populations fill a CU's LDS of
// 160 KB in FP64; in FP32 and FP16 four nodes per thread hold 4096.
constexpr int kResidentNodes64 = 2496, kResidentNodes32 = 4096;

// nsteps steps of every instance, one workgroup each; no instance has more than `most` nodes.
void launch_batch_resident_f64(const BatchPass& p, int nsteps, int most);
void launch_batch_resident_f32(const BatchPass& p, int nsteps, int most);
void launch_batch_resident_f16(const BatchPass& p, int nsteps, int most);

}  // namespace lbm
