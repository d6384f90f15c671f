// Walking passes of a batch (lbm_walk.hpp over many instances), for one precision; included by
// lbm_batch_walk_f64.hip, lbm_batch_walk_f32.hip and lbm_batch_walk_f16.hip, which are compiled side by side.
//
// A pass is an ordinary launch, ordered by the stream: unlike the persistent passes it needs neither barriers
// nor one owner XCD per instance, and every population is read and written once per 5 or 7 steps
// instead of 3.  An odd number of steps changes the copy as it changes the parity of the step, so any number
// of passes leaves a live state in the copy of its step's parity.
//
// What bounds it: as the walking launches of one grid, the vector ALU in FP32 and FP16 and its issue rate in
// FP64, times what lies outside the grid: strips are 112 columns wide whatever the instance's width, and each
// task first fills up its D steps in 2 (D - 1) rows.  The host cuts the instances into as many tasks as there
// are wave slots (deal_tasks).  Measured on MI355X, 56 grids of 64 to 512 nodes a side and all models (us per
// step, three steps per persistent pass before, 5 steps per walking pass now): FP64 51.9 -> 31.6, FP32 37.8 ->
// 23.7; 17 of them FP64 23.2 -> 11.4 (with tasks of equal rows, whatever the model: 32.1, 26.2 and
// 12.2).  Blocks of one wave instead of four measured the same.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm.h"
#include "lbm_batch_desc.hpp"
#include "lbm_cell.hpp"
#include "lbm_internal.hpp"
#include "lbm_walk.hpp"

namespace lbm {
namespace {

// Wave t of the launch advances task t by D steps.  The tasks are in order of the model, so that the waves of
// neighbouring CUs, which share an instruction cache, run the same one.
template <int PREC, int D>
__global__ __launch_bounds__(256) void k_batch_walk(char* __restrict__ base, long long copy_elems,
                                                    const BDesc<typename Store<PREC>::R>* __restrict__ desc,
                                                    const WalkTask* __restrict__ tasks, int ntasks,
                                                    int* __restrict__ blowup, const int* __restrict__ active,
                                                    int* __restrict__ lastcopy, const long long* __restrict__ step_ctr,
                                                    int first, int advance) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    unsigned b, none;
    tile_of_block(blockIdx.x, gridDim.x, gridDim.x, 1, b, none);
    const int t = __builtin_amdgcn_readfirstlane((int)(4u * b + (threadIdx.x >> 6)));
    if (t >= ntasks) return;
    const WalkTask task = tasks[t];
    if (task.j < 0) return;
    const long long n = *step_ctr + first;
    // blew up before this pass, or retired.  Another task's record of this pass is of a step >= n
    if ((long long)__hip_atomic_load(blowup + task.j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n || !active[task.j])
        return;
    const BDesc<R>& d = desc[task.j];
    const int sc = (int)(n & 1);
    if (advance && task.strip == 0 && task.y0 == 0 && (threadIdx.x & 63u) == 0) lastcopy[task.j] = sc ^ 1;
    const S* src = reinterpret_cast<const S*>(base) + sc * copy_elems + d.off;
    S* dst = reinterpret_cast<S*>(base) + (sc ^ 1) * copy_elems + d.off;
    constexpr int W = walk_width<PREC>();
    const int narrow = walk_narrow<PREC>(d.nx);
    const int x0 = max(0, task.strip * W - narrow), x1 = min((task.strip + 1) * W - narrow, d.nx);
    const Geom g{d.nx, d.ny, d.plane};
    const Ref<R> ref = d.ref;
    const Coef<R> c = d.c;
    const int N = d.N;
    auto walk = [&](auto model) __attribute__((always_inline)) {
        constexpr int M = decltype(model)::value;
        strip_walk<D, PREC>(src, dst, g, ref, x0, x1 - x0, task.y0, task.y1, (int)n, blowup + task.j,
                            [&](R(&h)[9], const Macro<R>& m) __attribute__((always_inline)) { collide<M>(h, m, ref, c, N); });
    };
    switch (d.model) {
        case kBGK: walk(std::integral_constant<int, kBGK>{}); break;
        case kRM: walk(std::integral_constant<int, kRM>{}); break;
        case kHM: walk(std::integral_constant<int, kHM>{}); break;
        case kCM: walk(std::integral_constant<int, kCM>{}); break;
        case kCHM: walk(std::integral_constant<int, kCHM>{}); break;
        case kK: walk(std::integral_constant<int, kK>{}); break;
        case kPR: walk(std::integral_constant<int, kPR>{}); break;
        default: walk(std::integral_constant<int, kRR>{}); break;
    }
}

template <int PREC, int D>
void launch_batch_walk_d(const BatchPass& p, const WalkTask* tasks, int ntasks) {
    hipLaunchKernelGGL((k_batch_walk<PREC, D>), dim3((unsigned)((ntasks + 3) / 4)), dim3(256), 0, p.stream, p.base,
                       p.copy_elems, static_cast<const BDesc<typename Store<PREC>::R>*>(p.desc), tasks, ntasks,
                       p.blowup, p.active, p.lastcopy, p.step_ctr, p.first, p.advance);
}

template <int PREC>
void launch_batch_walk_p(const BatchPass& p, int depth, const WalkTask* tasks, int ntasks) {
    switch (depth) {
        case 3: launch_batch_walk_d<PREC, 3>(p, tasks, ntasks); break;
        case 5: launch_batch_walk_d<PREC, 5>(p, tasks, ntasks); break;
        default:
            if constexpr (PREC != kF16) launch_batch_walk_d<PREC, 7>(p, tasks, ntasks);
            break;
    }
}

}  // namespace
}  // namespace lbm
