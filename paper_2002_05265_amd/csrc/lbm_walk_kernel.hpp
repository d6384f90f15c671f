// The walking kernel (lbm_walk.hpp) over a grid and its launch, for one precision; included by
// lbm_walk_f64.hip, lbm_walk_f32.hip and lbm_walk_f16.hip, which are compiled side by side.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm.h"
#include "lbm_cell.hpp"
#include "lbm_internal.hpp"
#include "lbm_walk.hpp"

namespace lbm {
namespace {

// D steps of the whole grid: wave t of the launch walks down strip t mod sx of the segment of hs rows
// t / sx.  The blocks are dealt to the XCDs in contiguous bands (the hardware hands block b to XCD
// b mod 8), so that the strips at the two sides of an edge run on one XCD at the same time.
template <int MODEL, int PREC, int D>
__global__ __launch_bounds__(256) void k_walk(const typename Store<PREC>::S* __restrict__ src,
                                              typename Store<PREC>::S* __restrict__ dst, Geom g,
                                              Coef<typename Store<PREC>::R> c, Ref<typename Store<PREC>::R> ref,
                                              int N, int step, int* __restrict__ blowup, unsigned sx, unsigned tasks,
                                              int hs) {
    using R = typename Store<PREC>::R;
    constexpr int W = walk_width<PREC>();
    unsigned b, none;
    tile_of_block(blockIdx.x, gridDim.x, gridDim.x, 1, b, none);
    const unsigned t = (unsigned)__builtin_amdgcn_readfirstlane((int)(4u * b + (threadIdx.x >> 6)));
    if (t >= tasks) return;
    const unsigned by = t / sx, bx = t - by * sx;
    const int d = walk_narrow<PREC>(g.nx);
    const int x0 = max(0, (int)bx * W - d), x1 = min((int)(bx + 1) * W - d, g.nx), ys = (int)by * hs;
    strip_walk<D, PREC>(src, dst, g, ref, x0, x1 - x0, ys, min(ys + hs, g.ny), step, blowup,
                        [&](R(&h)[9], const Macro<R>& m) { collide<MODEL>(h, m, ref, c, N); });
}

template <int MODEL, int PREC, int D>
void launch_walk_d(lbm_ctx* ctx, const double* w, int hs, const void* src, void* dst, int step) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    const unsigned sx = (unsigned)walk_strips(ctx->nx, walk_width<PREC>(), walk_cols<PREC>());
    const unsigned tasks = sx * (unsigned)((ctx->ny + hs - 1) / hs);
    hipLaunchKernelGGL((k_walk<MODEL, PREC, D>), dim3((tasks + 3) / 4), dim3(256), 0, ctx->stream,
                       reinterpret_cast<const S*>(src), reinterpret_cast<S*>(dst), ctx->geom(), make_coef<R>(w),
                       ref_as<R>(ctx->ref), ctx->eq_order, step, ctx->d_flag, sx, tasks, hs);
}

template <int MODEL, int PREC>
void launch_walk_m(lbm_ctx* ctx, const double* w, int depth, int hs, const void* src, void* dst, int step) {
    switch (depth) {
        case 4: launch_walk_d<MODEL, PREC, 4>(ctx, w, hs, src, dst, step); break;
        case 6: launch_walk_d<MODEL, PREC, 6>(ctx, w, hs, src, dst, step); break;
        default:
            if constexpr (PREC == kF16)
                launch_walk_d<MODEL, PREC, 5>(ctx, w, hs, src, dst, step);
            else
                launch_walk_d<MODEL, PREC, 8>(ctx, w, hs, src, dst, step);
            break;
    }
}

template <int PREC>
void launch_walk_p(lbm_ctx* ctx, int model, const double* w, int depth, int hs, const void* src, void* dst, int step) {
    switch (model) {
        case LBM_BGK: launch_walk_m<kBGK, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_RM: launch_walk_m<kRM, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_HM: launch_walk_m<kHM, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_CM: launch_walk_m<kCM, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_CHM: launch_walk_m<kCHM, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_K: launch_walk_m<kK, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_PR: launch_walk_m<kPR, PREC>(ctx, w, depth, hs, src, dst, step); break;
        case LBM_RR: launch_walk_m<kRR, PREC>(ctx, w, depth, hs, src, dst, step); break;
        default: launch_walk_m<kStreamOnly, PREC>(ctx, w, depth, hs, src, dst, step); break;
    }
}

}  // namespace
}  // namespace lbm
