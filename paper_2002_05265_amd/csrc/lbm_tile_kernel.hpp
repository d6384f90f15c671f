// Tile launches: several steps per launch on grids that are too small for the walking launches, for one
// precision; included by lbm_tile_f64.hip, lbm_tile_f32.hip and lbm_tile_f16.hip, which are compiled side
// by side.
//
// A workgroup pulls a patch of PW x PW nodes from memory (wrapped, so that it may be wider than the grid)
// and advances it by T steps, the valid part shrinking by one node on each side per step: it stores a tile
// of PW - 2 (T - 1) nodes a side.  The first step's streaming is the pull itself; between two steps the
// eight moving populations go through LDS in the stored type, the resting one stays in its register.
//
// What bounds it: on a small grid a step launched alone costs 2.6-3 us, nearly all of it launch and memory
// latency, and moves next to no bytes; a step of the patch costs two barriers, eight LDS words each way and
// the collision, 0.45-0.75 us.  So the halo is recomputed rather than exchanged, as deep as the workgroups
// still run at the same time (one per CU).  Measured on MI355X (us per step, BGK / K, strip launches -> tile launches
// in runs of 240 steps, 48 at 1024^2):
//   64^2    FP64 3.6  / 3.8  -> 0.79 / 0.86   FP32 3.3 / 3.7 -> 0.82 / 0.95   FP16 3.5 / 3.8 -> 0.89 / 1.03
//   256^2   FP64 4.6  / 4.7  -> 1.33 / 1.47   FP32 4.1 / 4.2 -> 1.10 / 1.26   FP16 4.2 / 4.4 -> 1.12 / 1.31
//   512^2   FP64 4.3  / 4.5  -> 2.82 / 3.14   FP32 2.7 / 3.0 -> 2.10 / 2.36   FP16 4.5 / 4.7 -> 1.92 / 2.21
//   768^2   FP64 7.7  / 7.9  -> 4.76 / 5.38   FP32 5.3 / 5.6 -> 3.62 / 4.17   FP16 5.9 / 6.1 -> 3.25 / 3.90
//   1024^2  FP64 12.9 / 13.5 -> 10.0 / 10.4   FP32 7.7 / 8.1 -> 6.20 / 6.60   FP16 9.0 / 9.0 -> 5.4  / 6.1
// (FP64 1024^2 takes walking launches: 8.9 / 10.2).  Two LDS buffers, for one barrier
// per step, gained nothing at any size (64^2 FP64 0.92 against 0.82) and halve the workgroups per CU; a patch
// of 48 (768 threads, three nodes each) was never faster than 44.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "lbm.h"
#include "lbm_cell.hpp"
#include "lbm_internal.hpp"

namespace lbm {
namespace {

// With KEEP the state after step s + 1 of the launch is also written to keep.state[s] where that is not NULL
// (each workgroup its tile): a run whose every state is kept costs its writes and nothing else.
template <int MODEL, int PREC, int PW, int NT, bool KEEP>
__global__ __launch_bounds__(NT) void k_tile(const typename Store<PREC>::S* __restrict__ src,
                                             typename Store<PREC>::S* __restrict__ dst, Geom g,
                                             Coef<typename Store<PREC>::R> c, Ref<typename Store<PREC>::R> ref, int N,
                                             int step, int* __restrict__ blowup, int nsteps, unsigned gx,
                                             std::conditional_t<KEEP, TileKeep, int> keep) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    constexpr int kNodes = PW * PW, kEach = (kNodes + NT - 1) / NT;
    __shared__ S lds[8][kNodes];
    unsigned bx, by;
    tile_of_block(blockIdx.x, gx, gridDim.x, 1, bx, by);  // neighbouring tiles, sharing lines, on one XCD
    const int e = nsteps - 1, tw = PW - 2 * e;
    const int x0 = (int)bx * tw, y0 = (int)by * tw;
    R h[kEach][9];
    int pi[kEach], pj[kEach];
    // whether node k of this thread is valid after `s` steps less one
    auto inside = [&](int k, int s) { return pi[k] >= s && pi[k] < PW - s && pj[k] >= s && pj[k] < PW - s; };
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int id = (int)threadIdx.x + k * NT;
        pj[k] = id / PW;
        pi[k] = id - pj[k] * PW;
        if (id < kNodes) {
            int x = (x0 - e + pi[k]) % g.nx, y = (y0 - e + pj[k]) % g.ny;
            x = x < 0 ? x + g.nx : x;
            y = y < 0 ? y + g.ny : y;
            pull_load(src, g.plane, neighbours(x, y, g.nx, g.ny), h[k]);
        } else {
            pi[k] = -1;  // none: never valid
        }
    }
    for (int s = 0;; ++s) {
        bool bad = false;
#pragma unroll
        for (int k = 0; k < kEach; ++k)
            if (inside(k, s)) {
                double rho_d;
                const Macro<R> m = macro_of<S>(h[k], ref, rho_d);
                bad = bad || !(rho_d > 0.0);
                collide<MODEL>(h[k], m, ref, c, N);
            }
        flag_bad(bad, blowup, step + s);
        if (s == e) break;
        if constexpr (KEEP) {
            if (keep.state[s]) {
#pragma unroll
                for (int k = 0; k < kEach; ++k) {
                    const int x = x0 + pi[k] - e, y = y0 + pj[k] - e;
                    if (inside(k, e) && x < g.nx && y < g.ny)
                        store_cell<S, R, false>(static_cast<S*>(keep.state[s]), g.plane,
                                                (unsigned)y * (unsigned)g.nx + (unsigned)x, h[k]);
                }
            }
        }
        if (s > 0) __syncthreads();  // the last step's values have been read
#pragma unroll
        for (int k = 0; k < kEach; ++k)
            if (inside(k, s)) {
                const int id = (int)threadIdx.x + k * NT;
                h[k][0] = R(to_store<S>(h[k][0]));
#pragma unroll
                for (int q = 1; q < 9; ++q) lds[q - 1][id] = to_store<S>(h[k][q]);
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kEach; ++k)
            if (inside(k, s + 1)) {
                const int id = (int)threadIdx.x + k * NT;
#pragma unroll
                for (int q = 1; q < 9; ++q) h[k][q] = R(lds[q - 1][id - cx(q) - PW * cy(q)]);
            }
    }
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int x = x0 + pi[k] - e, y = y0 + pj[k] - e;
        if (inside(k, e) && x < g.nx && y < g.ny)
            store_cell<S, R, false>(dst, g.plane, (unsigned)y * (unsigned)g.nx + (unsigned)x, h[k]);
    }
}

template <int MODEL, int PREC, int PW, int NT>
void launch_tile_w(lbm_ctx* ctx, const double* w, int nsteps, const void* src, void* dst, int step,
                   const TileKeep* keep) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    const int tw = PW - 2 * (nsteps - 1);
    const unsigned gx = (unsigned)((ctx->nx + tw - 1) / tw), gy = (unsigned)((ctx->ny + tw - 1) / tw);
    if (keep)
        hipLaunchKernelGGL((k_tile<MODEL, PREC, PW, NT, true>), dim3(gx * gy), dim3(NT), 0, ctx->stream,
                           reinterpret_cast<const S*>(src), reinterpret_cast<S*>(dst), ctx->geom(), make_coef<R>(w),
                           ref_as<R>(ctx->ref), ctx->eq_order, step, ctx->d_flag, nsteps, gx, *keep);
    else
        hipLaunchKernelGGL((k_tile<MODEL, PREC, PW, NT, false>), dim3(gx * gy), dim3(NT), 0, ctx->stream,
                           reinterpret_cast<const S*>(src), reinterpret_cast<S*>(dst), ctx->geom(), make_coef<R>(w),
                           ref_as<R>(ctx->ref), ctx->eq_order, step, ctx->d_flag, nsteps, gx, 0);
}

template <int MODEL, int PREC>
void launch_tile_m(lbm_ctx* ctx, const double* w, int nsteps, const void* src, void* dst, int step,
                   const TileKeep* keep) {
    switch (ctx->tile_patch) {
        case 22: launch_tile_w<MODEL, PREC, 22, 512>(ctx, w, nsteps, src, dst, step, keep); break;
        case 32: launch_tile_w<MODEL, PREC, 32, 1024>(ctx, w, nsteps, src, dst, step, keep); break;
        default: launch_tile_w<MODEL, PREC, 44, 1024>(ctx, w, nsteps, src, dst, step, keep); break;
    }
}

template <int PREC>
void launch_tile_p(lbm_ctx* ctx, int model, const double* w, int nsteps, const void* src, void* dst, int step,
                   const TileKeep* keep) {
    switch (model) {
        case LBM_BGK: launch_tile_m<kBGK, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_RM: launch_tile_m<kRM, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_HM: launch_tile_m<kHM, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_CM: launch_tile_m<kCM, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_CHM: launch_tile_m<kCHM, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_K: launch_tile_m<kK, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_PR: launch_tile_m<kPR, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        case LBM_RR: launch_tile_m<kRR, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
        default: launch_tile_m<kStreamOnly, PREC>(ctx, w, nsteps, src, dst, step, keep); break;
    }
}

}  // namespace
}  // namespace lbm
