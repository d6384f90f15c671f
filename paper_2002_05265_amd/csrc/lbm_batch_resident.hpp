// Resident passes of a batch of small instances, for one precision; included by lbm_batch_resident_f64.hip,
// lbm_batch_resident_f32.hip and lbm_batch_resident_f16.hip, which are compiled side by side.
//
// One workgroup keeps a whole instance and advances it all the steps of a run: it pulls the instance from
// memory once, passes the eight moving populations from step to step through LDS in the stored type (the
// resting one stays in its register), and writes the last step back.  No workgroup waits for another.
//
// What bounds it: the persistent passes read and write 144 bytes per node and step (FP64) through L2 and
// meet at an XCD-wide barrier each step or three; here a step touches no memory and costs two barriers of
// the workgroup, eight LDS words each way and the collision per node, so that the vector ALU is the bound
// once two instances share a CU.  512 threads of two nodes hold 1024 nodes, so two FP64 instances (64 KB
// each) fit a CU and one computes while the other waits; larger instances take 1024 threads (FP64 ones of 2049 to
// 2496 nodes three nodes each, at the 128 registers that 1024 threads leave with 56 bytes per lane in scratch).
// Measured on MI355X, 640 instances of all models, 64 steps (us per step, three steps per persistent pass before,
// resident now): 32^2 FP64 15.5 -> 3.8, FP32 18.0 -> 2.7; 40^2 FP64 18.2 -> 7.4, FP32 21.4 -> 5.6.
//
// An instance that blows up stops at the state after that step, as in passes of one step.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm.h"
#include "lbm_batch_desc.hpp"
#include "lbm_cell.hpp"
#include "lbm_internal.hpp"

namespace lbm {
namespace {

// src and dst are the same memory in a run of an even number of steps, so neither is declared restrict.
template <int MODEL, int PREC, int NT, int NPT, int CAP>
__device__ __forceinline__ void resident_steps(typename Store<PREC>::S (&lds)[8][CAP], int& stop,
                                               const typename Store<PREC>::S* src, typename Store<PREC>::S* dst,
                                               const BDesc<typename Store<PREC>::R>& d, int n, int nsteps,
                                               int* __restrict__ blowup) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    const int nx = d.nx, ny = d.ny, cells = d.cells, N = d.N;
    const long long plane = d.plane;
    const Ref<R> ref = d.ref;
    const Coef<R> c = d.c;
    R h[NPT][9];
    int xm[NPT], xp[NPT], ym[NPT], yp[NPT];  // from a node to its neighbours
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int id = (int)threadIdx.x + k * NT;
        if (id < cells) {
            const int y = row_of(id, nx, d.inv_nx), x = id - y * nx;
            xm[k] = x == 0 ? nx - 1 : -1;
            xp[k] = x == nx - 1 ? 1 - nx : 1;
            ym[k] = y == 0 ? (ny - 1) * nx : -nx;
            yp[k] = y == ny - 1 ? -(ny - 1) * nx : nx;
            pull_load(src, plane, neighbours(x, y, nx, ny), h[k]);
        }
    }
    for (int s = 0;; ++s) {
        bool bad = false;
#pragma unroll
        for (int k = 0; k < NPT; ++k)
            if ((int)threadIdx.x + k * NT < cells) {
                double rho_d;
                const Macro<R> m = macro_of<S>(h[k], ref, rho_d);
                bad = bad || !(rho_d > 0.0);
                collide<MODEL>(h[k], m, ref, c, N);
            }
        flag_bad(bad, blowup, n + s);
        if (bad) stop = 1;
        if (s == nsteps - 1) break;
        __syncthreads();  // the last step's values have been read
        if (stop) break;
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int id = (int)threadIdx.x + k * NT;
            if (id < cells) {
                h[k][0] = R(to_store<S>(h[k][0]));
#pragma unroll
                for (int q = 1; q < 9; ++q) lds[q - 1][id] = to_store<S>(h[k][q]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int id = (int)threadIdx.x + k * NT;
            if (id < cells) {
#pragma unroll
                for (int q = 1; q < 9; ++q)
                    h[k][q] = R(lds[q - 1][id + (cx(q) > 0 ? xm[k] : (cx(q) < 0 ? xp[k] : 0)) +
                                           (cy(q) > 0 ? ym[k] : (cy(q) < 0 ? yp[k] : 0))]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int id = (int)threadIdx.x + k * NT;
        if (id < cells) store_cell<S, R, false>(dst, plane, (unsigned)id, h[k]);
    }
}

// nsteps steps of instance blockIdx.x, whose nodes number at most CAP <= NT NPT.  The state may end in the
// copy it starts from: the workgroup has read all of it before the first barrier, and a run of one step,
// which has none, changes the copy.
template <int PREC, int NT, int NPT, int CAP>
__global__ __launch_bounds__(NT) void k_batch_resident(char* __restrict__ base, long long copy_elems,
                                                       const BDesc<typename Store<PREC>::R>* __restrict__ desc,
                                                       int* __restrict__ blowup, const int* __restrict__ active,
                                                       int* __restrict__ lastcopy,
                                                       const long long* __restrict__ step_ctr, int nsteps, int advance) {
    using S = typename Store<PREC>::S;
    using R = typename Store<PREC>::R;
    __shared__ S lds[8][CAP];
    __shared__ int stop;
    const int j = (int)blockIdx.x;
    const long long n = *step_ctr;
    if ((long long)blowup[j] < n || !active[j]) return;  // blew up earlier, or retired
    if (threadIdx.x == 0) stop = 0;
    __syncthreads();
    const BDesc<R>& d = desc[j];
    const int sc = (int)(n & 1), dc = advance ? (int)((n + nsteps) & 1) : sc ^ 1;
    if (advance && threadIdx.x == 0) lastcopy[j] = dc;
    const S* src = reinterpret_cast<const S*>(base) + sc * copy_elems + d.off;
    S* dst = reinterpret_cast<S*>(base) + dc * copy_elems + d.off;
    switch (d.model) {
#define LBM_RESIDENT(M) resident_steps<M, PREC, NT, NPT, CAP>(lds, stop, src, dst, d, (int)n, nsteps, blowup + j)
        case kBGK: LBM_RESIDENT(kBGK); break;
        case kRM: LBM_RESIDENT(kRM); break;
        case kHM: LBM_RESIDENT(kHM); break;
        case kCM: LBM_RESIDENT(kCM); break;
        case kCHM: LBM_RESIDENT(kCHM); break;
        case kK: LBM_RESIDENT(kK); break;
        case kPR: LBM_RESIDENT(kPR); break;
        default: LBM_RESIDENT(kRR); break;
#undef LBM_RESIDENT
    }
}

template <int PREC, int NT, int NPT, int CAP>
void launch_batch_resident_c(const BatchPass& p, int nsteps) {
    hipLaunchKernelGGL((k_batch_resident<PREC, NT, NPT, CAP>), dim3((unsigned)p.n), dim3(NT), 0, p.stream, p.base,
                       p.copy_elems, static_cast<const BDesc<typename Store<PREC>::R>*>(p.desc), p.blowup, p.active,
                       p.lastcopy, p.step_ctr, nsteps, p.advance);
}

template <int PREC>
void launch_batch_resident_p(const BatchPass& p, int nsteps, int most) {
    if (most <= 1024)
        launch_batch_resident_c<PREC, 512, 2, 1024>(p, nsteps);
    else if (most <= 2048)
        launch_batch_resident_c<PREC, 1024, 2, 2048>(p, nsteps);
    else if constexpr (PREC == kF64)
        launch_batch_resident_c<PREC, 1024, 3, kResidentNodes64>(p, nsteps);
    else
        launch_batch_resident_c<PREC, 1024, 4, kResidentNodes32>(p, nsteps);
}

}  // namespace
}  // namespace lbm
