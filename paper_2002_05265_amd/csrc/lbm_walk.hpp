// Several time steps per pass over memory in registers: one wave walks down a strip of columns row
// by row and runs step k of a row k - 1 rows behind step 1, so that every population is read from and
// written to memory once for all of them.
//
// What bounds it: with three steps per launch and rings in LDS (lbm_step3.hpp) every model ran at the
// rate of the pure pull, that is of HBM (5.4-5.6 TB/s), with the vector ALU idle 25-70% of the time; more
// rings do not fit the LDS of two or three workgroups.  Here nothing is kept in LDS and no wave waits
// for another, so the number of steps is limited by registers alone: nine values per column and step,
// 18 VGPRs in FP32 and 36 in FP64 for the two columns of a lane.  In FP32 and FP16 eight (six) steps leave
// two waves per SIMD, which issue vector instructions all the time: that is the bound (K: 139 per node and
// step, 72 us per step at 4096^2 where full issue would take 70).  In FP64 one wave per SIMD holds
// eight steps (some values in accumulation registers) and issues about 75% of the time; one column per
// lane and two waves took 8-9% longer (4096^2), as a quarter of its lanes is halo against an eighth.  Four columns
// per lane in FP32 ran 3-12% slower (one wave per SIMD).  Measured at 4096^2, us per step (BGK / K), against the strip
// launches: FP32 53 / 72 (82 / 85), FP64 75 / 93 (162 / 168), FP16 53 / 72 (75 / 79); the pure pull moves 4.7-4.9 TB/s
// in each.
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_cell.hpp"
#include "lbm_internal.hpp"
#include "lbm_step2.hpp"

namespace lbm {

// Columns per lane and halo columns on each side of a strip.  The halo takes one column per step; eight
// columns make a strip 112 columns wide, so that its row segments begin at multiples of 64 bytes in
// FP32 and FP64 wherever the rows do.
template <int PREC> constexpr int walk_cols() { return 2; }
constexpr int kWalkHalo = 8;
// Output columns of a strip: the wave's columns less the halo.
template <int PREC> constexpr int walk_width() { return 64 * walk_cols<PREC>() - 2 * kWalkHalo; }

// The strips of a row of nx columns, W wide but for the first, which is up to V - 1 columns narrower so
// that the last one, whose halo wraps around, begins and ends between two lanes' columns.
constexpr int walk_narrow_by(int nx, int V) { return (V - nx % V) % V; }
constexpr int walk_strips(int nx, int W, int V) { return (nx + walk_narrow_by(nx, V) + W - 1) / W; }
template <int PREC> __device__ __forceinline__ int walk_narrow(int nx) { return walk_narrow_by(nx, walk_cols<PREC>()); }

// Value of the previous / next lane (0 in the first / last lane of the wave).
__device__ __forceinline__ unsigned lane_prev(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ unsigned lane_next(unsigned v) {
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
template <bool PREV, typename R>
__device__ __forceinline__ R lane_shift(R v) {
    if constexpr (sizeof(R) == 4) {
        const unsigned u = __builtin_bit_cast(unsigned, v);
        return __builtin_bit_cast(R, PREV ? lane_prev(u) : lane_next(u));
    } else {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
        const unsigned lo = PREV ? lane_prev((unsigned)u) : lane_next((unsigned)u);
        const unsigned hi = PREV ? lane_prev((unsigned)(u >> 32)) : lane_next((unsigned)(u >> 32));
        return __builtin_bit_cast(R, ((unsigned long long)hi << 32) | lo);
    }
}
// v moved by one column: out[j] = value at column j - 1 (PREV) or j + 1 of the row that the lanes'
// V adjacent columns make up.
template <bool PREV, int V, typename R>
__device__ __forceinline__ void column_shift(const R (&v)[V], R (&out)[V]) {
    if constexpr (PREV) {
        out[0] = lane_shift<true>(v[V - 1]);
#pragma unroll
        for (int j = 1; j < V; ++j) out[j] = v[j - 1];
    } else {
        out[V - 1] = lane_shift<false>(v[0]);
#pragma unroll
        for (int j = 0; j < V - 1; ++j) out[j] = v[j + 1];
    }
}

// Has the loads of v waited for here: v is made an operand of an empty statement, as 32-bit words.
template <typename T>
__device__ __forceinline__ void loaded(T& v) {
    if constexpr (sizeof(T) == 4) {
        unsigned u = __builtin_bit_cast(unsigned, v);
        asm volatile("" : "+v"(u));
        v = __builtin_bit_cast(T, u);
    } else {
        typedef unsigned Words __attribute__((ext_vector_type(sizeof(T) / 4)));
        Words u = __builtin_bit_cast(Words, v);
        asm volatile("" : "+v"(u));
        v = __builtin_bit_cast(T, u);
    }
}

// The x part of the pull of population q: out[j] = v at column j - cx(q).
template <int V, typename R>
__device__ __forceinline__ void pull_x(int q, const R (&v)[V], R (&out)[V]) {
    if (cx(q) > 0)
        column_shift<true>(v, out);
    else if (cx(q) < 0)
        column_shift<false>(v, out);
    else
#pragma unroll
        for (int j = 0; j < V; ++j) out[j] = v[j];
}

// D steps of rows ys .. ye - 1 and columns x0 .. x0 + w - 1 of grid g by one wave: pulls
// from src, writes to dst, collides with coll(h, m).  Lane l holds columns x0 - kWalkHalo + V l .. + V - 1
// of each row it works on.  In an iteration step 1 collides row a, step 2 row a - 1, ... step
// D row a - D + 1, which is written; step k + 1 pulls its 4, 7, 8 from the row that step
// k has just collided, 0, 1, 3 from the one before and 2, 5, 6 from the one before that, so nine
// values per column are kept between two steps.  The x-neighbours are the lane's own columns and one
// column of the next lane (DPP).  Each step spoils one more column at both ends of the wave, which the
// halo columns absorb; rows ys - D + 1 .. and .. ye + D - 2 are collided by both strips
// that need them.  Every node is computed by the arithmetic of k_step on values of the storage type,
// so the result is bit-identical to D launches of it.
// Requires ny > D (one conditional wrap), x0 + w <= nx, and that no lane's columns straddle the periodic edge:
// nx a multiple of V, or nx >= 64 V and, for x0 + w = nx, w a multiple of V.
template <int D, int PREC, typename S, typename R, typename Coll>
__device__ __forceinline__ void strip_walk(const S* __restrict__ src, S* __restrict__ dst, const Geom& g,
                                           const Ref<R>& ref, int x0, int w, int ys, int ye, int step,
                                           int* __restrict__ blowup, Coll&& coll) {
    constexpr int V = walk_cols<PREC>(), H = kWalkHalo;
    static_assert(D >= 2 && D <= H, "the halo covers one column per step");
    constexpr unsigned E = sizeof(S);
    typedef S Vec __attribute__((ext_vector_type(V), aligned(sizeof(S))));
    const int lane = (int)(threadIdx.x & 63u);
    const int c0 = V * lane - H;  // first column of the lane, relative to x0
    // byte offset of the lane's columns in a row; lanes whose columns no step needs repeat the
    // nearest needed ones
    unsigned xo;
    {
        constexpr int lo = (H - D) / V * V - H;
        const int hi = (H + w + D - 1) / V * V - H;
        int x = x0 + min(max(c0, lo), hi);
        while (x < 0) x += g.nx;
        while (x >= g.nx) x -= g.nx;
        xo = (unsigned)x * E;
    }
    unsigned long long inside[V];  // lanes whose column j is an output column
#pragma unroll
    for (int j = 0; j < V; ++j) inside[j] = __ballot(c0 + j >= 0 && c0 + j < w);

    auto wrap_row = [&](int a) { return a < 0 ? a + g.ny : (a >= g.ny ? a - g.ny : a); };
    Vec raw[9];
    auto load_row = [&](int a) __attribute__((always_inline)) {  // the stored populations that step 1 pulls into row a, not yet shifted in x
        const int yw = wrap_row(a);
        const long long r0 = (long long)yw * g.nx;
        const long long rm = yw == 0 ? (long long)(g.ny - 1) * g.nx : r0 - g.nx;
        const long long rp = yw == g.ny - 1 ? 0 : r0 + g.nx;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const long long r = cy(q) == 0 ? r0 : (cy(q) > 0 ? rm : rp);
            unsigned o = xo;
            asm("" : "+v"(o));  // keeps the offset's widening out of the loop (scalar-base loads)
            raw[q] = *reinterpret_cast<const Vec*>(byte_off(wave_uniform(src + q * g.plane + r), o));
        }
    };
    // What step k + 1 needs of the rows that step k has collided: populations 0, 1, 3 of the last one
    // and 2, 5, 6 of the last two, these in two sets used in turn (the row loop is unrolled by two),
    // so that a value stays in its register until it is pulled.
    R A[D - 1][3][V], B[2][D - 1][3][V];
#pragma unroll
    for (int k = 0; k < D - 1; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < V; ++j) A[k][i][j] = B[0][k][i][j] = B[1][k][i][j] = R(0);

    // collide the row h in place (h[q][j]: population q of column j, already pulled)
    auto collide_row = [&](R(&h)[9][V], int n) __attribute__((always_inline)) {
        unsigned long long bad = 0;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            R c[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) c[q] = h[q][j];
            double rho_d;
            const Macro<R> m = macro_of<S>(c, ref, rho_d);
            bad |= __ballot(!(rho_d > 0.0)) & inside[j];
            coll(c, m);
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                h[q][j] = R(to_store<S>(c[q]));
                asm volatile("" : "+v"(h[q][j]));
            }
        }
        if (bad != 0ull) {
            if (lane == 0) atomicMin(blowup, n);
        }
    };
    auto store_row = [&](const R(&h)[9][V], int y) __attribute__((always_inline)) {
        const long long r = (long long)y * g.nx + x0;
        if (c0 >= 0 && c0 + V <= w) {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                Vec v;
#pragma unroll
                for (int j = 0; j < V; ++j) v[j] = S(h[q][j]);
                unsigned o = (unsigned)c0 * E;
                asm("" : "+v"(o));
                __builtin_nontemporal_store(v, reinterpret_cast<Vec*>(byte_off(wave_uniform(dst + q * g.plane + r), o)));
            }
        } else if (c0 >= 0 && c0 < w) {
#pragma unroll
            for (int q = 0; q < 9; ++q)
#pragma unroll
                for (int j = 0; j < V - 1; ++j)
                    if (c0 + j < w) dst[q * g.plane + r + c0 + j] = S(h[q][j]);
        }
    };
    // one iteration; with GUARD the steps that the rows above do not reach yet are left out
    const int a0 = ys - D + 1, a1 = ye + D - 2;
    auto row = [&](auto parity, auto guard, int a) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        R h[9][V];
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            R t[V];
#pragma unroll
            for (int j = 0; j < V; ++j) t[j] = R(raw[q][j]);
            pull_x<V>(q, t, h[q]);
        }
        collide_row(h, step);
        __builtin_amdgcn_sched_barrier(0);
        load_row(a + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 1; k < D; ++k) {
            // step k + 1 pulls row a - k: 0, 1, 3 kept from the last iteration, 2, 5, 6 from the one
            // before, 4, 7, 8 from the row just collided, which takes their places
            constexpr int near[3] = {0, 1, 3}, far[3] = {2, 5, 6}, now[3] = {4, 7, 8};
            R o[9][V];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                pull_x<V>(near[i], A[k - 1][i], o[near[i]]);
                pull_x<V>(far[i], B[P][k - 1][i], o[far[i]]);
                pull_x<V>(now[i], h[now[i]], o[now[i]]);
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    A[k - 1][i][j] = h[near[i]][j];
                    B[P][k - 1][i][j] = h[far[i]][j];
                }
            }
            if constexpr (decltype(guard)::value)
                if (a < a0 + 2 * k) return;
#pragma unroll
            for (int q = 0; q < 9; ++q)
#pragma unroll
                for (int j = 0; j < V; ++j) h[q][j] = o[q][j];
            collide_row(h, step + k);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the loads of the next row are waited for here, where they have had the other steps' time:
        // at the top of the next iteration the wait would include this row's stores
#pragma unroll
        for (int q = 0; q < 9; ++q) loaded(raw[q]);
        if (P == 0 || a <= a1) store_row(h, a - D + 1);
    };
    const std::integral_constant<int, 0> even{};
    const std::integral_constant<int, 1> odd{};
    load_row(a0);
    int a = a0;
    for (; a < a0 + 2 * (D - 1); a += 2) {
        row(even, std::true_type{}, a);
        row(odd, std::true_type{}, a + 1);
    }
    for (; a <= a1; a += 2) {
        row(even, std::false_type{}, a);
        row(odd, std::false_type{}, a + 1);
    }
}

}  // namespace lbm
