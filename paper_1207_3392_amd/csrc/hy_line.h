// A 1D patch advanced step by step by one workgroup, its state in registers
// (shared by the batched tubes and the 1D patch loop; internal).
//
// The cells are dealt to wavefronts in chunks of 56: lanes 4 .. 59 of a chunk
// own a cell each, lanes 0 .. 3 and 60 .. 63 hold copies of the four cells on
// either side.  Neighbouring cells are neighbouring lanes, reached by
// whole-wavefront DPP shifts, and four copies are what two stages of the
// two-cell stencil consume (stage 1 is repeated on the inner two), so a whole
// Runge-Kutta step needs one exchange of edge cells through LDS and one
// barrier.  (One cell per thread with primitives and fluxes in LDS took four
// barriers and formed each slope twice: 2.8 us a step for a few hundred
// cells, the latency of its four phases.)
#pragma once

#include "hy_internal.h"
#include "hy_face.h"
#include "hy_stage.h"

namespace hy {
namespace {

constexpr int LINE_OWN = 56;  // cells a chunk owns
constexpr int LINE_H = 4;     // copies on either side
constexpr int LINE_EDGE = 8 * 3;  // LDS words per chunk: its first four cells, its last four

__device__ __forceinline__ float lane_value(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double lane_value(double x, int l)
{
    return __longlong_as_double((long long)lane_u64((unsigned long long)__double_as_longlong(x), l));
}

// NW wavefronts with CPW chunks each (chunk c = wave + k NW).  PATCH: rounds a
// step as the 1D stage kernel (stage.hip) does, bit for bit, so that a patch's
// results do not depend on which of the two takes a step.  (The tubes' own
// order of operations rounds the second stage's change before it is added; a
// run of some 13,000 steps amplifies the difference to 5e-5, so they keep it.)
template <typename T, int SOLVER, int NW, int CPW, bool PATCH>
struct Line {
    T U[CPW][3];    // the lane's cell of each chunk
    int from[CPW];  // LDS word of the lane's copy (-1: an own cell, a wall ghost or unused)
    int n, nch, wave, lane;
    int bclo, bchi;
    bool walllo, wallhi;  // that end is a wall or outflow (its ghosts are formed from the state)
    T k, hs, sg, gamma, gm1, igm1, idx;
    bool bad;

    // Geometry: n cells; a shared end takes its copies from the mail slots
    // (after the chunks' edges in LDS), the end of a periodic line from its
    // other end.
    __device__ __forceinline__ void init(int n_, int bclo_, int bchi_, bool sharedlo, bool sharedhi, T gamma_, T gm1_, T igm1_, T theta,
                                         T idx_)
    {
        n = n_;
        nch = (n + LINE_OWN - 1) / LINE_OWN;
        lane = (int)threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        bclo = bclo_;
        bchi = bchi_;
        walllo = !sharedlo && bclo != BC_PERIODIC;
        wallhi = !sharedhi && bchi != BC_PERIODIC;
        gamma = gamma_;
        gm1 = gm1_;
        igm1 = igm1_;
        const ThetaLim<T> tl = theta_lim(theta);
        k = uniform_(tl.k);
        hs = uniform_(tl.hs);
        sg = uniform_(sqrt_gamma(gamma_));
        idx = idx_;
        bad = false;
#pragma unroll
        for (int q = 0; q < CPW; ++q) {
            const int c = wave + q * NW, j = cell(q), e = end(c);
            from[q] = -1;
            if (c < nch) {
                if (j < c * LINE_OWN) {
                    if (j >= 0) from[q] = c_word(c - 1, 4 + lane);
                    else if (sharedlo) from[q] = c_word(nch, lane);
                    else if (!walllo) from[q] = wrapped((j % n + n) % n);
                } else if (j >= e && j < e + LINE_H) {
                    if (j < n) from[q] = c_word(c + 1, j - e);
                    else if (sharedhi) from[q] = j - n < LINE_H ? c_word(nch, 4 + j - n) : -1;
                    else if (!wallhi) from[q] = wrapped(j % n);
                }
            }
        }
    }
    __device__ __forceinline__ int cell(int q) const { return (wave + q * NW) * LINE_OWN - LINE_H + lane; }
    __device__ __forceinline__ int end(int c) const { return (c + 1) * LINE_OWN < n ? (c + 1) * LINE_OWN : n; }
    __device__ __forceinline__ bool own(int q) const
    {
        const int c = wave + q * NW, j = cell(q);
        return c < nch && j >= c * LINE_OWN && j < end(c);
    }
    __device__ static __forceinline__ int c_word(int c, int slot) { return (c * 8 + slot) * 3; }
    // the word of a cell among the first or last four of its chunk
    __device__ __forceinline__ int wrapped(int j) const
    {
        const int c = j / LINE_OWN, p = j - c * LINE_OWN;
        return p < 4 ? c_word(c, p) : c_word(c, 8 - (end(c) - j));
    }
    // Once per step: what follows from the lane's number is formed again where
    // it is used (a few integer instructions) instead of being kept through
    // the loop in about 20 registers per chunk.
    __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(lane)); }
    // every chunk's first and last four cells to LDS
    __device__ __forceinline__ void send(T *edge) const
    {
#pragma unroll
        for (int q = 0; q < CPW; ++q) {
            const int c = wave + q * NW;
            if (c >= nch) break;
            const int p = lane - LINE_H, cnt = end(c) - c * LINE_OWN;
            if (p >= 0 && p < 4 && p < cnt) {
#pragma unroll
                for (int v = 0; v < 3; ++v) edge[c_word(c, p) + v] = U[q][v];
            }
            if (p >= 0 && p >= cnt - 4 && p < cnt) {
#pragma unroll
                for (int v = 0; v < 3; ++v) edge[c_word(c, 8 - cnt + p) + v] = U[q][v];
            }
        }
    }
    __device__ __forceinline__ void receive(int q, const T *edge)
    {
        if (from[q] >= 0) {
#pragma unroll
            for (int v = 0; v < 3; ++v) U[q][v] = edge[from[q] + v];
        }
    }
    // primitives of the chunk's lanes, wall ghosts included
    __device__ __forceinline__ void prims(int q, const T (&u)[3], T (&w)[3])
    {
        const bool ok = to_prim<1>(u, w, gm1);
        bad |= own(q) && !ok;
        const int c = wave + q * NW;
        if (walllo && c == 0) {
            const bool m = bclo == BC_REFLECT;
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                T a0 = lane_value(w[v], LINE_H), a1 = m ? lane_value(w[v], LINE_H + 1) : a0;
                if (m && v == 1) { a0 = -a0; a1 = -a1; }
                if (lane == LINE_H - 1) w[v] = a0;
                if (lane == LINE_H - 2) w[v] = a1;
            }
        }
        const int g = n - c * LINE_OWN + LINE_H;  // the lane of cell n
        if (wallhi && g < 64) {
            const bool m = bchi == BC_REFLECT;
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                T b0 = lane_value(w[v], g - 1), b1 = m ? lane_value(w[v], g - 2) : b0;
                if (m && v == 1) { b0 = -b0; b1 = -b1; }
                if (lane == g) w[v] = b0;
                if (lane == g + 1) w[v] = b1;
            }
        }
    }
    // D = flux through the low face minus flux through the high face
    __device__ __forceinline__ void flux_difference(const T (&w)[3], T (&D)[3]) const
    {
        T l[3], r[3], f[3];
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const T s = slope_d(w[v] - lane_dn(w[v]), lane_up(w[v]) - w[v], k);
            r[v] = fma_(-hs, s, w[v]);
            l[v] = lane_dn(fma_(hs, s, w[v]));
        }
        riemann<1, 0, SOLVER>(l, r, f, sg, igm1);
#pragma unroll
        for (int v = 0; v < 3; ++v) D[v] = f[v] - lane_up(f[v]);
    }
    __device__ __forceinline__ void stage1_flux(int q, T (&D)[3])
    {
        T w[3];
        prims(q, U[q], w);
        flux_difference(w, D);
    }
    // the rest of the step from stage 1's flux differences; c1 = dt / dx, ca =
    // dt a (uniform acceleration), c2 and cb the same of dt / 2; returns the
    // CFL rate of the new own cell
    __device__ __forceinline__ T finish(int q, const T (&D)[3], T c1, T ca, T c2, T cb)
    {
        T V[3], w[3], E[3];
#pragma unroll
        for (int v = 0; v < 3; ++v) V[v] = fma_(c1, D[v], U[q][v]);
        if (ca != T(0)) {
            V[1] = fma_(U[q][0], ca, V[1]);
            V[2] += U[q][1] * ca;
        }
        prims(q, V, w);
        flux_difference(w, E);
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            if constexpr (PATCH) U[q][v] = fma_(c2, E[v], T(0.5) * (U[q][v] + V[v]));
            else U[q][v] = fma_(T(0.5), U[q][v] + V[v], c2 * E[v]);
        }
        if (cb != T(0)) {
            U[q][1] = fma_(V[0], cb, U[q][1]);
            U[q][2] += V[1] * cb;
        }
        return rate(q);
    }
    __device__ __forceinline__ T speed(const T (&w)[3]) const  // |v| + c
    {
        if constexpr (!PATCH && sizeof(T) == 4) {
            const T gp = gamma * w[2];
            return fma_(gp, __builtin_amdgcn_rsqf(w[0] * gp), fabs(w[1]));
        }
        return fabs(w[1]) + sound_(gamma, w[2], w[0]);
    }
    // (|v| + c) / dx of the own cell, 0 elsewhere
    __device__ __forceinline__ T rate(int q)
    {
        T w[3];
        const bool o = own(q), ok = to_prim<1>(U[q], w, gm1);
        bad |= o && !ok;
        return o ? speed(w) * idx : T(0);
    }
};

}  // namespace
}  // namespace hy
