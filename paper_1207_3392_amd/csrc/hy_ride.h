// Device helpers of the multilevel step shared by the multilevel kernels
// and the stage kernel's padded launches (internal): the enumeration of a
// padded level's exterior shell, the clock updates, and the prolongation of
// the exterior from the parent (Sec. 2), which a launch of its own or extra
// workgroups of another launch (RideJob) carry out.
#pragma once

#include "hy_fmr.h"
#include "hy_face.h"

namespace hy {
namespace {

// The exterior cells of a padded array, enumerated flat: first the rows that
// lie wholly in the exterior (every x), then the NG cells at each x end of
// the remaining rows.
template <int ND>
__host__ __device__ inline int shell_full_rows(const Grid &g)
{
    if constexpr (ND == 1) return 0;
    if constexpr (ND == 2) return 2 * FMR_NG;
    return 2 * FMR_NG * g.m[1] + (g.m[2] - 2 * FMR_NG) * 2 * FMR_NG;
}

template <int ND>
__host__ __device__ inline int shell_cells(const Grid &g)
{
    int part = 1;
    if constexpr (ND >= 2) part *= g.m[1] - 2 * FMR_NG;
    if constexpr (ND >= 3) part *= g.m[2] - 2 * FMR_NG;
    return shell_full_rows<ND>(g) * g.m[0] + part * 2 * FMR_NG;
}

template <int ND>
__device__ __forceinline__ void shell_cell(const Grid &g, int s, int (&c)[3])
{
    const int full = shell_full_rows<ND>(g) * g.m[0];
    c[1] = 0;
    c[2] = 0;
    if (s < full) {
        const int r = s / g.m[0];
        c[0] = s - r * g.m[0];
        if constexpr (ND == 2) {
            c[1] = r < FMR_NG ? r : g.m[1] - 2 * FMR_NG + r;
        } else if constexpr (ND == 3) {
            const int slab = FMR_NG * g.m[1];  // rows of the low (or high) z exterior
            if (r < 2 * slab) {
                const int h = r / slab, rr = r - h * slab;
                c[2] = (h ? g.m[2] - FMR_NG : 0) + rr / g.m[1];
                c[1] = rr % g.m[1];
            } else {
                const int rr = r - 2 * slab, jj = rr % (2 * FMR_NG);
                c[2] = FMR_NG + rr / (2 * FMR_NG);
                c[1] = jj < FMR_NG ? jj : g.m[1] - 2 * FMR_NG + jj;
            }
        }
    } else {
        const int p = s - full, row = p / (2 * FMR_NG), x = p - row * 2 * FMR_NG;
        c[0] = x < FMR_NG ? x : g.m[0] - 2 * FMR_NG + x;
        if constexpr (ND == 2) c[1] = FMR_NG + row;
        if constexpr (ND == 3) {
            const int ny = g.m[1] - 2 * FMR_NG;
            c[2] = FMR_NG + row / ny;
            c[1] = FMR_NG + row % ny;
        }
    }
}

// Clock update op on level l, whose entry is a (and level l + 1's is n): the
// new entry in a and in memory.  rb: the largest rate (CLOCK_DEEPEST).
__device__ __forceinline__ void clock_op(FmrClock *c, int op, int l, FmrClock &a, const FmrClock &n,
                                         unsigned long long rb, double cfl, double dt_fixed)
{
    switch (op) {
    case CLOCK_DEEPEST:
    case CLOCK_DEEPEST_KEEP:
        a.dt = dt_fixed > 0.0 ? dt_fixed : cfl / __longlong_as_double((long long)rb);
        c[l].dt = a.dt;
        break;
    case CLOCK_COARSE:
        a.dt = n.t - a.t;
        c[l].dt = a.dt;
        break;
    case CLOCK_PROVISIONAL:
        a.dtp = n.t - a.t;
        c[l].dtp = a.dtp;
        break;
    case CLOCK_ADVANCE:
        a.t += a.dt;
        c[l].t = a.t;
        break;
    default: break;
    }
}

// Up to two clock updates in order (op < 0: none), by one thread.  Everything
// that they read is fetched at once: one memory latency, not one per value,
// since the launch that carries them waits for this thread.
__device__ __forceinline__ void clock_ops(FmrClock *c, int op0, int l0, int op1, int l1, int nlev,
                                          unsigned long long *rate_bits, double cfl, double dt_fixed)
{
    auto reset = [&]() {
        for (int i = 0; i < nlev; ++i) c[i].t = 0.0;
        for (int k = 0; k < FMR_RATE_SLOTS; ++k) rate_bits[k * RATE_STRIDE] = 0ull;
    };
    if (op0 == CLOCK_RESET) reset();
    auto entry = [&](int l) { return l >= 0 && l < nlev ? c[l] : FmrClock{}; };
    FmrClock a0 = entry(l0), n0 = entry(l0 + 1), a1 = entry(l1), n1 = entry(l1 + 1);
    const bool d0 = op0 == CLOCK_DEEPEST || op0 == CLOCK_DEEPEST_KEEP;
    const bool d1 = op1 == CLOCK_DEEPEST || op1 == CLOCK_DEEPEST_KEEP;
    unsigned long long rb = 0ull;
    if (d0 || d1) {
        unsigned long long r[FMR_RATE_SLOTS];
#pragma unroll
        for (int k = 0; k < FMR_RATE_SLOTS; ++k) r[k] = rate_bits[k * RATE_STRIDE];
#pragma unroll
        for (int k = 0; k < FMR_RATE_SLOTS; ++k) rb = rb > r[k] ? rb : r[k];
        if (op0 == CLOCK_DEEPEST || op1 == CLOCK_DEEPEST)
            for (int k = 0; k < FMR_RATE_SLOTS; ++k) rate_bits[k * RATE_STRIDE] = 0ull;
    }
    if (op0 >= 0) clock_op(c, op0, l0, a0, n0, rb, cfl, dt_fixed);
    if (op1 >= 0) {
        if (op0 >= 0 && l1 == l0) a1 = a0;
        if (op0 >= 0 && l1 + 1 == l0) n1 = a0;
        clock_op(c, op1, l1, a1, n1, rb, cfl, dt_fixed);
        if (op1 == CLOCK_RESET) reset();
    }
}

// One exterior cell (shell index sc) of the job's level: the parent cell's
// primitives plus +/- 1/4 of the parent's minmod-limited differences along
// each active dimension, stored as conserved variables into fine and, when
// not null, fine2 (the level's stage state).
template <int ND, typename T>
__device__ __forceinline__ void prolong_cell(const RideJob<T> &j, int sc)
{
    int c3[3];
    shell_cell<ND>(j.fg, sc, c3);
    int p3[3], s3[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (q < ND) {
            const int r = c3[q] - FMR_NG;  // offset from the first interior cell
            p3[q] = j.pb.lo[q] + (r >> 1);  // floor(r / 2)
            s3[q] = r & 1;                  // 0: low child, 1: high child
        } else {
            p3[q] = 0;
            s3[q] = 0;
        }
    }
    T w0[ND + 2], wc[ND + 2];
    load_prim<ND>(j.parent, j.pg, at(j.pg, p3[0], p3[1], p3[2]), j.gm1, w0);
#pragma unroll
    for (int v = 0; v < ND + 2; ++v) wc[v] = w0[v];
#pragma unroll
    for (int q = 0; q < ND; ++q) {
        int lo3[3] = {p3[0], p3[1], p3[2]}, hi3[3] = {p3[0], p3[1], p3[2]};
        lo3[q] -= 1;
        hi3[q] += 1;
        T wm[ND + 2], wp[ND + 2];
        load_prim<ND>(j.parent, j.pg, at(j.pg, lo3[0], lo3[1], lo3[2]), j.gm1, wm);
        load_prim<ND>(j.parent, j.pg, at(j.pg, hi3[0], hi3[1], hi3[2]), j.gm1, wp);
        // minmod (theta = 1) as twice the slope; the child sits at +/- 1/4
        // of the parent width, so it moves by +/- slope2 / 8
        const T h = s3[q] ? T(0.125) : T(-0.125);
#pragma unroll
        for (int v = 0; v < ND + 2; ++v) wc[v] = fma_(h, slope2_mm(wm[v], w0[v], wp[v], T(2)), wc[v]);
    }
    const int64_t c = at(j.fg, c3[0], c3[1], c3[2]);
    T uc[ND + 2], ke = T(0);
    uc[0] = wc[0];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        uc[1 + d] = wc[0] * wc[1 + d];
        ke = fma_(wc[1 + d], wc[1 + d], ke);
    }
    uc[ND + 1] = fma_(wc[ND + 1], j.inv_gm1, T(0.5) * wc[0] * ke);
#pragma unroll
    for (int v = 0; v < ND + 2; ++v) {
        j.fine[v * j.fg.vs + c] = uc[v];
        if (j.fine2) j.fine2[v * j.fg.vs + c] = uc[v];
    }
}

// Host: the workgroups (of nt threads) that a riding job takes: its shell
// cells', and one for the clock, so that neither waits for the other.
template <typename T>
inline int ride_blocks(const RideJob<T> &j, int nt)
{
    return (j.cells + nt - 1) / nt + (j.ck.c ? 1 : 0);
}

// Workgroup wg (of j.blocks, nthreads threads each) of a riding job: the last
// one carries out the clock updates if there are any, the others the shell
// cells.
template <int ND, typename T>
__device__ __forceinline__ void ride_run(const RideJob<T> &j, int wg, int tid, int nthreads)
{
    const int nb = j.blocks - (j.ck.c ? 1 : 0);
    if (wg >= nb) {
        if (tid == 0 && j.ck.c)
            clock_ops(j.ck.c, j.ck.op0, j.ck.l0, j.ck.op1, j.ck.l1, j.ck.nlev, j.ck.rate, j.ck.cfl, j.ck.dt_fixed);
        return;
    }
    for (int sc = wg * nthreads + tid; sc < j.cells; sc += nb * nthreads) prolong_cell<ND>(j, sc);
}

}  // namespace
}  // namespace hy
