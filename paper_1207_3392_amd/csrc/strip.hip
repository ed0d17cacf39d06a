// strip.hip -- one Runge-Kutta stage of the finite-volume update in 2D.
//
// The slopes, face states and fluxes are those of the 3D stage kernel
// (stage.hip; hy_face.h holds both); a cell's change is summed before its state
// is added, which rounds the state once a stage; and who computes what differs.
// A wavefront owns a strip of 60 columns (its 64 lanes are the columns from 2
// left of the strip to 2 right of it)
// and marches along y over a chunk of rows.  The y stencil lives in
// registers (two rows of primitives, the left state of the next y face, the
// carried y flux), so every y face is solved once; the x neighbours are the
// neighbouring lanes, reached by whole-wavefront DPP shifts that ride on the
// consuming instructions, so every x face is solved once as well.  Nothing
// goes through LDS and no wavefront waits for another.
//
// What bounds it: vector-instruction issue.  A tile of one plane (the 3D
// kernel's layout, which served 2D before) spends half of its instructions on
// what the 3D kernel spreads over a chunk of planes: boundary maps, halo and
// ring items, slopes and fluxes through LDS.  Here the redundant work is 4
// lanes of 64 and, per chunk, the 3 rows and the one face below its first
// row: 192 instructions per row of a wavefront (205 per cell) in the first
// stage, where the tile took 475.  HLLC, us per step in replayed
// graphs: Kelvin-Helmholtz 2048^2 FP32 83 against 128 with the tiles, a random field
// of 2048^2 75.5 / 123, of 1024^2 30 / 38, FP64 54 / 111.
#include "hy_internal.h"
#include "hy_face.h"
#include "hy_ride.h"
#include "hy_stage.h"

#include <limits>

namespace hy {
namespace {

constexpr int SC = 60;  // columns a wavefront updates: lanes 2 .. 61
constexpr int COLS = 64;  // StageArgs::zchunk holds the rows per chunk (1 .. 32) and this flag: chunks fastest

template <typename T, int SOLVER, int STAGE, int LIM>
__global__ void __launch_bounds__(512, sizeof(T) == 8 ? 2 : 4) k_strip(const StageArgs<T> a)
{
    constexpr int NP = 4, IP = 3;
    constexpr bool PAD = LIM == LIM_THETA_PADDED;
    constexpr bool SW = SOLVER == SOLVER_HLLC_SWITCH;
    constexpr int SV = SW ? SOLVER_HLLC : SOLVER;
    static_assert(!PAD || !SW, "padded arrays take HLL or HLLC");
    __shared__ double sRate[8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wpw = (int)blockDim.x >> 6;
    if constexpr (PAD) {
        if ((int)blockIdx.x >= a.ntiles) {
            const int fid = (int)blockIdx.x - a.ntiles;
            if (fid < a.nbfwg) stage_box_faces<2, SOLVER>(a, fid, tid, (int)blockDim.x);
            else ride_run<2>(a.ride, fid - a.nbfwg, tid, (int)blockDim.x);
            return;
        }
    }
    const int nx = (int)a.n[0], ny = (int)a.n[1];
    const int vx = PAD ? a.voff[0] : 0, vy = PAD ? a.voff[1] : 0;
    const int sx = PAD ? a.vm[0] : nx;
    // each XCD takes a contiguous band of the chunks: rows of them (strips
    // fastest), or, in patches lying along x, columns, so that the rows that two
    // chunks share come from one XCD's cache
    int wid;
    {
        const int lid = blockIdx.x, total = a.ntiles;
        const int per = total >> 3, rem = total & 7, xcd = lid & 7;
        const int logical = xcd * per + (xcd < rem ? xcd : rem) + (lid >> 3);
        wid = logical * wpw + __builtin_amdgcn_readfirstlane(tid >> 6);
    }
    // (the last workgroup's wavefronts past the last chunk repeat its first
    // rows' loads and update nothing)
    const bool idle = wid >= a.tiles_x * a.tiles_y;
    if (idle) wid = a.tiles_x * a.tiles_y - 1;
    const int major = wid / a.tiles_x, minor = wid - major * a.tiles_x;
    const bool cols = (a.zchunk & COLS) != 0;
    const int rows = a.zchunk & (COLS - 1);
    const int chunk = cols ? minor : major, strip = cols ? major : minor;
    const int y0 = chunk * rows;
    const int y1 = idle ? y0 : (y0 + rows < ny ? y0 + rows : ny);

    const T gamma = a.gamma, gm1 = a.gm1, igm1 = a.inv_gm1;
    const T sg = uniform_(sqrt_gamma(gamma));
    const ThetaLim<T> tl = theta_lim(a.theta);
    const T lk = uniform_(tl.k);
    const T hs = LIM == LIM_LEARNED ? T(0.5) : uniform_(tl.hs);
    const bool grav = a.accel[0] != T(0) || a.accel[1] != T(0);
    const bool mirx = (a.bc[0][0] == BC_REFLECT) | (a.bc[0][1] == BC_REFLECT);  // (uniform)
    const bool square = a.idx[1] == a.idx[0];

    // this lane's column: its source in storage, mirror sign, whether it is updated
    const int cx = strip * SC - 2 + lane;
    bool fx = false;
    const int mx = PAD ? (cx > nx + 1 ? nx + 1 : cx) + vx : map32(cx, nx, a.bc[0][0], a.bc[0][1], fx);
    const unsigned xoff = (unsigned)mx * (unsigned)sizeof(T);
    const T sgx = fx ? T(-1) : T(1);
    const bool own = lane >= 2 && lane < 2 + SC && cx < nx;

    // byte offset of a row in a variable's array (below 4 GiB: checked on the
    // host), boundary-mapped; flip: a mirror image.  Rows are wave-uniform.
    auto rowoff = [&](int r, bool &flip) -> unsigned {
        const int m = PAD ? r + vy : map32(r, ny, a.bc[1][0], a.bc[1][1], flip);
        return (unsigned)m * (unsigned)sx * (unsigned)sizeof(T);
    };
    auto at = [&](const T *base, unsigned ro) -> const T & { return *(const T *)((const char *)base + ro + xoff); };
    auto load = [&](int r, T (&u)[NP]) {
        bool f = false;
        const unsigned ro = rowoff(r, f);
#pragma unroll
        for (int v = 0; v < NP; ++v) u[v] = at(a.uin + v * a.vstride, ro);
    };
    bool bad = false;
    T rate = T(0);
    auto prim = [&](int r, const T (&u)[NP], T (&w)[NP]) {
        bad |= !to_prim<2>(u, w, gm1);
        if (!PAD) {
            if (mirx) w[1] *= sgx;
            bool f = false;
            (void)rowoff(r, f);
            if (f) w[2] = -w[2];
        }
    };
    // learned slopes of row r along Q: a ghost cell along Q takes its
    // source's slope (periodic), zero (outflow) or the mirrored one (the
    // normal velocity odd about the wall, the others even)
    auto learned = [&](int q, int r, T (&s)[NP]) {
        bool f = false;
        const unsigned ro = rowoff(r, f);
        T sn = T(1), so = T(1);
        const int i = q == 0 ? cx : r, n = q == 0 ? nx : ny;
        if (i < 0 || i >= n) {
            const int bc = a.bc[q][i < 0 ? 0 : 1];
            if (bc == BC_OUTFLOW) sn = so = T(0);
            else if (bc == BC_REFLECT) so = T(-1);
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) {
            const float *b = a.slopes + (int64_t)(q * NP + v) * a.vstride;
            s[v] = (T)(*(const float *)((const char *)b + ro + xoff)) * (v == 1 + q ? sn : so);
        }
    };

    // the first chunk rows and the flux through the face below them
    T WA[NP], WB[NP], WC[NP], UA[NP], UB[NP], UC[NP];
    T L[NP], d[NP], Flo[NP];
    T um[NP];
    T wb[NP];  // switch: the row below the current one
    // stage 2: the row of U^n, fetched a row ahead (fetched at its use's row,
    // the last of a row's work waited for it: 7 levels of 256^2 23.2 -> 22.1 ms)
    T u0[NP];
    auto load0 = [&](int r) {
        bool f = false;
        const unsigned ro = rowoff(r, f);
#pragma unroll
        for (int v = 0; v < NP; ++v) u0[v] = at(a.u0 + v * a.vstride, ro);
    };
    if constexpr (STAGE == 2) load0(y0);
    load(y0, UA);
    load(y0 - 1, um);
    {
        T um2[NP];
        load(y0 - 2, um2);
        load(y0 + 1, UB);
        load(y0 + 2, UC);
        T wm2[NP], wm1[NP], s[NP], R[NP];
        prim(y0 - 2, um2, wm2);
        prim(y0 - 1, um, wm1);
        prim(y0, UA, WA);
        prim(y0 + 1, UB, WB);
        if constexpr (LIM == LIM_LEARNED) {
            learned(1, y0 - 1, s);
#pragma unroll
            for (int v = 0; v < NP; ++v) L[v] = fma_(hs, s[v], wm1[v]);
            learned(1, y0, s);
        } else {
#pragma unroll
            for (int v = 0; v < NP; ++v) {
                d[v] = WA[v] - wm1[v];
                L[v] = fma_(hs, slope_d(wm1[v] - wm2[v], d[v], lk), wm1[v]);
                const T dp = WB[v] - WA[v];
                s[v] = slope_d(d[v], dp, lk);
                d[v] = dp;
            }
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) R[v] = fma_(-hs, s[v], WA[v]);
        riemann<2, 1, SV>(L, R, Flo, sg, igm1);
        if constexpr (SW) {
            // the face y0 - 1/2 takes HLL where a cell of rows y0 - 1, y0 is in a shock along x
            const bool hll = x_shock(lane_dn(wm1[IP]), lane_up(wm1[IP]), lane_dn(wm1[1]), lane_up(wm1[1])) |
                             x_shock(lane_dn(WA[IP]), lane_up(WA[IP]), lane_dn(WA[1]), lane_up(WA[1]));
            if (__builtin_amdgcn_ballot_w64(hll) != 0ull) {
                if (hll) riemann<2, 1, SOLVER_HLL>(L, R, Flo, sg, igm1);
            }
#pragma unroll
            for (int v = 0; v < NP; ++v) wb[v] = wm1[v];
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) L[v] = fma_(hs, s[v], WA[v]);
    }
    // the step, after the first loads are on their way
    const double dtd = stage_dt(a);
    if (STAGE == 1 && wid == 0 && lane < RATE_SLOTS) {
        a.ctl->rate[a.parity ^ 1][lane * RATE_STRIDE] = 0ull;
        if (lane == 0) a.ctl->time[a.parity ^ 1] = a.ctl->time[a.parity] + dtd;
    }
    const T dt = (T)dtd;
    const T wdt = STAGE == 1 ? dt : T(0.5) * dt;
    T cdt[2], cacc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        cdt[q] = uniform_(wdt * a.idx[q]);
        cacc[q] = uniform_(wdt * a.accel[q]);
    }

    // row r: W0/U0 hold it, W1/U1 row r + 1, U2 row r + 2 as loaded (its
    // primitives go to W2); the rows' registers are rotated by the caller
    auto body = [&](int r, T (&W0)[NP], T (&W1)[NP], T (&W2)[NP], T (&U0)[NP], T (&U1)[NP], T (&U2)[NP]) {
        (void)U1;
        bool nf = false;
        const unsigned ro = rowoff(r, nf);
        prim(r + 2, U2, W2);
        // ---- y face r + 1/2 ----
        T s[NP], R[NP], Fhi[NP];
        if constexpr (LIM == LIM_LEARNED) learned(1, r + 1, s);
        else {
#pragma unroll
            for (int v = 0; v < NP; ++v) {
                const T dp = W2[v] - W1[v];
                s[v] = slope_d(d[v], dp, lk);
                d[v] = dp;
            }
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) R[v] = fma_(-hs, s[v], W1[v]);
        riemann<2, 1, SV>(L, R, Fhi, sg, igm1);
        bool yb = false;  // switch: the own cell is in a shock along y
        if constexpr (SW) {
            const bool hll = x_shock(lane_dn(W0[IP]), lane_up(W0[IP]), lane_dn(W0[1]), lane_up(W0[1])) |
                             x_shock(lane_dn(W1[IP]), lane_up(W1[IP]), lane_dn(W1[1]), lane_up(W1[1]));
            if (__builtin_amdgcn_ballot_w64(hll) != 0ull) {
                if (hll) riemann<2, 1, SOLVER_HLL>(L, R, Fhi, sg, igm1);
            }
            yb = x_shock(wb[IP], W1[IP], wb[2], W1[2]);
#pragma unroll
            for (int v = 0; v < NP; ++v) wb[v] = W0[v];
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) L[v] = fma_(hs, s[v], W1[v]);
        // ---- x face between the lane below and the own column ----
        T Fx[NP];
        {
            T xl[NP], xr[NP], sx_[NP];
            if constexpr (LIM == LIM_LEARNED) learned(0, r, sx_);
            else {
#pragma unroll
                for (int v = 0; v < NP; ++v) sx_[v] = slope_d(W0[v] - lane_dn(W0[v]), lane_up(W0[v]) - W0[v], lk);
            }
#pragma unroll
            for (int v = 0; v < NP; ++v) {
                xr[v] = fma_(-hs, sx_[v], W0[v]);
                xl[v] = lane_dn(fma_(hs, sx_[v], W0[v]));
            }
            riemann<2, 0, SV>(xl, xr, Fx, sg, igm1);
            if constexpr (SW) {
                const unsigned long long m = __builtin_amdgcn_ballot_w64(yb);
                const unsigned long long f = m | (m << 1);
                if (f != 0ull) {
                    if ((f >> lane) & 1ull) riemann<2, 0, SOLVER_HLL>(xl, xr, Fx, sg, igm1);
                }
            }
        }
        // ---- divergence, source, Runge-Kutta combination ----
        // the change is summed first and added to the state last, so a stage
        // rounds the state once (stage 2: (U^n + U1 + dt L) / 2 as U^n +
        // [(U1 - U^n) / 2 + dt L / 2], the difference being exact)
        T out[NP];
#pragma unroll
        for (int v = 0; v < NP; ++v) {
            T ch = fma_(cdt[1], Flo[v] - Fhi[v], cdt[0] * (Fx[v] - lane_up(Fx[v])));
            if constexpr (STAGE == 2) ch = fma_(T(0.5), U0[v] - u0[v], ch);
            out[v] = ch;
            Flo[v] = Fhi[v];
        }
        if (grav) {
#pragma unroll
            for (int q = 0; q < 2; ++q) out[1 + q] = fma_(U0[0], cacc[q], out[1 + q]);
            out[IP] += fma_(U0[1], cacc[0], U0[2] * cacc[1]);
        }
#pragma unroll
        for (int v = 0; v < NP; ++v) out[v] += STAGE == 1 ? U0[v] : u0[v];
        // the row three ahead, into the registers this row leaves
        if (r + 3 <= y1 + 1) load(r + 3, U0);
        if constexpr (STAGE == 2)
            if (r + 1 < y1) load0(r + 1);
        if (own) {
#pragma unroll
            for (int v = 0; v < NP; ++v) *(T *)((char *)(a.uout + v * a.vstride) + ro + xoff) = out[v];
            if constexpr (STAGE == 2) {
                T wo[NP];
                bad |= !to_prim<2>(out, wo, gm1);
                const T cs = sound_(gamma, wo[IP], wo[0]);
                if (square) rate = fmax(rate, (fmax(fabs(wo[1]), fabs(wo[2])) + cs) * a.idx[0]);
                else rate = fmax(rate, fmax((fabs(wo[1]) + cs) * a.idx[0], (fabs(wo[2]) + cs) * a.idx[1]));
            }
        }
    };
    for (int r = y0; r < y1; r += 3) {
        body(r, WA, WB, WC, UA, UB, UC);
        if (r + 1 < y1) body(r + 1, WB, WC, WA, UB, UC, UA);
        if (r + 2 < y1) body(r + 2, WC, WA, WB, UC, UA, UB);
    }
    if (bad) atomicOr(&a.ctl->err, 1u);
    if constexpr (STAGE == 2) {
        double m = (double)lanes_max(rate);
        if (lane == 0) sRate[tid >> 6] = m;
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 1; w < 8; ++w) m = fmax(m, w < wpw ? sRate[w] : 0.0);
            if (m > 0.0)
                atomicMax(&a.ctl->rate[a.parity ^ 1][(blockIdx.x % RATE_SLOTS) * RATE_STRIDE],
                          (unsigned long long)__double_as_longlong(m));
        }
    }
}

}  // namespace

// Rows per chunk: a short chunk repeats its 3 rows and one face more often, a
// long one leaves few wavefronts to hide latency with, and a last round over the
// card's 1024 SIMDs that is nearly empty costs most of a full one.  The rows are
// those with the least (1 + k) (rows + 1.2), FP64 (0.7 + k) (rows + 2), k the
// wavefronts on a SIMD, three quarters the busiest one's and one the mean: over 54
// shapes of 10^4 to 10^7 cells the step is then within 2 % (FP64 7 %) of the best of
// 1 .. 32 rows, on average 0.1 % (0.8 %).  (Rows as the square root of the strips'
// length, picked before: 15 % and 31 %, on average 2 and 11 %.  us per step, HLLC: FP32
// 700^2 20.6 -> 17.9, FP64 38.7 -> 30.3; FP64 61 x 4000 32.4 -> 26.1; FP32 2048^2 75.8 and
// 512^2 14.2 as before.)
template <typename T>
int strip_rows(const int64_t n[3])
{
    const int ny = (int)n[1], strips = (int)((n[0] + SC - 1) / SC);
    const float a = sizeof(T) == 4 ? 1.f : 0.7f, b = sizeof(T) == 4 ? 1.2f : 2.f;
    int best = 1;
    float cost = std::numeric_limits<float>::max();
    for (int r = 1; r <= 32 && r <= ny; ++r) {
        const int waves = strips * ((ny + r - 1) / r);
        const float mean = (float)waves * (1.f / 1024.f);
        const float k = 0.75f * (float)((waves + 1023) >> 10) + 0.25f * (mean > 1.f ? mean : 1.f);
        const float c = (a + k) * ((float)r + b);
        if (c < cost) {
            cost = c;
            best = r;
        }
    }
    return best;
}
template int strip_rows<float>(const int64_t *);
template int strip_rows<double>(const int64_t *);

namespace {

template <typename T, int SOLVER, int STAGE, int LIM>
hipError_t launch_one(const LaunchCfg &cfg, StageArgs<T> a, hipStream_t s)
{
    const int nt = cfg.bx * cfg.by, wpw = nt / 64;
    const int rows = strip_rows<T>(a.n);
    const int strips = (int)((a.n[0] + SC - 1) / SC), chunks = (int)((a.n[1] + rows - 1) / rows);
    // (FP32, us per step: 20,000 x 8 16.0 strips fastest, 11.6 chunks fastest; 10,000 x 30
    // 17.5 / 14.9; 5000 x 32 13.6 / 11.8; 3000 x 100 15.2 / 15.2; 2000 x 16 9.2 / 9.4; 400^2 12.8 / 14.2)
    const bool cols = a.n[0] >= 128 * a.n[1];
    a.zchunk = rows | (cols ? COLS : 0);
    a.tiles_x = cols ? chunks : strips;
    a.tiles_y = cols ? strips : chunks;
    a.ntiles = (int)(((int64_t)strips * chunks + wpw - 1) / wpw);
    int64_t blocks = a.ntiles;
    if constexpr (LIM == LIM_THETA_PADDED) {
        const hipError_t e = stage_extra_blocks<2>(a, nt, &blocks);
        if (e != hipSuccess) return e;
    }
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_strip<T, SOLVER, STAGE, LIM>), dim3((unsigned)blocks), dim3(nt), 0, s, a);
    return hipGetLastError();
}

template <typename T, int SOLVER, int STAGE>
hipError_t launch_lim(int limiter, const LaunchCfg &cfg, const StageArgs<T> &a, hipStream_t s)
{
    if constexpr (sizeof(T) == 4) {
        if (limiter == LIM_LEARNED) return launch_one<T, SOLVER, STAGE, LIM_LEARNED>(cfg, a, s);
    }
    if constexpr (SOLVER != SOLVER_HLLC_SWITCH) {
        if (limiter == LIM_THETA_PADDED) return launch_one<T, SOLVER, STAGE, LIM_THETA_PADDED>(cfg, a, s);
    } else {
        if (limiter == LIM_THETA_PADDED) return hipErrorInvalidValue;
    }
    return launch_one<T, SOLVER, STAGE, LIM_THETA>(cfg, a, s);
}

}  // namespace

template <typename T>
hipError_t launch_strip(int solver, int stage, int limiter, const LaunchCfg &cfg, const StageArgs<T> &a, hipStream_t s)
{
    switch (solver) {
    case SOLVER_HLL: return stage == 1 ? launch_lim<T, 0, 1>(limiter, cfg, a, s) : launch_lim<T, 0, 2>(limiter, cfg, a, s);
    case SOLVER_HLLC_SWITCH:
        return stage == 1 ? launch_lim<T, 2, 1>(limiter, cfg, a, s) : launch_lim<T, 2, 2>(limiter, cfg, a, s);
    default: return stage == 1 ? launch_lim<T, 1, 1>(limiter, cfg, a, s) : launch_lim<T, 1, 2>(limiter, cfg, a, s);
    }
}

template hipError_t launch_strip<float>(int, int, int, const LaunchCfg &, const StageArgs<float> &, hipStream_t);
template hipError_t launch_strip<double>(int, int, int, const LaunchCfg &, const StageArgs<double> &, hipStream_t);

}  // namespace hy
