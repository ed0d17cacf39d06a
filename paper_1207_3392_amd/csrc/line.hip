// line.hip -- whole runs of steps of a 1D patch in one launch: the single-level
// loop (dt from the device, both Runge-Kutta stages, the CFL rate of the new
// state) on one workgroup, the state in registers (hy_line.h).
//
// What bounds it: the latency of one step's dependent instructions (0.9 us a
// step of 16 cells, 1.6 of 600), then the vector issue of one compute unit (1.8 us
// per 1000 cells, FP64 3.6), and per launch the loads, the stores and the ends
// (2.3 us and 0.5 us per 1000 cells).  us per step, HLLC, in runs of 400:
//   cells                    600  1000  1792  2200  2700  3584
//   FP32 here               1.61  2.39  3.54  4.49  5.62  7.04
//   FP32 stages, graph      7.72  7.71  7.69  7.80  7.77  7.59
//   FP64 here               3.16  4.82  7.28  8.96  11.3  13.9
//   FP64 stages, graph      8.78  8.80  8.70  8.69  8.80  8.62
// The host (takes_line) sends each run of steps to the faster of the two.
#include "hy_line.h"

namespace hy {
namespace {

template <typename T, int SOLVER, int NW, int CPW>
__global__ void __launch_bounds__(64 * NW) k_line(const StageArgs<T> a, int nsteps)
{
    __shared__ T sEdge[2][(NW * CPW + 1) * LINE_EDGE];
    __shared__ T sRate[2][NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Line<T, SOLVER, NW, CPW, true> ln;
    ln.init((int)a.n[0], a.bc[0][0], a.bc[0][1], false, false, a.gamma, a.gm1, a.inv_gm1, a.theta, a.idx[0]);
    T *u = a.uout;
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        const bool o = ln.own(k);
#pragma unroll
        for (int v = 0; v < 3; ++v) ln.U[k][v] = o ? u[v * a.vstride + ln.cell(k)] : T(1);
    }
    // the rate and time of the state as the last step (or hy_set_state) left them
    double t = a.ctl->time[a.parity], rmax;
    {
        const unsigned long long m = row_max(a.ctl->rate[a.parity][(lane & (RATE_SLOTS - 1)) * RATE_STRIDE]);
        const unsigned long long m0 = lane_u64(m, 0), m1 = lane_u64(m, 16);
        rmax = __longlong_as_double((long long)(m0 > m1 ? m0 : m1));
    }
    T rate = T(0);
    for (int s = 0; s < nsteps; ++s) {
        T *edge = sEdge[s & 1];
        if constexpr (CPW * NW > 32) ln.fresh();
        ln.send(edge);
        if (s > 0) {
            rate = lanes_max(rate);
            if (lane == 0) sRate[s & 1][wave] = rate;
        }
        __syncthreads();
        if (s > 0) rmax = (double)lanes_max(lane < NW ? sRate[s & 1][lane] : T(0));
        double dt = a.dt_host;
        if (a.dt_mode == DT_DEVICE) {
            dt = fmin(a.cfl / rmax, a.t_end - t);
            if (!(dt > 0.0)) dt = 0.0;
        }
        const T c1 = uniform_((T)dt * a.idx[0]), c2 = T(0.5) * c1;
        T ca = T(0), cb = T(0);
        if (a.accel[0] != T(0)) {
            ca = uniform_((T)dt * a.accel[0]);
            cb = uniform_(T(0.5) * (T)dt * a.accel[0]);
        }
        rate = T(0);
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            if (wave + k * NW >= ln.nch) break;
            T D[3];
            ln.receive(k, edge);
            ln.stage1_flux(k, D);
            rate = fmax(rate, ln.finish(k, D, c1, ca, c2, cb));
            __builtin_amdgcn_sched_barrier(0);
        }
        t += dt;
    }
#pragma unroll
    for (int k = 0; k < CPW; ++k) {
        if (ln.own(k))
#pragma unroll
            for (int v = 0; v < 3; ++v) u[v * a.vstride + ln.cell(k)] = ln.U[k][v];
    }
    if (ln.bad) atomicOr(&a.ctl->err, 1u);
    rate = lanes_max(rate);
    if (lane == 0) sRate[nsteps & 1][wave] = rate;
    __syncthreads();
    if (wave == 0) {
        const double m = (double)lanes_max(lane < NW ? sRate[nsteps & 1][lane] : T(0));
        const int par = a.parity ^ (nsteps & 1);
        if (lane < RATE_SLOTS)
            a.ctl->rate[par][lane * RATE_STRIDE] = lane == 0 && m > 0.0 ? (unsigned long long)__double_as_longlong(m) : 0ull;
        if (lane == 0) a.ctl->time[par] = t;
    }
}

// Register footprints: 16, 32 and 64 chunks over 16 wavefronts.
template <typename T, int SOLVER>
hipError_t launch_sized(const StageArgs<T> &a, int nsteps, hipStream_t s)
{
    const int nch = (int)((a.n[0] + LINE_OWN - 1) / LINE_OWN);
    const dim3 g(1), b(1024);
    if (nch <= 16) hipLaunchKernelGGL((k_line<T, SOLVER, 16, 1>), g, b, 0, s, a, nsteps);
    else if (nch <= 32) hipLaunchKernelGGL((k_line<T, SOLVER, 16, 2>), g, b, 0, s, a, nsteps);
    else hipLaunchKernelGGL((k_line<T, SOLVER, 16, 4>), g, b, 0, s, a, nsteps);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_line(int solver, const StageArgs<T> &a, int nsteps, hipStream_t s)
{
    if (nsteps < 1 || a.n[0] > LINE_CELLS || a.uout != a.u0) return hipErrorInvalidValue;
    return solver == SOLVER_HLL ? launch_sized<T, SOLVER_HLL>(a, nsteps, s) : launch_sized<T, SOLVER_HLLC>(a, nsteps, s);
}

template hipError_t launch_line<float>(int, const StageArgs<float> &, int, hipStream_t);
template hipError_t launch_line<double>(int, const StageArgs<double> &, int, hipStream_t);

}  // namespace hy
