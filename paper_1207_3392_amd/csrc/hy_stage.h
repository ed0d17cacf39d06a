// Device and launch helpers shared by the stage kernels (stage.hip, strip.hip).
#pragma once

#include "hy_internal.h"
#include "hy_face.h"

namespace hy {
namespace {

// The neighbouring lanes' values: lane l takes l - 1's (lane_dn) or l + 1's
// (lane_up); the end lane, which no cell that is stored depends on, takes 0.
__device__ __forceinline__ int dpp_shr(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_shl(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ float lane_dn(float x) { return __int_as_float(dpp_shr(__float_as_int(x))); }
__device__ __forceinline__ float lane_up(float x) { return __int_as_float(dpp_shl(__float_as_int(x))); }
__device__ __forceinline__ double lane_dn(double x)
{
    return __hiloint2double(dpp_shr(__double2hiint(x)), dpp_shr(__double2loint(x)));
}
__device__ __forceinline__ double lane_up(double x)
{
    return __hiloint2double(dpp_shl(__double2hiint(x)), dpp_shl(__double2loint(x)));
}

// The maximum of x over the lane's row of 16, in every lane of the row (bit
// patterns of non-negative doubles, which order like the doubles).
__device__ __forceinline__ unsigned long long row_max(unsigned long long x)
{
#define HY_ROW_STEP(ctrl)                                                                                      \
    {                                                                                                          \
        const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)x, ctrl, 0xf, 0xf, true);   \
        const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(x >> 32), ctrl, 0xf, 0xf, true);     \
        const unsigned long long y = ((unsigned long long)hi << 32) | lo;                                       \
        x = x > y ? x : y;                                                                                     \
    }
    HY_ROW_STEP(0x128)  // row_ror:8, 4, 2, 1
    HY_ROW_STEP(0x124)
    HY_ROW_STEP(0x122)
    HY_ROW_STEP(0x121)
#undef HY_ROW_STEP
    return x;
}

__device__ __forceinline__ unsigned long long lane_u64(unsigned long long x, int l)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(x >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

// The maximum of non-negative x over the wavefront, the same in every lane:
// 4 shifts within the rows of 16 and 4 lanes read (12 exchanges through LDS for
// a double by shuffles ended every workgroup: 180 x 150, 350 -> 345 us per pass; in
// the 1D runs, a floating-point maximum passed on from row to row, with its
// wait states, took 218 us for 100 steps of 600 cells, this 210).
__device__ __forceinline__ double lanes_max(double x)
{
    const unsigned long long m = row_max((unsigned long long)__double_as_longlong(x));
    const unsigned long long a = lane_u64(m, 0), b = lane_u64(m, 16), c = lane_u64(m, 32), d = lane_u64(m, 48);
    const unsigned long long e = a > b ? a : b, f = c > d ? c : d;
    return __longlong_as_double((long long)(e > f ? e : f));
}
__device__ __forceinline__ float lanes_max(float x)
{
    unsigned m = __float_as_uint(x);
#define HY_ROW_STEP(ctrl)                                                                                      \
    {                                                                                                          \
        const unsigned y = (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, ctrl, 0xf, 0xf, true);              \
        m = m > y ? m : y;                                                                                     \
    }
    HY_ROW_STEP(0x128)
    HY_ROW_STEP(0x124)
    HY_ROW_STEP(0x122)
    HY_ROW_STEP(0x121)
#undef HY_ROW_STEP
    const unsigned a = __builtin_amdgcn_readlane((int)m, 0), b = __builtin_amdgcn_readlane((int)m, 16);
    const unsigned c = __builtin_amdgcn_readlane((int)m, 32), d = __builtin_amdgcn_readlane((int)m, 48);
    const unsigned e = a > b ? a : b, f = c > d ? c : d;
    return __uint_as_float(e > f ? e : f);
}

// The stage's time step, the same in every lane.  Called by whole wavefronts:
// each lane reads one rate slot and the maximum is taken across lanes (one
// load and about 30 instructions, where a loop over the slots in every lane
// cost 32 loads and about 100).
template <typename T>
__device__ __forceinline__ double stage_dt(const StageArgs<T> &a)
{
    if (a.dt_mode == DT_HOST) return a.dt_host;
    if (a.dt_mode == DT_PTR) return *a.dt_dev;
    static_assert(RATE_SLOTS == 32, "two rows of 16 lanes hold the slots");
    const unsigned long long m = row_max(a.ctl->rate[a.parity][(__lane_id() & (RATE_SLOTS - 1)) * RATE_STRIDE]);
    const unsigned long long m0 = lane_u64(m, 0), m1 = lane_u64(m, 16);
    const double rate = __longlong_as_double((long long)(m0 > m1 ? m0 : m1));
    const double t = a.ctl->time[a.parity];
    const double dt = fmin(a.cfl / rate, a.t_end - t);
    return dt > 0.0 ? dt : 0.0;
}

// A value every lane holds alike, moved to a scalar register so the vector
// register budget of the per-cell work does not carry it.
__device__ __forceinline__ float uniform_(float x)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
__device__ __forceinline__ double uniform_(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Source of index i along a dimension of n interior cells; flip toggles when
// the source is a mirror image.  Indices far outside the ghost range (only
// met by the unused columns of partial tiles) are clamped into the array.
__device__ __forceinline__ int map32(int i, int n, int bclo, int bchi, bool &flip)
{
    if (i >= 0 && i < n) return i;
    int m;
    if (i < 0) {
        if (bclo == BC_PERIODIC) m = i + n;
        else if (bclo == BC_OUTFLOW) m = 0;
        else { m = -1 - i; flip = !flip; }
    } else {
        if (bchi == BC_PERIODIC) m = i - n;
        else if (bchi == BC_OUTFLOW) m = n - 1;
        else { m = 2 * n - 1 - i; flip = !flip; }
    }
    return m < 0 ? 0 : (m >= n ? n - 1 : m);
}

// The HLLC switch's detector along one dimension, from a cell's two
// neighbours: their pressures differ by more than eps of the smaller one and
// the velocity decreases from the lower (a) to the upper (b) one.
template <typename T>
__device__ __forceinline__ bool x_shock(T pa, T pb, T va, T vb)
{
    return (fabs(pb - pa) > (T)SHOCK_EPS * fmin(pa, pb)) & (vb - va < T(0));
}

// The face-flux workgroups of a padded launch (see BoxFluxes): workgroup fid
// after the tiles takes (box, q, side) = segment fid / blocks, nt faces of it.
template <int ND, int SOLVER, typename T>
__device__ __forceinline__ void stage_box_faces(const StageArgs<T> &a, int fid, int tid, int nt)
{
    const int seg = fid / a.bf.blocks;
    const int t = (fid - seg * a.bf.blocks) * nt + tid;
    const int side = seg & 1, bq = seg >> 1, k = bq / ND, q = bq - k * ND;
    const Grid g{{a.vm[0], a.vm[1], a.vm[2]}, a.vstride};
    const Box &b = a.bf.b[k];
    const double w = 0.5 * *a.dt_dev;
    const bool as = a.bf.assign[k] != 0;
    if (q == 0)
        box_faces<ND, 0, SOLVER>(a.uin, g, b, t, side, a.gamma, a.gm1, a.inv_gm1, a.theta, w, as, a.bf.acc[k][0][0],
                                 a.bf.acc[k][0][1]);
    if constexpr (ND >= 2)
        if (q == 1)
            box_faces<ND, 1, SOLVER>(a.uin, g, b, t, side, a.gamma, a.gm1, a.inv_gm1, a.theta, w, as,
                                     a.bf.acc[k][1][0], a.bf.acc[k][1][1]);
    if constexpr (ND >= 3)
        if (q == 2)
            box_faces<ND, 2, SOLVER>(a.uin, g, b, t, side, a.gamma, a.gm1, a.inv_gm1, a.theta, w, as,
                                     a.bf.acc[k][2][0], a.bf.acc[k][2][1]);
}

// Host: the workgroups (of nt threads) that a padded launch carries after its
// tiles, for the box face fluxes and the riding job.
template <int ND, typename T>
hipError_t stage_extra_blocks(StageArgs<T> &a, int nt, int64_t *blocks)
{
    a.nbfwg = 0;
    if (a.bf.nbox > 0) {
        if (a.bf.nbox > 2 || a.dt_mode != DT_PTR || !a.dt_dev) return hipErrorInvalidValue;
        int most = 0;
        for (int k = 0; k < a.bf.nbox; ++k)
            for (int q = 0; q < ND; ++q) {
                const int r1 = q == 0 ? 1 : 0, r2 = q == 2 ? 1 : 2;
                most = most > a.bf.b[k].n[r1] * a.bf.b[k].n[r2] ? most : a.bf.b[k].n[r1] * a.bf.b[k].n[r2];
            }
        a.bf.blocks = (most + nt - 1) / nt;
        a.nbfwg = a.bf.nbox * ND * 2 * a.bf.blocks;
        *blocks += a.nbfwg;
    }
    a.ride.blocks = ride_blocks(a.ride, nt);
    *blocks += a.ride.blocks;
    return hipSuccess;
}

}  // namespace
}  // namespace hy
