// Pointwise device math of the finite-volume update, shared by the stage
// kernels and the multilevel kernels so that both compute the same face
// fluxes: primitive recovery (Sec. 3.5), the generalised-minmod slope (eq.
// MinMod) and the HLL / HLLC fluxes (eqs. FluxHLL, FluxHLLC and the middle
// wave of eq. MiddleWaveSpeed).  Internal; every user gets its own copy.
#pragma once

#include "hy_internal.h"

#include <math.h>

namespace hy {
namespace {

// Every function here rounds the same way wherever it is inlined: contraction
// is off and each fused multiply-add is written out.  A face that two
// wavefronts (or the stage and the flux-replacement kernels) evaluate then has
// one flux, bit for bit, so what one cell loses its neighbour gains.  (Left to
// the compiler, contraction follows its basic blocks: the copies of one face
// differed in the last place.)
#pragma clang fp contract(off)

// ---------------------------------------------------------------- math ----

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// 1 / x.  FP64: two Newton steps on the hardware's estimate (relative error
// 2^-23 at most, so 2^-92 before the last rounding), 5 instructions where the
// IEEE division sequence takes 11; x normal and not 0.
template <typename T> __device__ __forceinline__ T rcp_(T x);
template <> __device__ __forceinline__ float rcp_<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <> __device__ __forceinline__ double rcp_<double>(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma_(fma_(-x, r, 1.0), r, r);
    return fma_(fma_(-x, r, 1.0), r, r);
}

// sqrt(p / r), evaluated as p rsqrt(p r).  FP64: y = 1 / sqrt(p r) from the
// hardware's reciprocal roots of p and of r, not of p r, which leaves the range
// long before the ratio does (densities and pressures near 1e-155 or 1e155); one
// Newton step on s = p y, with p r y^2 formed from p y and r y / 2, leaves about
// 2^-42, and the residual p - s^2 r, with s r carried in two parts, corrects s to
// the last rounding: 13 instructions where a division and a root take 25.  (One
// reciprocal root of p r saves 1 to 3 % of an FP64 step, 150 x 140 x 130, 10 steps:
// 2160 us against 2189, and gives a NaN where p r overflows or vanishes.)
__device__ __forceinline__ float root_ratio(float p, float r) { return p * __builtin_amdgcn_rsqf(p * r); }
__device__ __forceinline__ double root_ratio(double p, double r)
{
    const double y = __builtin_amdgcn_rsq(p) * __builtin_amdgcn_rsq(r), h = 0.5 * y, u = p * y;
    const double s = u * fma_(-u, r * h, 1.5), t = s * r;
    const double e = fma_(-fma_(s, r, -t), s, fma_(-t, s, p));
    return fma_(e, h, s);
}

// sqrt(p / rho), the sound speed divided by sqrt(gamma); the solvers fold
// sqrt(gamma) into the signal speeds
template <typename T> __device__ __forceinline__ T sound1_(T p, T rho) { return root_ratio(p, rho); }

// c_s = sqrt(gamma p / rho)
template <typename T> __device__ __forceinline__ T sound_(T gamma, T p, T rho) { return root_ratio(gamma * p, rho); }

template <typename T> __device__ __forceinline__ T max3_(T a, T b, T c) { return fmax(a, fmax(b, c)); }

// ------------------------------------------------------ fluid variables ----

// x > 0 and finite: one class test in FP32 (positive normal or subnormal)
template <typename T> __device__ __forceinline__ bool pos_finite(T x);
template <> __device__ __forceinline__ bool pos_finite<float>(float x) { return __builtin_amdgcn_classf(x, 0x180); }
template <> __device__ __forceinline__ bool pos_finite<double>(double x)
{
    return __builtin_amdgcn_class(x, 0x180);
}

// In 1D some sums below are fused in another order than in 2D and 3D (the
// branches on ND == 1): the order in which the compiler contracted the tubes'
// kernel while contraction was left to it.  A tube's run takes thousands of
// steps through shocks (512 tubes of up to 4096 cells: 13,000), which amplify a
// last place to 5e-5 of the state, so the order stays as it was.

// primitives (rho, v, p) from conserved (D, S, G), m = 1; returns false on
// rho <= 0, p <= 0 or a non-finite value
template <int ND, typename T>
__device__ __forceinline__ bool to_prim(const T (&u)[ND + 2], T (&w)[ND + 2], T gm1)
{
    const T ir = rcp_(u[0]);
    w[1] = u[1] * ir;
    if constexpr (ND == 1) {
        w[2] = gm1 * fma_(T(-0.5) * u[1], w[1], u[2]);
    } else {
        T ke = u[1] * w[1];
#pragma unroll
        for (int d = 1; d < ND; ++d) {
            w[1 + d] = u[1 + d] * ir;
            ke = fma_(u[1 + d], w[1 + d], ke);
        }
        w[ND + 1] = gm1 * fma_(T(-0.5), ke, u[ND + 1]);
    }
    w[0] = u[0];
    return pos_finite(w[0]) & pos_finite(w[ND + 1]);
}

// The two-argument minmod: the argument nearer to zero when they share a
// sign, else 0 (the median of x, y and 0).
__device__ __forceinline__ float minmod_(float x, float y) { return __builtin_amdgcn_fmed3f(x, y, 0.f); }
__device__ __forceinline__ double minmod_(double x, double y)
{
    return fmax(fmin(x, fmax(y, 0.0)), fmin(y, 0.0));
}
// The same where the arguments never differ in sign.
__device__ __forceinline__ float minmod_same(float x, float y) { return __builtin_amdgcn_fmed3f(x, y, 0.f); }
__device__ __forceinline__ double minmod_same(double x, double y) { return fabs(x) < fabs(y) ? x : y; }

// Twice the generalised-minmod slope of eq. MinMod as a per-cell difference:
// with a = 2 theta dm, b = dm + dp, c = 2 theta dp, MM(a, b, c) (the argument
// of least magnitude when all share a sign, else 0) = 2 MM(theta dm,
// (dm + dp) / 2, theta dp) exactly, evaluated as MM(MM(a, c), b) (b shares
// the sign of a and c when they agree; see slope_mm).  Face values are then
// w +/- slope / 4.
template <typename T>
__device__ __forceinline__ T slope2_mm(T wm, T w0, T wp, T theta2)
{
    const T dm = w0 - wm, dp = wp - w0;
    const T a = theta2 * dm, b = dm + dp, c = theta2 * dp;
    return minmod_same(minmod_(a, c), b);
}

// The generalised-minmod slope of eq. MinMod divided by theta: scaling every
// argument of MM by 1 / theta (a positive factor commutes with MM) gives
// MM(dm, (dm + dp) k, dp) with k = 1 / (2 theta); the face values are then
// w +/- hs * slope with hs = theta / 2.  The factors theta leave the per-cell
// work this way.  The middle argument b = (dm + dp) k carries the sign of
// dm and dp whenever those two agree, so MM(dm, b, dp) = MM(MM(dm, dp), b):
// two two-argument minmods (in FP32 two median instructions), the same value
// as med3(min3, max3, 0) bit for bit (each form selects one of its inputs).
template <typename T>
__device__ __forceinline__ T slope_d(T dm, T dp, T k)  // from the two differences
{
    return minmod_same(minmod_(dm, dp), (dm + dp) * k);
}
template <typename T>
__device__ __forceinline__ T slope_mm(T wm, T w0, T wp, T k)
{
    return slope_d(w0 - wm, wp - w0, k);
}

// The per-patch constants of slope_mm and of the face values, formed the
// same way by every kernel that computes a face flux of the same state.
template <typename T> struct ThetaLim {
    T k, hs;
};
template <typename T> __device__ __forceinline__ ThetaLim<T> theta_lim(T theta)
{
    return ThetaLim<T>{T(0.5) / theta, T(0.5) * theta};
}

// ------------------------------------------------------ Riemann solvers ----

// Flux normal to Q from the primitive face states wl (left), wr (right).
// sg = sqrt(gamma) (formed once per kernel by the caller, the same way
// everywhere: sqrt_gamma below).
template <int ND, int Q, int SOLVER, typename T>
__device__ __forceinline__ void riemann(const T (&wl)[ND + 2], const T (&wr)[ND + 2], T (&f)[ND + 2],
                                        T sg, T inv_gm1)
{
    constexpr int IP = ND + 1;
    const T rl = wl[0], vl = wl[1 + Q], pl = wl[IP];
    const T rr = wr[0], vr = wr[1 + Q], pr = wr[IP];
    const T ul = sound1_(pl, rl), ur = sound1_(pr, rr);
    // outer speed estimates alpha_+/- = max(0, +/-lambda_+/-(L), +/-lambda_+/-(R)),
    // c = sg u
    const T ap = max3_(T(0), fma_(sg, ul, vl), fma_(sg, ur, vr));
    const T am = max3_(T(0), fma_(sg, ul, -vl), fma_(sg, ur, -vr));
    if constexpr (SOLVER == 0) {
        T El, Er;
        if constexpr (ND == 1) {
            El = fma_(vl, T(0.5) * rl * vl, pl * inv_gm1);
            Er = fma_(vr, T(0.5) * rr * vr, pr * inv_gm1);
        } else {
            T kl = wl[1] * wl[1], kr = wr[1] * wr[1];
#pragma unroll
            for (int d = 1; d < ND; ++d) {
                kl = fma_(wl[1 + d], wl[1 + d], kl);
                kr = fma_(wr[1 + d], wr[1 + d], kr);
            }
            El = fma_(pl, inv_gm1, T(0.5) * rl * kl);
            Er = fma_(pr, inv_gm1, T(0.5) * rr * kr);
        }
        // F = (a+ F_L + a- F_R - a+ a- (U_R - U_L)) / (a+ + a-).  With the
        // physical flux F = v U + P (P: p in the normal momentum, p v in the
        // energy) each side's state enters once:
        //   F = cL U_L + cR U_R + wL P_L + wR P_R,
        //   wL = a+ / (a+ + a-), wR = a- / (a+ + a-),
        //   cL = wL (v_L + a-), cR = wR (v_R - a+).
        // a+ + a- = 0 (both sides at rest with c = 0, so a+ = a- = 0) takes
        // wL = wR = 1/2, which makes the same coefficients the mean of the
        // two fluxes.
        const T den = ap + am;
        const bool pos = den > T(0);
        const T inv = pos ? rcp_(den) : T(0);
        const T wL = pos ? ap * inv : T(0.5), wR = pos ? am * inv : T(0.5);
        const T cL = wL * (vl + am), cR = wR * (vr - ap);
        const T gL = cL * rl, gR = cR * rr;  // the coefficients of the velocities in the momentum
        f[0] = fma_(cL, rl, gR);
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            if (d == Q) f[1 + d] = fma_(gL, wl[1 + d], fma_(gR, wr[1 + d], fma_(wL, pl, wR * pr)));
            else f[1 + d] = fma_(gL, wl[1 + d], gR * wr[1 + d]);
        }
        f[IP] = fma_(cL, El, fma_(cR, Er, fma_(wL, pl * vl, wR * (pr * vr))));
    } else {
        // Batten's middle-wave speed (eq. MiddleWaveSpeed):
        // (A v_R + B v_L + p_L - p_R) / (A + B), A = rho_R (a+ - v_R), B = rho_L (a- + v_L)
        const T ql = am + vl, qr = ap - vr;
        const T A = rr * qr, B = rl * ql;
        const T am_ = fma_(A, vr, fma_(B, vl, pl - pr)) * rcp_(ND == 1 ? fma_(rr, qr, B) : A + B);
        // eq. FluxHLLC: alpha_- = 0 selects L, then alpha_+ = 0 selects R,
        // then the sign of alpha_m selects the middle state on its side
        const bool sup = (am == T(0)) | (ap == T(0));
        const bool useL = (am == T(0)) | ((ap != T(0)) & (am_ >= T(0)));
        T wk[ND + 2];
#pragma unroll
        for (int v = 0; v < ND + 2; ++v) wk[v] = useL ? wl[v] : wr[v];
        const T sK = useL ? -am : ap;
        const T rK = wk[0], vK = wk[1 + Q], pK = wk[IP];
        // supersonic (s_K = 0): a middle speed equal to v_K makes the middle
        // state U_K itself, so the flux below is F_K
        const T sm = sup ? vK : am_;
        T ek;  // rho v^2 / 2
        if constexpr (ND == 1) {
            ek = T(0.5) * rK * vK * vK;
        } else {
            T kk = wk[1] * wk[1];
#pragma unroll
            for (int d = 1; d < ND; ++d) kk = fma_(wk[1 + d], wk[1 + d], kk);
            ek = T(0.5) * rK * kk;
        }
        const T EK = fma_(pK, inv_gm1, ek);
        // middle state from the jump conditions across the K-side outer wave
        // (s_K - sm is nonzero: opposite signs, or v_K != 0 when supersonic):
        // rho* = rho_K q_K / (s_K - sm), p* = p_K + rho_K q_K (sm - v_K),
        // E* = (q_K E_K - p_K v_K + p* sm) / (s_K - sm), q_K = s_K - v_K
        const T qk = sK - vK;
        const T rq = rK * qk;
        const T ps = fma_(rq, sm - vK, pK);
        // F_K + s_K (U*_K - U_K) equals the physical flux of the middle state
        // (the jump conditions across the s_K wave), formed directly: mass
        // flux rho* sm, and energy flux (E* + p*) sm = (q_K E_K - p_K v_K +
        // p* s_K) sm / (s_K - sm) (the p* sm terms cancel)
        const T ism = rcp_(sK - sm) * sm;
        const T fd = rq * ism;
        f[0] = fd;
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            if (d == Q) f[1 + d] = fma_(fd, sm, ps);
            else f[1 + d] = fd * wk[1 + d];
        }
        f[IP] = fma_(ps, sK, fma_(qk, EK, -(pK * vK))) * ism;
    }
}

// Face flux for the kernel's solver: the HLLC switch takes HLL where hll is
// set (a shock flagged along a direction transverse to this face), HLLC
// elsewhere; the other solvers ignore hll.
template <int ND, int Q, int SOLVER, typename T>
__device__ __forceinline__ void face_flux(const T (&wl)[ND + 2], const T (&wr)[ND + 2], T (&f)[ND + 2], T sg,
                                          T inv_gm1, bool hll)
{
    if constexpr (SOLVER == SOLVER_HLLC_SWITCH) {
        if (hll) riemann<ND, Q, SOLVER_HLL>(wl, wr, f, sg, inv_gm1);
        else riemann<ND, Q, SOLVER_HLLC>(wl, wr, f, sg, inv_gm1);
    } else {
        (void)hll;
        riemann<ND, Q, SOLVER>(wl, wr, f, sg, inv_gm1);
    }
}

template <typename T> __device__ __forceinline__ T sqrt_gamma(T gamma) { return sqrt(gamma); }

// ------------------------------------------------ box face fluxes ----

__device__ __forceinline__ int64_t at(const Grid &g, int i, int j, int k)
{
    return ((int64_t)k * g.m[1] + j) * g.m[0] + i;
}

template <int ND, typename T>
__device__ __forceinline__ void load_prim(const T *u, const Grid &g, int64_t c, T gm1, T (&w)[ND + 2])
{
    T uu[ND + 2];
#pragma unroll
    for (int v = 0; v < ND + 2; ++v) uu[v] = u[v * g.vs + c];
    (void)to_prim<ND>(uu, w, gm1);
}

// The faces of one box normal to Q on one side (0: low, 1: high): one
// thread per face position transverse to Q.
template <int ND, int Q, int SOLVER, typename T>
__device__ __forceinline__ void box_faces(const T *u, const Grid &g, const Box &b, int t, int side, T gamma, T gm1,
                                          T inv_gm1, T theta, double w, bool assign, double *acc_lo, double *acc_hi)
{
    constexpr int R1 = Q == 0 ? 1 : 0, R2 = Q == 2 ? 1 : 2;  // transverse dimensions, the lower one fastest
    const int faces = b.n[R1] * b.n[R2];
    if (t >= faces) return;
    const int t1 = t % b.n[R1], t2 = t / b.n[R1];
    {
        const int f = side == 0 ? b.lo[Q] : b.lo[Q] + b.n[Q];  // face between cells f - 1 and f
        // the accumulators' values under way with the cells' (read one by one
        // between the stores, each would wait for the one before)
        double *acc = side == 0 ? acc_lo : acc_hi;
        double old[ND + 2];
#pragma unroll
        for (int v = 0; v < ND + 2; ++v) old[v] = assign ? 0.0 : acc[(int64_t)v * faces + t];
        T w4[4][ND + 2];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            int c3[3];
            c3[Q] = f - 2 + s;
            c3[R1] = b.lo[R1] + t1;
            c3[R2] = b.lo[R2] + t2;
            load_prim<ND>(u, g, at(g, c3[0], c3[1], c3[2]), gm1, w4[s]);
        }
        T wl[ND + 2], wr[ND + 2], fl[ND + 2];
        const ThetaLim<T> lim = theta_lim(theta);
#pragma unroll
        for (int v = 0; v < ND + 2; ++v) {
            wl[v] = fma_(lim.hs, slope_mm(w4[0][v], w4[1][v], w4[2][v], lim.k), w4[1][v]);
            wr[v] = fma_(-lim.hs, slope_mm(w4[1][v], w4[2][v], w4[3][v], lim.k), w4[2][v]);
        }
        face_flux<ND, Q, SOLVER>(wl, wr, fl, sqrt_gamma(gamma), inv_gm1, false);
#pragma unroll
        for (int v = 0; v < ND + 2; ++v) acc[(int64_t)v * faces + t] = fma_(w, (double)fl[v], old[v]);
    }
}

}  // namespace
}  // namespace hy
