// mlp.hip -- the learned slope limiter on gfx950 matrix cores.
//
// The network (4 -> 32 -> 32 -> 1, ReLU) replaces the generalised minmod of
// eq. MinMod.  Its inputs are the four one-sided differences of a 5-cell
// stencil of one primitive variable along one dimension, divided by
// s = max|d| + 1e-12 (|w_c| + 1e-30); its output times s is clamped to the TVD
// region 0 <= sign(D) sigma <= 2 min(|D-|, |D+|) (zero where the central
// differences D-, D+ disagree in sign), so the result never leaves the region
// that contains minmod and the monotonized-central limiter.
//
// All three layers run as bf16 MFMA with FP32 accumulation; biases enter as
// the accumulator input.  One wave evaluates 64 stencils at a time, one per lane,
// in the transposed orientation H^T = W X^T so that each layer's output
// registers are already the next layer's operand layout:
//   lane l = (grp = l / 16, col = l % 16) owns stencil (batch grp, column col);
//   layer 1: for each batch g, A = W1 placed in K-group g (zeros elsewhere),
//            B = the lanes' own bf16 inputs (K-group = grp), C = b1;
//   layer 2: A = W2 (one K = 32 block per output block), B = relu(H1) as
//            bf16, C = b2;
//   layer 3: A = w3 in every row (K = 32), B = relu(H2) as bf16, C = b3, so
//            every row of the result holds the outputs and each lane reads
//            its own stencil's value without a cross-lane reduction.
// The elementwise work between the layers (ReLU and bf16 packing) bounds the
// kernel, so the third layer is put on the matrix cores rather than the
// vector ALU.
#include "hy_internal.h"
#include "hy_mlp.h"

#include <hip/hip_bf16.h>
#include <cstring>

namespace hy {

void mlp_pack(const float *flat, MlpDevice *out)
{
    std::memset(out, 0, sizeof(*out));
    const float *p = flat;
    std::memcpy(out->w1, p, sizeof(out->w1)); p += MLP_H * MLP_IN;
    std::memcpy(out->b1, p, sizeof(out->b1)); p += MLP_H;
    std::memcpy(out->w2, p, sizeof(out->w2)); p += MLP_H * MLP_H;
    std::memcpy(out->b2, p, sizeof(out->b2)); p += MLP_H;
    std::memcpy(out->w3, p, sizeof(out->w3)); p += MLP_H;
    out->b3 = *p;
}

namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ short bf(float x)
{
    __hip_bfloat16 b = __float2bfloat16(x);  // round to nearest even
    unsigned short u;
    __builtin_memcpy(&u, &b, 2);
    return (short)u;
}

// Four floats to a bf16 MFMA operand, two per conversion instruction
// (round to nearest even, element 0 in the low half).
__device__ __forceinline__ s4 bf4(float a, float b, float c, float d)
{
    const u2 w = {__builtin_bit_cast(unsigned, __builtin_convertvector((f2){a, b}, b2)),
                  __builtin_bit_cast(unsigned, __builtin_convertvector((f2){c, d}, b2))};
    return __builtin_bit_cast(s4, w);
}

// Eight floats to a K = 32 bf16 operand (lane elements jj = 0..7).
__device__ __forceinline__ b8 bf8(const s4 lo, const s4 hi)
{
    const u2 l = __builtin_bit_cast(u2, lo), h = __builtin_bit_cast(u2, hi);
    const u4 w = {l[0], l[1], h[0], h[1]};
    return __builtin_bit_cast(b8, w);
}

// The K = 32 operand of the next layer from the two output blocks of a
// 16-stencil batch: every value packed to bf16 with the conversion's output
// clamped to [0, 1], which for pre-activations of magnitude below 1 (the
// scaled network) is the ReLU of the rounded value, bit for bit: negative
// values and -0 give +0.  The inputs are results of matrix instructions, which
// a vector instruction may read only 12 wait states after they issue, and the
// outputs feed matrix instructions, which may read a vector result only 2
// after it is written; the compiler's hazard tracking does not look into
// inline assembly, so the wait states are part of it: the last 2 here, the
// first 12 once per layer in results_settle.
__device__ __forceinline__ b8 relu_pack_clamped(const f4 lo, const f4 hi)
{
    unsigned r0, r1, r2, r3;
    asm volatile("v_cvt_pk_bf16_f32 %0, %4, %5 clamp\n\t"
                 "v_cvt_pk_bf16_f32 %1, %6, %7 clamp\n\t"
                 "v_cvt_pk_bf16_f32 %2, %8, %9 clamp\n\t"
                 "v_cvt_pk_bf16_f32 %3, %10, %11 clamp\n\t"
                 "s_nop 1"
                 : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3)
                 : "v"(lo[0]), "v"(lo[1]), "v"(lo[2]), "v"(lo[3]), "v"(hi[0]), "v"(hi[1]), "v"(hi[2]), "v"(hi[3]));
    const u4 w = {r0, r1, r2, r3};
    return __builtin_bit_cast(b8, w);
}

// Every matrix instruction above is issued above, everything below is issued
// below, and 12 wait states lie between them: 48 cycles that a wavefront spends
// once per layer (once per batch of 16 stencils they were a third of the
// network's latency: 1040 -> 950 us for the slopes of 256^3).
__device__ __forceinline__ void results_settle()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 11");
    __builtin_amdgcn_sched_barrier(0);
}

// Layer 2 runs as one K = 32 product per output block (v_mfma_f32_16x16x32_bf16:
// lane (grp, col) holds A[col][8 grp + jj] and B[8 grp + jj][col], jj = 0..7).
// Its K order is permuted so that B is exactly what layer 1 left in the lane:
// K index 8 grp + jj stands for hidden unit hk(grp, jj) = 4 grp + jj (jj < 4)
// or 16 + 4 grp + jj - 4 (jj >= 4), the units of both layer-1 output blocks.
// Layer 3 uses the same K permutation, with w3 replicated over the 16 rows.
struct MlpRegs {
    s4 a1[4][2];  // layer-1 weights placed in K-group g, per output block
    f4 c1[2];     // b1 as accumulator input
    b8 a2[2];     // layer-2 weights [out block], K permuted as above
    f4 c2[2];     // b2 as accumulator input
    b8 a3;        // w3, K permuted as above, the same in every row
    f4 c3;        // b3 as accumulator input
};

__device__ __forceinline__ float bf_value(float x)
{
    const unsigned u = (unsigned)(unsigned short)bf(x) << 16;
    return __uint_as_float(u);
}

// k with 2^k > 2 max(B1, B2), B1 = max_m sum_j |bf16(W1[m][j])| + |b1[m]|
// (inputs lie in [-1, 1]) and B2 = max_m sum_j |bf16(W2[m][j])| B1 + |b2[m]|
// (0 <= h1 <= B1): then every pre-activation times 2^-k lies in [-1/2, 1/2]
// (the factor 2 covers the FP32 accumulation and bf16 rounding).
__device__ __forceinline__ int mlp_upscale(const MlpDevice *m)
{
    float b1 = 0.f, b2 = 0.f;
    for (int r = 0; r < MLP_H; ++r) {
        float a = fabsf(m->b1[r]);
        for (int j = 0; j < MLP_IN; ++j) a += fabsf(bf_value(m->w1[r][j]));
        b1 = fmaxf(b1, a);
    }
    for (int r = 0; r < MLP_H; ++r) {
        float a = 0.f;
        for (int j = 0; j < MLP_H; ++j) a += fabsf(bf_value(m->w2[r][j]));
        b2 = fmaxf(b2, a * b1 + fabsf(m->b2[r]));
    }
    int e = 0;
    (void)frexpf(2.f * fmaxf(b1, b2), &e);  // 2 max(B1, B2) < 2^e
    return e < 0 ? 0 : e;
}

// The lane's operands of the network scaled by 2^-k (k = mlp_upscale): W1
// and every bias times 2^-k (exact: a power of two), W2 and w3 as they are.
__device__ __forceinline__ void load_regs(const MlpDevice *m, int grp, int col, int k, MlpRegs &R)
{
    const float dn = ldexpf(1.f, -k);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int j = 0; j < 4; ++j) R.a1[g][mb][j] = grp == g ? bf(m->w1[16 * mb + col][j] * dn) : (short)0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            R.c1[mb][j] = m->b1[16 * mb + 4 * grp + j] * dn;
            R.c2[mb][j] = m->b2[16 * mb + 4 * grp + j] * dn;
        }
        const float *w2r = m->w2[16 * mb + col];
        R.a2[mb] = bf8(bf4(w2r[4 * grp], w2r[4 * grp + 1], w2r[4 * grp + 2], w2r[4 * grp + 3]),
                       bf4(w2r[16 + 4 * grp], w2r[17 + 4 * grp], w2r[18 + 4 * grp], w2r[19 + 4 * grp]));
    }
    const float *w3 = m->w3;
    R.a3 = bf8(bf4(w3[4 * grp], w3[4 * grp + 1], w3[4 * grp + 2], w3[4 * grp + 3]),
               bf4(w3[16 + 4 * grp], w3[17 + 4 * grp], w3[18 + 4 * grp], w3[19 + 4 * grp]));
#pragma unroll
    for (int j = 0; j < 4; ++j) R.c3[j] = m->b3 * dn;
}

static_assert(sizeof(MlpRegs) == sizeof(uint4) * 12, "lane image layout");

// Network output for the lane's own input x[0..3] (all 64 lanes must be active,
// and every lane's input finite: 0 x inf in a zero block of an operand would
// spread a NaN to the other lanes of the same column).
// The four 16-stencil batches are independent: a layer's products of one batch
// run under the packing of the next one.
// Returns the output of the scaled network (the true output times 1 / up).
__device__ __forceinline__ float mlp_wave(const float (&x)[4], const MlpRegs &R)
{
    const s4 xb = bf4(x[0], x[1], x[2], x[3]);
    f4 d1[4][2];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
            d1[g][mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(R.a1[g][mb], xb, R.c1[mb], 0, 0, 0);
    results_settle();
    f4 d2[4][2];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const b8 h = relu_pack_clamped(d1[g][0], d1[g][1]);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
            d2[g][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(R.a2[mb], h, R.c2[mb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    results_settle();
    f4 d3[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const b8 h = relu_pack_clamped(d2[g][0], d2[g][1]);
        d3[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(R.a3, h, R.c3, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    // the unused elements stay allocated until here: a conversion above must
    // not be given a register that a product in flight still writes
    asm volatile("" ::"v"(d3[0]), "v"(d3[1]), "v"(d3[2]), "v"(d3[3]));
    int part[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) part[g] = __float_as_int(d3[g][0]);
    // lane group g takes batch g's value: moves that write one row of 16 lanes
    int y = part[0];
    y = __builtin_amdgcn_update_dpp(y, part[1], 0xe4, 0x2, 0xf, false);
    y = __builtin_amdgcn_update_dpp(y, part[2], 0xe4, 0x4, 0xf, false);
    y = __builtin_amdgcn_update_dpp(y, part[3], 0xe4, 0x8, 0xf, false);
    return __int_as_float(y);
}

// sigma from the 5-cell stencil w[0..4] (centre w[2]); up as in MlpImage
__device__ __forceinline__ float learned_sigma(const float (&w)[5], const MlpRegs &R, float up)
{
    float d[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) d[k] = w[k + 1] - w[k];
    const float s = fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fmaxf(fabsf(d[2]), fabsf(d[3]))) +
                    1e-12f * (fabsf(w[2]) + 1e-30f);
    // The floor term alone (a flat stencil of zeros) is below the FP32 normal
    // range, and 1/s would overflow; every input must stay finite because a
    // NaN or infinite input of one lane reaches the other lanes of its column
    // through the zero blocks of the matrix operands.  Inputs are unchanged
    // wherever s is a normal number and exact zeros for a flat stencil.
    const float rs = __builtin_amdgcn_rcpf(fmaxf(s, 1.17549435e-38f));  // 1 ulp
    float x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = d[k] * rs;
    const float sigma = s * (mlp_wave(x, R) * up);  // the product with up is exact
    // zero, or between zero and twice the smaller difference where their signs agree
    const float m = __builtin_amdgcn_fmed3f(d[1], d[2], 0.f);
    return __builtin_amdgcn_fmed3f(sigma, m + m, 0.f);
}

struct Bc {
    int v[3][2];
};

__device__ __forceinline__ int64_t map1(int64_t i, int64_t n, int lo, int hi, bool &flip)
{
    if (i >= 0 && i < n) return i;
    int64_t m;
    if (i < 0) {
        if (lo == BC_PERIODIC) m = i + n;
        else if (lo == BC_OUTFLOW) m = 0;
        else { m = -1 - i; flip = !flip; }
    } else {
        if (hi == BC_PERIODIC) m = i - n;
        else if (hi == BC_OUTFLOW) m = n - 1;
        else { m = 2 * n - 1 - i; flip = !flip; }
    }
    return m < 0 ? 0 : (m >= n ? n - 1 : m);
}

// One cell's primitives from its conserved values.
template <int ND>
__device__ __forceinline__ void prims(const float (&uu)[ND + 2], float gm1, float (&w)[ND + 2])
{
    float ir = __builtin_amdgcn_rcpf(uu[0]);
    ir = fmaf(fmaf(-uu[0], ir, 1.f), ir, ir);  // to the last bit, as a division gives
    float ke = 0.f;
    w[0] = uu[0];
#pragma unroll
    for (int d = 0; d < ND; ++d) {
        w[1 + d] = uu[1 + d] * ir;
        ke += uu[1 + d] * w[1 + d];
    }
    w[ND + 1] = gm1 * (uu[ND + 1] - 0.5f * ke);
}

template <int ND>
__device__ __forceinline__ void load_cell(const float *u, int64_t vs, unsigned cell, float (&uu)[ND + 2])
{
#pragma unroll
    for (int v = 0; v < ND + 2; ++v) uu[v] = *(const float *)((const char *)(u + v * vs) + cell * 4u);
}

template <int ND>
__device__ __forceinline__ void store_slope(float *slopes, int64_t svs, int qv, unsigned cell, float sg)
{
    // a variable's slope array is below 4 GiB (checked on the host): 32-bit
    // byte offsets from its (wave-uniform) base
    *(float *)((char *)(slopes + (int64_t)qv * svs) + cell * 4u) = sg;
}

// Slopes along Q, and with XS along x in the same pass.  A wavefront owns 64
// consecutive cells of the plane across Q (2D: of a row; 3D: of the plane's
// cells numbered x first, so that no lane idles at the end of a row) and
// marches along Q over R rows with the five rows of the stencil in registers:
// each cell is read and converted once per pass (and 4 more per R), the next
// row's loads are under way during the networks of this one, and no wavefront
// waits for another.  The x stencils come from a 68-cell line of the row in LDS,
// private to the wavefront; at the ends of a row of cells the two neighbours
// beyond are fetched by the lane itself (on both sides where a row has fewer
// than 4 cells: NARROW); where a lane's five cells lie in LDS is fixed for the
// march.
//
// What bounds it: the matrix and the vector units, which take turns more than
// they overlap at 3 wavefronts per SIMD: 330 cycles of products and about 290
// of vector work per network and wavefront, 590 measured.  Tiles of 16 rows in
// LDS, one launch per dimension with a barrier between conversion and networks,
// took 54 us for 1024^2 (now 42), 26 for 256^2 (6.7), 254 for 150 x 120 x 160
// (180) and 1083 for 256^3 (935).
template <int ND, int Q, bool XS, bool NARROW>
__global__ void __launch_bounds__(256)
    k_slopes_march(const float *__restrict__ u, float *__restrict__ slopes, int nx, int ny, int nz, int R, int nseg,
                   int ntask, int64_t vs, int64_t svs, float gm1, Bc bc, const MlpImage *__restrict__ img)
{
    constexpr int NP = ND + 2, NE = NARROW ? 4 : 2;
    __shared__ float sL[XS ? 4 : 1][NP][68 + 64 * NE];  // the line, then what each lane fetched beyond its ends
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task = blockIdx.x * 4 + wv;
    if (task >= ntask) return;
    MlpRegs M;
    __builtin_memcpy(&M, &img->lane[lane][0], sizeof(M));
    const float up = img->up;
    const int chunk = task / nseg, f0 = (task - chunk * nseg) * 64;
    const int nf = ND == 2 ? nx : (Q == 2 ? nx * ny : nx * nz);
    const int nq = Q == 1 ? ny : nz;
    const unsigned sq = Q == 1 ? (unsigned)nx : (unsigned)nx * (unsigned)ny;
    const int j0 = chunk * R, j1 = min(j0 + R, nq);
    const unsigned f = (unsigned)min(f0 + lane, nf - 1);
    unsigned c0 = f;  // the lane's cell in row 0
    if constexpr (ND == 3 && Q == 1) {
        const unsigned z = f / (unsigned)nx;
        c0 = z * (unsigned)nx * (unsigned)ny + (f - z * (unsigned)nx);
    }

    // x stencils: the line's ends (lanes 0 .. 3) and the row's, and where the
    // lane finds its five cells
    unsigned ch = 0, ce[NE] = {};
    float fl[NE] = {};
    int at[5] = {};
    bool edge = false;
    if constexpr (XS) {
        ch = (unsigned)min(max(lane < 2 ? f0 - 2 + lane : f0 + 62 + (lane & 3), 0), nf - 1);
        const int x = ND == 2 ? (int)f : (int)(f % (unsigned)nx);
        const bool lo = x < 2, hi = x >= nx - 2;
        edge = lo || hi;
#pragma unroll
        for (int k = 0; k < 5; ++k) at[k] = (int)f - f0 + k;
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int side = NARROW ? (e < 2 ? -1 : 1) : (lo ? -1 : 1), d = 1 + (e & 1);
            bool flip = false;
            const int xe = edge ? (int)map1(x + side * d, nx, bc.v[0][0], bc.v[0][1], flip) : x;
            ce[e] = f - (unsigned)x + (unsigned)xe;
            fl[e] = flip ? -1.f : 1.f;
            if (side < 0 ? lo : hi) at[side < 0 ? 2 - d : 2 + d] = 68 + 64 * e + lane;
        }
    }

    auto row = [&](int j, bool &flip) {  // offset of row j (mapped into the patch)
        return (unsigned)map1(j, nq, bc.v[Q][0], bc.v[Q][1], flip) * sq;
    };
    float W[5][NP], raw[NP];
    bool flipn = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        bool flip = false;
        load_cell<ND>(u, vs, c0 + row(j0 - 2 + k, flip), raw);
        prims<ND>(raw, gm1, W[k + 1]);
        if (flip) W[k + 1][1 + Q] = -W[k + 1][1 + Q];
    }
    load_cell<ND>(u, vs, c0 + row(j0 + 2, flipn), raw);
    for (int j = j0; j < j1; ++j) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < NP; ++v) W[k][v] = W[k + 1][v];
        prims<ND>(raw, gm1, W[4]);
        if (flipn) W[4][1 + Q] = -W[4][1 + Q];
        const unsigned cell = c0 + (unsigned)j * sq;
        if constexpr (XS) {
            float (*ln)[68 + 64 * NE] = sL[wv];
            const unsigned o = (unsigned)j * sq;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (the last row's reads)
            if (edge)
#pragma unroll
                for (int e = 0; e < NE; ++e) {
                    float re[NP], we[NP];
                    load_cell<ND>(u, vs, ce[e] + o, re);
                    prims<ND>(re, gm1, we);
                    we[1] *= fl[e];
#pragma unroll
                    for (int v = 0; v < NP; ++v) ln[v][68 + 64 * e + lane] = we[v];
                }
            if (lane < 4) {
                float rh[NP], wh[NP];
                load_cell<ND>(u, vs, ch + o, rh);
                prims<ND>(rh, gm1, wh);
#pragma unroll
                for (int v = 0; v < NP; ++v) ln[v][lane < 2 ? lane : 64 + lane] = wh[v];
            }
#pragma unroll
            for (int v = 0; v < NP; ++v) ln[v][lane + 2] = W[2][v];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        flipn = false;
        load_cell<ND>(u, vs, c0 + row(j + 3, flipn), raw);
#pragma unroll
        for (int v = 0; v < NP; ++v) {
            const float w5[5] = {W[0][v], W[1][v], W[2][v], W[3][v], W[4][v]};
            store_slope<ND>(slopes, svs, Q * NP + v, cell, learned_sigma(w5, M, up));
        }
        if constexpr (XS)
#pragma unroll
            for (int v = 0; v < NP; ++v) {
                float w5[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) w5[k] = sL[wv][v][at[k]];
                store_slope<ND>(slopes, svs, v, cell, learned_sigma(w5, M, up));
            }
    }
}

// 1D: 64 cells and two more on each side per wavefront, in LDS.
__global__ void __launch_bounds__(64)
    k_slopes_1d(const float *__restrict__ u, float *__restrict__ slopes, int nx, int64_t vs, int64_t svs, float gm1,
                Bc bc, const MlpImage *__restrict__ img)
{
    __shared__ float sW[3][68];
    const int lane = threadIdx.x, x0 = blockIdx.x * 64;
    MlpRegs M;
    __builtin_memcpy(&M, &img->lane[lane][0], sizeof(M));
    const float up = img->up;
    for (int c = lane; c < 68; c += 64) {
        bool flip = false;
        const unsigned cell = (unsigned)map1(x0 - 2 + c, nx, bc.v[0][0], bc.v[0][1], flip);
        float uu[3], w[3];
        load_cell<1>(u, vs, cell, uu);
        prims<1>(uu, gm1, w);
        sW[0][c] = w[0];
        sW[1][c] = flip ? -w[1] : w[1];
        sW[2][c] = w[2];
    }
    __syncthreads();
    for (int v = 0; v < 3; ++v) {
        float w5[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) w5[k] = sW[v][lane + k];
        const float sg = learned_sigma(w5, M, up);
        if (x0 + lane < nx) store_slope<1>(slopes, svs, v, (unsigned)(x0 + lane), sg);
    }
}

// Rows per wavefront of the marching kernel: what gives 3 wavefronts to each
// of the 1024 SIMDs (as many as the registers allow), at most 8.  Fewer rows
// mean four extra rows read and converted for fewer results, more rows a longer
// serial chain: 256^2 takes 6.7 us at 1 row and 15.1 at 4, 64^3 27 at 2 and
// 31 at 4, 1024^2 49 at 1, 42 at 4 and 43 at 8, 256^3 955 at 4 and 935 at 8,
// 2048^2 131 at 4, 133 at 8 and 165 at 16.
int march_rows(int64_t nseg, int nq)
{
    const int64_t r = (nseg * nq + 3071) / 3072;
    return (int)(r < 1 ? 1 : (r > 8 ? 8 : r));
}

template <int ND, int Q, bool XS, bool NARROW>
void march_launch(const float *u, float *slopes, int nx, int ny, int nz, int64_t vs, int64_t svs, float gm1,
                  const Bc &b, const MlpImage *img, hipStream_t s)
{
    const int64_t nf = ND == 2 ? nx : (Q == 2 ? (int64_t)nx * ny : (int64_t)nx * nz);
    const int nq = Q == 1 ? ny : nz;
    const int64_t nseg = (nf + 63) / 64;
    const int R = march_rows(nseg, nq);
    const int64_t ntask = nseg * ((nq + R - 1) / R);
    hipLaunchKernelGGL((k_slopes_march<ND, Q, XS, NARROW>), dim3((unsigned)((ntask + 3) / 4)), dim3(256), 0, s, u,
                       slopes, nx, ny, nz, R, (int)nseg, (int)ntask, vs, svs, gm1, b, img);
}

__global__ void __launch_bounds__(64) k_mlp_image(const MlpDevice *__restrict__ mlp, MlpImage *__restrict__ img)
{
    const int lane = threadIdx.x, grp = lane >> 4, col = lane & 15;
    const int k = mlp_upscale(mlp);
    MlpRegs R;
    load_regs(mlp, grp, col, k, R);
    __builtin_memcpy(&img->lane[lane][0], &R, sizeof(R));
    if (lane == 0) img->up = ldexpf(1.f, k);
}

__global__ void __launch_bounds__(256) k_mlp_forward(const MlpDevice *__restrict__ mlp, const float *__restrict__ x,
                                                     float *__restrict__ y, int64_t batch)
{
    const int lane = threadIdx.x & 63, grp = lane >> 4, col = lane & 15;
    const int k = mlp_upscale(mlp);
    const float up = ldexpf(1.f, k);
    MlpRegs R;
    load_regs(mlp, grp, col, k, R);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t ii = i < batch ? i : batch - 1;
    const float xi[4] = {x[4 * ii], x[4 * ii + 1], x[4 * ii + 2], x[4 * ii + 3]};
    const float out = mlp_wave(xi, R) * up;
    if (i < batch) y[i] = out;
}

}  // namespace

hipError_t launch_learned_slopes(const float *u, float *slopes, const int64_t n[3], int64_t vstride, int64_t svs,
                                 int ndim, float gm1, const int bc[3][2], const MlpImage *img, hipStream_t s)
{
    Bc b;
    for (int q = 0; q < 3; ++q) {
        b.v[q][0] = bc[q][0];
        b.v[q][1] = bc[q][1];
    }
    const int nx = (int)n[0], ny = (int)n[1], nz = (int)n[2];
    if (ndim == 1) {
        hipLaunchKernelGGL(k_slopes_1d, dim3((unsigned)((nx + 63) / 64)), dim3(64), 0, s, u, slopes, nx, vstride, svs,
                           gm1, b, img);
    } else if (ndim == 2) {
        if (nx < 4) march_launch<2, 1, true, true>(u, slopes, nx, ny, nz, vstride, svs, gm1, b, img, s);
        else march_launch<2, 1, true, false>(u, slopes, nx, ny, nz, vstride, svs, gm1, b, img, s);
    } else {
        if (nx < 4) march_launch<3, 2, true, true>(u, slopes, nx, ny, nz, vstride, svs, gm1, b, img, s);
        else march_launch<3, 2, true, false>(u, slopes, nx, ny, nz, vstride, svs, gm1, b, img, s);
        march_launch<3, 1, false, false>(u, slopes, nx, ny, nz, vstride, svs, gm1, b, img, s);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_image(const MlpDevice *mlp, MlpImage *img, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_image, dim3(1), dim3(64), 0, s, mlp, img);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpDevice *mlp, const float *x, float *y, int64_t batch, hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0, s, mlp, x, y, batch);
    return hipGetLastError();
}

}  // namespace hy
