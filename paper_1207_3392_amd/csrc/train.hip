// train.hip -- training the learned slope limiter on gfx950.
//
// Data: a fine run of the plain method is restricted to a grid four times
// coarser (the averaging of the restriction step, 4^d fine cells per coarse
// cell).  Each (coarse cell, primitive variable, dimension) gives one sample:
// the network inputs are the normalised one-sided differences of the 5-cell
// coarse stencil, and the target is the least-squares slope of the four fine
// sub-cell averages along the dimension (positions -3/8, -1/8, 1/8, 3/8 of the
// coarse cell, slope 0.4 (-3 w1 - w2 + w3 + 3 w4)), clamped to the TVD
// region and divided by the same normalisation s.
//
// Step: each wavefront takes tiles of 64 samples and runs the network forward
// and backward on the matrix cores (weights and activations in bfloat16,
// accumulation in FP32), accumulating its share of the gradient of the mean
// squared error in FP32; a second kernel adds the workgroup partials in a
// fixed order and applies Adam to the FP32 master weights.
#include "hy_internal.h"
#include "hy_mlp.h"
#include "hy_train.h"

#include <hip/hip_bf16.h>

#include <cmath>
#include <mutex>

namespace hy {
namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------ data ----

// U: conserved fine state (nv vars, stride vs), nf = fine cells per dim;
// out: coarse primitives (nv, nc) and, per dim q, the four sub-cell slab
// averages of each primitive (q, v, 4, nc) for the target slopes.
template <int ND>
__global__ void __launch_bounds__(256) k_coarsen4(const float *__restrict__ U, int64_t vs, int nfx, int nfy, int nfz,
                                                  float gm1, float *__restrict__ Wc, float *__restrict__ sub,
                                                  int64_t nc)
{
    constexpr int NP = ND + 2;
    const int ncx = nfx / 4, ncy = ND >= 2 ? nfy / 4 : 1, ncz = ND == 3 ? nfz / 4 : 1;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= nc) return;
    const int cx = (int)(c % ncx), cy = (int)((c / ncx) % ncy), cz = (int)(c / ((int64_t)ncx * ncy));
    constexpr int KY = ND >= 2 ? 4 : 1, KZ = ND == 3 ? 4 : 1;
    constexpr float inv = 1.0f / (4 * KY * KZ);
    // restriction: averages of the conserved (balanced) variables over the
    // coarse cell and over each quarter slab along every dimension, then the
    // primitives of those averages
    float acc[NP] = {};
    float slab[3][4][NP] = {};
    for (int kz = 0; kz < KZ; ++kz)
        for (int ky = 0; ky < KY; ++ky)
            for (int kx = 0; kx < 4; ++kx) {
                const int64_t f = ((int64_t)(cz * KZ + kz) * nfy + (cy * KY + ky)) * nfx + (cx * 4 + kx);
#pragma unroll
                for (int v = 0; v < NP; ++v) {
                    const float u = U[f + v * vs];
                    acc[v] += u;
                    slab[0][kx][v] += u;
                    if (ND >= 2) slab[1][ky][v] += u;
                    if (ND == 3) slab[2][kz][v] += u;
                }
            }
    auto prim = [&](const float (&u)[NP], float sc, float (&w)[NP]) {
        float uu[NP];
#pragma unroll
        for (int v = 0; v < NP; ++v) uu[v] = u[v] * sc;
        const float ir = 1.0f / uu[0];
        float ke = 0.f;
        w[0] = uu[0];
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            w[1 + d] = uu[1 + d] * ir;
            ke += uu[1 + d] * w[1 + d];
        }
        w[NP - 1] = gm1 * (uu[NP - 1] - 0.5f * ke);
    };
    float w[NP];
    prim(acc, inv, w);
#pragma unroll
    for (int v = 0; v < NP; ++v) Wc[v * nc + c] = w[v];
    const float sinv = 4.0f * inv;  // each slab holds a quarter of the fine cells
#pragma unroll
    for (int q = 0; q < ND; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            prim(slab[q][k], sinv, w);
#pragma unroll
            for (int v = 0; v < NP; ++v) sub[((int64_t)(q * NP + v) * 4 + k) * nc + c] = w[v];
        }
}

// samples from the coarse primitives (periodic coarse grid): x (nsamp, 4),
// target t (nsamp); sample index = (q * NP + v) * nc + c
template <int ND>
__global__ void __launch_bounds__(256) k_samples(const float *__restrict__ Wc, const float *__restrict__ sub, int ncx,
                                                 int ncy, int ncz, float *__restrict__ x, float *__restrict__ t)
{
    constexpr int NP = ND + 2;
    const int64_t nc = (int64_t)ncx * ncy * ncz;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nc * NP * ND) return;
    const int64_t c = i % nc;
    const int qv = (int)(i / nc);
    const int q = qv / NP, v = qv % NP;
    const int cx = (int)(c % ncx), cy = (int)((c / ncx) % ncy), cz = (int)(c / ((int64_t)ncx * ncy));
    float w[5];
    for (int s = 0; s < 5; ++s) {
        int p[3] = {cx, cy, cz};
        const int nn[3] = {ncx, ncy, ncz};
        p[q] = ((p[q] + s - 2) % nn[q] + nn[q]) % nn[q];
        w[s] = Wc[v * nc + ((int64_t)p[2] * ncy + p[1]) * ncx + p[0]];
    }
    float d[4];
    for (int k = 0; k < 4; ++k) d[k] = w[k + 1] - w[k];
    // s as in the limiter; the division uses s raised to the smallest normal
    // FP32 number, so a flat stencil of zeros gives x = t = 0, not 0/0
    const float s = fmaxf(fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fmaxf(fabsf(d[2]), fabsf(d[3]))) +
                              1e-12f * (fabsf(w[2]) + 1e-30f),
                          1.17549435e-38f);
    for (int k = 0; k < 4; ++k) x[i * 4 + k] = d[k] / s;
    const float *sb = sub + (int64_t)(q * NP + v) * 4 * nc;
    const float w1 = sb[c], w2 = sb[nc + c], w3 = sb[2 * nc + c], w4 = sb[3 * nc + c];
    float sg = 0.4f * (-3.f * w1 - w2 + w3 + 3.f * w4);
    const float dm = d[1], dp = d[2];
    const float sgn = dp > 0.f ? 1.f : -1.f;
    sg = (dm * dp > 0.f) ? sgn * fminf(fmaxf(sgn * sg, 0.f), 2.f * fminf(fabsf(dm), fabsf(dp))) : 0.f;
    t[i] = sg / s;
}

// ------------------------------------------------------------ step ----

constexpr int TS = 64;         // samples per wave tile
constexpr int H = MLP_H;       // 32

typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));

// two floats to bfloat16 (round to nearest even), the first in the low half
__device__ __forceinline__ unsigned pk(float a, float b)
{
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f2){a, b}, b2));
}
__device__ __forceinline__ u2 pk4(const f4 v) { return (u2){pk(v[0], v[1]), pk(v[2], v[3])}; }
__device__ __forceinline__ u2 pk4_relu(const f4 v)
{
    return (u2){pk(fmaxf(v[0], 0.f), fmaxf(v[1], 0.f)), pk(fmaxf(v[2], 0.f), fmaxf(v[3], 0.f))};
}
__device__ __forceinline__ b8 op8(const u2 lo, const u2 hi)
{
    return __builtin_bit_cast(b8, (u4){lo[0], lo[1], hi[0], hi[1]});
}

// x rounded to the nearest bfloat16 (ties to even), as a float: the third
// layer's operands, which the inference kernel feeds to the matrix cores
__device__ __forceinline__ float bfr(float x) { return __bfloat162float(__float2bfloat16(x)); }

__device__ __forceinline__ f4 mfma16(u2 a, u2 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, a), __builtin_bit_cast(s4, b), c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma32(b8 a, b8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f4 splat(float x) { return (f4){x, x, x, x}; }

// The gradient of the mean squared error over the batch: per-workgroup partial
// sums.  A wave takes 64 samples, lane (grp = lane / 16, col = lane % 16)
// owning sample 16 grp + col.  Every layer is evaluated twice on the matrix
// cores, with the operands swapped: once with the units along the result's
// rows (a lane holds 4 units of one sample: what the next layer and the
// backward product through W2 take as an operand) and once with the samples
// along the rows (a lane holds 4 samples of one unit: what the weight
// gradients, contractions over the samples, take as operands).  So nothing is
// transposed, activations stay in registers, and only the samples and targets
// go through LDS, within the wavefront.  K = 32 operands: K index 8 grp + jj
// stands for unit 4 grp + jj (jj < 4) or 16 + 4 grp + jj - 4, and in the
// weight gradients for those samples of two 16-sample batches.
//
// What bounds it: the latency of one wavefront's chain (gather, 64 matrix
// instructions, about 600 vector ones) under the weights' load, one tile per
// wavefront up to 65,536 samples, so four wavefronts per workgroup and as many
// workgroups as there are rows of partial sums.  65,536 samples: 18.3 -> 10.0 us
// per launch against operands staged element by element in LDS between seven
// workgroup barriers; a step with the sum below 23.5 -> 11.0 us.
constexpr int TW = TRAIN_WAVES;

__global__ void __launch_bounds__(64 * TW) k_train_grad(const MlpDevice *__restrict__ m, const float *__restrict__ x,
                                                        const float *__restrict__ t, const int *__restrict__ idx,
                                                        int64_t batch, float inv_batch, float *__restrict__ partial,
                                                        float *__restrict__ loss_partial)
{
    __shared__ float sg[TW][MLP_NPARAM + 3];
    __shared__ __align__(16) unsigned short sX[TW][MLP_IN][TS];  // the tile's inputs, bf16
    __shared__ __align__(16) float sT[TW][TS];     // and targets
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, grp = lane >> 4, col = lane & 15;
    const int64_t ntile = (batch + TS - 1) / TS;
    float xs[MLP_IN], ts;
    auto gather = [&](int64_t si) {
        xs[0] = xs[1] = xs[2] = xs[3] = ts = 0.f;
        if (si < batch) {
            const int64_t s = (int64_t)idx[si];
            __builtin_memcpy(xs, x + s * 4, sizeof(xs));
            ts = t[s];
        }
    };
    int64_t tile = (int64_t)blockIdx.x * TW + wv;
    gather(tile * TS + lane);  // two dependent fetches, under way while the weights arrive

    // the network as this lane's operands
    u2 w1v[2];
    b8 a2[2], a2t[2], a3;
    f4 c1[2], c2[2], w3a[2];
    float c1t[2], c2t[2], w3b[2];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
        const float *r = m->w1[16 * mb + col];
        w1v[mb] = (u2){pk(r[0], r[1]), pk(r[2], r[3])};
        const float *w = m->w2[16 * mb + col];
        a2[mb] = op8((u2){pk(w[4 * grp], w[4 * grp + 1]), pk(w[4 * grp + 2], w[4 * grp + 3])},
                     (u2){pk(w[16 + 4 * grp], w[17 + 4 * grp]), pk(w[18 + 4 * grp], w[19 + 4 * grp])});
        f4 lo, hi;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            lo[jj] = m->w2[4 * grp + jj][16 * mb + col];
            hi[jj] = m->w2[16 + 4 * grp + jj][16 * mb + col];
            c1[mb][jj] = m->b1[16 * mb + 4 * grp + jj];
            c2[mb][jj] = m->b2[16 * mb + 4 * grp + jj];
            w3a[mb][jj] = bfr(m->w3[16 * mb + 4 * grp + jj]);
        }
        a2t[mb] = op8(pk4(lo), pk4(hi));
        c1t[mb] = m->b1[16 * mb + col];
        c2t[mb] = m->b2[16 * mb + col];
        w3b[mb] = bfr(m->w3[16 * mb + col]);
    }
    a3 = op8(pk4(w3a[0]), pk4(w3a[1]));  // (already bf16 values)
    const float b3 = m->b3;

    f4 gW2[2][2] = {}, gW1[2] = {};
    float gb1[2] = {}, gb2[2] = {}, gw3[2] = {}, gb3 = 0.f, lsum = 0.f;
    for (; tile < ntile; tile += (int64_t)gridDim.x * TW) {
        const int nvalid = batch - tile * TS < TS ? (int)(batch - tile * TS) : TS;
        const u2 xb = {pk(xs[0], xs[1]), pk(xs[2], xs[3])};
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (the last tile's reads)
        sX[wv][0][lane] = (unsigned short)xb[0];
        sX[wv][1][lane] = (unsigned short)(xb[0] >> 16);
        sX[wv][2][lane] = (unsigned short)xb[1];
        sX[wv][3][lane] = (unsigned short)(xb[1] >> 16);
        sT[wv][lane] = ts;
        gather((tile + (int64_t)gridDim.x * TW) * TS + lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        b8 dz2s[4];              // dZ2, 4 units of a sample: backward operand
        u2 h1p[4][2], dz2p[4][2], dz1p[4][2];  // H1, dZ2, dZ1, 4 samples of a unit: gradient operands
        f4 e1[4][2];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u2 a1[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) a1[mb] = grp == g ? w1v[mb] : (u2){0u, 0u};
            const b8 h1 = op8(pk4_relu(mfma16(a1[0], xb, c1[0])), pk4_relu(mfma16(a1[1], xb, c1[1])));
            f4 d2[2], e2[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                e1[g][mb] = mfma16(xb, a1[mb], splat(c1t[mb]));
                d2[mb] = mfma32(a2[mb], h1, c2[mb]);
                e2[mb] = mfma32(h1, a2[mb], splat(c2t[mb]));
                h1p[g][mb] = pk4_relu(e1[g][mb]);
            }
            const b8 h2 = op8(pk4_relu(d2[0]), pk4_relu(d2[1]));
            const float y1 = mfma32(a3, h2, splat(b3))[0];  // sample 16 g + col
            const f4 y2 = mfma32(h2, a3, splat(b3));        // samples 16 g + 4 grp + jj
            const float r1 = 16 * g + col < nvalid ? y1 - sT[wv][16 * g + col] : 0.f;
            if (grp == g) lsum += r1 * r1;
            const float dy1 = 2.f * r1 * inv_batch;
            const f4 t2 = *(const f4 *)&sT[wv][16 * g + 4 * grp];
            f4 dy2;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                dy2[jj] = 16 * g + 4 * grp + jj < nvalid ? 2.f * (y2[jj] - t2[jj]) * inv_batch : 0.f;
                gb3 += dy2[jj];
            }
            f4 q[2];
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                f4 p;
                const u2 h2p = pk4_relu(e2[mb]);
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    q[mb][jj] = d2[mb][jj] > 0.f ? dy1 * w3a[mb][jj] : 0.f;
                    p[jj] = e2[mb][jj] > 0.f ? dy2[jj] * w3b[mb] : 0.f;
                    gb2[mb] += p[jj];
                    const unsigned hw = h2p[jj >> 1];
                    gw3[mb] += dy2[jj] * __uint_as_float((jj & 1) ? hw & 0xffff0000u : hw << 16);
                }
                dz2p[g][mb] = pk4(p);
            }
            dz2s[g] = op8(pk4(q[0]), pk4(q[1]));
        }
        // dH1 = dZ2 W2, dZ1 = dH1 (Z1 > 0)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                f4 d = mfma32(dz2s[g], a2t[nb], splat(0.f));
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    d[jj] = e1[g][nb][jj] > 0.f ? d[jj] : 0.f;
                    gb1[nb] += d[jj];
                }
                dz1p[g][nb] = pk4(d);
            }
        // g_W2 = dZ2^T H1, g_W1 = dZ1^T X over two batches of 16 samples each
#pragma unroll
        for (int P = 0; P < 2; ++P) {
            u2 x0 = {0u, 0u}, x1 = {0u, 0u};
            if (col < MLP_IN) {
                x0 = *(const u2 *)&sX[wv][col][32 * P + 4 * grp];
                x1 = *(const u2 *)&sX[wv][col][32 * P + 16 + 4 * grp];
            }
            const b8 xo = op8(x0, x1);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) {
                const b8 za = op8(dz2p[2 * P][mb], dz2p[2 * P + 1][mb]);
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    gW2[mb][nb] = mfma32(za, op8(h1p[2 * P][nb], h1p[2 * P + 1][nb]), gW2[mb][nb]);
                gW1[mb] = mfma32(op8(dz1p[2 * P][mb], dz1p[2 * P + 1][mb]), xo, gW1[mb]);
            }
        }
    }

    // the wave's sums in parameter order
    float *o = sg[wv];
    constexpr int B1 = H * MLP_IN, W2 = B1 + H, B2 = W2 + H * H, W3 = B2 + H;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int unit = 16 * mb + 4 * grp + jj;
            if (col < MLP_IN) o[unit * MLP_IN + col] = gW1[mb][jj];
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) o[W2 + unit * H + 16 * nb + col] = gW2[mb][nb][jj];
        }
        float u = gb1[mb], v = gb2[mb], w = gw3[mb];
        u += __shfl_xor(u, 16, 64);
        v += __shfl_xor(v, 16, 64);
        w += __shfl_xor(w, 16, 64);
        u += __shfl_xor(u, 32, 64);
        v += __shfl_xor(v, 32, 64);
        w += __shfl_xor(w, 32, 64);
        if (grp == 0) {
            o[B1 + 16 * mb + col] = u;
            o[B2 + 16 * mb + col] = v;
            o[W3 + 16 * mb + col] = w;
        }
    }
    gb3 += __shfl_xor(gb3, 16, 64);
    gb3 += __shfl_xor(gb3, 32, 64);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
    if (lane == 0) {
        o[MLP_NPARAM - 1] = gb3;
        o[MLP_NPARAM] = lsum;
    }
    __syncthreads();
    // workgroup partial (fixed wave order)
    for (int i = threadIdx.x; i <= MLP_NPARAM; i += 64 * TW) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < TW; ++w) v += sg[w][i];
        if (i < MLP_NPARAM) partial[(int64_t)blockIdx.x * MLP_NPARAM + i] = v;
        else loss_partial[blockIdx.x] = v * inv_batch;
    }
}

// Fixed-order sum of the workgroup partials.  Workgroup g takes parameters
// 16 g .. 16 g + 15 (the loss counts as one more), 64 rows at a time: thread
// (slot = thread / 16, column = thread % 16) adds rows slot, slot + 64, ...,
// and the 64 slots are added as a tree within each wavefront and in wave order
// after it: the same order on every call.  One launch's latency bounds it, so
// at the most rows (256) each thread has its four loads under way at once and
// 79 workgroups share them (20 workgroups of 64 columns, 16 loads a thread,
// took 6.7 us).  With ad.m set, the thread that formed a parameter's gradient
// also takes that parameter's Adam step (elementwise, so no other workgroup
// waits), on values it has loaded meanwhile.
constexpr int GR_C = 16, GR_S = 64;
static_assert(TRAIN_BLOCKS <= 4 * GR_S, "k_grad_reduce takes 4 rows per thread");

__global__ void __launch_bounds__(GR_C *GR_S) k_grad_reduce(const float *__restrict__ partial, int nblocks,
                                                            const float *__restrict__ loss_partial,
                                                            float *__restrict__ grad, float *__restrict__ loss,
                                                            AdamStep ad)
{
    __shared__ float sp[GR_S / 4][GR_C];
    const int col = threadIdx.x & 15, slot = threadIdx.x >> 4;
    const int i = (int)blockIdx.x * GR_C + col;
    const bool is_loss = i == MLP_NPARAM, on = i <= MLP_NPARAM;
    const float *src = is_loss ? loss_partial : partial + i;
    const int64_t st = is_loss ? 1 : MLP_NPARAM;
    float r[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (on && slot + GR_S * k < nblocks) r[k] = src[(slot + GR_S * k) * st];
    const bool adam = ad.m && threadIdx.x < GR_C && i < MLP_NPARAM;
    float *p = reinterpret_cast<float *>(ad.m) + i;  // MlpDevice is the flat parameter vector (ABI order)
    float a0 = 0.f, v0 = 0.f, p0 = 0.f;
    if (adam) {
        a0 = ad.m1[i];
        v0 = ad.m2[i];
        p0 = *p;
    }
    float s = (r[0] + r[1]) + (r[2] + r[3]);
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if ((slot & 3) == 0) sp[slot >> 2][col] = s;
    __syncthreads();
    if (threadIdx.x >= GR_C || !on) return;
    float g = 0.f;
#pragma unroll
    for (int k = 0; k < GR_S / 4; ++k) g += sp[k][col];
    if (is_loss) {
        *loss = g;
        return;
    }
    grad[i] = g;
    if (adam) {
        const float a = ad.b1 * a0 + ad.ob1 * g;
        const float v = ad.b2 * v0 + ad.ob2 * g * g;
        ad.m1[i] = a;
        ad.m2[i] = v;
        *p = p0 - ad.lr * (a * ad.c1) / (sqrtf(v * ad.c2) + ad.eps);
    }
}

}  // namespace

hipError_t launch_coarsen4(const float *U, int64_t vs, int ndim, const int nf[3], float gm1, float *Wc, float *sub,
                           hipStream_t s)
{
    int64_t nc = nf[0] / 4;
    if (ndim >= 2) nc *= nf[1] / 4;
    if (ndim == 3) nc *= nf[2] / 4;
    const dim3 grid((unsigned)((nc + 255) / 256));
    if (ndim == 1) hipLaunchKernelGGL(k_coarsen4<1>, grid, dim3(256), 0, s, U, vs, nf[0], 1, 1, gm1, Wc, sub, nc);
    else if (ndim == 2) hipLaunchKernelGGL(k_coarsen4<2>, grid, dim3(256), 0, s, U, vs, nf[0], nf[1], 1, gm1, Wc, sub, nc);
    else hipLaunchKernelGGL(k_coarsen4<3>, grid, dim3(256), 0, s, U, vs, nf[0], nf[1], nf[2], gm1, Wc, sub, nc);
    return hipGetLastError();
}

hipError_t launch_samples(const float *Wc, const float *sub, int ndim, const int nc[3], float *x, float *t,
                          hipStream_t s)
{
    const int64_t ncell = (int64_t)nc[0] * nc[1] * nc[2];
    const int64_t ns = ncell * (ndim + 2) * ndim;
    const dim3 grid((unsigned)((ns + 255) / 256));
    if (ndim == 1) hipLaunchKernelGGL(k_samples<1>, grid, dim3(256), 0, s, Wc, sub, nc[0], 1, 1, x, t);
    else if (ndim == 2) hipLaunchKernelGGL(k_samples<2>, grid, dim3(256), 0, s, Wc, sub, nc[0], nc[1], 1, x, t);
    else hipLaunchKernelGGL(k_samples<3>, grid, dim3(256), 0, s, Wc, sub, nc[0], nc[1], nc[2], x, t);
    return hipGetLastError();
}

hipError_t launch_train_grad(const MlpDevice *m, const float *x, const float *t, const int *idx, int64_t batch,
                             float *partial, float *loss_partial, int nblocks, float *grad, float *loss,
                             const AdamStep &adam, hipStream_t s)
{
    // one tile per wavefront as far as the partial rows (TRAIN_BLOCKS) go
    const int64_t want = (batch + TS * TW - 1) / (TS * TW);
    if (want < nblocks) nblocks = (int)want;
    hipLaunchKernelGGL(k_train_grad, dim3(nblocks), dim3(64 * TW), 0, s, m, x, t, idx, batch, 1.0f / (float)batch,
                       partial, loss_partial);
    hipLaunchKernelGGL(k_grad_reduce, dim3(MLP_NPARAM / GR_C + 1), dim3(GR_C * GR_S), 0, s, partial, nblocks,
                       loss_partial, grad, loss, adam);
    return hipGetLastError();
}

// Staging of hy_lim_make_samples_noalloc: the coarse primitives and sub-cell
// averages live in this library-owned array instead of a caller scratch.
// Host code never passes the symbol itself to a kernel (on the host it names
// a stand-in, not device memory); it uses the per-device address that
// hipGetSymbolAddress returns.
static __device__ __align__(256) float scratch[SAMPLES_STATIC_BYTES / sizeof(float)];

hipError_t samples_static_scratch(int device, float **ptr)
{
    static std::mutex mu;
    static float *addr[MAX_DEVICES] = {};
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e == hipSuccess && cur != device) e = hipSetDevice(device);
        void *a = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
        if (cur >= 0 && cur != device) {
            const hipError_t er = hipSetDevice(cur);
            if (e == hipSuccess) e = er;
        }
        if (e != hipSuccess) return e;
        addr[device] = (float *)a;
    }
    *ptr = addr[device];
    return hipSuccess;
}

AdamStep adam_step(MlpDevice *m, float *m1, float *m2, float lr, double b1, double b2, float eps, int step)
{
    AdamStep a{};
    a.m = m;
    a.m1 = m1;
    a.m2 = m2;
    a.lr = lr;
    a.b1 = (float)b1;
    a.b2 = (float)b2;
    a.ob1 = (float)(1.0 - b1);
    a.ob2 = (float)(1.0 - b2);
    a.eps = eps;
    a.c1 = (float)(1.0 / (1.0 - std::pow(b1, (double)step)));
    a.c2 = (float)(1.0 / (1.0 - std::pow(b2, (double)step)));
    return a;
}

}  // namespace hy
