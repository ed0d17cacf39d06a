// batch.hip -- many independent 1D patches ("tubes") advanced to a common end
// time in one persistent launch.
//
// Each workgroup pulls an entry from a device-side atomic queue (longest
// first), holds the tube, or its share of it, in registers (hy_line.h) and
// runs the full single-level loop of Alg. 2: dt = min(C dt_CFL, t_end - t)
// from a max-reduction (eq. courantTimeStep), then the two Runge-Kutta stages
// (eqs. RungeKutta1-3) of the same finite-volume update as the patch kernels
// (hy_face.h).  When the queue is empty every workgroup exits.  The host
// captures the reset and this kernel in a hipGraph once and replays it.
//
// What bounds it: the longest tube.  On one compute unit its steps are bound
// by vector issue, so tubes that would outlast the rest are split over a team
// of workgroups.  A member owns a run of cells and, once per step, takes from
// each neighbour the 4 cells beyond its own (two stages of a two-cell
// stencil: stage 1 is repeated on two of them) and from every member the CFL
// rate.
//
// The exchange needs no fence and no flag: each value travels in a 64-bit
// word with the step number beside it, stored and polled with relaxed
// device-scope atomics, so it has arrived when its number has.  Words of
// consecutive steps alternate between two places: a member overwrites the
// words of step k at step k + 2, which it reaches only after every member has
// sent its rate of step k + 1, that is, has read the words of step k.  One
// wavefront polls while the others compute the first stage's fluxes away from
// the ends, which need neither the neighbours nor dt.
//
// Every wait ends: a team consists of the workgroups that have joined it by
// the time its first member closes it (all of them running; a listed
// workgroup that comes later finds the team closed and goes on to the next
// entry), and members take the same number of steps, because each computes
// dt from the same rates.  Polls are bounded all the same; a member that
// reaches the bound marks the tube as stopped early.
#include "hy_batch.h"
#include "hy_internal.h"
#include "hy_line.h"

namespace hy {
namespace {

// Polls before giving up: about a second for a member (a step takes a few
// microseconds), about 50 us for a team's first member waiting for the others.
constexpr int POLL_LIMIT = 1 << 21;
constexpr int JOIN_POLLS = 64;
constexpr unsigned TEAM_CLOSED = 1u << 16;

__device__ __forceinline__ void mail_put(unsigned long long *w, unsigned tag, float v)
{
    __hip_atomic_store(w, ((unsigned long long)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long mail_get(const unsigned long long *w)
{
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void __launch_bounds__(256) k_batch_reset(BatchCtl *ctl, unsigned *join, unsigned long long *mail,
                                                      TubeStatus *status, int ntubes)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) ctl->next = 0u;
    if (i < TEAM_SLOTS) join[i] = 0u;
    if (i < TEAM_SLOTS * 2 * MAIL_WORDS) mail[i] = 0ull;
    for (int k = i; k < ntubes; k += gridDim.x * 256) status[k].err = 0;
}

// A tube's state from pinned host memory (3 x n, read over the bus) into the
// concatenated device arrays, primitives converted on the way.  One launch in
// place of three copies and a conversion: 46 us per call with its wait
// before.
__global__ void __launch_bounds__(256) k_tube_put(const float *__restrict__ host, float *__restrict__ U, int64_t ntot,
                                                   int n, int prim, float inv_gm1)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float a = host[i], b = host[n + i], c = host[2 * n + i];
    U[i] = a;
    U[ntot + i] = prim ? a * b : b;
    U[2 * ntot + i] = prim ? fma_(0.5f * a, b * b, c * inv_gm1) : c;
}

// A tube's state, as primitives when asked, and its status into pinned host memory.
__global__ void __launch_bounds__(256) k_tube_get(const float *__restrict__ U, int64_t ntot, int n, int prim, float gm1,
                                                   const TubeStatus *st, float *__restrict__ host, TubeStatus *hst)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) *hst = *st;
    if (i >= n) return;
    const float D = U[i], S = U[ntot + i], G = U[2 * ntot + i];
    host[i] = D;
    host[n + i] = prim ? S / D : S;
    host[2 * n + i] = prim ? gm1 * (G - 0.5f * (S * S) / D) : G;
}

// NW wavefronts per workgroup, CPW chunks of 56 cells each (NW * CPW * 56 >=
// the batch's longest tube; the smaller CPW that fits keeps the state in
// fewer registers)
template <int SOLVER, int NW, int CPW>
__global__ void __launch_bounds__(64 * NW) k_batch(const TubeDesc *__restrict__ tubes,
                                                   const BatchItem *__restrict__ items, float *__restrict__ U,
                                                   int64_t ntot, BatchCtl *ctl, unsigned *join,
                                                   unsigned long long *mail, TubeStatus *__restrict__ status)
{
    constexpr int NCH = NW * CPW;
    __shared__ float sEdge[2][(NCH + 1) * LINE_EDGE];  // by step parity: the chunks' edge cells, then the mail's
    __shared__ float sRate[2][NW];
    __shared__ float sAll;      // a team's rate
    __shared__ int sNext[3];    // entry, rank, members
    __shared__ int sStop;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool mailer = wave == NW - 1;  // (the wavefront with the fewest chunks)
    const double t_end = ctl->t_end, cfl = ctl->cfl;
    const int nitems = ctl->nitems, max_steps = ctl->max_steps;

    for (;;) {
        if (tid == 0) {
            // the next entry that is still open, and this workgroup's place in its team
            int q, rank, members;
            for (;;) {
                rank = 0;
                members = 1;
                q = (int)atomicAdd(&ctl->next, 1u);
                if (q >= nitems) break;
                const BatchItem it = items[q];
                if (it.parts <= 1) break;
                unsigned *j = join + it.team;
                unsigned long long *count = mail + (int64_t)it.slot * 2 * MAIL_WORDS + MAIL_WORDS - 1;
                unsigned c = __hip_atomic_fetch_add(j, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (c & TEAM_CLOSED) continue;
                rank = (int)c;
                if (rank == 0) {
                    for (int k = 0; k < JOIN_POLLS; ++k) {
                        if ((int)__hip_atomic_load(j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= it.parts) break;
                        __builtin_amdgcn_s_sleep(8);
                    }
                    members = (int)__hip_atomic_fetch_or(j, TEAM_CLOSED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    mail_put(count, 1u, (float)members);
                    break;
                }
                unsigned long long m = 0ull;
                for (int k = 0; k < POLL_LIMIT && (m >> 32) != 1ull; ++k) m = mail_get(count);
                if ((m >> 32) == 1ull) {
                    members = (int)__uint_as_float((unsigned)m);
                    break;
                }
            }
            sNext[0] = q;
            sNext[1] = rank;
            sNext[2] = members;
            sStop = 0;
        }
        __syncthreads();
        const int q = sNext[0], rank = sNext[1], M = sNext[2];
        if (q >= nitems) break;
        const BatchItem it = items[q];
        const TubeDesc d = tubes[it.tube];
        // this workgroup's cells of the tube: s0 .. s0 + nl - 1
        const int base = d.n / M, rem = d.n - base * M;
        const int s0 = rank * base + (rank < rem ? rank : rem);
        const int nl = base + (rank < rem ? 1 : 0);
        const bool ring = M > 1 && d.bclo == BC_PERIODIC;
        const bool hasl = M > 1 && (rank > 0 || ring), hasr = M > 1 && (rank < M - 1 || ring);
        const int left = rank > 0 ? rank - 1 : M - 1, right = rank < M - 1 ? rank + 1 : 0;
        auto slot = [&](int r, unsigned tag) -> unsigned long long * {
            return mail + ((int64_t)(it.slot + r) * 2 + (tag & 1u)) * MAIL_WORDS;
        };
        Line<float, SOLVER, NW, CPW, false> ln;
        ln.init(nl, d.bclo, d.bchi, hasl, hasr, d.gamma, d.gamma - 1.f, 1.f / (d.gamma - 1.f), d.theta, d.idx);
        float rate = 0.f;
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            const bool o = ln.own(k);
#pragma unroll
            for (int v = 0; v < 3; ++v) ln.U[k][v] = o ? U[v * ntot + d.off + s0 + ln.cell(k)] : 1.f;
            rate = fmaxf(rate, ln.rate(k));
        }

        double t = 0.0;
        int steps = 0;
        bool stop = false;
        for (;;) {
            const unsigned tag = (unsigned)steps + 1u;
            float *edge = sEdge[tag & 1u];
            if constexpr (CPW * NW > 32) ln.fresh();
            // the state's rate and edge cells, to LDS and to the neighbours
            ln.send(edge);
            if (M > 1) {
#pragma unroll
                for (int k = 0; k < CPW; ++k) {
                    if (wave + k * NW >= ln.nch) break;
                    const int j = ln.cell(k);
                    if (!ln.own(k)) continue;
                    if (hasl && j < LINE_H) {
#pragma unroll
                        for (int v = 0; v < 3; ++v) mail_put(slot(rank, tag) + 3 * j + v, tag, ln.U[k][v]);
                    }
                    if (hasr && j >= nl - LINE_H) {
#pragma unroll
                        for (int v = 0; v < 3; ++v)
                            mail_put(slot(rank, tag) + 12 + 3 * (j - nl + LINE_H) + v, tag, ln.U[k][v]);
                    }
                }
            }
            rate = lanes_max(rate);
            if (lane == 0) sRate[tag & 1u][wave] = rate;
            __syncthreads();
            float r = lanes_max(lane < NW ? sRate[tag & 1u][lane] : 0.f);
            if (M > 1 && mailer) {
                // this workgroup's rate out; the neighbours' cells (lanes 0 ..
                // 7, three words each) and every member's rate (lanes 8 ..) in
                if (lane == 0) mail_put(slot(rank, tag) + 24, tag, r);
                const bool cell = lane < 2 * LINE_H && (lane < LINE_H ? hasl : hasr);
                const bool rt = lane >= 8 && lane < 8 + M;
                const unsigned long long *w = lane < LINE_H ? slot(left, tag) + 12 + 3 * lane
                                              : (lane < 8 ? slot(right, tag) + 3 * (lane - LINE_H)
                                                          : slot(rt ? lane - 8 : 0, tag) + 24);
                float x[3] = {0.f, 0.f, 0.f};
                bool wait = cell || rt;
                for (int k = 0; k < POLL_LIMIT && __builtin_amdgcn_ballot_w64(wait) != 0ull; ++k) {
                    if (wait) {
                        unsigned long long m[3];
#pragma unroll
                        for (int v = 0; v < 3; ++v) m[v] = mail_get(w + (cell ? v : 0));
                        wait = (unsigned)(m[0] >> 32) != tag || (unsigned)(m[1] >> 32) != tag ||
                               (unsigned)(m[2] >> 32) != tag;
#pragma unroll
                        for (int v = 0; v < 3; ++v) x[v] = __uint_as_float((unsigned)m[v]);
                    }
                }
                if (__builtin_amdgcn_ballot_w64(wait) != 0ull && lane == 0) sStop = 1;
                if (cell) {
#pragma unroll
                    for (int v = 0; v < 3; ++v) edge[ln.c_word(ln.nch, lane) + v] = x[v];
                }
                r = lanes_max(rt ? x[0] : 0.f);
                if (lane == 0) sAll = r;
            }
            // stage 1's fluxes need neither dt nor, away from the ends, the mail
            float D[CPW][3];
            auto late = [&](int c) { return M > 1 && ((hasl && c == 0) || (hasr && (c + 1) * LINE_OWN + LINE_H > nl)); };
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                const int c = wave + k * NW;
                if (c >= ln.nch) break;
                if (!late(c)) {
                    ln.receive(k, edge);
                    ln.stage1_flux(k, D[k]);
                }
                // (chunk by chunk: interleaving them only raises register pressure)
                __builtin_amdgcn_sched_barrier(0);
            }
            if (M > 1) {
                __syncthreads();
                r = sAll;
#pragma unroll
                for (int k = 0; k < CPW; ++k) {
                    const int c = wave + k * NW;
                    if (c >= ln.nch) break;
                    if (late(c)) {
                        ln.receive(k, edge);
                        ln.stage1_flux(k, D[k]);
                    }
                }
            }
            if (!(t < t_end)) break;
            const double dt = fmin(cfl / (double)r, t_end - t);
            if (!(dt > 0.0) || steps >= max_steps || sStop) {  // non-finite rate, step cap: stop this tube
                stop = true;
                break;
            }
            const float c1 = uniform_((float)dt * d.idx);
            rate = 0.f;
#pragma unroll
            for (int k = 0; k < CPW; ++k) {
                if (wave + k * NW >= ln.nch) break;
                rate = fmaxf(rate, ln.finish(k, D[k], c1, 0.f, 0.5f * c1, 0.f));
                __builtin_amdgcn_sched_barrier(0);
            }
            t += dt;
            ++steps;
        }
#pragma unroll
        for (int k = 0; k < CPW; ++k) {
            if (ln.own(k))
#pragma unroll
                for (int v = 0; v < 3; ++v) U[v * ntot + d.off + s0 + ln.cell(k)] = ln.U[k][v];
        }
        // per-tube status: any thread's bad flag, steps and time reached
        if (ln.bad) atomicOr(&status[it.tube].err, 1);
        if (tid == 0) {
            if (stop) atomicOr(&status[it.tube].err, 2);
            if (rank == 0) {
                status[it.tube].steps = steps;
                status[it.tube].t = t;
                status[it.tube].members = M;
            }
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_batch_reset(BatchCtl *ctl, unsigned *join, unsigned long long *mail, TubeStatus *status, int ntubes,
                              hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_reset, dim3((TEAM_SLOTS * 2 * MAIL_WORDS + 255) / 256), dim3(256), 0, s, ctl, join, mail,
                       status, ntubes);
    return hipGetLastError();
}

hipError_t launch_tube_put(const float *host, float *U, int64_t ntot, int n, bool prim, float inv_gm1, hipStream_t s)
{
    hipLaunchKernelGGL(k_tube_put, dim3((n + 255) / 256), dim3(256), 0, s, host, U, ntot, n, prim ? 1 : 0, inv_gm1);
    return hipGetLastError();
}

hipError_t launch_tube_get(const float *U, int64_t ntot, int n, bool prim, float gm1, const TubeStatus *st, float *host,
                           TubeStatus *hst, hipStream_t s)
{
    hipLaunchKernelGGL(k_tube_get, dim3((n + 255) / 256), dim3(256), 0, s, U, ntot, n, prim ? 1 : 0, gm1, st, host, hst);
    return hipGetLastError();
}

namespace {
// Register footprints by the batch's longest tube: 16, 32, 64, 80 or 112
// chunks over the workgroup's wavefronts (896, 1792, 3584, 4480, 6272 cells).
template <int SOLVER, int BT>
const void *batch_kernel_bt(int nmax)
{
    constexpr int NW = BT / 64;
    const int nch = (nmax + LINE_OWN - 1) / LINE_OWN;
    if (nch <= 16) return (const void *)k_batch<SOLVER, NW, 16 / NW>;
    if (nch <= 32) return (const void *)k_batch<SOLVER, NW, 32 / NW>;
    if (nch <= 64) return (const void *)k_batch<SOLVER, NW, 64 / NW>;
    if (nch <= 80) return (const void *)k_batch<SOLVER, NW, 80 / NW>;
    return (const void *)k_batch<SOLVER, NW, 112 / NW>;
}

template <int SOLVER>
const void *batch_kernel_s(int bt, int nmax)
{
    switch (bt) {
    case 256: return batch_kernel_bt<SOLVER, 256>(nmax);
    case 512: return batch_kernel_bt<SOLVER, 512>(nmax);
    default: return batch_kernel_bt<SOLVER, 1024>(nmax);
    }
}

const void *batch_kernel(int solver, int bt, int nmax)
{
    return solver == SOLVER_HLL ? batch_kernel_s<SOLVER_HLL>(bt, nmax) : batch_kernel_s<SOLVER_HLLC>(bt, nmax);
}
static_assert(112 * LINE_OWN >= BATCH_NMAX, "the longest tube fits");
}  // namespace

bool batch_bt_supported(int bt) { return bt == 256 || bt == 512 || bt == 1024; }

hipError_t launch_batch(const TubeDesc *tubes, const BatchItem *items, float *U, int64_t ntot, BatchCtl *ctl,
                        unsigned *join, unsigned long long *mail, TubeStatus *status, int solver, int nmax, int nblocks,
                        int bt, hipStream_t s)
{
    if (nmax < 1 || nmax > BATCH_NMAX || !batch_bt_supported(bt)) return hipErrorInvalidValue;
    void *args[] = {(void *)&tubes, (void *)&items, (void *)&U,    (void *)&ntot,
                    (void *)&ctl,   (void *)&join,  (void *)&mail, (void *)&status};
    const hipError_t e = hipLaunchKernel(batch_kernel(solver, bt, nmax), dim3(nblocks), dim3(bt), args, 0, s);
    return e != hipSuccess ? e : hipGetLastError();
}

int batch_blocks_per_cu(int nmax, int bt)
{
    int most = 1 << 30;
    for (int solver : {SOLVER_HLL, SOLVER_HLLC}) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch_kernel(solver, bt, nmax), bt, 0) != hipSuccess) return 1;
        most = nb < most ? nb : most;
    }
    return most > 0 ? most : 1;
}

}  // namespace hy
