// Batched 1D tubes: device records and launchers (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hy {

constexpr int BATCH_NMAX = 6144;  // cells per tube (register-resident)

struct TubeDesc {
    int n;
    int bclo, bchi;
    float idx;    // 1 / dx
    float gamma;
    float theta;
    int64_t off;  // first cell in the concatenated state arrays
};

struct TubeStatus {
    int steps;
    int err;      // bit 0: rho <= 0, p <= 0 or non-finite met; bit 1: stopped early (dt not > 0 or step cap)
    double t;
    int members;  // workgroups that shared the tube in its last run
    int pad;
};

// Teams: a long tube may be split over up to TEAM_MAX workgroups, each of
// which owns a run of its cells.  A queue entry names the tube, how many
// workgroups may share it, and (for more than one) its team's join word and
// first mail slot.  Each entry is listed once per workgroup wanted.
constexpr int TEAM_MAX = 16;
constexpr int TEAM_SLOTS = 512;   // mail slots of all teams together
constexpr int TEAM_MIN_CELLS = 128;  // a member's cells at least
constexpr int MAIL_WORDS = 32;    // per slot and step parity: 12 low-edge values, 12 high-edge values, the rate
struct BatchItem {
    int tube, parts, team, slot;
};

struct BatchCtl {
    unsigned next;  // queue head
    int nitems;
    int max_steps;
    int pad;
    double t_end;
    double cfl;
};

// Clears the queue head, the teams' join words and mail, and the tubes' error flags.
hipError_t launch_batch_reset(BatchCtl *ctl, unsigned *join, unsigned long long *mail, TubeStatus *status, int ntubes,
                              hipStream_t s);
// One tube's state (U: its first cell) from and to pinned host memory
// (3 x n floats), primitives converted on the way; get also fetches its status.
hipError_t launch_tube_put(const float *host, float *U, int64_t ntot, int n, bool prim, float inv_gm1, hipStream_t s);
hipError_t launch_tube_get(const float *U, int64_t ntot, int n, bool prim, float gm1, const TubeStatus *st, float *host,
                           TubeStatus *hst, hipStream_t s);
// bt = threads per workgroup: 256, 512 or 1024
bool batch_bt_supported(int bt);
hipError_t launch_batch(const TubeDesc *tubes, const BatchItem *items, float *U, int64_t ntot, BatchCtl *ctl,
                        unsigned *join, unsigned long long *mail, TubeStatus *status, int solver, int nmax, int nblocks,
                        int bt, hipStream_t s);
int batch_blocks_per_cu(int nmax, int bt);

}  // namespace hy
