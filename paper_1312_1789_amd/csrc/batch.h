// batch.h -- device-side plan and launch arguments of the batched form (many
// independent clusters in one step sequence).  Not part of the public C-ABI.
#pragma once

#include "internal.h"

namespace nb {

constexpr int kBatchITileMax = 256;   // largest i-tile: active rows per work item
constexpr int64_t kBatchMaxRows = int64_t(1) << 22;   // items aimed for in one step x i-tile, at most
constexpr int kBatchMaxPerWG = 32;     // most items aimed for per persistent workgroup
constexpr int kBatchSchedBlock = 1024;  // particles per scheduling block
constexpr int kXcds = 8;                // XCDs of the device: work queues of the persistent force kernel

// The work of the cluster of one rank (plan order) in a step, written by
// the plan for the persistent force kernel: one 64-byte load per work item.
struct BatchRank {
    int64_t i0, i1;   // its work items [i0, i1)
    int64_t base;     // first particle
    int64_t jc;       // j-range per split
    int64_t poff;     // offset of its split partials (doubles)
    int64_t aoff;     // offset of its active list
    int32_t nn, na;   // particles, active rows
    int32_t sp, c;    // j-splits, cluster index
};
static_assert(sizeof(BatchRank) == 64, "one 64-byte record per rank");

// Written by the plan kernel of every batched step and read by the kernels
// after it.  Arrays sized n_clusters + 1 (the last entry of a scanned array
// holds its total).
struct BatchPlan {
    int64_t t_end;              // clusters whose next time exceeds this do not step
    int64_t n_live;             // clusters that stepped in the last plan
    int64_t pad[6];
    int64_t *nact;              // [nc]   active particles per cluster
    int64_t *aoff;              // [nc+1] offsets of the clusters' active lists
    int64_t *ioff;              // [nc+1] first work item of each cluster rank
    int64_t *poff;              // [nc+1] offsets of the clusters' split partials (doubles)
    int64_t *jchunk;            // [nc]   j-range per split
    int32_t *split;             // [nc]   j-splits per cluster
    int64_t *tcur;              // [nc]   time of the cluster's last completed step
    BatchRank *rank;            // [nc]   work of each cluster rank
    // items taken from each XCD's eighth of the step's items (one 64-byte
    // line per counter); reset by the plan
    unsigned queue[kXcds * 16];
};

struct BatchCounters {
    int64_t steps;
    int64_t sum_n_act;
    int64_t interactions;
    unsigned long long underflow;
    unsigned long long nonfinite;
    int64_t pad[3];
};

// Everything a batched launch needs; all pointers are device addresses inside
// the batch workspace except the state, which the caller passes per call.
struct BatchLaunch {
    int nc;                     // clusters
    int nb;                     // scheduling blocks per cluster (largest cluster / 1024, rounded up)
    int nblk;                   // scheduling blocks of all clusters
    const int32_t *blk;         // [nblk][2] (cluster, block) of each
    int64_t n;                  // particles in all clusters
    const int64_t *off;         // [nc+1] cluster offsets
    const int32_t *ord;         // [nc]   clusters by decreasing size
    int32_t *cid;               // [n]    cluster of each particle
    int64_t *tnext;             // [nc]   next block time of each cluster
    int64_t *bmin;              // [nc][nb]
    int32_t *bcnt;              // [nc][nb]
    int32_t *brow;              // [nblk]  first row of each scheduling block in the active list
    unsigned *arrive;           // arrival counters of the schedule (zero between launches)
    BatchPlan *plan;
    BatchCounters *ctr;
    int32_t *act;               // [n] concatenated active lists
    double *part;               // split partials
    double *force;              // [12][n] step forces by active row
    double eps2;
    int64_t n_hard;             // per cluster; every pair is unsoftened when eps2 == 0
    int force_grid;             // workgroups of the persistent force kernel
    int per_wg;                 // work items aimed for per persistent workgroup
    int k_items;                // items aimed for in one step: min(force_grid * per_wg, kBatchMaxRows / itile)
    int itile;                  // active rows per work item: 64, 128 or 256
    int halves;                 // items per 64-row tile and split: 2 = half its rows each, one row per lane
    int grain;                  // shortest j-split: MIXED an FP32 chunk, FP64 and DS two tiles
};

// How a step's work is cut (also compiled for the host, which tests it).
constexpr int64_t kBItemMin = 32768;   // pair evaluations of a work item worth claiming

// Work items of a row tile and split.
__host__ __device__ __forceinline__ int b_tile_items(const BatchLaunch &L) { return L.itile == 64 ? L.halves : 1; }

// The work of one cluster in a step: row tiles, j-splits sp of jc particles.
struct BatchCut {
    int32_t tiles, sp, jc;
};
__host__ __device__ __forceinline__ BatchCut b_cut(int64_t na, int64_t nn, int itile, int grain, int64_t w_item)
{
    BatchCut k;
    k.tiles = int32_t((unsigned(na) + unsigned(itile) - 1u) / unsigned(itile));
    int64_t sp = (int64_t(itile) * nn + w_item - 1) / w_item;
    const int64_t sp_max = (nn + grain - 1) / grain;   // pieces of at least a grain (MIXED: an FP32 chunk)
    sp = sp < 1 ? 1 : (sp > sp_max ? sp_max : sp);
    unsigned jc = (unsigned(nn) + unsigned(sp) - 1u) / unsigned(sp);
    jc = (jc + unsigned(grain) - 1u) / unsigned(grain) * unsigned(grain);
    k.jc = int32_t(jc);
    k.sp = int32_t((unsigned(nn) + jc - 1u) / jc);
    return k;
}

// Pair evaluations per item for W in all.  Items of at least kBItemMin pairs (an
// item costs a few microseconds of loads before its first pair, and the claim
// of one from a counter that an eighth of the chip shares some 50 ns), up to the
// number asked for; a step of less than four such items per workgroup is cut
// into as many as there are workgroups (an eighth less, as the cuts round up),
// all dealt, and at least into one (a single workgroup).
__host__ __device__ __forceinline__ int64_t b_item_size(const BatchLaunch &L, int64_t W)
{
    int64_t k = W / kBItemMin;
    if (k < 4 * int64_t(L.force_grid)) k = int64_t(L.force_grid) * 7 / 8;
    if (k > L.k_items) k = L.k_items;
    if (k < 1) k = 1;
    return W * b_tile_items(L) / k + 1;
}

hipError_t batch_cid(const BatchLaunch &L, hipStream_t s);
// The step's schedule and plan (order: of the pair terms the partials hold);
// all_active: every particle at t = 0.
hipError_t batch_schedule(const BatchLaunch &L, const nbody_state &st, int all_active, int order, hipStream_t s);
// The active lists of a schedule: of all particles (initialisation), or of a
// step with every particle of the stepping clusters predicted.
hipError_t batch_list_all(const BatchLaunch &L, const nbody_state &st, hipStream_t s);
hipError_t batch_advance(const BatchLaunch &L, const nbody_state &st, int order, int precision, void *rec,
                         hipStream_t s);
// Reset the work queues (a second force pass on the same plan).
hipError_t batch_requeue(const BatchLaunch &L, hipStream_t s);
hipError_t batch_force(const BatchLaunch &L, int order, int precision, const void *rec, hipStream_t s);
hipError_t batch_reduce(const BatchLaunch &L, int order, double *o0, double *o1, double *o2, double *o3,
                        hipStream_t s);
// Split sums and corrector of the step.
hipError_t batch_finish(const BatchLaunch &L, const nbody_config &c, const nbody_state &st, hipStream_t s);
// Workgroups of the persistent force kernel (i-tile itile) that fit on the
// device at once.
int batch_force_resident(int order, int precision, int itile, int halves, int device);

}  // namespace nb
