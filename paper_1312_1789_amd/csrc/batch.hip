// batch.hip -- many independent clusters advanced together: every call of a
// batched step gives each cluster one block step of its own (its own t_next
// and active set), with a fixed sequence of launches whose grids do not
// depend on the data, so one step can be captured in a HIP graph and
// replayed without the host.
//
// Sequence of one batched step:
//   k_b_schedule         per (cluster, 1024-particle block): next-time minima and
//                        counts, the clusters' t_next and active counts (by each
//                        cluster's last workgroup), the plan (by the last of all:
//                        active offsets, j-splits and work items per cluster,
//                        largest clusters first, counters, work queues);
//   k_b_advance          ordered active lists, and every particle predicted to
//                        its cluster's t_next;
//   k_b_force            persistent: workgroups take (cluster, i-tile, j-split)
//                        items from per-XCD queues until all are empty;
//   k_b_finish           split partials summed in split order, corrector,
//                        interpolation and new steps.
// Most steps of a small ensemble are a few microseconds of work per kernel: as
// eight kernels (three for the schedule, compaction, predictor, force, split sum,
// corrector) the seven small ones took 42 us a step at 32 clusters of 2^10 to
// 2^14, with 2 us between kernels and 9 between graphs of one step; the three
// take 27, in graphs of eight steps without gaps: t = 1/256 in 13.3 ms instead of
// 16.2 with the same force kernel.
// Method as in the single-system kernels (paper: Abstract; Sec. "Codes
// description"): Hermite block steps of order 4, 6 or 8 and direct-summation
// softened gravity with its derivatives (Nitadori & Makino 2008).
#include <climits>

#include "batch.h"
#include "hermite.h"
#include "pairwise.h"

namespace nb {
namespace {

constexpr int kBBlock = kBatchSchedBlock;
constexpr int kBTile = 32;   // records per LDS tile of the one-wave force workgroups
constexpr int kBSub = 32;               // clusters per arrival counter
constexpr int kBThreads = 256;  // threads per scheduling block (4 particles each)

__device__ __forceinline__ int64_t b_next(const int64_t *t_tick, const int32_t *level, int64_t i)
{
    return t_tick[i] + (int64_t(1) << (kLevelMax - level[i]));
}

// Accesses that other workgroups of the same launch see, and the wait that
// orders them before an arrival is counted (as in the single-system step).
template <class T> __device__ __forceinline__ T shared_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void shared_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

constexpr int kBWaves = kBThreads / 64;

// Least time and number of particles at it over the block; every thread gets
// both.
__device__ __forceinline__ void block_min_count(int64_t &m, int64_t &c, int64_t *sm, int64_t *sc)
{
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t m2 = __shfl_xor(m, o, 64), c2 = __shfl_xor(c, o, 64);
        c = m2 < m ? c2 : (m2 == m ? c + c2 : c);
        m = m2 < m ? m2 : m;
    }
    __syncthreads();   // sm, sc are no longer read
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        sc[threadIdx.x >> 6] = c;
    }
    __syncthreads();
    m = sm[0];
    c = sc[0];
    for (int k = 1; k < kBWaves; ++k) {
        c = sm[k] < m ? sc[k] : (sm[k] == m ? c + sc[k] : c);
        m = sm[k] < m ? sm[k] : m;
    }
}

// Exclusive scan of one value per thread over the block; *total the sum.
__device__ __forceinline__ int64_t block_excl(int64_t x, int64_t *sh, int64_t *total)
{
    const int lane = int(threadIdx.x) & 63, w = int(threadIdx.x) >> 6;
    int64_t incl = x;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    __syncthreads();   // sh is no longer read
    if (lane == 63) sh[w] = incl;
    __syncthreads();
    int64_t before = 0, tot = 0;
    for (int k = 0; k < kBWaves; ++k) {
        if (k < w) before += sh[k];
        tot += sh[k];
    }
    *total = tot;
    return before + incl - x;
}

// Exclusive scan of v[0..n) in one block (chunks of kBThreads, running carry).
__device__ void block_scan(int64_t *v, int n, int64_t *sh)
{
    int64_t carry = 0;
    for (int c0 = 0; c0 < n; c0 += kBThreads) {
        const int c = c0 + threadIdx.x;
        int64_t tot = 0;
        const int64_t ex = block_excl(c < n ? v[c] : 0, sh, &tot);
        if (c < n) v[c] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) v[n] = carry;
    __syncthreads();
}

// Sum over the block of one value per thread (the result is returned to
// every thread).
__device__ int64_t block_sum(int64_t v, int64_t *sh)
{
    int64_t tot = 0;
    (void)block_excl(v, sh, &tot);
    return tot;
}

// Workgroups of range x's XCD: the items of the range that are dealt to them.
__host__ __device__ __forceinline__ int b_dealt(int grid, int x) { return (grid - x + kXcds - 1) / kXcds; }

// Start of range x's counter for `total` items.
__device__ __forceinline__ uint32_t b_queue_start(int64_t total, int grid, int x)
{
    const int64_t len = total * (x + 1) / kXcds - total * x / kXcds;
    const int dealt = b_dealt(grid, x);
    return uint32_t(len < dealt ? len : dealt);
}

// The plan of one batched step (one block).  For every cluster: active
// offset, j-splits and work items.  Items are sized by cost: the step's
// padded work W = sum_c tiles_c * itile * N_c is cut into about k_items items
// of W / k_items pair evaluations each (a cluster's j-range is split into s_c
// pieces of at least 128), so no item is much longer than the average and the
// persistent kernel ends evenly.  Items are numbered in the cluster order
// ord[] (largest clusters first).  Bound used for the partial buffer:
// s_c <= itile N_c k_items / W + 1, so sum_c s_c a_c <= itile k_items + n.
// Also resets the work queues and adds the step's interactions to the counters.
__device__ __forceinline__ void plan_step(const BatchLaunch &L, int ncomp, int64_t *sh)
{
    const int nc = L.nc, itile = L.itile, grid = L.force_grid, grain = L.grain;
    const int64_t *off = L.off;
    const int32_t *ord = L.ord;
    BatchPlan *pl = L.plan;
    int64_t w = 0, inter = 0, live = 0;
    for (int c = threadIdx.x; c < nc; c += kBThreads) {
        const int64_t a = shared_load(&pl->nact[c]), nn = off[c + 1] - off[c];
        pl->aoff[c] = a;
        if (a > 0) pl->tcur[c] = shared_load(&L.tnext[c]);
        w += (a + itile - 1) / itile * itile * nn;
        inter += a * nn;
        live += a > 0 ? 1 : 0;
    }
    const int64_t W = block_sum(w, sh);
    inter = block_sum(inter, sh);
    live = block_sum(live, sh);
    const int64_t w_item = b_item_size(L, W);
    block_scan(pl->aoff, nc, sh);
    // splits, items (in rank order), partial rows (in cluster order)
    for (int r = threadIdx.x; r < nc; r += kBThreads) {
        const int c = ord[r];
        const int64_t na = shared_load(&pl->nact[c]), nn = off[c + 1] - off[c];
        const BatchCut k = b_cut(na, nn, itile, grain, w_item);
        pl->split[c] = k.sp;
        pl->jchunk[c] = k.jc;
        pl->ioff[r] = int64_t(k.tiles) * k.sp * b_tile_items(L);
        pl->poff[c] = int64_t(k.sp) * na * ncomp;
    }
    __syncthreads();
    block_scan(pl->ioff, nc, sh);
    block_scan(pl->poff, nc, sh);
    for (int r = threadIdx.x; r < nc; r += kBThreads) {
        const int c = ord[r];
        BatchRank d;
        d.i0 = pl->ioff[r];
        d.i1 = pl->ioff[r + 1];
        d.base = off[c];
        d.jc = pl->jchunk[c];
        d.poff = pl->poff[c];
        d.aoff = pl->aoff[c];
        d.nn = int32_t(off[c + 1] - off[c]);
        d.na = int32_t(shared_load(&pl->nact[c]));
        d.sp = pl->split[c];
        d.c = c;
        pl->rank[r] = d;
    }
    if (threadIdx.x < kXcds) pl->queue[threadIdx.x * 16] = b_queue_start(pl->ioff[nc], grid, int(threadIdx.x));
    if (threadIdx.x == 0) {
        pl->n_live = live;
        L.ctr->interactions += inter;
        L.ctr->sum_n_act += pl->aoff[nc];
        L.ctr->steps += 1;
    }
}

// The same plan for up to kBThreads clusters, one per thread: the values stay in
// registers and LDS instead of passing through memory between the scans (14 us
// for the schedule kernel at 32 clusters with plan_step, 12 with this).
__device__ __forceinline__ void plan_small(const BatchLaunch &L, int ncomp, int64_t *sh)
{
    __shared__ int64_t s_base[kBThreads], s_aoff[kBThreads];
    __shared__ int32_t s_nn[kBThreads], s_na[kBThreads];
    const int t = int(threadIdx.x), nc = L.nc, itile = L.itile;
    BatchPlan *pl = L.plan;
    const bool on = t < nc;
    const int cr = on ? L.ord[t] : 0;   // cluster of rank t
    const int64_t a = on ? shared_load(&pl->nact[t]) : 0, tn = on ? shared_load(&L.tnext[t]) : 0;
    const int64_t base = on ? L.off[t] : 0, nn = on ? L.off[t + 1] - base : 0;
    int64_t n_act = 0;
    const int64_t aoff = block_excl(a, sh, &n_act);
    const int64_t W = block_sum(int64_t((unsigned(a) + unsigned(itile) - 1u) / unsigned(itile)) * itile * nn, sh);
    const int64_t inter = block_sum(a * nn, sh), live = block_sum(a > 0 ? 1 : 0, sh);
    const int64_t w_item = b_item_size(L, W);
    if (on) {
        pl->aoff[t] = aoff;
        if (a > 0) pl->tcur[t] = tn;
        s_base[t] = base;
        s_aoff[t] = aoff;
        s_nn[t] = int32_t(nn);
        s_na[t] = int32_t(a);
    }
    __syncthreads();
    BatchRank d{};
    BatchCut k{0, 0, 0};
    if (on) {
        d.c = cr;
        d.base = s_base[cr];
        d.aoff = s_aoff[cr];
        d.nn = s_nn[cr];
        d.na = s_na[cr];
        k = b_cut(d.na, d.nn, itile, L.grain, w_item);
        d.sp = k.sp;
        d.jc = k.jc;
    }
    const int64_t items = int64_t(k.tiles) * k.sp * b_tile_items(L);
    int64_t n_items = 0, n_part = 0;
    d.i0 = block_excl(items, sh, &n_items);
    d.i1 = d.i0 + items;
    d.poff = block_excl(int64_t(d.sp) * d.na * ncomp, sh, &n_part);
    if (on) {
        pl->rank[t] = d;
        pl->split[cr] = d.sp;
        pl->poff[cr] = d.poff;
    }
    if (t < kXcds) pl->queue[t * 16] = b_queue_start(n_items, L.force_grid, t);
    if (t == 0) {
        pl->aoff[nc] = n_act;
        pl->ioff[nc] = n_items;
        pl->n_live = live;
        L.ctr->interactions += inter;
        L.ctr->sum_n_act += n_act;
        L.ctr->steps += 1;
    }
}

// Block b of cluster c covers [off[c] + b*kBBlock, min(off[c] + (b+1)*kBBlock, off[c+1])); the
// launch has one workgroup per such block, (c, b) = blk[2x], blk[2x + 1].  Each
// takes its block's least next time and the particles at it; the last of a
// cluster's workgroups takes the cluster's (clusters past t_end rest: no
// active particles), and the last of all makes the step's plan.  all_active
// marks every particle active at t = 0 (initialisation).  Arrivals are counted
// per cluster, per kBSub clusters, and in all.
__global__ void __launch_bounds__(kBThreads)
k_b_schedule(BatchLaunch L, const int64_t *__restrict__ t_tick, const int32_t *__restrict__ level, int all_active,
             int ncomp)
{
    __shared__ int64_t sm[kBWaves], sc[kBWaves], sh[kBWaves];
    __shared__ int s_last;
    const int c = L.blk[2 * blockIdx.x], b = L.blk[2 * blockIdx.x + 1], tid = int(threadIdx.x);
    const int64_t lo = L.off[c] + int64_t(b) * kBBlock, hi = L.off[c + 1];
    const int nbc = int((hi - L.off[c] + kBBlock - 1) / kBBlock);   // the cluster's blocks
    int64_t mn = INT64_MAX, cn = 0;
#pragma unroll
    for (int k = 0; k < kBBlock / kBThreads; ++k) {
        const int64_t i = lo + int64_t(k) * kBThreads + tid;
        if (i < hi && i < lo + kBBlock) {
            const int64_t t = all_active ? 0 : b_next(t_tick, level, i);
            cn = t < mn ? 1 : (t == mn ? cn + 1 : cn);
            mn = t < mn ? t : mn;
        }
    }
    block_min_count(mn, cn, sm, sc);
    unsigned *of_cluster = L.arrive, *of_sub = L.arrive + L.nc, *of_all = of_sub + (L.nc + kBSub - 1) / kBSub;
    if (tid == 0) {
        shared_store(&L.bmin[int64_t(c) * L.nb + b], mn);
        shared_store(&L.bcnt[int64_t(c) * L.nb + b], int32_t(cn));
        bool last = true;
        if (nbc > 1) {
            stores_done();
            last = atomicAdd(&of_cluster[c], 1u) == unsigned(nbc) - 1;
            if (last) shared_store(&of_cluster[c], 0u);   // for the next launch
        }
        s_last = last ? 1 : 0;
    }
    __syncthreads();
    if (!s_last) return;
    if (nbc > 1) {
        mn = INT64_MAX;
        cn = 0;
        for (int k = tid; k < nbc; k += kBThreads) {
            const int64_t t = shared_load(&L.bmin[int64_t(c) * L.nb + k]);
            const int64_t q = shared_load(&L.bcnt[int64_t(c) * L.nb + k]);
            cn = t < mn ? q : (t == mn ? cn + q : cn);
            mn = t < mn ? t : mn;
        }
        block_min_count(mn, cn, sm, sc);
    }
    __syncthreads();   // s_last has been read
    if (tid == 0) {
        const bool live = all_active || mn <= L.plan->t_end;
        shared_store(&L.tnext[c], mn);
        shared_store(&L.plan->nact[c], live ? cn : int64_t(0));
        stores_done();
        const int sub = c / kBSub, subs = (L.nc + kBSub - 1) / kBSub;
        const unsigned size = unsigned(L.nc - sub * kBSub < kBSub ? L.nc - sub * kBSub : kBSub);
        bool last = atomicAdd(&of_sub[sub], 1u) == size - 1;
        if (last) {
            shared_store(&of_sub[sub], 0u);
            last = subs == 1 || atomicAdd(of_all, 1u) == unsigned(subs) - 1;
            if (last) shared_store(of_all, 0u);
        }
        s_last = last ? 1 : 0;
    }
    __syncthreads();
    if (!s_last) return;
    if (L.nc <= kBThreads) plan_small(L, ncomp, sh);
    else plan_step(L, ncomp, sh);
}

// The active particles of block (c, b), written after those of the cluster's
// earlier blocks, at aoff[c] + the sum of their counts at the cluster's time (kept
// in brow[] for the step's end); and, unless PREC is negative (initialisation),
// every particle of the block predicted to the cluster's time.  Workgroup y of a
// block predicts a quarter of it; the first writes the list as well.
template <int P, int PREC>
__global__ void __launch_bounds__(kBThreads)
k_b_advance(BatchLaunch L, nbody_state st, int all_active, void *__restrict__ rec_out)
{
    __shared__ int64_t sh[kBWaves];
    constexpr int PER = kBBlock / kBThreads;
    const int c = L.blk[2 * blockIdx.x], b = L.blk[2 * blockIdx.x + 1], tid = int(threadIdx.x);
    const BatchPlan *pl = L.plan;
    if (pl->nact[c] == 0) return;   // a resting cluster: its records are not read
    const int64_t tn = L.tnext[c];
    const int64_t *bmin = L.bmin + int64_t(c) * L.nb;
    const int32_t *bcnt = L.bcnt + int64_t(c) * L.nb;
    const int64_t lo = L.off[c] + int64_t(b) * kBBlock;
    const int64_t hi = L.off[c + 1] < lo + kBBlock ? L.off[c + 1] : lo + kBBlock;
    if constexpr (PREC >= 0) {
        const double *ds[6] = {st.d[0], st.d[1], st.d[2], st.d[3], st.d[4], st.d[5]};
        const int64_t i = lo + int64_t(blockIdx.y) * kBThreads + tid;
        if (i < hi) {
            const double dt = double(tn - st.t_tick[i]) * (1.0 / double(kTicksPerUnit));
            predict_one<P, PREC>(L.n, i, dt, st.m, st.x, st.v, ds, rec_out);
        }
    }
    if (blockIdx.y != 0 || bmin[b] != tn) return;   // uniform over the workgroup
    {
        int64_t before = 0;
        for (int k = tid; k < b; k += kBThreads) before += bmin[k] == tn ? bcnt[k] : 0;
        const int64_t row0 = pl->aoff[c] + block_sum(before, sh);
        if (tid == 0) L.brow[blockIdx.x] = int32_t(row0);
        const int64_t base = lo + int64_t(tid) * PER;
        int flags[PER];
        int k0 = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int64_t i = base + k;
            flags[k] = (i < hi && (all_active || b_next(st.t_tick, st.level, i) == tn)) ? 1 : 0;
            k0 += flags[k];
        }
        int64_t tot = 0;
        int64_t pos = row0 + block_excl(k0, sh, &tot);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (flags[k]) L.act[pos++] = int32_t(base + k);
    }
}

__device__ __forceinline__ int find_cluster(const int64_t *__restrict__ off, int nc, int64_t i)
{
    int lo = 0, hi = nc;   // off[lo] <= i < off[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (off[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

__global__ void __launch_bounds__(256)
k_b_cid(const int64_t *__restrict__ off, int nc, int64_t n, int32_t *__restrict__ cid)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) cid[i] = find_cluster(off, nc, i);
}

// One work item of a 64-lane workgroup: the rows of one i-tile against the
// j-range [j0, j1) of its cluster (cluster particles [base, base + nn), the
// first nh unsoftened).  The 64 lanes form R = 64 / JS groups of JS
// consecutive lanes; group r holds the tile's rows r and r + R (two rows per
// lane, so one record read from LDS serves two rows) and lane sl of the group
// takes j0 + sl, j0 + sl + JS, ... .  The JS lanes' sums are folded with a
// fixed butterfly and lane sl = 0 stores the group's rows.  A tile of `rows`
// active rows takes the largest JS (at most 64 and the tile length) with
// 2R >= rows, so a cluster's last, partly filled tile leaves at most half of
// its lanes idle (b_item_rows).
//
// NR = 1: the item is one of the two halves of the tile's rows (rows r + half R),
// one row per lane; each row's sums are the same bits.
template <class Pol, int P, int JS, int TILE, int NR>
__device__ __forceinline__ void b_item(const typename Pol::Rec *__restrict__ rec, const int32_t *__restrict__ al,
                                       int64_t na, int64_t row0, int64_t base, int64_t nn, int64_t nh, int64_t j0,
                                       int64_t j1, typename Pol::ET e2, int half, typename Pol::Rec (*tile)[TILE],
                                       double *__restrict__ dst)
{
    using Rec = typename Pol::Rec;
    using Part = typename Pol::Part;
    using ET = typename Pol::ET;
    static_assert(!Pol::kWithPot, "the batched force sums no potential");
    static_assert(TILE % JS == 0, "tile shape");
    constexpr int R = 64 / JS;
    constexpr int NV = 3 * (P / 2);
    constexpr int PIECES = int(sizeof(Rec) / 16);       // 16-byte pieces per record
    constexpr int PER_T = (TILE * PIECES + 63) / 64;     // pieces each lane moves per tile
    typedef uint4 __attribute__((may_alias)) piece_t;
    const int lane = int(threadIdx.x);
    const int r = lane / JS, sl = lane % JS;
    row0 += half * R;
    if (row0 >= na) return;   // no rows in this half (uniform over the workgroup)
    typename Pol::I ip[NR];
    int64_t iidx[NR];
    double acc[NR][NV];
    Part pt[NR][13];
#pragma unroll
    for (int k = 0; k < NR; ++k) {
        const int64_t q0 = row0 + r + k * R;
        const int64_t q = q0 < na ? q0 : na - 1;   // padding rows recompute the last row; never stored
        const int64_t ia = al[q];
        iidx[k] = (ia >= base && ia < base + nn) ? ia : base;
        ip[k] = Pol::load(rec[iidx[k]]);
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[k][c] = 0.0;
    }
    // unsoftened pairs among the cluster's first nh particles: this lane's j
    // of [j0, min(j1, base + nh)), each added into FP64 on its own
    const int64_t jh1 = j1 < base + nh ? j1 : base + nh;
    for (int64_t j = j0 + sl; j < jh1; j += JS) {
        const Rec rj = rec[j];
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            Part ph[13];
#pragma unroll
            for (int c = 0; c < 13; ++c) zero_part(ph[c]);
            const ET el = (iidx[k] - base < nh) ? ET(0) : e2;
            Pol::template pair<true>(ip[k], rj, el, j != iidx[k], ph);
#pragma unroll
            for (int c = 0; c < NV; ++c) acc[k][c] += to_double(ph[c]);
        }
    }
    // the softened rest through double-buffered LDS tiles; slots of the last
    // tile past j1 hold zero records (mass 0), which add exact zeros, as does
    // the row's own particle (zero separation, softened r^2 > 0)
    const int64_t js0 = j0 > base + nh ? j0 : base + nh;
    piece_t pre[PER_T];
    auto fetch = [&](int64_t jt) {
        const piece_t *src = reinterpret_cast<const piece_t *>(rec + jt);
        const int64_t avail = (j1 - jt) * PIECES;
#pragma unroll
        for (int k = 0; k < PER_T; ++k) {
            const int pc = lane + k * 64;
            if (pc < avail && pc < TILE * PIECES) pre[k] = src[pc];
            else pre[k] = piece_t{0u, 0u, 0u, 0u};
        }
    };
    if (js0 < j1) fetch(js0);
#pragma unroll
    for (int k = 0; k < NR; ++k)
#pragma unroll
        for (int c = 0; c < 13; ++c) zero_part(pt[k][c]);
    // every tile is taken whole (IT records per lane): the slots of the last
    // tile past j1 hold zero records.  The FP32 sums are added into FP64
    // every kChunk / TILE tiles (kChunk consecutive j of the range).
    constexpr int IT = TILE / JS;
    constexpr int FL = Pol::kChunk > 0 ? Pol::kChunk / TILE : (1 << 30);
    static_assert(Pol::kChunk % TILE == 0, "whole tiles per FP32 chunk");
    int since = 0;   // tiles since the last flush
    int buf = 0;
    for (int64_t jt = js0; jt < j1; jt += TILE) {
        piece_t *tw = reinterpret_cast<piece_t *>(tile[buf]);
#pragma unroll
        for (int k = 0; k < PER_T; ++k)
            if (lane + k * 64 < TILE * PIECES) tw[lane + k * 64] = pre[k];
        __syncthreads();   // tile ready; the other buffer is no longer read
        if (jt + TILE < j1) fetch(jt + TILE);
        const Rec *tr = tile[buf] + sl;
#pragma unroll 8
        for (int u = 0; u < IT; ++u) {
            const Rec rj = tr[u * JS];
#pragma unroll
            for (int k = 0; k < NR; ++k) Pol::template pair<false>(ip[k], rj, e2, true, pt[k]);
        }
        if (++since == FL) {
#pragma unroll
            for (int k = 0; k < NR; ++k)
#pragma unroll
                for (int c = 0; c < NV; ++c) {
                    acc[k][c] += to_double(pt[k][c]);
                    zero_part(pt[k][c]);
                }
            since = 0;
        }
        buf ^= 1;
    }
#pragma unroll
    for (int k = 0; k < NR; ++k)
#pragma unroll
        for (int c = 0; c < NV; ++c) acc[k][c] += to_double(pt[k][c]);
    // fold the group's JS lanes (consecutive lanes: xor offsets below JS stay in the group)
#pragma unroll
    for (int m = JS / 2; m > 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < NR; ++k)
#pragma unroll
            for (int c = 0; c < NV; ++c) acc[k][c] += __shfl_xor(acc[k][c], m, 64);
    if (sl == 0) {
#pragma unroll
        for (int k = 0; k < NR; ++k) {
            const int64_t q0 = row0 + r + k * R;
            if (q0 < na)
#pragma unroll
                for (int c = 0; c < NV; ++c) dst[int64_t(c) * na + q0] = acc[k][c];
        }
    }
}

// b_item with the largest lane group JS (at most 64 and the tile length)
// whose 2 * 64 / JS rows hold the tile's `rows` active rows.
template <class Pol, int P, int TILE, int ROWS, int NR>
__device__ __forceinline__ void b_item_rows(int rows, const typename Pol::Rec *__restrict__ rec,
                                            const int32_t *__restrict__ al, int64_t na, int64_t row0, int64_t base,
                                            int64_t nn, int64_t nh, int64_t j0, int64_t j1, typename Pol::ET e2,
                                            int half, typename Pol::Rec (*tile)[TILE], double *__restrict__ dst)
{
    constexpr int J2 = 2 < TILE ? 2 : TILE, J4 = 4 < TILE ? 4 : TILE, J8 = 8 < TILE ? 8 : TILE;
    constexpr int J16 = 16 < TILE ? 16 : TILE, J32 = 32 < TILE ? 32 : TILE, J64 = 64 < TILE ? 64 : TILE;
    if (ROWS == 128 && rows > 64) b_item<Pol, P, 1, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else if (rows > 32) b_item<Pol, P, J2, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else if (rows > 16) b_item<Pol, P, J4, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else if (rows > 8) b_item<Pol, P, J8, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else if (rows > 4) b_item<Pol, P, J16, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else if (rows > 2) b_item<Pol, P, J32, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    else b_item<Pol, P, J64, TILE, NR>(rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
}

// Measured (32 clusters of 2^10 to 2^14, MIXED order 6, to t = 1/256, 208 steps):
// 20578 us with two rows per lane, pieces of at least 256 particles (the cut
// rounded up) and every item claimed, 17464 with one row per lane, pieces of
// 128 and first items dealt; the median step's force kernel 42 -> 16 us.
// 128 clusters of 2^10 to 2^16 (two rows per lane, kHalfTilesBelow) 49.5 -> 49.5
// ms.
//
// Persistent force kernel.  The step's items (in cluster rank order: item
// = cluster ord[rank], i-tile, j-split) form 8 contiguous ranges, one per
// XCD, each with its own queue counter.  The dispatcher places workgroup g on
// XCD g mod 8: a workgroup takes items from its own XCD's range (a few
// clusters, whose j records that XCD's L2 then holds), then from the other
// ranges in turn, and leaves when all eight are empty.  Its first item is
// dealt by its number, without the counter, which an eighth of the workgroups
// would ask at once (some 0.1 us each; a step of 3600 items took 80 us that
// way).  Every wave reaches the exit: the counters only grow.  Tiles of ROWS = 64 or 128 rows run as one wave
// with two rows per lane (b_item); 256-row tiles as four waves with one row
// per lane.

// Waves per SIMD the register allocation of k_b_force aims for: the
// one-wave workgroups of the FP32 pair arithmetic (MIXED) at orders 4 and 6
// fit 3 without spills (otherwise the compiler's own choice).
template <class Pol, int P, int BLOCK, int NR>
constexpr int b_waves() { return BLOCK == 64 && NR == 2 && sizeof(typename Pol::Part) == 4 && P <= 6 ? 3 : 1; }

// One work item: the i-tile and j-split `local` of the cluster described by d.
template <class Pol, int P, int BLOCK, int TILE, int ROWS, int NR>
__device__ __forceinline__ void b_run(const BatchRank &d, int64_t local, const typename Pol::Rec *__restrict__ rec,
                                      const int32_t *__restrict__ act, typename Pol::ET e2, int64_t n_hard, int ncomp,
                                      double *__restrict__ part, typename Pol::Rec (*tile)[TILE])
{
    constexpr bool kHalves = ROWS == 64 && NR == 1;   // two items per row tile and split
    const int half = kHalves ? int(local & 1) : 0;
    const uint32_t lq = uint32_t(kHalves ? local >> 1 : local), sp = uint32_t(d.sp);
    const int64_t tile_i = lq / sp, split = lq % sp;
    const int64_t na = d.na, base = d.base, nn = d.nn, jc = d.jc;
    const int64_t j0 = base + split * jc;
    const int64_t j1 = (split + 1) * jc < nn ? base + (split + 1) * jc : base + nn;
    const int64_t nh = n_hard < nn ? n_hard : nn;
    double *dst = part + d.poff + split * ncomp * na;
    const int32_t *al = act + d.aoff;
    if constexpr (BLOCK == 64) {
        const int64_t row0 = tile_i * ROWS;
        const int64_t rows = na - row0 < ROWS ? na - row0 : ROWS;
        b_item_rows<Pol, P, TILE, ROWS, NR>(int(rows), rec, al, na, row0, base, nn, nh, j0, j1, e2, half, tile, dst);
    } else {
        // this lane's active row
        const int64_t q0 = tile_i * BLOCK + threadIdx.x;
        const int64_t q = q0 < na ? q0 : na - 1;
        typename Pol::I ip[1];
        int64_t iidx[1];
        double acc[1][13];
        const int64_t ia = al[q];
        iidx[0] = (ia >= base && ia < base + nn) ? ia : base;
        ip[0] = Pol::load(rec[iidx[0]]);
#pragma unroll
        for (int cc = 0; cc < 13; ++cc) acc[0][cc] = 0.0;
        hard_pairs<Pol, 1>(rec, j0, (j1 < base + nh) ? j1 : base + nh, base, nh, e2, ip, iidx, acc);
        const int64_t js0 = (j0 > base + nh) ? j0 : base + nh;
        lds_tiles<Pol, 1, BLOCK, 2, TILE>(rec, js0, j1, e2, ip, iidx, tile, acc);
        if (q0 < na) {
#pragma unroll
            for (int cc = 0; cc < 3 * (P / 2); ++cc) dst[int64_t(cc) * na + q0] = acc[0][cc];
        }
    }
}

__device__ __forceinline__ int64_t wave_uniform(uint32_t v) { return int64_t(uint32_t(__builtin_amdgcn_readfirstlane(v))); }

template <class Pol, int P, int BLOCK, int TILE, int ROWS, int NR>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(b_waves<Pol, P, BLOCK, NR>())))
k_b_force(const typename Pol::Rec *__restrict__ rec, int nc, const int32_t *__restrict__ act,
          BatchPlan *__restrict__ pl, double eps2, int64_t n_hard, int ncomp, double *__restrict__ part)
{
    using Rec = typename Pol::Rec;
    using ET = typename Pol::ET;
    __shared__ Rec tile[2][TILE];
    __shared__ uint32_t s_take;
    const ET e2 = ET(eps2);
    const BatchRank *__restrict__ rk = pl->rank;
    const int64_t total = rk[nc - 1].i1;
    const int x0 = int(blockIdx.x) % kXcds;
    const int64_t ahead = 2 * ((int64_t(gridDim.x) + kXcds - 1) / kXcds);   // two items per workgroup of an XCD
    for (int v = 0; v < kXcds; ++v) {
        const int xr = (x0 + v) % kXcds;
        const int64_t r0 = total * xr / kXcds, len = total * (xr + 1) / kXcds - r0;
        uint32_t *q = &pl->queue[xr * 16];
        int64_t take;
        if (v == 0) {
            // the first item is dealt: the range's counter starts past the
            // items of its XCD's workgroups (b_dealt)
            take = int64_t(blockIdx.x) / kXcds;
        } else {
            // an exhausted range is seen with a load, without adding to its counter
            __syncthreads();   // the previous item's tiles and s_take are no longer read
            if (threadIdx.x == 0) {
                const uint32_t seen = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s_take = seen >= uint32_t(len) ? uint32_t(len) : atomicAdd(q, 1u);
            }
            __syncthreads();
            take = wave_uniform(s_take);   // scalar: the cluster, ranges and loop bounds stay in SGPRs
        }
        if (take < len) {
            // rank of the item's cluster: rk[lo].i0 <= item < rk[lo].i1; the
            // items a workgroup takes from one range only increase
            int lo = 0;
            {
                int hi = nc;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) / 2;
                    if (rk[mid].i0 <= r0 + take) lo = mid; else hi = mid;
                }
            }
            const bool one = len <= b_dealt(int(gridDim.x), xr);   // every item of the range was dealt
            for (;;) {
                const int64_t item = r0 + take;
                while (rk[lo].i1 <= item) ++lo;
                const BatchRank d = rk[lo];
                // one wave, far from the range's end: the next item is claimed
                // now and its number read after this one, so the atomic's latency
                // is not waited for (near the end a claimed item would wait for
                // this one while other workgroups idle)
                const bool early = BLOCK == 64 && take + ahead < len;
                uint32_t nxt = 0u;
                if (early && threadIdx.x == 0) nxt = atomicAdd(q, 1u);
                b_run<Pol, P, BLOCK, TILE, ROWS, NR>(d, item - d.i0, rec, act, e2, n_hard, ncomp, part, tile);
                if (one) break;
                if (early) {
                    take = wave_uniform(nxt);
                } else {
                    __syncthreads();   // the item's tiles and s_take are no longer read
                    if (threadIdx.x == 0) s_take = atomicAdd(q, 1u);
                    __syncthreads();
                    take = wave_uniform(s_take);
                }
                if (take >= len) break;
            }
        }
        // a step with no more items than workgroups is all dealt: nothing is
        // left in the other ranges
        if (total <= int64_t(gridDim.x) / kXcds * kXcds) return;
    }
}

// Row r of the concatenated active list: sum of its cluster's split partials
// into outputs [3][stride] (acc, jerk, snap, crackle).  A group of kRedLanes
// consecutive lanes owns a row (its cluster found through the row's particle):
// for every component, lane l adds splits l, l + kRedLanes, ... in order,
// then the group folds its sums with a fixed butterfly (the order depends
// only on the cluster's split count).
constexpr int kRedLanes = 16;

template <int P>
__global__ void __launch_bounds__(256)
k_b_reduce(int nc, int64_t n, const BatchPlan *__restrict__ pl, const int32_t *__restrict__ act,
           const int32_t *__restrict__ cid, int ncomp, const double *__restrict__ part, double *__restrict__ o0,
           double *__restrict__ o1, double *__restrict__ o2, double *__restrict__ o3, int64_t stride)
{
    constexpr int NV = 3 * (P / 2);
    const int64_t total = pl->aoff[nc];
    const int l = int(threadIdx.x) % kRedLanes;
    const int64_t groups = int64_t(gridDim.x) * blockDim.x / kRedLanes;
    double *outs[4] = {o0, o1, o2, o3};
    // the lanes of a group share r, so they run the same iterations and their
    // exchanges (within the group) always find their partners active
    for (int64_t r = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kRedLanes; r < total; r += groups) {
        const int64_t i = act[r];
        const int c = (i >= 0 && i < n) ? cid[i] : 0;
        const int64_t na = pl->nact[c], q = r - pl->aoff[c];
        if (q < 0 || q >= na) continue;   // never for a consistent plan; the whole group skips together
        const double *src = part + pl->poff[c];
        const int sp = pl->split[c];
        double s[NV];
#pragma unroll
        for (int cc = 0; cc < NV; ++cc) s[cc] = 0.0;
        for (int k = l; k < sp; k += kRedLanes)
#pragma unroll
            for (int cc = 0; cc < NV; ++cc) s[cc] += src[(int64_t(k) * ncomp + cc) * na + q];
#pragma unroll
        for (int m = kRedLanes / 2; m > 0; m >>= 1)
#pragma unroll
            for (int cc = 0; cc < NV; ++cc) s[cc] += __shfl_xor(s[cc], m, 64);
        // lane l of the group stores component l
#pragma unroll
        for (int cc = 0; cc < NV; ++cc) {
            double *o = outs[cc / 3];
            if (l == cc % kRedLanes && o) o[(cc % 3) * stride + r] = s[cc];
        }
    }
}

// The end of a step for block (c, b): the split partials of its active rows
// summed (as k_b_reduce: a group of kRedLanes lanes per row, the same order) to the
// step's forces, then the rows corrected, kFinRows at a time.  The workgroups y of
// a block share its rows.
constexpr int kFinRows = 128;

template <int P>
__global__ void __launch_bounds__(kBThreads)
k_b_finish(BatchLaunch L, nbody_state st, double eta, int rule, int k_min, int k_max)
{
    constexpr int NV = 3 * (P / 2);
    __shared__ double f[NV][kFinRows];
    const int c = L.blk[2 * blockIdx.x], b = L.blk[2 * blockIdx.x + 1], tid = int(threadIdx.x);
    const BatchPlan *pl = L.plan;
    const int64_t na = pl->nact[c];
    if (na == 0) return;
    const int64_t tn = L.tnext[c];
    if (L.bmin[int64_t(c) * L.nb + b] != tn) return;
    const int all = L.bcnt[int64_t(c) * L.nb + b], first = all * int(blockIdx.y) / int(gridDim.y);
    const int cnt = all * (int(blockIdx.y) + 1) / int(gridDim.y) - first;
    const int64_t row0 = L.brow[blockIdx.x] + first;   // of the step's active list
    const int64_t q0 = row0 - pl->aoff[c];         // of the cluster's
    const double *src = L.part + pl->poff[c];
    const int sp = pl->split[c], ncomp = NV;
    double *const d[6] = {st.d[0], st.d[1], st.d[2], st.d[3], st.d[4], st.d[5]};
    const double *const fnew[4] = {f[0], f[3], NV > 6 ? f[6 % NV] : nullptr, NV > 9 ? f[9 % NV] : nullptr};
    const int l = tid % kRedLanes;
    for (int r0 = 0; r0 < cnt; r0 += kFinRows) {
        const int rows = cnt - r0 < kFinRows ? cnt - r0 : kFinRows;
        for (int r = tid / kRedLanes; r < rows; r += kBThreads / kRedLanes) {
            const int64_t q = q0 + r0 + r;
            double s[NV];
#pragma unroll
            for (int cc = 0; cc < NV; ++cc) s[cc] = 0.0;
            for (int k = l; k < sp; k += kRedLanes)
#pragma unroll
                for (int cc = 0; cc < NV; ++cc) s[cc] += src[(int64_t(k) * ncomp + cc) * na + q];
#pragma unroll
            for (int m = kRedLanes / 2; m > 0; m >>= 1)
#pragma unroll
                for (int cc = 0; cc < NV; ++cc) s[cc] += __shfl_xor(s[cc], m, 64);
            // lane l of the group stores component l
#pragma unroll
            for (int cc = 0; cc < NV; ++cc)
                if (l == cc % kRedLanes) {
                    f[cc][r] = s[cc];
                    L.force[int64_t(cc) * L.n + row0 + r0 + r] = s[cc];
                }
        }
        __syncthreads();
        if (tid < rows) {
            const int64_t i = L.act[row0 + r0 + tid];
            const int fl = correct_one<P>(L.n, i, tn, fnew, kFinRows, tid, st.x, st.v, d, st.t_tick, st.level, eta, rule,
                                          k_min, k_max);
            if (fl & 2) atomicAdd(&L.ctr->underflow, 1ull);
            if (fl & 1) atomicAdd(&L.ctr->nonfinite, 1ull);
        }
        __syncthreads();   // f is no longer read
    }
}

// Work queues back to their start (a second force pass on the same plan).
__global__ void k_b_requeue(BatchPlan *__restrict__ pl, int nc, int grid)
{
    if (threadIdx.x < kXcds) pl->queue[threadIdx.x * 16] = b_queue_start(pl->ioff[nc], grid, int(threadIdx.x));
}

unsigned nblk(int64_t n, int b) { return unsigned((n + b - 1) / b); }

// Workgroups of the grid-stride kernels whose work is bounded by the step's
// active count (at most n rows): enough to fill the chip, few enough that a
// step with a small active set does not pay for launching idle workgroups.
constexpr unsigned kStrideGrid = 2048;

template <class Pol, int P>
hipError_t force_p(const BatchLaunch &L, const void *rec, hipStream_t s)
{
    const auto *r = static_cast<const typename Pol::Rec *>(rec);
    if (L.itile == 64 && L.halves == 2)
        hipLaunchKernelGGL((k_b_force<Pol, P, 64, kBTile, 64, 1>), dim3(L.force_grid), dim3(64), 0, s, r, L.nc, L.act,
                           L.plan, L.eps2, L.n_hard, 3 * (P / 2), L.part);
    else if (L.itile == 64)
        hipLaunchKernelGGL((k_b_force<Pol, P, 64, kBTile, 64, 2>), dim3(L.force_grid), dim3(64), 0, s, r, L.nc, L.act,
                           L.plan, L.eps2, L.n_hard, 3 * (P / 2), L.part);
    else if (L.itile == 128)
        hipLaunchKernelGGL((k_b_force<Pol, P, 64, kBTile, 128, 2>), dim3(L.force_grid), dim3(64), 0, s, r, L.nc, L.act,
                           L.plan, L.eps2, L.n_hard, 3 * (P / 2), L.part);
    else
        hipLaunchKernelGGL((k_b_force<Pol, P, 256, 128, 256, 1>), dim3(L.force_grid), dim3(256), 0, s, r, L.nc, L.act,
                           L.plan, L.eps2, L.n_hard, 3 * (P / 2), L.part);
    return hipGetLastError();
}

template <int P>
hipError_t force_prec(int precision, const BatchLaunch &L, const void *rec, hipStream_t s)
{
    if (precision == NBODY_MIXED) return force_p<PolMx<P, false>, P>(L, rec, s);
    if (precision == NBODY_DS) return force_p<PolDS<P, false>, P>(L, rec, s);
    return force_p<PolF64<P, false>, P>(L, rec, s);
}

template <int P>
hipError_t reduce_p(const BatchLaunch &L, double *o0, double *o1, double *o2, double *o3, hipStream_t s)
{
    const unsigned g = nblk(L.n * kRedLanes, 256);
    hipLaunchKernelGGL((k_b_reduce<P>), dim3(g < kStrideGrid ? g : kStrideGrid), dim3(256), 0, s, L.nc, L.n, L.plan,
                       L.act, L.cid, 3 * (P / 2), L.part, o0, o1, o2, o3, L.n);
    return hipGetLastError();
}

}  // namespace

hipError_t batch_requeue(const BatchLaunch &L, hipStream_t s)
{
    hipLaunchKernelGGL(k_b_requeue, dim3(1), dim3(64), 0, s, L.plan, L.nc, L.force_grid);
    return hipGetLastError();
}

template <class Pol, int P>
int resident_p(int itile, int halves, int device)
{
    int per_cu = 0, cus = 0;
    hipError_t e;
    if (itile == 64 && halves == 2)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_b_force<Pol, P, 64, kBTile, 64, 1>, 64, 0);
    else if (itile == 64)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_b_force<Pol, P, 64, kBTile, 64, 2>, 64, 0);
    else if (itile == 128)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_b_force<Pol, P, 64, kBTile, 128, 2>, 64, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_b_force<Pol, P, 256, 128, 256, 1>, 256, 0);
    if (e != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}

template <int P>
int resident_prec(int precision, int itile, int halves, int device)
{
    if (precision == NBODY_MIXED) return resident_p<PolMx<P, false>, P>(itile, halves, device);
    if (precision == NBODY_DS) return resident_p<PolDS<P, false>, P>(itile, halves, device);
    return resident_p<PolF64<P, false>, P>(itile, halves, device);
}

int batch_force_resident(int order, int precision, int itile, int halves, int device)
{
    if (order == 4) return resident_prec<4>(precision, itile, halves, device);
    if (order == 6) return resident_prec<6>(precision, itile, halves, device);
    return resident_prec<8>(precision, itile, halves, device);
}

hipError_t batch_cid(const BatchLaunch &L, hipStream_t s)
{
    hipLaunchKernelGGL(k_b_cid, dim3(nblk(L.n, 256)), dim3(256), 0, s, L.off, L.nc, L.n, L.cid);
    return hipGetLastError();
}

hipError_t batch_schedule(const BatchLaunch &L, const nbody_state &st, int all_active, int order, hipStream_t s)
{
    hipLaunchKernelGGL(k_b_schedule, dim3(unsigned(L.nblk)), dim3(kBThreads), 0, s, L, st.t_tick, st.level, all_active,
                       3 * (order / 2));
    return hipGetLastError();
}

hipError_t batch_list_all(const BatchLaunch &L, const nbody_state &st, hipStream_t s)
{
    hipLaunchKernelGGL((k_b_advance<4, -1>), dim3(unsigned(L.nblk)), dim3(kBThreads), 0, s, L, st, 1, nullptr);
    return hipGetLastError();
}

hipError_t batch_advance(const BatchLaunch &L, const nbody_state &st, int order, int precision, void *rec,
                         hipStream_t s)
{
#define NB_BP(P, PREC) \
    hipLaunchKernelGGL((k_b_advance<P, PREC>), dim3(unsigned(L.nblk), kBBlock / kBThreads), dim3(kBThreads), 0, s, L, st, \
                       0, rec)
#define NB_BP_P(P)                                          \
    if (precision == NBODY_FP64) NB_BP(P, NBODY_FP64);     \
    else NB_BP(P, NBODY_MIXED)
    if (order == 4) { NB_BP_P(4); }
    else if (order == 6) { NB_BP_P(6); }
    else { NB_BP_P(8); }
#undef NB_BP_P
#undef NB_BP
    return hipGetLastError();
}

hipError_t batch_force(const BatchLaunch &L, int order, int precision, const void *rec, hipStream_t s)
{
    if (order == 4) return force_prec<4>(precision, L, rec, s);
    if (order == 6) return force_prec<6>(precision, L, rec, s);
    return force_prec<8>(precision, L, rec, s);
}

hipError_t batch_reduce(const BatchLaunch &L, int order, double *o0, double *o1, double *o2, double *o3,
                        hipStream_t s)
{
    if (order == 4) return reduce_p<4>(L, o0, o1, o2, o3, s);
    if (order == 6) return reduce_p<6>(L, o0, o1, o2, o3, s);
    return reduce_p<8>(L, o0, o1, o2, o3, s);
}

hipError_t batch_finish(const BatchLaunch &L, const nbody_config &c, const nbody_state &st, hipStream_t s)
{
    // workgroups per block: enough that a block of 1024 active rows is not one
    // workgroup's 64 rounds of row sums, few enough that a large ensemble does
    // not launch mostly empty ones
    const unsigned y = L.nblk <= 512 ? 8u : (L.nblk <= 2048 ? 4u : 2u);
#define NB_BC(P)                                                                                               \
    hipLaunchKernelGGL((k_b_finish<P>), dim3(unsigned(L.nblk), y), dim3(kBThreads), 0, s, L, st, c.eta, dt_rule_of(c), \
                       int(c.k_min), int(c.k_max))
    if (c.order == 4) NB_BC(4);
    else if (c.order == 6) NB_BC(6);
    else NB_BC(8);
#undef NB_BC
    return hipGetLastError();
}

}  // namespace nb
