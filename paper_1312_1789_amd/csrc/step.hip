// step.hip -- the end of a block step and the schedule of the next one in one
// kernel, for runs of block steps (paper: Abstract; Sec. "Codes description":
// individual hierarchical block time steps).
//
// A small block step is bound by launches: its arithmetic takes a few
// microseconds, a kernel launch about four from the host and one or two of idle
// device after its predecessor.  Separate kernels for the split reduction, the
// post-Newtonian terms, the corrector and the scheduler's two passes made a
// step six or seven launches and one round trip to the host between them.
// Here one workgroup owns 256 consecutive particles: it sums its active rows'
// partial forces, corrects them, takes the block's next time and lists the
// particles at it.  The last workgroup to arrive takes the least of the block
// times, numbers the active particles, writes their list and publishes the
// schedule to the host.  No workgroup waits for another.
//
// The scheduler's result is also what the next small step's kernels read on the
// device (DevScalars), so the host may enqueue them before it has seen it.
//
// A small step is then the force kernel and this one, 6 and 10 us at n = 1024,
// 8 and 12 at n = 30000 (9 to 14 dependent memory round trips), with 1 to 2 us
// between kernels: whole runs (n = 1024 FP64 order 4, t = 1/32) 7632 -> 4252 us,
// (n = 30002 FP64 order 4 with a post-Newtonian binary, t = 1/128) 22202 -> 14532
// us, (n = 80000 MIXED order 6, t = 1/512) 14861 -> 14297 us.
#include <climits>

#include "pn.h"

namespace nb {
namespace {

constexpr int kSW = kStepBlock / 64;   // waves per workgroup
constexpr int kStepBlocks = int(kStepMaxN / kStepBlock);

__device__ __forceinline__ int64_t next_of(int64_t t, int32_t level) { return t + (int64_t(1) << (kLevelMax - level)); }

// Rank of this thread among the threads of the block with `flag`, in thread
// order, and their number.  Synchronises the block twice.
__device__ __forceinline__ int block_rank(bool flag, int *wcnt, int *total)
{
    const int lane = int(threadIdx.x) & 63, w = int(threadIdx.x) >> 6;
    const unsigned long long m = __ballot(flag);
    __syncthreads();   // wcnt is no longer read
    if (lane == 0) wcnt[w] = __popcll(m);
    __syncthreads();
    int before = __popcll(m & ((1ull << lane) - 1ull)), tot = 0;
    for (int k = 0; k < kSW; ++k) {
        if (k < w) before += wcnt[k];
        tot += wcnt[k];
    }
    *total = tot;
    return before;
}

__device__ __forceinline__ int64_t block_min(int64_t v, int64_t *wm)
{
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t u = __shfl_xor(v, o, 64);
        v = u < v ? u : v;
    }
    __syncthreads();   // wm is no longer read
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t r = wm[0];
    for (int k = 1; k < kSW; ++k) r = wm[k] < r ? wm[k] : r;
    return r;
}

// Sums of the partial groups of rows [q0, q0 + cnt), in the order of k_reduce, to
// f[component][row].
template <int L, int NV>
__device__ __forceinline__ void sum_rows(const double *__restrict__ part, int64_t na, int ng, int q0, int cnt,
                                         double (*f)[kSmallMax])
{
    const int l = int(threadIdx.x) % L;
    for (int e = int(threadIdx.x) / L; e < cnt * NV; e += kStepBlock / L) {
        const int c = e / cnt, row = e - c * cnt;
        const double *src = part + (int64_t(c) * na + q0 + row) * ng;
        double s = 0.0;
        int k = l;
        for (; k + 7 * L < ng; k += 8 * L) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[k + u * L];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; k < ng; k += L) s += src[k];
        // the lanes of a group share e, so their partners run the same iterations
#pragma unroll
        for (int m = L / 2; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
        if (l == 0) f[c][row] = s;
    }
}

// What workgroups tell each other goes through agent-scope atomic accesses, which
// are performed where all XCDs see them, and is ordered by waiting for the
// stores before the arrival is counted.  (Fences instead make every wave write
// back and invalidate its XCD's L2: this kernel then took 24 us at n = 80000.)
template <class T> __device__ __forceinline__ T shared_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void shared_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The last workgroup: t_next, the active particles before each block, their
// number, the published schedule, and the list when it is short enough.  PER
// consecutive blocks per thread.
template <int PER>
__device__ __forceinline__ void schedule(const StepArgs &a, int nb, int64_t *wm, int *wcnt, int32_t *soff)
{
    const int tid = int(threadIdx.x);
    const StepScratch &w = a.w;
    const int b0 = tid * PER;
    int64_t bt[PER];
    int bc[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int bb = b0 + k < nb ? b0 + k : nb - 1;
        bt[k] = shared_load(&w.blk[bb].t_next);
        bc[k] = int(shared_load(&w.blk[bb].count));
    }
    int64_t mn = INT64_MAX;
#pragma unroll
    for (int k = 0; k < PER; ++k) mn = bt[k] < mn ? bt[k] : mn;   // (a repeated last block changes nothing)
    const int64_t tn = block_min(mn, wm);
    int mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (b0 + k >= nb || bt[k] != tn) bc[k] = 0;
        mine += bc[k];
    }
    // exclusive prefix over the threads
    const int lane = tid & 63, wv = tid >> 6;
    int incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wcnt[wv] = incl;
    __syncthreads();
    int off = incl - mine, total = 0;
    for (int k = 0; k < kSW; ++k) {
        if (k < wv) off += wcnt[k];
        total += wcnt[k];
    }
    if (tid == 0) {
        DevScalars *sc = a.sc;
        const unsigned long long nf = shared_load(&sc->nonfinite), uf = shared_load(&sc->underflow);
        const int64_t seq = a.mode == kStepSchedule ? a.seq : sc->seq + 1;
        HostScalars *pub = a.pub + (seq & (kPubSlots - 1));
        __hip_atomic_store(&pub->t_next, tn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->n_act, int64_t(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->underflow, uf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->nonfinite, nf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        if (a.mode == kStepSchedule) sc->nonfinite0 = nf;
        sc->halt = (a.mode == kStepSchedule || nf == sc->nonfinite0) ? 0 : 1;
        sc->seq = seq;
        sc->t_next = tn;
        sc->n_act = total;
        stores_done();
        __hip_atomic_store(&pub->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (b0 + k < nb) {
            soff[b0 + k] = off;
            w.boff[b0 + k] = off;
            off += bc[k];
        }
    __syncthreads();
    if (total > kStepGather) return;   // listed by k_step_gather
    for (int e = tid; e < total; e += kStepBlock) {
        // the block of entry e: the last one with soff <= e (blocks without
        // active particles share their successor's offset)
        int lo = 0, hi = nb;
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (soff[mid] <= e) lo = mid; else hi = mid;
        }
        w.act[e] = shared_load(&w.cand[int64_t(lo) * kStepBlock + (e - soff[lo])]);
    }
}

template <int P, bool PN>
__global__ void __launch_bounds__(kStepBlock)
k_step(StepArgs a)
{
    constexpr int NV = 3 * (P / 2);
    __shared__ double f[NV][kSmallMax];
    __shared__ int64_t wm[kSW];
    __shared__ int wcnt[kSW];
    __shared__ int32_t soff[kStepBlocks];
    __shared__ int s_last;
    const int64_t n = a.cfg.n;
    const int b = int(blockIdx.x), nb = int(gridDim.x), tid = int(threadIdx.x);
    const int64_t i = int64_t(b) * kStepBlock + tid;
    if (a.mode == kStepSmall && !small_step(*a.sc, a.tab, a.t_limit)) return;
    int64_t *t_tick = a.st.t_tick;
    int32_t *level = a.st.level;
    int64_t next = i < n ? next_of(t_tick[i], level[i]) : INT64_MAX;
    if (a.mode != kStepSchedule) {
        const int64_t na = a.sc->n_act, tn = a.sc->t_next;
        const bool active = i < n && next == tn;
        int cnt = 0;
        const int rank = block_rank(active, wcnt, &cnt);
        if (cnt > 0) {   // uniform over the block
            const int64_t q0 = a.w.boff[b];
            double *fp[4];
            int64_t stride, row;
            if (a.mode == kStepSmall) {
                const int gs = na <= 16 ? 8 : (na <= 32 ? 4 : 2);   // small_group
                const int ng = (a.tab.n_split[na - 1] + gs - 1) / gs;
                const int L = reduce_lanes(ng);
                if (L == 1) sum_rows<1, NV>(a.part, na, ng, int(q0), cnt, f);
                else if (L == 4) sum_rows<4, NV>(a.part, na, ng, int(q0), cnt, f);
                else if (L == 16) sum_rows<16, NV>(a.part, na, ng, int(q0), cnt, f);
                else sum_rows<64, NV>(a.part, na, ng, int(q0), cnt, f);
                __syncthreads();
                stride = kSmallMax;
                row = rank;
#pragma unroll
                for (int k = 0; k < 4; ++k) fp[k] = k < P / 2 ? f[3 * k] : nullptr;
            } else {
                stride = na;
                row = q0 + rank;
#pragma unroll
                for (int k = 0; k < 4; ++k) fp[k] = a.f[k];
            }
            double *x = a.st.x, *v = a.st.v;
            double *const d[6] = {a.st.d[0], a.st.d[1], a.st.d[2], a.st.d[3], a.st.d[4], a.st.d[5]};
            if constexpr (PN) {
                // the hard particles are all in the first block: their terms from
                // the stored state, before any of them is corrected
                if (b == 0) {
                    if (active && i < a.cfg.n_hard) {
                        double w[4][3];
                        const PnDs ds{{d[0], d[1], d[2], d[3], d[4], d[5]}};
                        pn_row<P>(n, a.cfg.n_hard, i, a.st.m, x, v, ds, t_tick, tn, a.cfg.c_light, int(a.cfg.pn_terms),
                                  w);
#pragma unroll
                        for (int k = 0; k < P / 2; ++k)
#pragma unroll
                            for (int l = 0; l < 3; ++l) fp[k][l * stride + row] += w[k][l];
                    }
                    __syncthreads();
                }
            }
            if (active) {
                const double *const fnew[4] = {fp[0], fp[1], fp[2], fp[3]};
                const int fl = correct_one<P>(n, i, tn, fnew, stride, row, x, v, d, t_tick, level, a.cfg.eta,
                                              a.rule, int(a.cfg.k_min), int(a.cfg.k_max));
                if (fl & 2) atomicAdd(&a.sc->underflow, 1ull);
                if (fl & 1) atomicAdd(&a.sc->nonfinite, 1ull);
                next = next_of(t_tick[i], level[i]);
            }
        }
    }
    // the block's next time, and its particles at it in increasing order
    const int64_t bm = block_min(next, wm);
    int cnt = 0;
    const int rank = block_rank(i < n && next == bm, wcnt, &cnt);
    if (i < n && next == bm) shared_store(&a.w.cand[int64_t(b) * kStepBlock + rank], int32_t(i));
    if (tid == 0) {
        shared_store(&a.w.blk[b].t_next, bm);
        shared_store(&a.w.blk[b].count, int64_t(cnt));
    }
    // arrival: the last of each kStepSub workgroups counts for them all
    stores_done();
    __syncthreads();
    if (tid == 0) {
        const int sub = b / kStepSub, subs = (nb + kStepSub - 1) / kStepSub;
        const unsigned size = unsigned(nb - sub * kStepSub < kStepSub ? nb - sub * kStepSub : kStepSub);
        bool last = atomicAdd(&a.w.arrive[1 + sub], 1u) == size - 1;
        if (last) {
            shared_store(&a.w.arrive[1 + sub], 0u);   // for the next launch
            if (subs > 1) {
                last = atomicAdd(&a.w.arrive[0], 1u) == unsigned(subs) - 1;
                if (last) shared_store(&a.w.arrive[0], 0u);
            }
        }
        s_last = last ? 1 : 0;
    }
    __syncthreads();
    if (!s_last) return;
    if (nb <= kStepBlock) schedule<1>(a, nb, wm, wcnt, soff);
    else if (nb <= 4 * kStepBlock) schedule<4>(a, nb, wm, wcnt, soff);
    else schedule<kStepBlocks / kStepBlock>(a, nb, wm, wcnt, soff);
}

__global__ void __launch_bounds__(kStepBlock)
k_step_gather(StepScratch w, const DevScalars *__restrict__ sc)
{
    const int b = int(blockIdx.x);
    if (w.blk[b].t_next != sc->t_next) return;
    if (int(threadIdx.x) < int(w.blk[b].count))
        w.act[w.boff[b] + threadIdx.x] = w.cand[int64_t(b) * kStepBlock + threadIdx.x];
}

}  // namespace

hipError_t launch_step(const StepArgs &a, hipStream_t s)
{
    const unsigned nb = unsigned((a.cfg.n + kStepBlock - 1) / kStepBlock);
#define NB_STEP(P)                                                                             \
    if (a.pn) hipLaunchKernelGGL((k_step<P, true>), dim3(nb), dim3(kStepBlock), 0, s, a);      \
    else hipLaunchKernelGGL((k_step<P, false>), dim3(nb), dim3(kStepBlock), 0, s, a)
    if (a.cfg.order == 4) { NB_STEP(4); }
    else if (a.cfg.order == 6) { NB_STEP(6); }
    else { NB_STEP(8); }
#undef NB_STEP
    return hipGetLastError();
}

hipError_t launch_step_gather(const StepScratch &w, int64_t n, const DevScalars *sc, hipStream_t s)
{
    const unsigned nb = unsigned((n + kStepBlock - 1) / kStepBlock);
    hipLaunchKernelGGL(k_step_gather, dim3(nb), dim3(kStepBlock), 0, s, w, sc);
    return hipGetLastError();
}

}  // namespace nb
