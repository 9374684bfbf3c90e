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
// A small step is then the force kernel and this one, with 1 to 2 us between
// kernels: whole runs against the separate kernels (n = 1024 FP64 order 4, t = 1/32)
// 6573 -> 2873 us, (n = 30002 FP64 order 4 with a post-Newtonian binary, t = 1/128)
// 21570 -> 12664 us, (n = 80000 MIXED order 6, t = 1/512) 15245 -> 14083 us.
//
// It is a chain of dependent round trips to memory, most of them to lines that
// another XCD has written (about 1 us each), and of serial arithmetic on a few
// lanes.  So all that a stage reads is loaded together with what decides whether
// it is needed: the particles' times with the scheduler's result, the active
// ones' state before their forces are summed, the first candidates of every
// block with its time; least times and prefix sums are taken with moves between
// lanes, the corrector multiplies by powers of two instead of dividing, and the
// words for the host are stored without an order.  5.9 us at n = 1024, 9.3 at n =
// 30002 with the binary and 9.8 at n = 80000 (with one load waiting for another 7.2,
// 10.4 and 10.8).
#include <climits>

#include "pn.h"

namespace nb {
namespace {

constexpr int kSW = kStepBlock / 64;   // waves per workgroup
constexpr int kStepBlocks = int(kStepMaxN / kStepBlock);

__device__ __forceinline__ int64_t next_of(int64_t t, int32_t level) { return t + (int64_t(1) << (kLevelMax - level)); }

// Rank of this thread among the threads of the block with `flag`, in thread
// order, and their number.  Synchronises the block once (wcnt is not used again).
__device__ __forceinline__ int block_rank(bool flag, int *wcnt, int *total)
{
    const int lane = int(threadIdx.x) & 63, w = int(threadIdx.x) >> 6;
    const unsigned long long m = __ballot(flag);
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

// Wave-wide least value and inclusive sum by moves between lanes inside the VALU
// (a quarter of the latency of cross-lane exchanges through the LDS unit).
// Control words: shifts right by 1, 2, 4, 8 within rows of 16 lanes, then the
// last lane of a row to the next row (rows 1 and 3), and lane 31 to rows 2 and 3.
template <int CTRL, int ROWS> __device__ __forceinline__ int lane_move(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS> __device__ __forceinline__ int64_t min_move(int64_t v)
{
    const int lo = int(uint32_t(uint64_t(v))), hi = int(v >> 32);
    const int64_t u = int64_t(uint64_t(uint32_t(lane_move<CTRL, ROWS>(lo, lo))) |
                              (uint64_t(uint32_t(lane_move<CTRL, ROWS>(hi, hi))) << 32));
    return u < v ? u : v;
}
__device__ __forceinline__ int64_t wave_min(int64_t v)   // of all 64 lanes, to all
{
    v = min_move<0x111, 0xf>(v);
    v = min_move<0x112, 0xf>(v);
    v = min_move<0x114, 0xf>(v);
    v = min_move<0x118, 0xf>(v);
    v = min_move<0x142, 0xa>(v);
    v = min_move<0x143, 0xc>(v);
    const int lo = of_lane(int(uint32_t(uint64_t(v))), 63), hi = of_lane(int(v >> 32), 63);
    return int64_t(uint64_t(uint32_t(lo)) | (uint64_t(uint32_t(hi)) << 32));
}
__device__ __forceinline__ int wave_sum_to(int v)   // inclusive, in lane order
{
    v += lane_move<0x111, 0xf>(0, v);
    v += lane_move<0x112, 0xf>(0, v);
    v += lane_move<0x114, 0xf>(0, v);
    v += lane_move<0x118, 0xf>(0, v);
    v += lane_move<0x142, 0xa>(0, v);
    v += lane_move<0x143, 0xc>(0, v);
    return v;
}

// Sums of the partial groups of rows [q0, q0 + cnt), in the order of k_reduce, to
// f[component][row].  Every load of up to three passes over the outputs is in
// flight before the first sum (k_step at n = 80000 order 6, 64 lanes an output: 10.1
// -> 9.0 us; with the ends of the sums one load after another it had been up to
// twelve round trips).
template <int L, int NV>
__device__ __forceinline__ void sum_rows(const double *__restrict__ part, int64_t na, int ng, int q0, int cnt,
                                         double (*f)[kSmallMax])
{
    // outputs a pass, and passes in flight together (short sums have enough outputs to a pass)
    constexpr int G = kStepBlock / L, E = L >= 16 ? 3 : 1;
    const int l = int(threadIdx.x) % L;
    for (int e0 = int(threadIdx.x) / L; e0 < cnt * NV; e0 += G * E) {
        // (the last output again where there are fewer)
        const double *src[E];
        int c[E], row[E];
        double s[E];
#pragma unroll
        for (int x = 0; x < E; ++x) {
            const int e = e0 + x * G < cnt * NV ? e0 + x * G : cnt * NV - 1;
            c[x] = e / cnt, row[x] = e - c[x] * cnt;
            src[x] = part + (int64_t(c[x]) * na + q0 + row[x]) * ng;
            s[x] = 0.0;
        }
        for (int k = l; k < ng; k += 8 * L) {
            double v[E][8];
#pragma unroll
            for (int x = 0; x < E; ++x)
#pragma unroll
                for (int u = 0; u < 8; ++u) v[x][u] = k + u * L < ng ? src[x][k + u * L] : 0.0;
#pragma unroll
            for (int x = 0; x < E; ++x)
#pragma unroll
                for (int u = 0; u < 8; ++u) s[x] += v[x][u];
        }
        // the lanes of a group share e0, so their partners run the same iterations
#pragma unroll
        for (int m = L / 2; m > 0; m >>= 1)
#pragma unroll
            for (int x = 0; x < E; ++x) s[x] += __shfl_xor(s[x], m, 64);
        if (l == 0)
#pragma unroll
            for (int x = 0; x < E; ++x) f[c[x]][row[x]] = s[x];
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
__device__ __forceinline__ void schedule(const StepArgs &a, int nb, int64_t *wm, int *wcnt, int *wbig, int32_t *soff)
{
    const int tid = int(threadIdx.x);
    const StepScratch &w = a.w;
    const int b0 = tid * PER;
    // all that it reads, in flight together
    DevScalars *sc = a.sc;
    const unsigned long long nf = shared_load(&sc->nonfinite), uf = shared_load(&sc->underflow);
    unsigned long long nf0 = a.nonfinite;
    // (taken into registers here: a choice between its address and the other's
    // would put the launch's arguments into scratch memory, 832 bytes a lane)
    asm volatile("" : "+s"(nf0));
    if (a.mode != kStepSchedule) nf0 = sc->nonfinite0;
    const int64_t seq = a.mode == kStepSchedule ? a.seq : sc->seq + 1;
    int64_t bt[PER];
    int bc[PER];
    constexpr int kAhead = 2;   // candidates of each block loaded with its time
    int32_t c0[PER][kAhead];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int bb = b0 + k < nb ? b0 + k : nb - 1;
        bt[k] = shared_load(&w.blk[bb].t_next);
        bc[k] = int(shared_load(&w.blk[bb].count));
#pragma unroll
        for (int u = 0; u < kAhead; ++u) c0[k][u] = shared_load(&w.cand[int64_t(bb) * kStepBlock + u]);
    }
    // each wave's least time, its active particles and their prefix; then the
    // block's from the four waves'
    int64_t mn = INT64_MAX;
#pragma unroll
    for (int k = 0; k < PER; ++k) mn = bt[k] < mn ? bt[k] : mn;   // (a repeated last block changes nothing)
    const int64_t wmin = wave_min(mn);
    int mine = 0;
    bool more = false;   // a block with more candidates than are here
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        if (b0 + k >= nb || bt[k] != wmin) bc[k] = 0;
        mine += bc[k];
        more = more || bc[k] > kAhead;
    }
    const int lane = tid & 63, wv = tid >> 6;
    const int incl = wave_sum_to(mine);
    const bool wmore = __ballot(more) != 0;
    if (lane == 63) {
        wm[wv] = wmin;
        wcnt[wv] = incl;
        wbig[wv] = wmore ? 1 : 0;
    }
    __syncthreads();
    int64_t tn = wm[0];
    for (int k = 1; k < kSW; ++k) tn = wm[k] < tn ? wm[k] : tn;
    // (a wave whose least time is not the step's has no active particles: its
    // prefix counts others, and its blocks share their successor's offset)
    int off = wmin == tn ? incl - mine : 0, total = 0, search = 0;
    for (int k = 0; k < kSW; ++k) {
        const int c = wm[k] == tn ? wcnt[k] : 0;
        if (k < wv) off += c;
        total += c;
        search |= wm[k] == tn ? wbig[k] : 0;
    }
    if (wmin != tn)
#pragma unroll
        for (int k = 0; k < PER; ++k) bc[k] = 0;
    // the last wave publishes, without an order among the words: the host waits
    // for each of them (read_published); the others go on to the list
    if (tid == kStepBlock - 64) {
        HostScalars *pub = a.pub + (seq & (kPubSlots - 1));
        __hip_atomic_store(&pub->t_next, tn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->n_act, int64_t(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->underflow, uf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->nonfinite, nf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&pub->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        sc->nonfinite0 = nf0;
        sc->halt = nf == nf0 ? 0 : 1;
        sc->seq = seq;
        sc->t_next = tn;
        sc->n_act = total;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (b0 + k < nb) {
            soff[b0 + k] = off;
            w.boff[b0 + k] = off;
            if (total <= kStepGather)
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
                    if (u < bc[k]) w.act[off + u] = c0[k][u];
            off += bc[k];
        }
    if (total > kStepGather || !search) return;   // listed by k_step_gather, or already
    __syncthreads();
    for (int e = tid; e < total; e += kStepBlock) {
        // the block of entry e: the last one with soff <= e (blocks without
        // active particles share their successor's offset)
        int lo = 0, hi = nb;
        while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (soff[mid] <= e) lo = mid; else hi = mid;
        }
        if (e - soff[lo] >= kAhead) w.act[e] = shared_load(&w.cand[int64_t(lo) * kStepBlock + (e - soff[lo])]);
    }
}

template <int P, bool PN>
__global__ void __launch_bounds__(kStepBlock)
k_step(StepArgs a)
{
    constexpr int NV = 3 * (P / 2);
    __shared__ double f[NV][kSmallMax];
    __shared__ int64_t wm[kSW];
    __shared__ int wcnt[kSW], wbig[kSW], wact[kSW];
    __shared__ int32_t soff[kStepBlocks];
    __shared__ int s_last;
    const int64_t n = a.cfg.n;
    const int b = int(blockIdx.x), nb = int(gridDim.x), tid = int(threadIdx.x);
    const int64_t i = int64_t(b) * kStepBlock + tid;
    int64_t *t_tick = a.st.t_tick;
    int32_t *level = a.st.level;
    int64_t t0 = i < n ? t_tick[i] : 0;
    int l0 = i < n ? level[i] : 0;
    int q0 = a.w.boff[b];   // of the step to end
    int sp = a.tab.n_split[tid & 63];
    asm volatile("" : "+v"(t0), "+v"(l0), "+v"(q0), "+v"(sp));   // in flight together with what the next line reads
    if (a.mode == kStepSmall && !small_step(*a.sc, sp, a.t_limit)) return;
    int64_t next = i < n ? next_of(t0, l0) : INT64_MAX;
    if (a.mode != kStepSchedule) {
        const int64_t na = a.sc->n_act, tn = a.sc->t_next;
        const bool active = i < n && next == tn;
        double *x = a.st.x, *v = a.st.v;
        double *const d[6] = {a.st.d[0], a.st.d[1], a.st.d[2], a.st.d[3], a.st.d[4], a.st.d[5]};
        HermiteState<P> s0;
        if (active) load_state<P>(s0, n, i, x, v, d, t0, l0);   // in flight while the partial forces are summed
        int cnt = 0;
        const int rank = block_rank(active, wact, &cnt);
        if (cnt > 0) {   // uniform over the block
            double *fp[4];
            int64_t stride, row;
            if (a.mode == kStepSmall) {
                const int nsp = of_lane(sp, na - 1), gs = small_group(na, nsp);
                const int ng = (nsp + gs - 1) / gs;
                const int L = reduce_lanes(ng);
                if (L == 1) sum_rows<1, NV>(a.part, na, ng, q0, cnt, f);
                else if (L == 4) sum_rows<4, NV>(a.part, na, ng, q0, cnt, f);
                else if (L == 16) sum_rows<16, NV>(a.part, na, ng, q0, cnt, f);
                else sum_rows<64, NV>(a.part, na, ng, q0, cnt, f);
                __syncthreads();
                stride = kSmallMax;
                row = rank;
#pragma unroll
                for (int k = 0; k < 4; ++k) fp[k] = k < P / 2 ? f[3 * k] : nullptr;
            } else {
                stride = na;
                row = int64_t(q0) + rank;
#pragma unroll
                for (int k = 0; k < 4; ++k) fp[k] = a.f[k];
            }
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
                int l1;
                const int fl = correct_state<P, true>(s0, n, i, tn, fnew, stride, row, x, v, d, t_tick, level, a.cfg.eta,
                                                      a.rule, int(a.cfg.k_min), int(a.cfg.k_max), &l1);
                if (fl & 2) atomicAdd(&a.sc->underflow, 1ull);
                if (fl & 1) atomicAdd(&a.sc->nonfinite, 1ull);
                next = next_of(tn, l1);
            }
        }
    }
    // the block's next time, and its particles at it in increasing order
    const int64_t wmin = wave_min(next);
    const int lane = tid & 63, wv = tid >> 6;
    const unsigned long long at = __ballot(i < n && next == wmin);
    if (lane == 0) {
        wm[wv] = wmin;
        wcnt[wv] = __popcll(at);
    }
    __syncthreads();
    int64_t bm = wm[0];
    for (int k = 1; k < kSW; ++k) bm = wm[k] < bm ? wm[k] : bm;
    int cnt = 0, rank = __popcll(at & ((1ull << lane) - 1ull));
    for (int k = 0; k < kSW; ++k) {
        const int c = wm[k] == bm ? wcnt[k] : 0;
        if (k < wv) rank += c;
        cnt += c;
    }
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
    if (nb <= kStepBlock) schedule<1>(a, nb, wm, wcnt, wbig, soff);
    else schedule<kStepBlocks / kStepBlock>(a, nb, wm, wcnt, wbig, soff);
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
