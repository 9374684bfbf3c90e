// force_small.hip -- the wave j-split force kernel with the j-particle
// predictor folded into its j loads, for block steps with few active
// particles.
//
// Each block step predicts every particle to the block time and then sums the
// force on the active ones over all of them (paper: Sec. "Codes
// description").  With few active particles the separate predictor pass
// (read the stored state, write a record) and the force pass (read the
// records back) are both bound by HBM traffic over all n particles.  Here
// each workgroup predicts the j-particles of its splits itself as it walks
// them: the stored state is read once, no record is written or read.
//
// The arithmetic is the predictor's (predict_state) and the pair term's
// (Pol::pair), and every lane visits its j-particles in the order of the
// unfused wave j-split kernel, with the same FP32 chunk boundaries; the
// splits' sums are added in the order of the grouped split reduction.  The
// results equal, bit for bit, those of the predictor, that kernel and that
// reduction.
#include <type_traits>

#include "hermite.h"
#include "pairwise.h"

namespace nb {
namespace {

constexpr int kWaves = 8;                  // waves per workgroup
constexpr int kSlots = 128;                // (split, row) pairs of a workgroup, at most

// The waves of a workgroup against a set of n_act rows.  A row's j-particles of
// a split are dealt to JS lanes (64, 16 or 4: fixed by the row count, for the
// FP32 sums), R = 64 / (JS G) rows fill the rest of the wave, G splits where the
// rows would fill half of it only; T waves take the same splits for T tiles of
// 16 rows each and share the predicted particles through LDS (each predicts one
// tile of 64 in T).  gs splits (small_group) make gs T / G waves; others of the
// workgroup (a launch sized for another row count) have nothing to do.
template <int JS_, int G_, int T_> struct Cut {
    static constexpr int JS = JS_, G = G_, T = T_;
    static constexpr int R = 64 / (JS * G);           // rows per wave
    static constexpr int kRows = R * T;               // rows per workgroup
    static constexpr int kMost = T == 1 ? 8 : 8 / T;  // splits per workgroup, at most
    static_assert(kMost * kRows <= kSlots && kMost * T / G <= kWaves, "slots and waves");
};
using Cut1 = Cut<64, 1, 1>;
using Cut2 = Cut<16, 2, 1>;
using Cut4 = Cut<16, 1, 1>;
using Cut8 = Cut<4, 2, 1>;
using Cut16 = Cut<4, 1, 1>;
using Cut32 = Cut<4, 1, 2>;
using Cut64 = Cut<4, 1, 4>;   // and more rows, 64 to a workgroup
static_assert(Cut16::kMost == 8 && Cut32::kMost == 4 && Cut64::kMost == 2, "small_group");

// One workgroup: rows [row0, row0 + kRows) against the splits [s0, s0 + gs).
// The sums of (local split, local row, component) end in red[c][slot], slot
// = split * kRows + row.
template <class C, class Pol, int P, int PREC>
__device__ __forceinline__ void walk(const PredIn &in, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
                                     typename Pol::ET e2, int64_t n_hard, int64_t j_chunk, int n_split, int s0,
                                     int gs, int64_t row0, typename Pol::Rec *tiles, double (*red)[kSlots])
{
    using Rec = typename Pol::Rec;
    using Part = typename Pol::Part;
    using ET = typename Pol::ET;
    constexpr int JS = C::JS, G = C::G, T = C::T, R = C::R;
    constexpr int NT = 64 / JS;          // j-particles of a tile per lane
    constexpr int UN = sizeof(Rec) > 80 ? 1 : (sizeof(Rec) > 64 ? 2 : 4);   // as many records as registers hold
    constexpr int NV = 3 * (P / 2);
    constexpr double kInvTick = 1.0 / double(kTicksPerUnit);
    const int lane = int(threadIdx.x) & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int g = lane / (JS * R), r = (lane / JS) % R, sl = lane % JS;
    const int sub = wave % T, grp = wave / T;
    const bool used = wave * G < gs * T;   // uniform over the wave
    const int sw = s0 + grp * G;         // the wave's first split
    const int64_t q = row0 + sub * R + r;
    const int64_t qq = q < n_act ? q : n_act - 1;   // padding rows recompute the last row; never stored
    double acc[13];
    const int64_t steps = (j_chunk + 64 * T - 1) / (64 * T);   // the same for every wave
    if (used) {
        const int64_t ia = act[qq];
        const int64_t i = (ia >= 0 && ia < n) ? ia : 0;
        const typename Pol::I ip = Pol::load(predict_state<P, PREC>(load_pstate<P>(n, i, in.m, in.x, in.v, in.d),
                                                                    double(in.t - in.t_tick[i]) * kInvTick));
        const bool i_hard = i < n_hard;
        Part p[13];
#pragma unroll
        for (int c = 0; c < 13; ++c) {
            acc[c] = 0.0;
            zero_part(p[c]);
        }
        constexpr int CH = Pol::kChunk > 0 ? Pol::kChunk : (1 << 30);
        static_assert(CH % NT == 0, "chunk length a multiple of a lane's share of a tile");
        int since = 0;
        // ends of the wave's splits (empty past the last split)
        int64_t b0[G], b1[G];
#pragma unroll
        for (int k = 0; k < G; ++k) {
            b0[k] = int64_t(sw + k) * j_chunk;
            b1[k] = b0[k] + j_chunk < n ? b0[k] + j_chunk : n;
            if (sw + k >= n_split) b0[k] = b1[k] = n;
        }
        const int64_t j1 = b1[g < G ? g : 0];
        // the stored state of this lane's next j-particle of each split, one
        // tile ahead (lanes past the end load the last particle; never used)
        PState<P> nx[G];
        int64_t tn[G];
        auto fetch = [&](int64_t step) {
#pragma unroll
            for (int k = 0; k < G; ++k) {
                const int64_t j = b0[k] + (step * T + sub) * 64 + lane;
                const int64_t jj = j < b1[k] ? j : n - 1;
                nx[k] = load_pstate<P>(n, jj, in.m, in.x, in.v, in.d);
                tn[k] = in.t_tick[jj];
            }
        };
        // (loaded in place where the registers would not hold it beside the pair loop's)
        constexpr bool kAhead = T == 1 || P == 4 || (P == 6 && std::is_same<Part, float>::value);
        if constexpr (kAhead) fetch(0);
        for (int64_t step = 0; step < steps; ++step) {
            Rec mine[G];
            if constexpr (!kAhead) fetch(step);
#pragma unroll
            for (int k = 0; k < G; ++k) mine[k] = predict_state<P, PREC>(nx[k], double(in.t - tn[k]) * kInvTick);
            if (kAhead && step + 1 < steps) fetch(step + 1);
            if constexpr (JS == 64) {
                const int64_t j = b0[0] + step * 64 + lane;
                if (j < j1) {
                    const ET el = (i_hard && j < n_hard) ? ET(0) : e2;
                    Pol::template pair<true>(ip, mine[0], el, j != i, p);
                    if (++since == CH) {
                        flush<Part, 1>(&p, &acc);
                        since = 0;
                    }
                }
            } else {
                Rec *tw = tiles + (wave * G) * 64;   // T > 1: the T waves of a group write T tiles in a row
#pragma unroll
                for (int k = 0; k < G; ++k) tw[k * 64 + lane] = mine[k];
                if constexpr (T > 1) __syncthreads();
                else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
                for (int k = 0; k < T; ++k) {
                    const Rec *tr = tiles + (T > 1 ? grp * T + k : wave * G + g) * 64;
                    const int64_t jt = b0[G == 1 ? 0 : g] + (step * T + k) * 64;
                    const int cnt = j1 - jt < 64 ? int(j1 - jt) : 64;
                    // A full tile without the row's own particle and without hard
                    // pairs needs no per-pair checks; the chunk counter then moves
                    // by NT at once (the chunk length is a multiple of NT, and only
                    // the split's last tile can be partial, so the flushes fall on
                    // the same pairs as with per-pair counting).  Not with the
                    // potential: without the self-pair select the compiler may
                    // fuse m_j / r into the potential sum as one FMA, which
                    // rounds differently.
                    const bool plain =
                        !Pol::kWithPot && cnt == 64 && (i < jt || i >= jt + 64) && !(i_hard && jt < n_hard);
                    if (plain) {
#pragma unroll UN
                        for (int u = 0; u < NT; ++u) Pol::template pair<false>(ip, tr[sl + u * JS], e2, true, p);
                        since += NT;
                        if (since == CH) {
                            flush<Part, 1>(&p, &acc);
                            since = 0;
                        }
                    } else {
#pragma unroll 1
                        for (int u = sl; u < cnt; u += JS) {
                            const int64_t j = jt + u;
                            const ET el = (i_hard && j < n_hard) ? ET(0) : e2;
                            Pol::template pair<true>(ip, tr[u], el, j != i, p);
                            if (++since == CH) {
                                flush<Part, 1>(&p, &acc);
                                since = 0;
                            }
                        }
                    }
                }
                if constexpr (T > 1) __syncthreads();
                else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        }
        flush<Part, 1>(&p, &acc);
        // fold the row's JS lanes
#pragma unroll
        for (int m = JS / 2; m > 0; m >>= 1)
#pragma unroll
            for (int c = 0; c < 13; ++c) acc[c] += __shfl_xor(acc[c], m, 64);
    } else if constexpr (T > 1) {
        for (int64_t step = 0; step < steps; ++step) {   // the barriers of the others
            __syncthreads();
            __syncthreads();
        }
    }
    __syncthreads();   // the tiles are no longer read: red shares their LDS
    if (used && sl == 0) {
        const int slot = (grp * G + g) * C::kRows + sub * R + r;
#pragma unroll
        for (int c = 0; c < NV; ++c) red[c][slot] = acc[c];
        if (Pol::kWithPot) red[NV][slot] = -acc[kPot];
    }
    __syncthreads();
}

// Sums of the workgroup's splits, in order, to partial group `grp` of ng (or to
// the outputs when the launch has one group and out is given).
template <class C, class Pol, int P>
__device__ __forceinline__ void put(int64_t n_act, int64_t row0, int splits, int grp, int ng, bool direct,
                                    const OutPtrs &o, double *__restrict__ part, const double (*red)[kSlots])
{
    constexpr int NV = 3 * (P / 2), NC = NV + (Pol::kWithPot ? 1 : 0);
    const int64_t left = n_act - row0;
    const int rows = left < C::kRows ? int(left) : C::kRows;
    for (int e = int(threadIdx.x); e < rows * NC; e += int(blockDim.x)) {
        const int c = e / rows, row = e - c * rows;
        double s = 0.0;
        for (int k = 0; k < splits; ++k) s += red[c][k * C::kRows + row];
        const int64_t q = row0 + row;
        if (!direct) part[(int64_t(c) * n_act + q) * ng + grp] = s;
        else if (c == NV) { if (o.p[4]) o.p[4][q] = s; }
        else if (double *d = o.p[c / 3]) d[(c % 3) * n_act + q] = s;
    }
}

template <class C, class Pol, int P, int PREC>
__device__ __forceinline__ void small_run(const PredIn &in, int64_t n, const int32_t *act, int64_t n_act, double eps2,
                                          int64_t n_hard, int64_t j_chunk, int n_split, int gs, bool to_part,
                                          const OutPtrs &o, double *part, typename Pol::Rec *tiles, double (*red)[kSlots])
{
    const int ng = (n_split + gs - 1) / gs;
    const int grp = int(blockIdx.y);
    if (grp >= ng) return;
    const int64_t row0 = int64_t(blockIdx.x) * 64;
    const int s0 = grp * gs;
    walk<C, Pol, P, PREC>(in, n, act, n_act, typename Pol::ET(eps2), n_hard, j_chunk, n_split, s0, gs, row0, tiles, red);
    put<C, Pol, P>(n_act, row0, n_split - s0 < gs ? n_split - s0 : gs, grp, ng, !to_part && ng == 1, o, part, red);
}

// Bound by HBM for up to four rows (every particle's stored state is read
// once: n = 2^20, order 6, 168 MB) and by VALU issue and latency for more, where
// a particle meets up to 16 rows in a wave.  Up to eight waves per workgroup, whose
// splits' sums are added in LDS, leave an eighth of the partial sums to the
// reduction, and up to 8 rows share a wave between two splits instead of leaving
// half its lanes to padding rows (n = 2^20, 5 rows, MIXED order 6: 53.4 us for the
// call with one wave per workgroup and 16 rows to it, 43.8 now; the state alone
// takes 33 us to read at the rate of a large copy).  Where eight splits to a
// workgroup would leave CUs without one, a workgroup takes fewer (small_group), and
// a wave one: n = 3000, one row MIXED order 8 14.1 -> 8.8 us for the call, n = 600000,
// one row 44.9 -> 23.8, n = 500, 5 rows MIXED order 6 30.0 -> 22.1; a bound of 512
// workgroups instead of 256 loses 10% at n = 120000.  With `dev` the active set,
// its time and its split come from the
// device (the block step that the scheduler has just found), and nothing is
// done when that step is not one for this kernel.
template <class Pol, int P, int PREC>
__global__ void __launch_bounds__(kWaves * 64)
k_force_small(PredIn in, int64_t n, const int32_t *__restrict__ act, int64_t n_act, double eps2, int64_t n_hard,
              int64_t j_chunk, int n_split, OutPtrs o, double *__restrict__ part, const DevScalars *__restrict__ dev,
              SmallTable tab, int64_t t_limit)
{
    using Rec = typename Pol::Rec;
    static_assert(std::is_same<Rec, typename PredRec<P, PREC>::type>::value, "record type of the precision");
    constexpr int kTileBytes = int(sizeof(Rec)) * 64 * kWaves, kRedBytes = 13 * kSlots * 8;
    __shared__ __attribute__((aligned(16))) char lds[kTileBytes > kRedBytes ? kTileBytes : kRedBytes];
    Rec *tiles = reinterpret_cast<Rec *>(lds);
    double(*red)[kSlots] = reinterpret_cast<double(*)[kSlots]>(lds);
    if (dev) {
        int sp = tab.n_split[threadIdx.x & 63], jc = tab.j_chunk[threadIdx.x & 63];
        asm volatile("" : "+v"(sp), "+v"(jc));   // in flight together with the scheduler's result
        if (!small_step(*dev, sp, t_limit)) return;
        n_act = dev->n_act;
        in.t = dev->t_next;
        n_split = of_lane(sp, n_act - 1);
        j_chunk = of_lane(jc, n_act - 1);
    }
#define NB_SMALL(CUT) small_run<CUT, Pol, P, PREC>(in, n, act, n_act, eps2, n_hard, j_chunk, n_split, gs, dev != nullptr, \
                                                   o, part, tiles, red)
    const int gs = small_group(n_act, n_split);
    // Two splits to a wave where all waves would be more than the chip holds two to
    // a SIMD (gs is 8 then), and the registers hold two splits' states in flight:
    // order 4, and order 6 beside FP32 sums.
    constexpr bool kTwo = P == 4 || (P == 6 && std::is_same<typename Pol::Part, float>::value);
    const bool two = kTwo && gs == 8;
    if (n_act <= 1) NB_SMALL(Cut1);
    else if (two && n_act <= 2) NB_SMALL(Cut2);
    else if (n_act <= 4) NB_SMALL(Cut4);
    else if (two && n_act <= 8) NB_SMALL(Cut8);
    else if (n_act <= 16) NB_SMALL(Cut16);
    else if (n_act <= 32) NB_SMALL(Cut32);
    else NB_SMALL(Cut64);
#undef NB_SMALL
}

struct Launch {
    const ForceArgs *a;
    const PredIn *in;
    int n_split;
    int64_t j_chunk;
    unsigned tiles, groups;   // the grid: tiles of 64 rows (up to 2^20) by groups of splits (up to 2^16)
    int waves;                // per workgroup
    const DevScalars *dev;
    const SmallTable *tab;
    int64_t t_limit;
};

template <class Pol, int P, int PREC>
hipError_t run(const Launch &L, hipStream_t s)
{
    const ForceArgs &a = *L.a;
    const OutPtrs o{{a.out[0], a.out[1], a.out[2], a.out[3], a.out[4]}};
    hipLaunchKernelGGL((k_force_small<Pol, P, PREC>), dim3(L.tiles, L.groups), dim3(unsigned(L.waves) * 64u), 0, s, *L.in, a.n, a.act,
                       a.n_act, a.eps2, a.n_hard, L.j_chunk, L.n_split, o, a.part, L.dev, *L.tab, L.t_limit);
    return hipGetLastError();
}

template <int P, bool POT>
hipError_t run_pot(int precision, const Launch &L, hipStream_t s)
{
    switch (precision) {
    case NBODY_MIXED: return run<PolMx<P, POT>, P, NBODY_MIXED>(L, s);
    case NBODY_DS: return run<PolDS<P, POT>, P, NBODY_DS>(L, s);
    default: return run<PolF64<P, POT>, P, NBODY_FP64>(L, s);
    }
}

template <int P>
hipError_t run_prec(int precision, const Launch &L, hipStream_t s)
{
    return L.a->out[4] ? run_pot<P, true>(precision, L, s) : run_pot<P, false>(precision, L, s);
}

hipError_t run_order(int order, int precision, const Launch &L, hipStream_t s)
{
    switch (order) {
    case 4: return run_prec<4>(precision, L, s);
    case 6: return run_prec<6>(precision, L, s);
    default: return run_prec<8>(precision, L, s);
    }
}

// Waves of a workgroup that adds gs splits, at most (two splits to a wave take half).
int small_waves(int64_t n_act, int gs) { return n_act <= 16 ? gs : (n_act <= 32 ? 2 * gs : 4 * gs); }

}  // namespace

hipError_t launch_force_pred(int order, int precision, const ForceArgs &a, const PredIn &in, hipStream_t s,
                             UsedShape *used)
{
    int n_split = 1;
    int64_t j_chunk = 0;
    split_shape(precision, a.n, a.n_act, a.n_split, a.fine, 1, 3, a.part_rows, &n_split, &j_chunk);
    if (used) *used = UsedShape{1, 64, n_split, 3};
    const int gs = small_group(a.n_act, n_split), ng = (n_split + gs - 1) / gs;
    const SmallTable none{};
    const Launch L{&a, &in, n_split, j_chunk, unsigned((a.n_act + 63) / 64), unsigned(ng), small_waves(a.n_act, gs), nullptr, &none, 0};
    const hipError_t e = run_order(order, precision, L, s);
    if (e != hipSuccess || ng == 1) return e;
    return launch_split_reduce_sf(order, a, ng, s);
}

hipError_t launch_force_small_dev(int order, int precision, const ForceArgs &a, const PredIn &in,
                                  const DevScalars *dev, const SmallTable &tab, int64_t t_limit, hipStream_t s)
{
    int groups = 1, waves = 1;
    for (int k = 0; k < kSmallMax; ++k) {
        if (tab.n_split[k] == 0) continue;
        const int gs = small_group(k + 1, tab.n_split[k]), ng = (tab.n_split[k] + gs - 1) / gs;
        if (ng > groups) groups = ng;
        if (small_waves(k + 1, gs) > waves) waves = small_waves(k + 1, gs);
    }
    const Launch L{&a, &in, 0, 0, 1u, unsigned(groups), waves, dev, &tab, t_limit};
    return run_order(order, precision, L, s);
}

}  // namespace nb
