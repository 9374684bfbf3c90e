// force.hip -- the O(n_act * n) pairwise force kernels (acceleration, jerk,
// snap, crackle, potential) for gfx950, in FP64, MIXED and DS arithmetic.
//
// Direct summation of softened gravity over all j != i (paper: Abstract,
// where correlations between distant particles rule out approximations), with
// the time derivatives a Hermite scheme of order 4, 6 or 8 needs (paper:
// Sec. "Codes description").  Derivative recursion: Nitadori & Makino (2008).
//
// Launch shape: grid (i-tiles, j-splits).  A lane holds NI active particles
// in registers and the block walks its split's j range; the j records reach
// the lanes either through wave-uniform scalar loads (kernel A) or through
// LDS tiles (kernel B).  For active sets smaller than a wavefront, kernel C
// spreads each active row over several lanes instead.  With one split the
// kernel writes the final FP64 sums; with several, each split writes its
// partial sums and a second kernel adds them in a fixed order.
#include "pairwise.h"

namespace nb {
namespace {

// --------------------------------------------------------------------------
// Pieces shared by both force kernels.  A workgroup (place) has an i-tile of
// blockDim.x * NI active particles (lane t holds rows t, t + blockDim.x, ...) and a
// j-split [split * j_chunk, min(n, (split+1) * j_chunk)).  Pairs with both
// indices below n_hard are unsoftened and their self pair is masked; above
// n_hard the self pair is evaluated with eps2 > 0 (its acceleration and
// derivatives are exactly zero, every difference being zero), except in the
// kernels that also sum the potential, which mask it by index.
//
// Partial sums of launches with more than kSplitFastestAbove splits are
// stored split-fastest, part[component][row][split], so that the lanes
// reducing one output read consecutive splits; with fewer splits (one lane
// or four per output) row-fastest, part[split][component][row], so that a
// workgroup's stores are coalesced.
constexpr int kSplitFastestAbove = 32;

template <class Pol, int P, int NI>
__device__ __forceinline__ void store_rows(int64_t n_act, int64_t row0, int split, int n_split,
                                           double (*acc)[13], double *__restrict__ o_acc,
                                           double *__restrict__ o_jrk, double *__restrict__ o_snp,
                                           double *__restrict__ o_crk, double *__restrict__ o_pot,
                                           double *__restrict__ part)
{
    constexpr int NV = 3 * (P / 2), C0 = Pol::kFirst;
#pragma unroll
    for (int k = 0; k < NI; ++k) {
        const int64_t q = row0 + int64_t(k) * blockDim.x;
        if (q >= n_act) continue;
        const double pot = acc[k][kPot];
        if (n_split == 1) {
            double *outs[4] = {o_acc, o_jrk, o_snp, o_crk};
#pragma unroll
            for (int c = C0; c < NV; ++c) {
                double *o = outs[c / 3];
                if (o) o[(c % 3) * n_act + q] = acc[k][c];
            }
            if (Pol::kWithPot && o_pot) o_pot[q] = -pot;
        } else if (n_split > kSplitFastestAbove) {
            double *base = part + q * n_split + split;
            const int64_t cs = n_act * n_split;
#pragma unroll
            for (int c = C0; c < NV; ++c) base[(c - C0) * cs] = acc[k][c];
            if (Pol::kWithPot) base[NV * cs] = -pot;
        } else {
            constexpr int NC = NV + 1;
            double *base = part + int64_t(split) * NC * n_act;
#pragma unroll
            for (int c = C0; c < NV; ++c) base[int64_t(c - C0) * n_act + q] = acc[k][c];
            if (Pol::kWithPot) base[int64_t(NV) * n_act + q] = -pot;
        }
    }
}

// Kernel A (scalar j path): every lane walks the same j range, so each j
// record is read with a wave-uniform address into SGPRs and feeds the VALU
// directly.  Suits FP64 arithmetic, which issues at one wave instruction per
// four cycles whatever the operand source.
template <class Pol, int P, int NI>
__global__ void __launch_bounds__(256)
k_force(const typename Pol::Rec *__restrict__ rec, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
        double eps2, int64_t n_hard, int64_t j_chunk, int n_split, double *__restrict__ o_acc,
        double *__restrict__ o_jrk, double *__restrict__ o_snp, double *__restrict__ o_crk,
        double *__restrict__ o_pot, double *__restrict__ part, Places places)
{
    using Rec = typename Pol::Rec;
    using Part = typename Pol::Part;
    using ET = typename Pol::ET;
    const ET e2 = ET(eps2);
    int64_t tile_i;
    int split;
    if (!place(places, n_split, &tile_i, &split)) return;
    const int64_t row0 = tile_i * blockDim.x * NI + threadIdx.x;
    if (row0 - int64_t(threadIdx.x & 63) >= n_act) return;   // a wave of padding rows only (no barrier follows)
    const int64_t j0 = int64_t(split) * j_chunk;
    const int64_t j1 = (j0 + j_chunk < n) ? j0 + j_chunk : n;

    typename Pol::I ip[NI];
    int64_t iidx[NI];
    double acc[NI][13];
    load_rows<Pol, NI>(rec, n, act, n_act, row0, ip, iidx, acc);
    hard_pairs<Pol, NI>(rec, j0, (j1 < n_hard) ? j1 : n_hard, 0, n_hard, e2, ip, iidx, acc);

    const int64_t js0 = (j0 > n_hard) ? j0 : n_hard;
    constexpr int64_t CH = Pol::kChunk > 0 ? Pol::kChunk : (int64_t(1) << 40);
    Part p[NI][13];
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
        for (int c = 0; c < 13; ++c) zero_part(p[k][c]);
    for (int64_t jc = js0; jc < j1; jc += CH) {
        const int cnt = int(((jc + CH < j1) ? jc + CH : j1) - jc);   // <= n <= 2^26
#pragma unroll 2
        for (int u = 0; u < cnt; ++u) {
            const int64_t j = jc + u;
            const Rec rj = rec[j];
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                // the self pair adds nothing to a, jerk, ...; only the potential needs it masked
                if constexpr (Pol::kWithPot) Pol::template pair<true>(ip[k], rj, e2, j != iidx[k], p[k]);
                else Pol::template pair<false>(ip[k], rj, e2, true, p[k]);
            }
        }
        flush<Part, NI>(p, acc);
    }
    store_rows<Pol, P, NI>(n_act, row0, split, n_split, acc, o_acc, o_jrk, o_snp, o_crk,
                           o_pot, part);
}

// Kernel B (LDS j path): the block stages BLOCK j records at a time in LDS
// (double-buffered, the next tile's global loads in flight during the
// current tile's arithmetic) and every lane reads them with same-address
// (broadcast) LDS loads into VGPRs.  All VALU operands are then VGPRs, which
// lets FP32 instructions of two waves on a SIMD issue together -- about twice
// the FP32 rate of SGPR-operand instructions on gfx950.  The FP32 chunk
// boundaries are those of kernel A, so both give identical bits.
template <class Pol, int P, int NI, int BLOCK, int UNROLL, int TILE>
__global__ void __launch_bounds__(BLOCK)
k_force_lds(const typename Pol::Rec *__restrict__ rec, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
            double eps2, int64_t n_hard, int64_t j_chunk, int n_split, double *__restrict__ o_acc,
            double *__restrict__ o_jrk, double *__restrict__ o_snp, double *__restrict__ o_crk,
            double *__restrict__ o_pot, double *__restrict__ part, Places places)
{
    using Rec = typename Pol::Rec;
    using ET = typename Pol::ET;
    __shared__ Rec tile[2][TILE];
    const ET e2 = ET(eps2);
    int64_t tile_i;
    int split;
    if (!place(places, n_split, &tile_i, &split)) return;   // the whole workgroup
    const int64_t row0 = tile_i * BLOCK * NI + threadIdx.x;
    const int64_t j0 = int64_t(split) * j_chunk;
    const int64_t j1 = (j0 + j_chunk < n) ? j0 + j_chunk : n;

    typename Pol::I ip[NI];
    int64_t iidx[NI];
    double acc[NI][13];
    load_rows<Pol, NI>(rec, n, act, n_act, row0, ip, iidx, acc);
    hard_pairs<Pol, NI>(rec, j0, (j1 < n_hard) ? j1 : n_hard, 0, n_hard, e2, ip, iidx, acc);

    const int64_t js0 = (j0 > n_hard) ? j0 : n_hard;
    lds_tiles<Pol, NI, BLOCK, UNROLL, TILE>(rec, js0, j1, e2, ip, iidx, tile, acc);
    store_rows<Pol, P, NI>(n_act, row0, split, n_split, acc, o_acc, o_jrk, o_snp, o_crk,
                           o_pot, part);
}

// Kernel C (wave j-split, for active sets smaller than a wavefront): a
// 64-lane workgroup holds R active rows, each on JS = 64 / R lanes; lane s of
// a row takes j = j0 + s, j0 + s + JS, ... of the split's range, with vector
// loads (the JS lanes of a row read consecutive records; the rows share
// them).  The row's JS partial sums are then folded with a fixed cross-lane
// butterfly, so a workgroup's serial work is 1/JS of kernels A and B and the
// result is the same for every run.  Hard pairs (both indices below n_hard)
// and the self pair are handled per pair.
template <class Pol, int P, int R>
__global__ void __launch_bounds__(64)
k_force_ws(const typename Pol::Rec *__restrict__ rec, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
           double eps2, int64_t n_hard, int64_t j_chunk, int n_split, double *__restrict__ o_acc,
           double *__restrict__ o_jrk, double *__restrict__ o_snp, double *__restrict__ o_crk,
           double *__restrict__ o_pot, double *__restrict__ part)
{
    using Rec = typename Pol::Rec;
    using Part = typename Pol::Part;
    using ET = typename Pol::ET;
    constexpr int JS = 64 / R;
    constexpr int NV = 3 * (P / 2);
    const ET e2 = ET(eps2);
    const int lane = int(threadIdx.x);
    const int r = lane / JS, sl = lane % JS;
    const int64_t q = int64_t(blockIdx.x) * R + r;
    const int split = blockIdx.y;
    const int64_t j0 = int64_t(split) * j_chunk;
    const int64_t j1 = (j0 + j_chunk < n) ? j0 + j_chunk : n;
    const int64_t qq = q < n_act ? q : n_act - 1;   // padding rows recompute the last row; never stored
    const int64_t ia = act[qq];
    const int64_t i = (ia >= 0 && ia < n) ? ia : 0;
    const typename Pol::I ip = Pol::load(rec[i]);
    const bool i_hard = i < n_hard;
    double acc[13];
    Part p[13];
#pragma unroll
    for (int c = 0; c < 13; ++c) {
        acc[c] = 0.0;
        zero_part(p[c]);
    }
    constexpr int CH = Pol::kChunk > 0 ? Pol::kChunk : (1 << 30);
    int since = 0;
    int64_t j = j0 + sl;
    Rec nxt = rec[j < j1 ? j : j1 - 1];
    for (; j < j1; j += JS) {
        const Rec rj = nxt;
        nxt = rec[j + JS < j1 ? j + JS : j1 - 1];
        const ET el = (i_hard && j < n_hard) ? ET(0) : e2;
        Pol::template pair<true>(ip, rj, el, j != i, p);
        if (++since == CH) {
            flush<Part, 1>(&p, &acc);
            since = 0;
        }
    }
    flush<Part, 1>(&p, &acc);
    // fold the JS lanes of the row (lanes r*JS .. r*JS + JS - 1)
#pragma unroll
    for (int m = JS / 2; m > 0; m >>= 1)
#pragma unroll
        for (int c = 0; c < 13; ++c) acc[c] += __shfl_xor(acc[c], m, 64);
    if (sl != 0 || q >= n_act) return;
    if (n_split == 1) {
        double *outs[4] = {o_acc, o_jrk, o_snp, o_crk};
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            double *o = outs[c / 3];
            if (o) o[(c % 3) * n_act + q] = acc[c];
        }
        if (Pol::kWithPot && o_pot) o_pot[q] = -acc[kPot];
    } else {
        // split-fastest partial sums: the reduction's lanes then read
        // consecutive splits of one output
        double *base = part + q * n_split + split;
        const int64_t cs = n_act * n_split;
#pragma unroll
        for (int c = 0; c < NV; ++c) base[c * cs] = acc[c];
        if (Pol::kWithPot) base[NV * cs] = -acc[kPot];
    }
}

// Sum of the j-split partial results.  A group of L lanes (L = 1, 4, 16 or
// 64, consecutive lanes of one wavefront) owns one output value: lane l adds
// splits l, l + L, l + 2L, ... in order, then the group folds its L sums with
// a fixed butterfly of cross-lane exchanges.  The order depends only on
// n_split and L, so reruns are bitwise identical.  Layouts: SF = false,
// part[split][component][row] (kernels A and B with at most
// kSplitFastestAbove splits: a workgroup's lanes write consecutive rows);
// SF = true, part[component][row][split] (kernels A and B with more splits,
// and the wave j-split kernels: a group's lanes read consecutive splits).
// C0: the first component of the launch (Pol::kFirst); the partials hold
// those from it on.
template <int P, int L, bool SF, int C0>
__global__ void __launch_bounds__(256)
k_reduce(const double *__restrict__ part, int64_t n_act, int n_split, double *__restrict__ o_acc,
         double *__restrict__ o_jrk, double *__restrict__ o_snp, double *__restrict__ o_crk,
         double *__restrict__ o_pot)
{
    constexpr int NV = 3 * (P / 2);
    constexpr int NC = NV + 1;
    const int64_t g = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / L;   // output index
    const int l = int(threadIdx.x) % L;
    const bool valid = g < n_act * (o_pot ? NC : NV - C0);   // the potential's sums exist only when asked for
    const int64_t gg = valid ? g : 0;
    const int c = int(gg / n_act);
    const int64_t q = gg - int64_t(c) * n_act;
    double s = 0.0;
    if (valid) {
        const double *src = SF ? part + (int64_t(c) * n_act + q) * n_split : part + int64_t(c) * n_act + q;
        s = lane_sum<L>(src, l, n_split, SF ? 1 : int64_t(NC) * n_act);
    }
#pragma unroll
    for (int m = L / 2; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
    if (!valid || l != 0) return;
    if (!C0 && c == NV) {
        if (o_pot) o_pot[q] = s;
        return;
    }
    double *outs[4] = {o_acc, o_jrk, o_snp, o_crk};
    double *o = outs[(c + C0) / 3];
    if (o) o[(c % 3) * n_act + q] = s;
}

// Lane l of the L that share a sum over groups of GS consecutive partials
// src[0..n): groups l, l + L, ..., each added in order, sixteen loads in flight
// together (the zeros past the end change nothing).
template <int L, int GS>
__device__ __forceinline__ double lane_group_sum(const double *__restrict__ src, int l, int n)
{
    constexpr int U = 16 / GS;
    double s = 0.0;
    for (int k = l; k * GS < n; k += U * L) {
        double v[U][GS];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < GS; ++g) {
                const int at = (k + u * L) * GS + g;
                v[u][g] = at < n ? src[at] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double t = 0.0;
#pragma unroll
            for (int g = 0; g < GS; ++g) t += v[u][g];
            s += t;
        }
    }
    return s;
}

// Sum of kernel C's partial results (split-fastest), in the order of the kernel
// that predicts inside: groups of gs consecutive splits first, each in order,
// then lane l of an output's L lanes adds groups l, l + L, ... and the lanes
// are folded as in k_reduce.
template <int P, int L>
__global__ void __launch_bounds__(256)
k_reduce_groups(const double *__restrict__ part, int64_t n_act, int n_split, int gs, double *__restrict__ o_acc,
                double *__restrict__ o_jrk, double *__restrict__ o_snp, double *__restrict__ o_crk,
                double *__restrict__ o_pot)
{
    constexpr int NV = 3 * (P / 2);
    const int64_t g = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / L;   // output index
    const int l = int(threadIdx.x) % L;
    const bool valid = g < n_act * (o_pot ? NV + 1 : NV);
    const int64_t gg = valid ? g : 0;
    const int c = int(gg / n_act);
    const int64_t q = gg - int64_t(c) * n_act;
    const double *src = part + (int64_t(c) * n_act + q) * n_split;
    double s = 0.0;
    if (valid)
        s = gs == 2   ? lane_group_sum<L, 2>(src, l, n_split)
            : gs == 4 ? lane_group_sum<L, 4>(src, l, n_split)
                      : lane_group_sum<L, 8>(src, l, n_split);
#pragma unroll
    for (int m = L / 2; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
    if (!valid || l != 0) return;
    if (c == NV) {
        o_pot[q] = s;
        return;
    }
    double *outs[4] = {o_acc, o_jrk, o_snp, o_crk};
    double *o = outs[c / 3];
    if (o) o[(c % 3) * n_act + q] = s;
}

template <int P, bool SF, int C0 = 0>
hipError_t launch_reduce(const ForceArgs &a, int n_split, hipStream_t s)
{
    static_assert(C0 % 3 == 0, "whole vectors");
    const int64_t outs = a.n_act * (3 * (P / 2) - C0 + (a.out[4] ? 1 : 0));
    const int L = reduce_lanes(n_split);
    const unsigned blocks = unsigned((outs * L + 255) / 256);
#define NB_RED(LL) hipLaunchKernelGGL((k_reduce<P, LL, SF, C0>), dim3(blocks), dim3(256), 0, s, a.part, a.n_act, n_split, \
                                      a.out[0], a.out[1], a.out[2], a.out[3], a.out[4])
    if (L == 1) NB_RED(1);
    else if (L == 4) NB_RED(4);
    else if (L == 16) NB_RED(16);
    else NB_RED(64);
#undef NB_RED
    return hipGetLastError();
}

template <int P>
hipError_t launch_reduce_groups(const ForceArgs &a, int n_split, hipStream_t s)
{
    const int gs = small_group(a.n_act, n_split), ng = (n_split + gs - 1) / gs;
    if (gs == 1) return launch_reduce<P, true>(a, n_split, s);
    const int64_t outs = a.n_act * (3 * (P / 2) + (a.out[4] ? 1 : 0));
    const int L = reduce_lanes(ng);
    const unsigned blocks = unsigned((outs * L + 255) / 256);
#define NB_RED(LL) hipLaunchKernelGGL((k_reduce_groups<P, LL>), dim3(blocks), dim3(256), 0, s, a.part, a.n_act, n_split, \
                                      gs, a.out[0], a.out[1], a.out[2], a.out[3], a.out[4])
    if (L == 1) NB_RED(1);
    else if (L == 4) NB_RED(4);
    else if (L == 16) NB_RED(16);
    else NB_RED(64);
#undef NB_RED
    return hipGetLastError();
}

// Whether a launch places units of consecutive splits: its partial sums are
// split-fastest.  Not on the scalar path, whose splits are long: there the tiles of
// a split had better run side by side, n = 262144, 3001 rows 932 us in the plain
// order, 942 by units.
bool spread(int jpath, int n_split) { return jpath == 2 && n_split > kSplitFastestAbove; }

struct Shape {
    int ni, block, n_split, jpath;
    int64_t j_chunk;
};

template <class Pol, int P, int NI>
hipError_t run(const ForceArgs &a, hipStream_t s, const Shape &sh)
{
    const int64_t per_block = int64_t(sh.block) * NI;
    const int64_t tiles = (a.n_act + per_block - 1) / per_block;
    const Places pl = places_for(tiles, sh.n_split, spread(sh.jpath, sh.n_split));
    const dim3 grid{place_grid(pl), 1u, 1u};
    const auto *rec = static_cast<const typename Pol::Rec *>(a.rec);
#define NB_FORCE_ARGS rec, a.n, a.act, a.n_act, a.eps2, a.n_hard, sh.j_chunk, sh.n_split, a.out[0], a.out[1], \
                      a.out[2], a.out[3], a.out[4], a.part
    if (sh.jpath == 3) {
        // rows per wave for the active set: 1, 4 or 16
        const int rw = a.n_act <= 1 ? 1 : (a.n_act <= 4 ? 4 : 16);
        const dim3 g3{unsigned((a.n_act + rw - 1) / rw), unsigned(sh.n_split), 1u};
        if (rw == 1) hipLaunchKernelGGL((k_force_ws<Pol, P, 1>), g3, dim3(64), 0, s, NB_FORCE_ARGS);
        else if (rw == 4) hipLaunchKernelGGL((k_force_ws<Pol, P, 4>), g3, dim3(64), 0, s, NB_FORCE_ARGS);
        else hipLaunchKernelGGL((k_force_ws<Pol, P, 16>), g3, dim3(64), 0, s, NB_FORCE_ARGS);
    } else if (sh.jpath == 1) {
        hipLaunchKernelGGL((k_force<Pol, P, NI>), grid, dim3(sh.block), 0, s, NB_FORCE_ARGS, pl);
    } else if (sh.block == 64) {
        hipLaunchKernelGGL((k_force_lds<Pol, P, NI, 64, 2, 64>), grid, dim3(64), 0, s, NB_FORCE_ARGS, pl);
    } else if (sh.block == 128) {
        hipLaunchKernelGGL((k_force_lds<Pol, P, NI, 128, 2, 128>), grid, dim3(128), 0, s, NB_FORCE_ARGS, pl);
    } else {
        hipLaunchKernelGGL((k_force_lds<Pol, P, NI, 256, 2, 128>), grid, dim3(256), 0, s, NB_FORCE_ARGS, pl);
    }
#undef NB_FORCE_ARGS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || sh.n_split == 1) return e;
    if (sh.jpath == 3) return launch_reduce_groups<P>(a, sh.n_split, s);
    if (sh.n_split > kSplitFastestAbove) return launch_reduce<P, true>(a, sh.n_split, s);
    return launch_reduce<P, false>(a, sh.n_split, s);
}

template <class Pol, int P>
hipError_t run_ni(const ForceArgs &a, hipStream_t s, const Shape &sh)
{
    if (sh.ni == 2 && sh.jpath != 3) return run<Pol, P, 2>(a, s, sh);
    return run<Pol, P, 1>(a, s, sh);
}

template <int P, bool POT>
hipError_t run_pot(int precision, const ForceArgs &a, hipStream_t s, const Shape &sh)
{
    switch (precision) {
    case NBODY_MIXED: return run_ni<PolMx<P, POT>, P>(a, s, sh);
    case NBODY_DS: return run_ni<PolDS<P, POT>, P>(a, s, sh);
    default: return run_ni<PolF64<P, POT>, P>(a, s, sh);
    }
}

// The potential is accumulated only when it is asked for.
template <int P>
hipError_t run_prec(int precision, const ForceArgs &a, hipStream_t s, const Shape &sh)
{
    return a.out[4] ? run_pot<P, true>(precision, a, s, sh) : run_pot<P, false>(precision, a, s, sh);
}

// The default j-split of kernels A and B, sized in waves of 64 NI rows (wt row
// tiles) that walk c particles each:
//  - many (wt n / 128 >= 16384, several rounds of waves on the chip): about
//    32768 waves of at least 256 particles (128 in FP64 with fewer than 32 row tiles
//    unless 256 still give 16384 waves), so that the last round is a small part
//    of the call, and at most 8192 (a wave is then some microseconds of work to a
//    100-byte partial row; n = 32768, n_act = 4096 MIXED order 8 with the potential
//    334 us with 256 splits, 297 with 128; n = n_act = 16000 FP64 order 8 908 with
//    125 splits, 861 with 63; but n = 600000, 200 rows FP64 order 4 220 with 128
//    particles to a wave, 241 with 256).  About 8192 waves, two or
//    three rounds, had cost 10-30% of it: n_act = n = 90000 MIXED order 6 11219
//    us with 6 splits, 9280 with 23; n = 262144, n_act = 3001 994 with 171, 926
//    with 683;
//  - otherwise a MIXED row takes its FP32 chunks (128 particles) one to a wave (two
//    cost 12% between 4096 and 8192 waves, 20 to 60% below; mean of orders 4 to 8 over
//    n = 8000 to 120000), and two above 8192 waves: there two cost 4% as long as the
//    partial sums stay in cache, but less memory (n = 32768, 2048 rows order 8 with the
//    potential, other inputs on every call: 169 us with one, 162 with two; n = 600000,
//    65 rows order 8 185 and 171);
//  - FP64 and DS sums have no chunks to keep, and a wave that walks 128
//    particles alone on its SIMD is all latency (28 us at order 4, FP64, for
//    any n): as few as 32 each, about 3072 waves, at most about 1250 splits (the
//    sum of the partials grows with them).  n = 1024, n_act = 100 FP64 order 4:
//    20.2 us with 8 splits of 128, 9.1 with 32 of 32 (order 8: 40.9, 13.1); n =
//    16384, n_act = 400: 26.0 with 128, 22.6 with 64.  But 128 where the 1024 SIMDs'
//    waves then add up to fewer particles: n = 16000, 1000 rows DS order 6 59 us with
//    three waves of 96 to a SIMD, 51 with two of 128.  Over n = 8000 to 120000 and
//    200 to 4000 rows DS and FP64 are within 5% of the best of 32 to 256 particles in the
//    mean; 256 instead of 128 cost 2 to 6% just below wt n / 128 = 16384 and more below.
int64_t default_chunk(int precision, int64_t n, int64_t n_act, int ni)
{
    const int64_t wt = (n_act + 64 * ni - 1) / (64 * ni);
    const auto up = [](int64_t v, int64_t g) { return (v + g - 1) / g * g; };
    if (wt * n >= int64_t(16384) * 128) {
        int64_t c = up(wt * n / 32768, 128);
        if (c < 256 && (precision != NBODY_FP64 || wt >= 32 || wt * n >= int64_t(16384) * 256)) c = 256;
        return c < 8192 ? c : 8192;
    }
    if (precision == NBODY_MIXED) return wt * n >= int64_t(8192) * kMixedChunk ? 2 * kMixedChunk : kMixedChunk;
    int64_t c = wt * n / 3072 > n / 1250 ? wt * n / 3072 : n / 1250;
    c = up(c, 32);
    c = c < 32 ? 32 : (c > 128 ? 128 : c);
    const auto rounds = [&](int64_t v) { return (wt * ((n + v - 1) / v) + 1023) / 1024 * v; };
    return rounds(c) > rounds(128) ? 128 : c;
}

}  // namespace

int record_bytes(int order, int precision)
{
    if (precision == NBODY_FP64) return order == 4 ? 64 : order == 6 ? 80 : 112;
    return order == 8 ? 80 : 64;
}

// Shortest j-split: a MIXED split holds whole FP32 chunks; the others' default
// and tuned splits may be shorter (kernel C walks tiles of 64).
int64_t split_grain(int precision, int jpath, bool fine)
{
    if (precision == NBODY_MIXED || !fine) return kMixedChunk;
    return jpath == 3 ? 64 : 32;
}

int auto_split(int precision, int64_t n, int64_t n_act, int ni, int jpath, int64_t part_rows)
{
    int64_t sp;
    if (jpath == 3) {
        // kernel C: one 64-lane workgroup per 1, 4 or 16 rows and split.  Split
        // counts giving about 512, 1024 and 2048 workgroups were the fastest on
        // MI355X (n = 2^17 and 2^20, orders 6 and 8, with and without the
        // predictor inside): shorter splits cost more in per-workgroup set-up and
        // in the split reduction than they add in parallelism.
        const int64_t rw = n_act <= 1 ? 1 : (n_act <= 4 ? 4 : 16);
        const int64_t tiles = (n_act + rw - 1) / rw;
        const int64_t target = rw == 1 ? 512 : (rw == 4 ? 1024 : 2048);
        const int64_t g = split_grain(precision, 3, true);
        sp = (target + tiles - 1) / tiles;
        if (sp > n / g) sp = n / g;
    } else {
        const int64_t c = default_chunk(precision, n, n_act, ni);
        sp = (n + c - 1) / c;
    }
    if (sp * n_act > part_rows) sp = part_rows / n_act;
    if (sp > 65535) sp = 65535;
    return sp < 1 ? 1 : int(sp);
}

void split_shape(int precision, int64_t n, int64_t n_act, int n_split_req, bool fine, int ni, int jpath,
                 int64_t part_rows, int *n_split, int64_t *j_chunk)
{
    int sp = n_split_req > 0 ? n_split_req : auto_split(precision, n, n_act, ni, jpath, part_rows);
    if (n_act > 0 && int64_t(sp) * n_act > part_rows) sp = int(part_rows / n_act);
    if (sp < 1) sp = 1;
    const int64_t g = split_grain(precision, jpath, fine || n_split_req <= 0);
    int64_t jc = (n + sp - 1) / sp;
    jc = (jc + g - 1) / g * g;
    *j_chunk = jc;
    *n_split = int((n + jc - 1) / jc);
}

// The launch shape of an untuned call.  Kernel C up to 32 rows; FP64 and DS
// up to 64 (one row per lane leaves a chip of 1024 SIMDs nearly idle there: n =
// 30000, 64 rows, FP64 order 8 45.7 us with kernel A, 19.9 with C; MIXED keeps
// the order of its FP32 sums, which costs a run of n = 80000 order 6 0 to 2%); but in
// systems above kWaveMaxN only up to 32 (n = 600000, 64 rows FP64 order 4 144 us with
// C, 115 with A; 33 rows DS order 8 with the predictor 238 and 206; n = 120000, 64 rows
// FP64 order 8 C is the faster one by a third).  One row per lane beyond: with many waves
// the scalar path, whose j records cost no LDS bandwidth (90000 rows MIXED order 4:
// LDS 6261, scalar 5459 us), in workgroups of 128 (MIXED from twice as many on: n =
// 32768, 4096 rows order 6 scalar 205, LDS 196 us, n = 120000, 2500 rows 384 and 398; and
// from 16 row tiles on: n = 2^20, 500 rows order 6 716 and 674, 300 rows order 8 705
// and 685, but 1000 rows order 6 1248 and 1275);
// but DS, whose
// adds keep more registers, and MIXED order 4 with the potential, whose self pairs
// are compared in scalar registers, stay on LDS tiles (n = 120000, 2500 rows DS order
// 8 scalar 1150, LDS 970 us, order 4 with the potential 538 and 501; MIXED order 4 with it
// 343 and 312; DS order 4 without it is the exception, 433 and 454); with few waves,
// the LDS path, whose loads run ahead (n = 80000, 200 rows FP64 order 8: scalar
// 107, LDS 91 us).  On the LDS path four waves share a tile where there are many
// row tiles (padded by a sixteenth at most) and three waves to a SIMD: 2 to 5%
// faster for 28 to 65 tiles (n = 20000, 4000 rows MIXED order 8 184 us with one wave to a
// workgroup, 176 with four), but up to 40% slower with fewer rows or more padding.
constexpr int64_t kWaveMaxN = 200000;
void default_shape(int precision, int order, bool pot, int64_t n, int64_t n_act, int *ni, int *block, int *jpath)
{
    *ni = 1;
    if (n_act <= (precision == NBODY_MIXED || n > kWaveMaxN ? 32 : 64)) {
        *block = 64;
        *jpath = 3;
        return;
    }
    const int64_t wt = (n_act + 63) / 64;
    const bool scalar = precision == NBODY_FP64    ? wt * n >= int64_t(16384) * 128
                        : precision == NBODY_MIXED ? wt >= 16 && wt * n >= int64_t(32768) * 128 && !(order == 4 && pot)
                                                   : false;
    if (scalar) {
        *block = 128;
        *jpath = 1;
        return;
    }
    const int64_t c = default_chunk(precision, n, n_act, 1);
    const bool share = wt >= 24 && wt * ((n + c - 1) / c) >= 3072 && 16 * ((wt + 3) / 4 * 4) <= 17 * wt;
    *block = share ? 256 : 64;
    *jpath = 2;
}

hipError_t launch_split_reduce_sf(int order, const ForceArgs &a, int n_split, hipStream_t s)
{
    if (order == 4) return launch_reduce<4, true>(a, n_split, s);
    if (order == 6) return launch_reduce<6, true>(a, n_split, s);
    return launch_reduce<8, true>(a, n_split, s);
}

hipError_t launch_force_high(const ForceArgs &a, hipStream_t s, UsedShape *used)
{
    Shape sh{};
    sh.block = (a.block == 64 || a.block == 128) ? a.block : 256;
    split_shape(NBODY_FP64, a.n, a.n_act, a.n_split, a.fine, 1, 1, a.part_rows, &sh.n_split, &sh.j_chunk);
    if (used) *used = UsedShape{1, sh.block, sh.n_split, 1};
    const Places pl = places_for((a.n_act + sh.block - 1) / sh.block, sh.n_split, false);
    hipLaunchKernelGGL((k_force<PolF64High, 8, 1>), dim3(place_grid(pl)), dim3(sh.block), 0, s, static_cast<const RecF64<8> *>(a.rec),
                       a.n, a.act, a.n_act, a.eps2, a.n_hard, sh.j_chunk, sh.n_split, nullptr, nullptr, a.out[2],
                       a.out[3], nullptr, a.part, pl);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || sh.n_split == 1) return e;
    return sh.n_split > kSplitFastestAbove ? launch_reduce<8, true, PolF64High::kFirst>(a, sh.n_split, s)
                                           : launch_reduce<8, false, PolF64High::kFirst>(a, sh.n_split, s);
}

hipError_t launch_force(int order, int precision, const ForceArgs &a, hipStream_t s, UsedShape *used)
{
    Shape sh{};
    sh.ni = (a.ni == 2) ? 2 : 1;
    sh.block = (a.block == 64 || a.block == 128) ? a.block : 256;
    // j path: FP64 reads j records from SGPRs, the FP32 modes from LDS
    sh.jpath = a.jpath >= 1 && a.jpath <= 3 ? a.jpath : (precision == NBODY_FP64 ? 1 : 2);
    split_shape(precision, a.n, a.n_act, a.n_split, a.fine, sh.ni, sh.jpath, a.part_rows, &sh.n_split, &sh.j_chunk);
    if (used) *used = UsedShape{sh.jpath == 3 ? 1 : sh.ni, sh.jpath == 3 ? 64 : sh.block, sh.n_split, sh.jpath};
    switch (order) {
    case 4: return run_prec<4>(precision, a, s, sh);
    case 6: return run_prec<6>(precision, a, s, sh);
    default: return run_prec<8>(precision, a, s, sh);
    }
}

}  // namespace nb
