// force_nb.hip -- the pairwise force split by neighbour spheres, with the
// neighbour lists (the Ahmad & Cohen 1973 scheme of the paper's second code,
// NBODY6++GPU, Sec. "Results": the GPU evaluates the force from the distant
// particles and the neighbour lists; the near, fast-changing part is summed
// over the list on its own shorter steps).
//
// For active particle i with neighbour radius squared h2[q], particle j != i
// is a neighbour when its unsoftened squared distance is below h2[q]; the
// kernel tests r^2 + eps_ij^2 < h2[q] + eps_ij^2 in its own precision, on the
// sum the pair term forms anyway.  Acceleration and jerk (the terms of the 4th-order
// scheme, softened as in the full force) are summed over the other particles
// (regular part) and over the neighbours (irregular part); the neighbour list
// holds their indices in increasing order.
//
// Kernel 1, a workgroup per i-tile of kNbBlock rows and j-split: each lane holds one
// active row and walks its split in increasing j, adding the pair terms of
// the non-neighbours (the neighbours are masked out of the same FMA sequence
// as the full force) and appending the neighbours to its split's part of the
// list.  The j below n_hard (unsoftened when i is hard too) are taken one by
// one with their checks; the rest streams through double-buffered LDS tiles of
// kNbTile records with no per-pair index test: the self pair (difference zero,
// r^2 = eps^2 > 0) either is a neighbour, and is dropped at the append, or adds
// exact zeros to the regular part.  Bound by VALU issue (3.7 cycles an
// instruction with 342 splits, 5.3 waves to a SIMD; 3.2 with 1024), so: one wave
// to a workgroup with tiles of 32, which leaves six waves (MIXED) or five (FP64)
// to a SIMD (tiles of 64 left four); neighbours, rare in a wave, are masked and noted under one wave-wide
// test of two pairs, and their list entries are written after the tile; entries
// of two bytes (offsets in the split) where a split is short enough, so that the
// scratch holds more splits.  The call at n = 131072, 1024 rows, lists of 128, MIXED
// 167 -> 152 us (512 splits instead of 342), n = 262144, 2048 rows MIXED 510 -> 475, FP64
// 716 -> 670, n = 8192, 64 rows MIXED 38 -> 32.  One
// scalar load of each record by the wave instead of LDS tiles: 206 us.  Kernel 2, one wave per
// row: the regular partial sums added in split order, the split lists
// concatenated, and the irregular part summed over the list (lanes take
// every 64th entry, then a fixed butterfly).  A row whose list was cut at
// max_nb gets NaN for its irregular part.
#include "pairwise.h"

namespace nb {
namespace {

constexpr int kNbBlock = 64;
constexpr int kNbChunk = 128;   // j of one FP32 sum
constexpr int kNbTile = 32;     // j of one LDS tile, a bit each in a lane's word of neighbours
constexpr int kNbGroup = 2;     // j of one test for neighbours
constexpr int64_t kShortChunk = 65536;   // j of a split whose list entries take two bytes, at most

// One pair of the regular sum: the differences, the softened r^2 + eps_ij^2,
// the neighbour test r^2 + eps_ij^2 < h^2 + eps_ij^2 (the unsoftened test,
// written on the sum the pair term forms anyway), and the pair's order-4
// terms added when j is valid and not a neighbour.  Returns whether j is a
// neighbour.  hh_e = h^2 + eps_ij^2 for the pair's softening.
__device__ __forceinline__ bool nb_pair(const typename PolF64<4, false>::I &i, const RecF64<4> &j, double el,
                                        double hh_e, bool valid, double *A)
{
    const double dx = j.x - i.x, dy = j.y - i.y, dz = j.z - i.z;
    const double wx = j.vx - i.vx, wy = j.vy - i.vy, wz = j.vz - i.vz;
    const double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, el)));
    const bool is_nb = valid && r2 < hh_e;
    const bool ok = valid && !is_nb;
    const double rinv = rsqrt64(ok ? r2 : 1.0);
    const double mr = ok ? j.m * rinv : 0.0;
    core_fma<4, false, double>(dx, dy, dz, wx, wy, wz, 0, 0, 0, 0, 0, 0, mr, rinv * rinv, A);
    return is_nb;
}

// A pair of the LDS-tile loop: softened (eps2 > 0, so r^2 > 0), no validity
// test (the self pair is handled as stated above).  set() forms all that the
// neighbour test and the sums need; add() adds the order-4 terms of mr = m / r
// (zeroed by the caller for a neighbour).
template <class T> struct SoftPair {
    T dx, dy, dz, wx, wy, wz, mr, rinv2;
    bool is_nb;
    __device__ __forceinline__ void finish(T r2, T rinv, T m, T hh_e)
    {
        is_nb = r2 < hh_e;
        mr = m * rinv;
        rinv2 = rinv * rinv;
    }
    __device__ __forceinline__ void set(const typename PolF64<4, false>::I &i, const RecF64<4> &j, double e2, double hh_e)
    {
        dx = j.x - i.x, dy = j.y - i.y, dz = j.z - i.z;
        wx = j.vx - i.vx, wy = j.vy - i.vy, wz = j.vz - i.vz;
        const double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, e2)));
        finish(r2, rsqrt64(r2), j.m, hh_e);
    }
    __device__ __forceinline__ void set(const typename DSIn<4>::I &i, const RecDS<4> &j, float e2, float hh_e)
    {
        dx = (j.xh - i.xh) + (j.xl - i.xl);
        dy = (j.yh - i.yh) + (j.yl - i.yl);
        dz = (j.zh - i.zh) + (j.zl - i.zl);
        wx = (j.vxh - i.vxh) + (j.vxl - i.vxl);
        wy = (j.vyh - i.vyh) + (j.vyl - i.vyl);
        wz = (j.vzh - i.vzh) + (j.vzl - i.vzl);
        const float r2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, __builtin_fmaf(dz, dz, e2)));
        finish(r2, __builtin_amdgcn_rsqf(r2), j.m, hh_e);
    }
    __device__ __forceinline__ void add(T *A) const
    {
        core_fma<4, false, T>(dx, dy, dz, wx, wy, wz, 0, 0, 0, 0, 0, 0, mr, rinv2, A);
    }
};

__device__ __forceinline__ bool nb_pair(const typename DSIn<4>::I &i, const RecDS<4> &j, float el, float hh_e,
                                        bool valid, float *A)
{
    const float dx = (j.xh - i.xh) + (j.xl - i.xl);
    const float dy = (j.yh - i.yh) + (j.yl - i.yl);
    const float dz = (j.zh - i.zh) + (j.zl - i.zl);
    const float wx = (j.vxh - i.vxh) + (j.vxl - i.vxl);
    const float wy = (j.vyh - i.vyh) + (j.vyl - i.vyl);
    const float wz = (j.vzh - i.vzh) + (j.vzl - i.vzl);
    const float r2 = __builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, __builtin_fmaf(dz, dz, el)));
    const bool is_nb = valid && r2 < hh_e;
    const bool ok = valid && !is_nb;
    const float rinv = __builtin_amdgcn_rsqf(ok ? r2 : 1.0f);
    const float mr = ok ? j.m * rinv : 0.0f;
    core_fma<4, false, float>(dx, dy, dz, wx, wy, wz, 0, 0, 0, 0, 0, 0, mr, rinv * rinv, A);
    return is_nb;
}

// SegT: the type of a list entry, j minus the split's first j.
template <class Pol, class SegT>
__global__ void __launch_bounds__(kNbBlock, Pol::kChunk ? 6 : 5)
k_force_nb(const typename Pol::Rec *__restrict__ rec, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
           const double *__restrict__ h2, double eps2, int64_t n_hard, int64_t j_chunk, int max_nb, int n_split,
           double *__restrict__ part, int32_t *__restrict__ seg_cnt, SegT *__restrict__ seg, Places places)
{
    using Rec = typename Pol::Rec;
    using ET = typename Pol::ET;
    using Part = typename Pol::Part;
    int64_t tile_i;
    int split;
    if (!place(places, n_split, &tile_i, &split)) return;   // the whole workgroup
    const int64_t q = tile_i * kNbBlock + threadIdx.x;
    const int64_t j0 = int64_t(split) * j_chunk;
    const int64_t j1 = (j0 + j_chunk < n) ? j0 + j_chunk : n;   // j0 < n for every split
    const bool row = q < n_act;
    const int64_t qq = row ? q : n_act - 1;   // padding lanes recompute the last row; never stored
    const int64_t ia = act[qq];
    const int64_t i = (ia >= 0 && ia < n) ? ia : 0;
    const typename Pol::I ip = Pol::load(rec[i]);
    const ET e2 = ET(eps2);
    const ET hh_e = ET(h2[qq] + eps2), hh_0 = ET(h2[qq]);   // h^2 + eps_ij^2 for soft and hard pairs
    const bool i_hard = i < n_hard;
    double acc[13];
    Part p[13];
#pragma unroll
    for (int c = 0; c < 13; ++c) {
        acc[c] = 0.0;
        zero_part(p[c]);
    }
    static_assert(Pol::kChunk == 0 || Pol::kChunk == kNbChunk, "the FP32 chunk");
    int cnt = 0;
    SegT *my_seg = seg + (int64_t(split) * n_act + qq) * max_nb;
    // j below n_hard: each pair's terms added into FP64 on their own
    const int64_t jh1 = j1 < n_hard ? j1 : n_hard;
    for (int64_t j = j0; j < jh1; ++j) {
        const Rec rj = rec[j];
        Part ph[13];
#pragma unroll
        for (int c = 0; c < 13; ++c) zero_part(ph[c]);
        const bool is_nb = nb_pair(ip, rj, i_hard ? ET(0) : e2, i_hard ? hh_0 : hh_e, j != i, ph);
        if (is_nb) {
            if (row && cnt < max_nb) my_seg[cnt] = SegT(j - j0);
            ++cnt;
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) acc[c] += to_double(ph[c]);
    }
    // the rest (softened pairs) through double-buffered LDS tiles; the FP32 sums
    // are flushed after every chunk
    constexpr int PIECES = int(sizeof(Rec) / 16) * kNbTile / kNbBlock;   // 16-byte pieces a lane moves per tile
    typedef uint4 __attribute__((may_alias)) piece_t;
    __shared__ Rec tile[2][kNbTile];
    const int64_t js0 = j0 > n_hard ? j0 : n_hard;
    const int left0 = int(j1 - js0);   // at most one split
    const piece_t *src = reinterpret_cast<const piece_t *>(rec + js0) + threadIdx.x;
    const int64_t last = int64_t(left0) * int(sizeof(Rec) / 16) - 1 - int(threadIdx.x);   // of src's pieces
    piece_t pre[PIECES];
#pragma unroll
    for (int k = 0; k < PIECES; ++k) pre[k] = piece_t{0u, 0u, 0u, 0u};
    if (left0 > 0)
#pragma unroll
        for (int k = 0; k < PIECES; ++k)
            if (k * kNbBlock <= last) pre[k] = src[k * kNbBlock];
    const int self = int(i - js0);   // |i - js0| < 2^26
    int buf = 0;
    for (int t = 0; t < left0; t += kNbTile) {
        piece_t *dst = reinterpret_cast<piece_t *>(tile[buf]) + threadIdx.x;
#pragma unroll
        for (int k = 0; k < PIECES; ++k) dst[k * kNbBlock] = pre[k];
        __syncthreads();
        const int at = (t + kNbTile) * int(sizeof(Rec) / 16);
#pragma unroll
        for (int k = 0; k < PIECES; ++k)
            if (at + k * kNbBlock <= last) pre[k] = src[at + k * kNbBlock];
        const Rec *tr = tile[buf];
        unsigned hits = 0;
        if (left0 - t >= kNbTile) {
#pragma unroll 1
            for (int u = 0; u < kNbTile; u += kNbGroup) {
                SoftPair<ET> sp[kNbGroup];
                bool any = false;
#pragma unroll
                for (int k = 0; k < kNbGroup; ++k) {
                    sp[k].set(ip, tr[u + k], e2, hh_e);
                    any = any || sp[k].is_nb;
                }
                if (__builtin_amdgcn_ballot_w64(any)) {
#pragma unroll
                    for (int k = 0; k < kNbGroup; ++k) {
                        sp[k].mr = sp[k].is_nb ? ET(0) : sp[k].mr;
                        hits |= sp[k].is_nb ? 1u << (u + k) : 0u;
                    }
                }
#pragma unroll
                for (int k = 0; k < kNbGroup; ++k) sp[k].add(p);
            }
        } else {
            for (int u = 0; u < left0 - t; ++u) {
                SoftPair<ET> sp;
                sp.set(ip, tr[u], e2, hh_e);
                sp.mr = sp.is_nb ? ET(0) : sp.mr;
                hits |= sp.is_nb ? 1u << u : 0u;
                sp.add(p);
            }
        }
        while (hits) {
            const int u = t + __builtin_ctz(hits);
            hits &= hits - 1;
            if (u == self) continue;
            if (row && cnt < max_nb) my_seg[cnt] = SegT(js0 - j0 + u);
            ++cnt;
        }
        if (((t + kNbTile) & (kNbChunk - 1)) == 0) flush<Part, 1>(&p, &acc);
        buf ^= 1;
    }
    flush<Part, 1>(&p, &acc);
    if (!row) return;
    // split-fastest: the finishing kernel's lanes read consecutive splits
#pragma unroll
    for (int c = 0; c < 6; ++c) part[(int64_t(c) * n_act + q) * n_split + split] = acc[c];
    seg_cnt[q * n_split + split] = cnt;
}

// One 64-lane workgroup per active row: for each of the 6 regular
// components, lane l adds the row's partial sums of splits l, l + 64, ... in
// order and a fixed butterfly folds the lanes; all lanes copy the splits'
// neighbour lists one after the other (increasing j, at most max_nb entries);
// then lane l adds the irregular terms of list entries l, l + 64, ... and the
// lanes' sums are folded with a fixed butterfly.
// Bound by the latency of its dependent loads (one wave per row, a wave or two per
// SIMD): with the loads of all splits and of the lists' first entries in flight
// together 14.9 us at 342 splits of 1024 rows instead of 22.7.
template <class Pol, class SegT>
__global__ void __launch_bounds__(64)
k_nb_finish(const typename Pol::Rec *__restrict__ rec, int64_t n, const int32_t *__restrict__ act, int64_t n_act,
            double eps2, int64_t n_hard, int n_split, int64_t j_chunk, int max_nb, const double *__restrict__ part,
            const int32_t *__restrict__ seg_cnt, const SegT *__restrict__ seg, double *__restrict__ acc_irr,
            double *__restrict__ jrk_irr, double *__restrict__ acc_reg, double *__restrict__ jrk_reg,
            int32_t *__restrict__ nb_count, int32_t *__restrict__ nb_list)
{
    using ET = typename Pol::ET;
    using Part = typename Pol::Part;
    const int64_t q = blockIdx.x;
    const int l = int(threadIdx.x);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        double s = lane_sum<64>(part + (int64_t(c) * n_act + q) * n_split, l, n_split, 1);
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) s += __shfl_xor(s, m, 64);
        if (l == 0) (c < 3 ? acc_reg : jrk_reg)[(c % 3) * n_act + q] = s;
    }
    // the lists: 64 splits at a time, lane l taking split s0 + l; a prefix sum
    // over the lanes places each split's entries after those of the splits
    // before it, and at most max_nb entries are kept in all.  The counts of
    // up to kNbPass passes are loaded together first, then the first entries of
    // the lists that have one (most have none or one): two memory round trips for
    // them instead of two per pass.
    constexpr int kNbPass = 16;
    int64_t total = 0;
    int written = 0;
    int cnts[kNbPass], firsts[kNbPass];
    for (int s0 = 0; s0 < n_split; s0 += 64) {
        const int pass = (s0 / 64) % kNbPass;
        if (pass == 0) {
#pragma unroll
            for (int k = 0; k < kNbPass; ++k) {
                const int spk = s0 + 64 * k + l;
                cnts[k] = spk < n_split ? seg_cnt[q * n_split + spk] : 0;
            }
#pragma unroll
            for (int k = 0; k < kNbPass; ++k) {
                const int spk = s0 + 64 * k + l;
                firsts[k] = cnts[k] > 0 && max_nb > 0 ? int(seg[(int64_t(spk) * n_act + q) * max_nb]) : 0;
            }
        }
        const int sp = s0 + l;
        int c = 0, first = 0;
#pragma unroll
        for (int k = 0; k < kNbPass; ++k) {
            c = k == pass ? cnts[k] : c;
            first = k == pass ? firsts[k] : first;
        }
        const int stored = c < max_nb ? c : max_nb;
        int incl = stored;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(incl, o, 64);
            if (l >= o) incl += t;
        }
        const int base = written + (incl - stored);
        const int room = max_nb - base;
        const int take = room <= 0 ? 0 : (stored < room ? stored : room);
        const int32_t j0 = int32_t(sp * j_chunk);   // (only used when the split is there)
        const SegT *src = seg + (int64_t(sp < n_split ? sp : 0) * n_act + q) * max_nb;
        if (take > 0) nb_list[q * max_nb + base] = j0 + first;
        for (int k = 1; k < take; ++k) nb_list[q * max_nb + base + k] = j0 + int32_t(src[k]);
        const int all = __shfl(incl, 63, 64);
        written = written + all < max_nb ? written + all : max_nb;
        int64_t cs = c;
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) cs += __shfl_xor(cs, m, 64);
        total += cs;
    }
    if (l == 0) nb_count[q] = int32_t(total);
    __syncthreads();   // the row's list is complete in memory
    const int64_t ia = act[q];
    const int64_t i = (ia >= 0 && ia < n) ? ia : 0;
    const typename Pol::I ip = Pol::load(rec[i]);
    const ET e2 = ET(eps2);
    const bool i_hard = i < n_hard;
    double acc[13];
    Part p[13];
#pragma unroll
    for (int c = 0; c < 13; ++c) {
        acc[c] = 0.0;
        zero_part(p[c]);
    }
    for (int k = l; k < written; k += 64) {   // at most 64 terms per lane: one FP32 chunk
        const int64_t j = nb_list[q * max_nb + k];
        Pol::template pair<true>(ip, rec[j], (i_hard && j < n_hard) ? ET(0) : e2, true, p);
    }
    flush<Part, 1>(&p, &acc);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1)
#pragma unroll
        for (int c = 0; c < 6; ++c) acc[c] += __shfl_xor(acc[c], m, 64);
    if (l < 6) {
        const double v = total > written ? __builtin_nan("") : acc[l];   // a cut list: no irregular part
        (l < 3 ? acc_irr : jrk_irr)[(l % 3) * n_act + q] = v;
    }
}

template <class Pol, class SegT>
hipError_t run_nb(const NbArgs &a, hipStream_t s, int n_split, int64_t j_chunk)
{
    const Places places = places_for((a.n_act + kNbBlock - 1) / kNbBlock, n_split, true);
    double *part = a.scratch;
    int32_t *seg_cnt = reinterpret_cast<int32_t *>(part + int64_t(n_split) * 6 * a.n_act);
    SegT *seg = reinterpret_cast<SegT *>(seg_cnt + int64_t(n_split) * a.n_act);
    hipLaunchKernelGGL((k_force_nb<Pol, SegT>), dim3(place_grid(places)), dim3(kNbBlock), 0, s,
                       static_cast<const typename Pol::Rec *>(a.rec), a.n, a.act, a.n_act, a.h2, a.eps2, a.n_hard,
                       j_chunk, a.max_nb, n_split, part, seg_cnt, seg, places);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_nb_finish<Pol, SegT>), dim3(unsigned(a.n_act)), dim3(64), 0, s,
                       static_cast<const typename Pol::Rec *>(a.rec), a.n, a.act, a.n_act, a.eps2, a.n_hard, n_split,
                       j_chunk, a.max_nb, part, seg_cnt, seg, a.acc_irr, a.jrk_irr, a.acc_reg, a.jrk_reg, a.nb_count,
                       a.nb_list);
    return hipGetLastError();
}

template <class Pol> hipError_t run_seg(const NbArgs &a, hipStream_t s, int n_split, int64_t j_chunk)
{
    if (j_chunk <= kShortChunk) return run_nb<Pol, uint16_t>(a, s, n_split, j_chunk);
    return run_nb<Pol, int32_t>(a, s, n_split, j_chunk);
}

// Splits are whole FP32 chunks in MIXED; FP64 has none to keep.
int64_t nb_grain(int precision) { return precision == NBODY_MIXED ? kNbChunk : 32; }

int64_t nb_chunk(int precision, int64_t n, int64_t n_split)
{
    const int64_t g = nb_grain(precision), c = (n + n_split - 1) / n_split;
    return (c + g - 1) / g * g;
}

// Bytes of scratch one (split, row) pair needs: 6 partial sums, a count and
// max_nb list entries.
int64_t nb_scratch_per_row(int max_nb, int64_t entry) { return 6 * 8 + 4 + entry * int64_t(max_nb); }

}  // namespace

// About 8192 waves (8 to a SIMD, where five or six fit: the ends of the first
// fill with the rest), splits of at least one grain, and what the scratch
// holds: it must hold one split with entries of four bytes.
int nb_split(int precision, int64_t n, int64_t n_act, int max_nb, int64_t scratch_bytes)
{
    const int64_t rows = n_act > 0 ? n_act : 1;
    const int64_t tiles = (rows + kNbBlock - 1) / kNbBlock;
    const int64_t fit4 = scratch_bytes / (nb_scratch_per_row(max_nb, 4) * rows);
    const int64_t fit2 = scratch_bytes / (nb_scratch_per_row(max_nb, 2) * rows);
    if (fit4 < 1) return 0;
    int64_t sp = (8192 + tiles - 1) / tiles;
    // (FP64: shorter than 128 particles only up to 512 splits, whose sums and lists
    // kernel 2 adds up: n = 40000, 300 rows 56 us with 313 splits, 80 with 1250, and
    // with three waves to a SIMD at most: n = 3000, 3000 rows 48 us with 94 splits, 35
    // with 47)
    const int64_t by_n = (n + kNbChunk - 1) / kNbChunk, by_grain = (n + nb_grain(precision) - 1) / nb_grain(precision);
    const int64_t few = 3072 / tiles > 1 ? 3072 / tiles : 1;   // (three such waves to a SIMD)
    int64_t fine = by_grain < 512 ? by_grain : 512;
    if (fine > few) fine = few;
    if (sp > (by_n > fine ? by_n : fine)) sp = by_n > fine ? by_n : fine;
    if (sp > 65535) sp = 65535;
    const int64_t sp2 = sp < fit2 ? sp : fit2;
    if (nb_chunk(precision, n, sp2) <= kShortChunk) return int(sp2);
    return int(sp < fit4 ? sp : fit4);
}

hipError_t launch_force_nb(int precision, const NbArgs &a, int n_split, hipStream_t s)
{
    const int64_t j_chunk = nb_chunk(precision, a.n, n_split);
    const int sp = int((a.n + j_chunk - 1) / j_chunk);
    if (precision == NBODY_MIXED) return run_seg<PolMx<4, false>>(a, s, sp, j_chunk);
    return run_seg<PolF64<4, false>>(a, s, sp, j_chunk);
}

}  // namespace nb
