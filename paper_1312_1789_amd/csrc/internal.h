// internal.h -- shared definitions of the gfx950 N-body library (not part of
// the public C-ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "nbody.h"

namespace nb {

// Record an error message (thread-local, returned by nbody_last_error) and
// return s.
nbody_status fail(nbody_status s, const char *fmt, ...);
const char *last_error();
// Validate a configuration (records the message on failure).
nbody_status check_config_checked(const nbody_config *c);

#define NB_HIP(call)                                                                                 \
    do {                                                                                             \
        hipError_t e_ = (call);                                                                      \
        if (e_ != hipSuccess) return nb::fail(NBODY_E_HIP, "%s: %s", #call, hipGetErrorString(e_));  \
    } while (0)

constexpr int kLevelMax = 40;               // time tick = 2^-40 time units; levels k <= 40
constexpr int64_t kTicksPerUnit = int64_t(1) << kLevelMax;
constexpr int kSchedBlock = 256;            // threads per scheduler block
constexpr int kSchedPerThread = 4;          // particles per scheduler thread
constexpr int kSchedChunk = kSchedBlock * kSchedPerThread;
constexpr int kMixedChunk = 128;            // FP32 partial-sum length in MIXED mode
constexpr int64_t kPartEntries = int64_t(1) << 21;  // j-split partial rows (n_act * n_split), at least
// Rows of j-split partial sums a context keeps (n_act * n_split <= rows): 16 per
// particle, so that an all-active force call can still take 16 splits, at
// least kPartEntries and at most 2^26 (7 GB of doubles).
inline int64_t part_rows_for(int64_t n)
{
    const int64_t r = 16 * n;
    return r < kPartEntries ? kPartEntries : (r > (int64_t(1) << 26) ? (int64_t(1) << 26) : r);
}
constexpr int kMaxComp = 13;                // acc3 + jerk3 + snap3 + crackle3 + pot
constexpr int kMaxNeighbours = 4096;        // neighbour-list capacity per row, at most

// Time-step rule in use (orders 6, 8): 1 = generalised criterion of the
// scheme's order, 2 = its order-4 form.  dt_rule 0 picks the order-4 form
// where the interpolated derivatives of the full-order criterion are
// dominated by rounding noise at short steps: a force with single-precision
// arithmetic, or order 8.
inline int dt_rule_of(const nbody_config &c)
{
    if (c.dt_rule != 0) return c.dt_rule;
    return (c.precision != NBODY_FP64 || c.order == 8) ? 2 : 1;
}

// Post-Newtonian terms between hard particles switched on.
inline bool pn_on(const nbody_config &c) { return c.c_light > 0.0 && c.pn_terms != 0 && c.n_hard >= 2; }

// Components of a force result for a Hermite order: 3 per derivative + pot.
inline int n_comp(int order) { return 3 * (order / 2) + 1; }

// Bytes of one predicted j-particle record.
int record_bytes(int order, int precision);

// Offsets of the sub-buffers inside the caller's workspace (bytes).
struct Layout {
    size_t rec;        // predicted records, n * record_bytes
    size_t part;       // j-split partial sums, part_rows_for(n) * kMaxComp doubles
    size_t force;      // step force outputs, kMaxComp-1 rows of n doubles ([12][n])
    size_t act;        // active indices, n int32
    size_t sched;      // scheduler per-block scratch (min ticks, counts, offsets)
    size_t scal;       // device scalars: t_next, n_act, counters; the step kernel's arrival counters
    size_t init;       // init scratch: 4 x [3][n] doubles (a, j, s, c of the two passes)
    size_t irec;       // init records (FP64 order-8 layout), n * 112
    size_t total;
};
Layout make_layout(const nbody_config &c);

// Device scalars at Layout::scal.
struct DevScalars {
    int64_t t_next;
    int64_t n_act;
    unsigned long long underflow;
    unsigned long long nonfinite;
    int64_t seq;                    // of the last schedule published by the step kernel
    int64_t halt;                   // a corrected value was not finite: no further small step
    unsigned long long nonfinite0;  // nonfinite as the host last read it before the run
    int64_t pad;
};

// Active sets that the small-step kernels take, and the split of each size
// (n_split 0: not taken).
constexpr int kSmallMax = 64;   // a lane of a wave each
struct SmallTable {
    int32_t n_split[kSmallMax];
    int32_t j_chunk[kSmallMax];
};

// The value lane `lane` (uniform) holds.  (The small-step kernels load their table
// into the lanes of a wave while the scheduler's result, its index, is in
// flight: a launch's arguments are as far away as any memory.)
__device__ __forceinline__ int of_lane(int v, int64_t lane) { return __builtin_amdgcn_readlane(v, int(lane)); }

// Whether the step the scheduler found is one for the small-step kernels;
// lane l holds n_split[l] of their table.
__device__ __forceinline__ bool small_step(const DevScalars &d, int n_split, int64_t t_limit)
{
    const int64_t na = d.n_act;
    return (na >= 1) & (na <= kSmallMax) & (d.t_next <= t_limit) & !d.halt & (of_lane(n_split, (na - 1) & 63) > 0);
}

// Lanes that share the sum of one output over n partials: each adds at most about 8.
__host__ __device__ constexpr int reduce_lanes(int n) { return n <= 8 ? 1 : n <= 32 ? 4 : n <= 128 ? 16 : 64; }

// Lane l of the L that share a sum over n partials: src[k * step], k = l, l + L, ...,
// added in order, eight loads in flight together (one memory round trip for
// all of them, also where fewer are left; the zeros in their place change
// nothing).
template <int L>
__device__ __forceinline__ double lane_sum(const double *__restrict__ src, int l, int n, int64_t step)
{
    double s = 0.0;
    for (int k = l; k < n; k += 8 * L) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = k + u * L < n ? src[int64_t(k + u * L) * step] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    return s;
}

// Which i-tile and split a workgroup of a force kernel has.  The dispatcher places
// workgroup g on XCD g mod 8.  Stored split-fastest, 16 consecutive splits of a row
// share a memory line, and 8-byte stores to one line from several XCDs reach memory
// one by one; so each unit of 2^shift consecutive splits of an i-tile goes to one
// XCD, as large (up to 16) as leaves 256 units.  In the plain order (units of one)
// the splits of a tile lie on one XCD only where 8 divides the number of tiles: n =
// 32768, 17 tiles of 64 rows MIXED order 4, 256 splits: 60 us, 47 by units (16 tiles:
// 46 and 45).
constexpr int kXcdCount = 8;
struct Places {
    unsigned tiles, units;
    int shift;
};
inline Places places_for(int64_t tiles, int n_split, bool units)
{
    Places p{unsigned(tiles), 0, 0};
    while (units && p.shift < 4 && tiles * n_split >= (int64_t(256) << (p.shift + 1))) ++p.shift;
    p.units = p.tiles * ((unsigned(n_split) + (1u << p.shift) - 1u) >> p.shift);
    return p;
}
inline unsigned place_grid(const Places &p) { return (p.units + kXcdCount - 1) / kXcdCount * kXcdCount << p.shift; }

// False for a workgroup past the last unit or split.
__device__ __forceinline__ bool place(const Places &p, int n_split, int64_t *tile, int *split)
{
    const unsigned slot = blockIdx.x / kXcdCount, u = (slot >> p.shift) * kXcdCount + blockIdx.x % kXcdCount;
    const unsigned group = u / p.tiles;
    *tile = u - group * p.tiles;
    *split = int((group << p.shift) + (slot & ((1u << p.shift) - 1u)));
    return u < p.units && *split < n_split;
}

// Force launch request.
struct ForceArgs {
    const void *rec;        // predicted records
    int64_t n;
    const int32_t *act;
    int64_t n_act;
    double eps2;
    int64_t n_hard;         // already n when eps2 == 0
    double *out[5];         // acc, jrk, snp, crk, pot ([3][n_act] / [n_act]); may be null
    double *part;           // partial-sum scratch
    int64_t part_rows;      // its capacity in rows of kMaxComp doubles (n_act * n_split <= part_rows)
    int ni, block, n_split; // launch shape (n_split 0 = auto)
    bool fine;              // n_split is a tuned count: splits may be as short as the default ones
    int jpath;              // 0 auto, 1 scalar loads, 2 LDS tiles, 3 wave j-split
};

// The launch shape a force call ran with (n_split after the scratch bound).
struct UsedShape {
    int ni, block, n_split, jpath;
};

hipError_t launch_force(int order, int precision, const ForceArgs &a, hipStream_t s, UsedShape *used);

// Snap and crackle alone, FP64 order 8 (a.rec: RecF64<8>, outputs a.out[2] and
// a.out[3]): the second initialisation pass.  One row per lane, scalar j path.
// With the first pass at order 4 (it had run the order-8 kernel too) nbody_init
// at order 6 and n = 40961 takes 6999 us instead of 10880.
hipError_t launch_force_high(const ForceArgs &a, hipStream_t s, UsedShape *used);

// j-splits and split length of a force launch: n_split_req > 0 is taken as
// given, bounded by the partial-sum scratch (n_act * n_split <= part_rows) and by
// the split length (at least one MIXED chunk, less when `fine`); 0 chooses from
// n_act and the shape.
void split_shape(int precision, int64_t n, int64_t n_act, int n_split_req, bool fine, int ni, int jpath,
                 int64_t part_rows, int *n_split, int64_t *j_chunk);
// The shape of an untuned call.
void default_shape(int precision, int order, bool pot, int64_t n, int64_t n_act, int *ni, int *block, int *jpath);

// Fixed-order sum of n_split partial results in part[component][row][split]
// into a.out.
hipError_t launch_split_reduce_sf(int order, const ForceArgs &a, int n_split, hipStream_t s);

// The stored state the predictor reads, and the time it predicts to.
struct PredIn {
    const double *m, *x, *v;
    const double *d[6];      // stored derivatives a^(0..p-3), [3][n] each
    const int64_t *t_tick;
    int64_t t;
};

struct OutPtrs {
    double *p[5];
};

// The wave j-split force (ForceArgs.jpath 3) with the predictor in its j
// loads: a.rec is not read; the j-particles and the active i-particles are
// predicted from `in` to in.t, exactly as the predictor kernel writes them.
hipError_t launch_force_pred(int order, int precision, const ForceArgs &a, const PredIn &in, hipStream_t s,
                             UsedShape *used);
// The same for the step that the scheduler has written to dev (active set
// a.act, split from tab); leaves the partial sums of each group of
// small_group splits in a.part, and does nothing when the step is not
// small or past t_limit.
hipError_t launch_force_small_dev(int order, int precision, const ForceArgs &a, const PredIn &in,
                                  const DevScalars *dev, const SmallTable &tab, int64_t t_limit, hipStream_t s);
// Consecutive splits whose sums that kernel adds in one workgroup: as few as give
// each of the 256 CUs a workgroup, at most 8 (4, 2: a split is then two or four
// waves).  A CU takes some 40 GB/s from HBM or another XCD's L2, so that 8 splits
// to a workgroup left calls of few splits waiting for a part of the chip.
__host__ __device__ inline int small_group(int64_t n_act, int n_split)
{
    const int most = n_act <= 16 ? 8 : (n_act <= 32 ? 4 : 2);
    const int64_t wgs = n_split * ((n_act + 63) / 64);
    int gs = 1;
    while (gs < most && wgs > 256 * gs) gs *= 2;
    return gs;
}

// The end of a block step and the schedule of the next one (step.hip).
constexpr int kStepBlock = 256;                    // particles (and threads) per workgroup
// Systems it takes: its last workgroup goes over the times of all blocks, which
// costs as much as the launches saved at about n = 220000 (a step of a run, MIXED order
// 4: n = 131072 32 us, separate kernels 44; n = 180000 57 and 59; n = 262144 49 and 45;
// n = 2^20 111 and 77).
constexpr int64_t kStepMaxN = 3 * (int64_t(1) << 16);
constexpr int kStepGather = 4096;                  // active sets it lists itself
constexpr int kStepSub = 64;                       // workgroups per arrival counter
constexpr int kStepCounters = int(kStepMaxN / kStepBlock) / kStepSub + 1;
struct StepBlock {
    int64_t t_next;     // next time of a block of kStepBlock particles
    int64_t count;      // its particles at it
};
struct StepScratch {
    StepBlock *blk;     // [nb]
    int32_t *boff;      // [nb] active particles before the block
    int32_t *cand;      // [nb][kStepBlock] the block's particles at its next time
    unsigned *arrive;   // [kStepCounters], zero between launches
    int32_t *act;       // [n] the active list
};
enum StepMode {
    kStepSchedule,      // only the schedule (starts a run: seq is the first sequence number)
    kStepSmall,         // a small step from the partial sums of launch_force_small_dev
    kStepForces         // any step from its forces f[k] ([3][n_act])
};
struct StepArgs {
    nbody_config cfg;
    int rule;                    // dt_rule_of(cfg)
    nbody_state st;
    StepScratch w;
    DevScalars *sc;
    struct HostScalars *pub;     // slots of the published schedules
    StepMode mode;
    int64_t seq;
    unsigned long long nonfinite;   // kStepSchedule: non-finite values the host knows of
    SmallTable tab;              // kStepSmall
    const double *part;          // kStepSmall
    double *f[4];                // kStepForces
    int64_t t_limit;             // kStepSmall
    bool pn;                     // add the post-Newtonian terms (n_hard <= kStepBlock)
};
hipError_t launch_step(const StepArgs &a, hipStream_t s);
// The active list of n_act > kStepGather particles.
hipError_t launch_step_gather(const StepScratch &w, int64_t n, const DevScalars *sc, hipStream_t s);

// Force split by neighbour spheres (order-4 terms) with the neighbour lists.
struct NbArgs {
    const void *rec;        // predicted records (order 4)
    int64_t n;
    const int32_t *act;
    int64_t n_act;
    const double *h2;       // neighbour radius squared per active row
    double eps2;
    int64_t n_hard;         // already n when eps2 == 0
    int max_nb;             // list capacity per row
    double *scratch;        // partial sums and per-split lists
    double *acc_irr, *jrk_irr, *acc_reg, *jrk_reg;   // [3][n_act]
    int32_t *nb_count;      // [n_act]
    int32_t *nb_list;       // [n_act][max_nb] (may be null when max_nb == 0)
};
// The split count for a scratch of the given size (0 when it cannot hold one
// split); the launch (FP64 or MIXED).
int nb_split(int precision, int64_t n, int64_t n_act, int max_nb, int64_t scratch_bytes);
hipError_t launch_force_nb(int precision, const NbArgs &a, int n_split, hipStream_t s);

// The default split count of a j path.
int auto_split(int precision, int64_t n, int64_t n_act, int ni, int jpath, int64_t part_rows);

// One row of the force-launch table filled by nbody_autotune.
struct TuneRow {
    int64_t n_act;
    int ni, block, n_split, jpath;
    double ms;
};
constexpr int kTuneRows = 32;

// Pack FP64 records from state arrays: order 4 {x, m, v} (a and j null), or
// order 8 {x, m, v, a, j}.
hipError_t launch_pack_f64(int64_t n, const double *m, const double *x, const double *v, const double *a,
                           const double *j, void *rec, hipStream_t s);

hipError_t launch_predict(int order, int precision, int64_t n, const nbody_state &st, int64_t t_tick,
                          void *rec, hipStream_t s);

// Corrector for act[0..n_act); when src is non-null the count and the end
// time are read from it on the device (n_act is then an upper bound).
hipError_t launch_correct(const nbody_config &c, const nbody_state &st, int64_t n_act, const int32_t *act,
                          const DevScalars *src, int64_t t_tick_host, const double *const f[4],
                          DevScalars *sc, hipStream_t s);

hipError_t launch_iota(int64_t n, int32_t *a, hipStream_t s);

// Adds the post-Newtonian terms of the hard pairs to acc, jrk and, when not
// null, snp and crk ([3][n_act]) for the rows of act (increasing indices; the hard particles,
// indices below n_hard, come first) predicted to t_tick (t_tick_of null: the
// state as it is).
hipError_t launch_pn(const nbody_config &c, const nbody_state &st, const int64_t *t_tick_of, int64_t t_tick,
                     const int32_t *act, int64_t n_act, double *acc, double *jrk, double *snp, double *crk,
                     hipStream_t s);

hipError_t launch_unpack(int order, int precision, int64_t n, const void *rec, double *xp, double *vp, double *ap,
                         double *jp, hipStream_t s);

// The scheduler's result for the host: written by the scheduler into
// pinned, coherent host memory, so that the host can wait for it by polling
// (all words written, see read_published) instead of a copy and a stream
// synchronisation.
// One slot per sequence number modulo kPubSlots (a run has a few steps in
// flight).
constexpr int kPubSlots = 8;
constexpr int64_t kPubEmpty = INT64_MIN;   // a word not written yet: no time, count or counter has this value
struct HostScalars {
    int64_t t_next;
    int64_t n_act;
    unsigned long long underflow;
    unsigned long long nonfinite;
    int64_t seq;
    int64_t pad[3];
};

// pub (device address of a HostScalars, may be null) receives the result
// with sequence number seq.
hipError_t launch_schedule(int64_t n, const int64_t *t_tick, const int32_t *level, void *sched_scratch,
                           int32_t *act_out, DevScalars *sc, HostScalars *pub, int64_t seq, hipStream_t s);

hipError_t launch_init_levels(const nbody_config &c, const nbody_state &st, const double *a, const double *j,
                              hipStream_t s);

// Energy of n particles whose [3][.] arrays have row stride `stride`:
// energy_partials(n) pairs (kinetic, potential), to be summed in order.
int energy_partials(int64_t n);
hipError_t launch_energy(int64_t n, int64_t stride, int64_t n_hard, double eps2, const double *m, const double *x,
                         const double *v, double *partials, hipStream_t s);

}  // namespace nb

struct nbody_ctx {
    nbody_config cfg;
    hipStream_t stream;
    char *ws;
    size_t ws_bytes;
    nb::Layout lay;
    int device;
    nb::HostScalars *pub_host;        // pinned host copy of the scheduler result (null: copy path)
    nb::HostScalars *pub_dev;         // its device address
    int64_t pub_seq;                  // the last schedule's number, and that of the last one read from its slot
    int64_t pub_read;
    bool predicted;
    bool fuse;                        // predictor folded into the wave j-split force (nbody_set_fusion)
    int ni, block, n_split, jpath;   // launch shape fixed by nbody_set_launch (when manual)
    nb::UsedShape last_shape;         // shape of the last force launch (nbody_get_last_launch)
    bool manual;
    bool tuned;                       // tune[] filled by nbody_autotune
    int n_tune;
    nb::TuneRow tune[nb::kTuneRows];
    nbody_stats stats;
    bool timing;              // record phase events in nbody_step
    hipEvent_t ev[6];         // phase boundaries (created on first enable)
    bool ev_made;
    double phase_ms[5];
    int64_t timed_steps;
};
