// How the batched step's plan cuts its work, on the host: the sums that the
// scheduling kernel makes over the clusters, for a launch shape and active
// counts given as arguments.
#include <algorithm>

#include "batch.h"

// out: items, partial rows (sum of splits x active rows), least and most splits
// of a cluster with active rows; nn and na: [nc] particles and active rows.
extern "C" void batch_plan(int nc, const int64_t *nn, const int64_t *na, int force_grid, int per_wg, int itile,
                           int halves, int grain, int64_t out[4])
{
    nb::BatchLaunch L{};
    L.force_grid = force_grid;
    L.per_wg = per_wg;
    L.k_items = int(std::min<int64_t>(int64_t(force_grid) * per_wg, nb::kBatchMaxRows / itile));
    L.itile = itile;
    L.halves = halves;
    L.grain = grain;
    int64_t W = 0;
    for (int c = 0; c < nc; ++c) W += (na[c] + itile - 1) / itile * itile * nn[c];
    const int64_t w_item = nb::b_item_size(L, W);
    out[0] = out[1] = 0;
    out[2] = INT64_MAX;
    out[3] = 0;
    for (int c = 0; c < nc; ++c) {
        const nb::BatchCut k = nb::b_cut(na[c], nn[c], itile, grain, w_item);
        out[0] += int64_t(k.tiles) * k.sp * nb::b_tile_items(L);
        out[1] += int64_t(k.sp) * na[c];
        if (na[c] > 0) {
            out[2] = std::min<int64_t>(out[2], k.sp);
            out[3] = std::max<int64_t>(out[3], k.sp);
        }
    }
}
