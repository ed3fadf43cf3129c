// Order of the work items of the kernels with tiles of a panel or part of one (gemm_mid.hip, gemm_small.hip).
#pragma once
#include "ss_common.h"
#include "mma_types.h"

namespace ss {

// What the workgroups of a launch need to find their items, prepared on the host (Div): nt tiles, tiles_t of them along the tokens, in `bands` bands of `width` token
// tiles (the last one of last_width), S ranges of k.
struct MidOrder {
    int nt, S, by_range, tiles_t, bands, width, last_width, per_band;
    Div by_nt, by_band, by_width, by_last;
    KRanges k;
};
struct MidItem { int panel, tt, range, tile; };
__device__ inline MidItem mid_item(const MidOrder& g)
{
    const int item = g.by_range ? xcd_run(blockIdx.y * g.nt + blockIdx.x, g.nt * g.S) : blockIdx.y * g.nt + xcd_run(blockIdx.x, g.nt);
    const int range = quot(item, g.by_nt), k = item - range * g.nt;
    const int band = quot(k, g.by_band), within = k - band * g.per_band;
    const bool last = band == g.bands - 1;
    const int panel = quot(within, last ? g.by_last : g.by_width), tt = band * g.width + within - panel * (last ? g.last_width : g.width);
    return {panel, tt, range, panel * g.tiles_t + tt};
}

inline MidOrder mid_order(int64_t ntiles, int tiles_t, int S, bool by_range, int64_t units, int widest = 8)
{
    const int bands = (tiles_t + widest - 1) / widest, width = (tiles_t + bands - 1) / bands, last = tiles_t - (bands - 1) * width;
    const int per_band = (int)(width * (ntiles / tiles_t));
    return {(int)ntiles, S, by_range, tiles_t, bands, width, last, per_band, make_div(ntiles), make_div(per_band), make_div(width), make_div(last), k_ranges(units, S)};
}

}  // namespace ss
