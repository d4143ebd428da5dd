// Launch of the convolution kernel that keeps the input rows of a tile in LDS.
#include <hip/hip_runtime.h>

#include "conv_rows.hip.h"

namespace tt {

namespace {

struct RowsTile {
    int tile_m, tile_n, threads;
    int (*lds)(const ContractArgs &);
    int (*grid)(const ContractArgs &, int count, int lds);
    int (*launch)(const ContractArgs &, const PointerSets &, void *);
};
#define TT_ROWS(TM_, TN_) {TM_, TN_, RowsShape<TM_, TN_>::THREADS, rows_lds<TM_, TN_>, rows_grid<TM_, TN_>, launch_rows<TM_, TN_>}

// The record's tile, where it has 128 rows or more: what a workgroup does once, and the input rows that neighbouring tiles
// share, count for less there.  Register pipeline -> this (us): 7x7 filters over 3 channels, stride 2, 32 x 224x224 to 64
// channels 128x64 46.8 -> 34.4, 128x32 65.3 -> 45.8, 256x32 72.6 -> 37.4, but 64x64 46.9 -> 46.7 and 64x32 64 -> 91; one
// image 128x64 8.8 -> 8.1, 256x32 10.8 -> 6.8, 32x32 8.9 -> 12.9; 3x3 over 17 channels, 4 x 56x56, 128x32 8.2 -> 6.0; 5x5
// over 9 channels, 8 x 56x56, 128x32 15.5 -> 11.0.  Single precision gained nothing (one image: 12.5 -> 13.5).
const RowsTile *find_tile(const ContractArgs &g)
{
    static const RowsTile tiles[] = {TT_ROWS(128, 32), TT_ROWS(256, 32), TT_ROWS(128, 64), TT_ROWS(256, 64), TT_ROWS(128, 128)};
    if (g.dtype != TT_BF16) return nullptr;
    for (const RowsTile &t : tiles)
        if (t.tile_m == g.map.tile_m && t.tile_n == g.map.tile_n) return &t;
    return nullptr;
}
#undef TT_ROWS

} // namespace

LaunchShape rows_shape(const ContractArgs &args, int count)
{
    const RowsTile *t = find_tile(args);
    const int lds = t ? t->lds(args) : 0;
    return {TT_LAUNCH_ROWS, lds > 0 ? t->grid(args, count, lds) : 0, t ? t->threads : 0, lds};
}

int launch_conv_rows(const ContractArgs &args, const PointerSets &sets, void *stream)
{
    const RowsTile *t = find_tile(args);
    return t ? t->launch(args, sets, stream) : TT_ERR_UNSUPPORTED;
}

} // namespace tt
