// Launches of contractions of different shapes, one instance per tile of the list rule (run_list.cpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "contract_launch.hip.h"
#include "contract_list.hip.h"
#include "contract_thin.hip.h"

namespace tt {

namespace {

template <typename Kernel> int launch_listed(Kernel kern, const ContractList &list, int grid, int threads, int lds_bytes, DynamicLdsLimit &limit, void *stream)
{
    if (const int rc = limit.raise_to(reinterpret_cast<const void *>(kern), lds_bytes); rc != TT_OK) return rc;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds_bytes, static_cast<hipStream_t>(stream), list);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, "contract_list_kernel launch");
}

template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF> int launch_tiles(const ContractList &list, int grid, void *stream)
{
    static DynamicLdsLimit limit; // per kernel instance
    constexpr int LDS = std::max(3 * RingLayout<DT, TM, TN, TK>::STAGE_BYTES, epilogue_bytes(TM, TN, WM, WN, MF));
    return launch_listed(contract_list_kernel<DT, FAM, TM, TN, TK, WM, WN, MF>, list, grid, (TM / WM) * (TN / WN) * 64, LDS, limit, stream);
}

template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF> int launch_group_list(const ContractList &list, int grid, void *stream)
{
    static DynamicLdsLimit limit;
    using S = GroupShape<DT, TM, TN, WM, WN, MF>;
    static_assert(S::KG > 1, "");
    return launch_listed(contract_groups_list_kernel<DT, FAM, TM, TN, WM, WN, MF>, list, grid, S::THREADS, S::LDS, limit, stream);
}

template <int FAM> int launch_block_list(const ContractList &list, int grid, void *stream)
{
    static DynamicLdsLimit limit;
    using S = BlockShape<FAM>;
    return launch_listed(contract_block_list_kernel<FAM>, list, grid, S::THREADS, S::LDS, limit, stream);
}

} // namespace

#define TT_TILE(DT_, TM_, TN_, TK_, WM_, WN_, FIXED_, PER_K_, ALONE_)                                                                  \
    {                                                                                                                                  \
        DT_, TM_, TN_, TK_, FIXED_, PER_K_, ALONE_, false,                                                                             \
        {                                                                                                                              \
            launch_tiles<DT_, FAM_CONV, TM_, TN_, TK_, WM_, WN_, 16>, launch_tiles<DT_, FAM_GEMM_TN, TM_, TN_, TK_, WM_, WN_, 16>      \
        }                                                                                                                              \
    }

#define TT_GROUPS(DT_, TM_, TN_, WM_, WN_, FIXED_, PER_K_, ALONE_)                                                                     \
    {                                                                                                                                  \
        DT_, TM_, TN_, GroupShape<DT_, TM_, TN_, WM_, WN_, 16>::TKI, FIXED_, PER_K_, ALONE_, false,                                    \
        {                                                                                                                              \
            launch_group_list<DT_, FAM_CONV, TM_, TN_, WM_, WN_, 16>, launch_group_list<DT_, FAM_GEMM_TN, TM_, TN_, WM_, WN_, 16>      \
        }                                                                                                                              \
    }

// Tiles and what a compute unit spends on one (us), measured in launches of many rounds (outputs streaming to memory, K from
// 64 to 4608): `fixed` + `per_k` * K while the chip is full, `alone` * K where a workgroup has its CU to itself.
const ListTile *list_tiles(int *count)
{
    static const ListTile tiles[] = {
        TT_TILE(TT_BF16, 128, 256, 64, 32, 64, 5.2f, 0.0146f, 0.0146f),
        TT_TILE(TT_BF16, 128, 256, 32, 64, 64, 3.7f, 0.0196f, 0.0160f),
        TT_TILE(TT_BF16, 128, 128, 64, 64, 32, 3.4f, 0.0097f, 0.0097f),
        TT_TILE(TT_BF16, 64, 128, 64, 32, 32, 1.6f, 0.0047f, 0.0066f),
        TT_TILE(TT_BF16, 64, 128, 32, 32, 64, 1.0f, 0.0068f, 0.0100f),
        TT_TILE(TT_BF16, 128, 64, 64, 32, 32, 1.7f, 0.0047f, 0.0066f),
        TT_TILE(TT_BF16, 64, 64, 64, 32, 32, 0.85f, 0.0027f, 0.0050f),
        TT_TILE(TT_BF16, 32, 32, 64, 16, 16, 0.42f, 0.00125f, 0.0042f),
        TT_TILE(TT_F32, 64, 64, 32, 16, 32, 2.0f, 0.0180f, 0.0230f),
        TT_TILE(TT_F32, 32, 32, 32, 16, 16, 0.55f, 0.0052f, 0.0115f),
        TT_TILE(TT_F32, 16, 32, 16, 16, 32, 0.23f, 0.0036f, 0.0200f),
        TT_TILE(TT_F32, 16, 16, 16, 16, 16, 0.13f, 0.0022f, 0.0190f),
        // the reduction split inside the workgroup
        TT_GROUPS(TT_BF16, 64, 64, 32, 32, 3.0f, 0.0030f, 0.0042f),
        TT_GROUPS(TT_F32, 32, 32, 16, 16, 3.2f, 0.0056f, 0.0065f),
        // the 256 x 256 block kernel
        {TT_BF16, 256, 256, 64, 11.0f, 0.0225f, 0.0185f, true, {launch_block_list<FAM_CONV>, launch_block_list<FAM_GEMM_TN>}},
    };
    static_assert(sizeof tiles / sizeof tiles[0] <= kMaxListTiles, "");
    *count = (int)(sizeof tiles / sizeof tiles[0]);
    return tiles;
}
#undef TT_TILE
#undef TT_GROUPS

// Columns: as many as 48 KB of weights hold (three workgroups on a CU), in equal chunks.  Rows: eight turns of the four waves;
// four, two or one where the entry would have less than 384 workgroups, half as many again as CUs.
void thin_layout(ThinEntry *e)
{
    const int pieces = (e->K + 15) / 16, blocks = (e->N + 15) / 16, most = std::max(1, 48 * 1024 / (pieces * 1024));
    e->chunks = (blocks + most - 1) / most;
    e->columns = (blocks + e->chunks - 1) / e->chunks * 16;
    e->chunks = (e->N + e->columns - 1) / e->columns;
    e->rows = 512;
    while (e->rows > 64 && (int64_t)e->chunks * ((e->M + e->rows - 1) / e->rows) < 384) e->rows /= 2;
}

int launch_thin_list(ThinList &list, int count, int pieces, void *stream)
{
    int64_t grid = 0;
    int lds = 0;
    for (int i = 0; i < kMaxThin; ++i) {
        list.first[i] = i < count ? (int32_t)grid : INT32_MAX;
        if (i >= count) continue;
        const ThinEntry &e = list.e[i];
        grid += thin_workgroups(e);
        lds = std::max(lds, e.columns / 16 * ((e.K + 15) / 16) * 1024 + e.columns * 4);
    }
    const int instance = pieces == kThinPieces[0] ? 0 : 1;
    auto kern = instance == 0 ? contract_thin_list_kernel<kThinPieces[0]> : contract_thin_list_kernel<kThinPieces[1]>;
    static DynamicLdsLimit limits[2];
    DynamicLdsLimit &limit = limits[instance];
    if (const int rc = limit.raise_to(reinterpret_cast<const void *>(kern), lds); rc != TT_OK) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, static_cast<hipStream_t>(stream), list);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, "contract_thin_list_kernel launch");
}

} // namespace tt
