// One launch for contractions of DIFFERENT shapes: the independent entries of a list (see run_list.cpp).
//
// A launch costs the chip 2 to 4 us of filling and draining, and a layer of a network at a small batch fills a part of the
// chip for 5 to 30 us.  Entries that do not touch each other's tensors need no launch of their own: the workgroups of up to
// kMaxListed of them, each with its own shape, share one launch of a tile that suits them together.  The tile code is that of
// the ring, groups and block kernels; a workgroup only looks up whose tile it is first.
#pragma once

#include "contract.hip.h"
#include "contract_block.hip.h"
#include "contract_groups.hip.h"

namespace tt {

// The arguments of an entry as the tile code knows them.  What all entries of a launch have in common (tile, raster, ring of
// three, unrolled steps) is constant here, so the tile code is compiled for it.
template <int DT, int FAM, int TM, int TN, int TK> __device__ __forceinline__ ContractArgs args_of(const ListEntry &e)
{
    ContractArgs g = {};
    g.a = e.a, g.b = e.b, g.bias = e.bias, g.res = e.res, g.out = e.out, g.ws = e.ws;
    g.batch = e.batch, g.M = e.M, g.N = e.N, g.K = e.K, g.k_walk = e.K;
    g.map.sketch = TT_SK_MFMA, g.map.order = kListOrder, g.map.grid = e.grid;
    g.map.tiles_m = e.tiles_m, g.map.tiles_n = e.tiles_n, g.map.tile_m = TM, g.map.tile_n = TN, g.map.tile_k = TK;
    g.map.M = e.M, g.map.N = e.N, g.map.K = e.K;
    g.map.eff_split_k = e.splits, g.map.k_iters = e.k_iters, g.map.k_tiles = e.k_tiles;
    g.map.div_tiles = e.div_tiles, g.map.div_n = e.div_n, g.map.div_split = e.div_split;
    g.C = e.C, g.H = e.H, g.W = e.W, g.R = e.R, g.S = e.S, g.Ho = e.Ho, g.Wo = e.Wo;
    g.stride_h = e.stride_h, g.stride_w = e.stride_w, g.pad_h = e.pad_h, g.pad_w = e.pad_w;
    g.run = g.runp = e.S * e.C;
    g.div_hw = e.div_hw, g.div_wo = e.div_wo;
    g.a_bytes = e.a_bytes, g.b_bytes = e.b_bytes;
    g.eff_vec_a = g.eff_vec_b = ElemOf<DT>::CH, g.eff_vec_c = e.vec_c;
    g.stages = 3, g.unroll = 8, g.dtype = DT;
    g.act = e.act, g.has_bias = e.bias != nullptr, g.has_res = e.res != nullptr;
    return g;
}

// Entry of workgroup `wg`, and its first workgroup.
__device__ __forceinline__ int entry_of(const ContractList &list, int wg, int *first)
{
    int e = 0;
#pragma unroll
    for (int i = 1; i < kMaxListed; ++i) e += wg >= list.first[i]; // (entries past the last start past every workgroup)
    *first = list.first[e];
    return e;
}

// (waves a SIMD as without the epilogue of odd rows, see waves_kept: 140 registers for 124 without, 68 for 64)
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF>
__global__ void __launch_bounds__((TM / WM) * (TN / WN) * 64, DT == TT_BF16 ? (TM == 64 && TN == 128 && TK == 32 ? 4 : 1) : (TM == 16 && TN == 32 ? 8 : 1)) contract_list_kernel(const ContractList list)
{
    int first;
    const ListEntry &e = list.e[entry_of(list, (int)blockIdx.x, &first)];
    const int wg = (int)blockIdx.x - first;
    if (wg >= e.grid) return; // (entries begin at multiples of the number of XCDs)
    contract_async_tile<DT, FAM, TM, TN, TK, WM, WN, MF, true>(args_of<DT, FAM, TM, TN, TK>(e), wg);
}

template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF>
__global__ void __launch_bounds__((GroupShape<DT, TM, TN, WM, WN, MF>::THREADS)) contract_groups_list_kernel(const ContractList list)
{
    int first;
    const ListEntry &e = list.e[entry_of(list, (int)blockIdx.x, &first)];
    const int wg = (int)blockIdx.x - first;
    if (wg >= e.grid) return;
    contract_groups_tile<DT, FAM, TM, TN, WM, WN, MF, true>(args_of<DT, FAM, TM, TN, GroupShape<DT, TM, TN, WM, WN, MF>::TKI>(e), wg);
}

template <int FAM> __global__ void __launch_bounds__(512) contract_block_list_kernel(const ContractList list)
{
    int first;
    const ListEntry &e = list.e[entry_of(list, (int)blockIdx.x, &first)];
    const int wg = (int)blockIdx.x - first;
    if (wg >= e.grid) return;
    using S = BlockShape<FAM>;
    contract_block<FAM>(args_of<TT_BF16, FAM, S::BM, S::BN, S::TK>(e), e.tiles_m, e.tiles_n, wg);
}

} // namespace tt
