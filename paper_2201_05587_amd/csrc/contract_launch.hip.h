// Launchers of the contraction kernels, one per compiled instance: the kernel the record names, or the one that
// splits the reduction inside the workgroup where the record's launch would leave most of the chip idle.
#pragma once

#include "contract.hip.h"
#include "contract_groups.hip.h"
#include "contract_taps.hip.h"

namespace tt {

// LDS the epilogue stages one band of MF rows per wave in (the operands' own).
constexpr int epilogue_bytes(int TM, int TN, int WM, int WN, int MF) { return (TM / WM) * (TN / WN) * MF * (WN + (MF == 32 ? 8 : 4)) * 4; }

// Whether there is a walk by taps in these tiles: beyond, sums and slices do not fit the registers.
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int AM> constexpr bool taps_built()
{
    constexpr int WAVES = (TM / WM) * (TN / WN), ITEMS = (TM + TN) * TK / ElemOf<DT>::CH / (WAVES * 64); // of a slice, for a lane
    return ((FAM == FAM_CONV && AM != 16) || FAM == FAM_GEMM_TN) && WM * WN <= 4096 && WAVES <= 8 && ITEMS <= 8;
}

// What a launch of `count` sets runs on, and the shape it has there.
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF, int AM>
int kernel_contract(const ContractArgs &args, int count, int grid)
{
    if constexpr (FAM == FAM_GEMM_TN || (FAM == FAM_CONV && AM == 16)) {
        if (groups_apply<DT, FAM, TM, TN, WM, WN, MF>(args, grid * count, 0)) return TT_LAUNCH_GROUPS;
    } else if constexpr (FAM == FAM_CONV) {
        if (rows_shape(args, count).grid > 0) return TT_LAUNCH_ROWS;
    }
    if constexpr (taps_built<DT, FAM, TM, TN, TK, WM, WN, AM>())
        if (taps_apply<DT, FAM>(args, (int64_t)grid * count, DT == TT_F32 && TK == 16 && WM * WN == 256 && TM * TN == 1024)) return TT_LAUNCH_TAPS;
    return TT_LAUNCH_RECORD;
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF>
int kernel_contract_async(const ContractArgs &args, int count, int grid, int lds_bytes)
{
    if constexpr (DT == TT_BF16)
        if (block_applies(args, FAM, count, TM * TN)) return TT_LAUNCH_BLOCKS;
    if (groups_apply<DT, FAM, TM, TN, WM, WN, MF>(args, grid * count, lds_bytes)) return TT_LAUNCH_GROUPS;
    return TT_LAUNCH_RECORD;
}
template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF>
LaunchShape shape_on(int kernel, const ContractArgs &args, int count, int grid, int lds_bytes)
{
    using S = GroupShape<DT, TM, TN, WM, WN, MF>;
    if (kernel == TT_LAUNCH_BLOCKS) return blocks_shape(args, FAM);
    if (kernel == TT_LAUNCH_ROWS) return rows_shape(args, count);
    if (kernel == TT_LAUNCH_GROUPS) return {TT_LAUNCH_GROUPS, grid, S::THREADS, S::LDS};
    return {kernel, grid, (TM / WM) * (TN / WN) * 64, std::max(lds_bytes, epilogue_bytes(TM, TN, WM, WN, MF))};
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF, int AM>
LaunchShape shape_contract(const ContractArgs &args, int count, int grid, int lds_bytes)
{
    return shape_on<DT, FAM, TM, TN, WM, WN, MF>(kernel_contract<DT, FAM, TM, TN, TK, WM, WN, MF, AM>(args, count, grid), args, count, grid, lds_bytes);
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF>
LaunchShape shape_contract_async(const ContractArgs &args, int count, int grid, int lds_bytes)
{
    return shape_on<DT, FAM, TM, TN, WM, WN, MF>(kernel_contract_async<DT, FAM, TM, TN, TK, WM, WN, MF>(args, count, grid, lds_bytes), args, count, grid, lds_bytes);
}

// A launch of one kernel.  The LDS it has been allowed so far is the kernel's own, whatever else the record can come to.
template <auto KERNEL> int launch_tiles(const ContractArgs &args, const PointerSets &sets, int grid, int threads, int lds_bytes, void *stream, const char *where)
{
    static DynamicLdsLimit limit;
    if (const int rc = limit.raise_to(reinterpret_cast<const void *>(KERNEL), lds_bytes); rc != TT_OK) return rc;
    hipLaunchKernelGGL(KERNEL, dim3(grid, sets.count), dim3(threads), lds_bytes, static_cast<hipStream_t>(stream), args, sets);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, where);
}

template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF, int AM>
int launch_contract(const ContractArgs &args, const PointerSets &sets, int grid, int lds_bytes, void *stream)
{
    constexpr int THREADS = (TM / WM) * (TN / WN) * 64;
    const int kernel = kernel_contract<DT, FAM, TM, TN, TK, WM, WN, MF, AM>(args, sets.count, grid);
    if constexpr (FAM == FAM_GEMM_TN || (FAM == FAM_CONV && AM == 16))
        if (kernel == TT_LAUNCH_GROUPS) return launch_groups<DT, FAM, TM, TN, WM, WN, MF>(args, sets, grid, stream);
    if constexpr (FAM == FAM_CONV && AM != 16)
        if (kernel == TT_LAUNCH_ROWS) return launch_conv_rows(args, sets, stream);
    lds_bytes = std::max(lds_bytes, epilogue_bytes(TM, TN, WM, WN, MF));
    if constexpr (taps_built<DT, FAM, TM, TN, TK, WM, WN, AM>())
        if (kernel == TT_LAUNCH_TAPS)
            return launch_tiles<contract_taps_kernel<DT, FAM, TM, TN, TK, WM, WN, MF>>(args, sets, grid, THREADS, lds_bytes, stream, "contract_taps_kernel launch");
    return launch_tiles<contract_kernel<DT, FAM, TM, TN, TK, WM, WN, MF, AM>>(args, sets, grid, THREADS, lds_bytes, stream, "contract_kernel launch");
}

// What the host's resource check multiplies by the number of stages.
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF, int AM> int stage_bytes_contract()
{
    return StageLayout<DT, FAM, TM, TN, TK, MF>::STAGE_BYTES;
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF> int stage_bytes_contract_async()
{
    return RingLayout<DT, TM, TN, TK>::STAGE_BYTES;
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF, int AM> int lds_bytes_contract(int stages)
{
    return stages * StageLayout<DT, FAM, TM, TN, TK, MF>::STAGE_BYTES;
}
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF> int lds_bytes_contract_async(int stages)
{
    return stages * RingLayout<DT, TM, TN, TK>::STAGE_BYTES;
}

template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF>
int launch_contract_async(const ContractArgs &args, const PointerSets &sets, int grid, int lds_bytes, void *stream)
{
    const int kernel = kernel_contract_async<DT, FAM, TM, TN, TK, WM, WN, MF>(args, sets.count, grid, lds_bytes);
    if constexpr (DT == TT_BF16)
        if (kernel == TT_LAUNCH_BLOCKS) return launch_blocks(args, sets, FAM, stream);
    if (kernel == TT_LAUNCH_GROUPS) return launch_groups<DT, FAM, TM, TN, WM, WN, MF>(args, sets, grid, stream);
    return launch_tiles<contract_async_kernel<DT, FAM, TM, TN, TK, WM, WN, MF>>(args, sets, grid, (TM / WM) * (TN / WN) * 64,
                                                                                std::max(lds_bytes, epilogue_bytes(TM, TN, WM, WN, MF)), stream,
                                                                                "contract_async_kernel launch");
}

} // namespace tt
