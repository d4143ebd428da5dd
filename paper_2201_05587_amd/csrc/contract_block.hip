// Launch of the 256 x 256 block kernel.
#include <hip/hip_runtime.h>

#include "contract_block.hip.h"

namespace tt {

// Whether a launch of `count` pointer sets is run in blocks instead of the tiles its record names: whole 16-byte items
// and rows, no split of the reduction, K of at least 1024, and enough outputs that blocks keep the chip busy.  `share`
// is the part of the blocks' rounds over all CUs that holds outputs of the matrix: larger tiles waste more of the last
// round, and need less of the bandwidth into a CU, so a record of small tiles gives way earlier.  Measured on M x N
// between 512 x 256 and 8192 x 4096, K = 1024 and 3072, blocks against the best ring record of a tile (us):
//   share 0.50 (4096 x 2048 x 1024)  64x64 27.1, 128x64 28.3, 128x128 22.2, 128x256 18.5   blocks 26.5
//   share 0.56 (3072 x 3072 x 1024)  64x64 29.4, 128x64 34.6, 128x128 31.6, 128x256 32.2   blocks 26.5
//   share 1.00 (4096 x 4096 x 1024)  64x64 48.3, 128x64 54.6, 128x128 49.4, 128x256 34.8   blocks 35.9
//   share 0.75, two rounds (8192 x 3072 x 3072)  the best record of all 135.3              blocks 140.9
// and 4096 x 4096 x 4096: 128x64 166, blocks 105 (1.31 PFLOP/s; operands of zeros: 78, the chip's power sets the
// clock).  Register-pipeline records keep their own kernel; the default schedule comes here as a ring record (launch_plan_of).
bool block_applies(const ContractArgs &a, int family, int count, int tile_outputs)
{
    if (a.dtype != TT_BF16 || a.batch != 1 || a.map.eff_split_k != 1 || a.K < 1024) return false;
    if (a.eff_vec_a != 8 || a.eff_vec_b != 8 || a.eff_vec_c != 8) return false;
    if (family == FAM_GEMM_TN && ((int64_t)a.M * a.K >= (1ll << 30) || (int64_t)a.N * a.K >= (1ll << 30))) return false;
    const int64_t blocks = (int64_t)((a.M + 255) / 256) * ((a.N + 255) / 256) * count;
    const int64_t cus = compute_units(), rounds = (blocks + cus - 1) / cus;
    const double share = (double)a.M * a.N * count / (65536.0 * (double)(cus * rounds));
    if (tile_outputs <= 64 * 128) return share >= 0.5;
    if (tile_outputs <= 128 * 128) return share >= 0.55;
    return share >= (rounds == 1 ? 0.55 : 0.95);
}

namespace {

template <int FAM> int launch(const ContractArgs &args, const PointerSets &sets, void *stream)
{
    auto kern = contract_block_kernel<FAM>;
    using S = BlockShape<FAM>;
    static DynamicLdsLimit limit;
    if (const int rc = limit.raise_to(reinterpret_cast<const void *>(kern), S::LDS); rc != TT_OK) return rc;
    const int bm = (args.M + S::BM - 1) / S::BM, bn = (args.N + S::BN - 1) / S::BN;
    hipLaunchKernelGGL(kern, dim3(bm * bn, sets.count), dim3(S::THREADS), S::LDS, static_cast<hipStream_t>(stream), args, bm, bn, sets);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, "contract_block_kernel launch");
}

} // namespace

namespace {
template <int FAM> LaunchShape shape_of(const ContractArgs &a)
{
    using S = BlockShape<FAM>;
    return {TT_LAUNCH_BLOCKS, ((a.M + S::BM - 1) / S::BM) * ((a.N + S::BN - 1) / S::BN), S::THREADS, S::LDS};
}
} // namespace

LaunchShape blocks_shape(const ContractArgs &args, int family)
{
    return family == FAM_CONV ? shape_of<FAM_CONV>(args) : shape_of<FAM_GEMM_TN>(args);
}

int launch_blocks(const ContractArgs &args, const PointerSets &sets, int family, void *stream)
{
    return family == FAM_CONV ? launch<FAM_CONV>(args, sets, stream) : launch<FAM_GEMM_TN>(args, sets, stream);
}

} // namespace tt
