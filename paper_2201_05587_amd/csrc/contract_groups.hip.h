// Matrix-core contraction with the reduction split INSIDE the workgroup, for launches that leave the chip idle.
//
// A launch of fewer workgroups than the chip has CUs runs one workgroup of 1 to 8 waves per CU.  Such a CU pays
// every latency in full, once per K slice: the slice's arrival, the barrier, the LDS reads, the chain of matrix
// products.  Here KG groups of waves own the SAME output tile: every slice is KG times as deep (or is shared), the
// groups take one part of it each, and their sums meet in LDS at the end.  One barrier then covers KG times the
// matrix work, KG times the bytes are in flight, and four waves per SIMD overlap each other's LDS reads and
// products.  A launch under a record keeps what the record defines (tile, grid, split of the reduction across
// workgroups); only how many waves work on a tile changes.  In a launch of several shapes the list rule names the tile
// (run_list.cpp).
//
// Operands go through the asynchronous ring of contract.hip.h (same loaders, same chunk swizzle).  The epilogue
// is shared by all groups too: each dumps its sums to LDS as a row-major tile, then every thread finishes whole
// 8-column pieces, adding the KG copies.
#pragma once

#include "contract.hip.h"

namespace tt {

// How a tile is run in groups: KG groups, slices of TKI elements; KG = 1 where no split fits the loaders' rules
// (whole 16-byte items per thread, one swizzle for all of a thread's rows) or the LDS.
template <int DT, int TM, int TN, int WM, int WN, int MF> struct GroupShape {
    static constexpr int CH = ElemOf<DT>::CH, ES = 16 / CH, WAVES = (TM / WM) * (TN / WN);
    static constexpr int PAD = MF == 32 ? 8 : 4;
    static constexpr int stage_bytes(int cpr) { return (TM + TN) * cpr * 16; }
    static constexpr int sums_bytes(int kg) { return kg * TM * (TN + PAD) * 4; }
    static constexpr bool fits(int kg, int cpr)
    {
        const int threads = WAVES * kg * 64;
        return threads <= 1024 && (WAVES <= 4 || TM + TN <= 128) && (TM * cpr) % threads == 0 && (TN * cpr) % threads == 0 && (threads / 16) % cpr == 0 &&
               (cpr * CH) % (kg * k_granule(DT, MF)) == 0 && 3 * stage_bytes(cpr) <= kLdsBudget && sums_bytes(kg) <= kLdsBudget;
    }
    // As many groups as fit 16 waves; tiles of 8 waves only up to 64 x 64 (larger ones: a workgroup of 8 waves already
    // overlaps, and the deeper slices leave a ring of three: 0.97 to 1.02 of the plain kernel's speed); 256-byte slices of a row where they can be shared out, else 512- or 128-byte ones
    static constexpr int pick()
    {
        for (int kg = 4; kg >= 2; kg /= 2)
            for (int cpr : {16, 32, 8})
                if (fits(kg, cpr)) return kg * 64 + cpr;
        return 64 + 16;
    }
    static constexpr int KG = pick() / 64, CPR = pick() % 64, TKI = CPR * CH;
    static constexpr int THREADS = WAVES * KG * 64;
    static constexpr int STAGES = 4 * stage_bytes(CPR) <= kLdsBudget ? 4 : 3;
    static constexpr int LDS = STAGES * stage_bytes(CPR) > sums_bytes(KG) ? STAGES * stage_bytes(CPR) : sums_bytes(KG);
};

// Tile `wg` of a contraction, in groups.  LISTED: the arguments are looked up in the launch, and the compiler has to be told that
// addresses in LDS are the same for all lanes; where it knows, saying so costs two instructions a request (7.35 -> 7.40 us for
// 64 channels on 56 x 56, 3x3, single precision).  There the arguments come by value: by reference the same statements were
// scheduled otherwise, twelve instructions longer, and 128 channels on 8 x 28 x 28, 3x3, bf16, took 7.41 us where this took 7.36
// (the same record with a residual, 88 to 104 channels on 5 x 31 x 45: 7.07 and 7.01; both with the divisions that lone
// launches make no longer, see AsyncGather).
template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF, bool LISTED>
__device__ __forceinline__ void contract_groups_tile(std::conditional_t<LISTED, const ContractArgs &, const ContractArgs> g, int32_t wg)
{
    using S = GroupShape<DT, TM, TN, WM, WN, MF>;
    using E = typename ElemOf<DT>::type;
    constexpr int CH = S::CH, ES = S::ES, KG = S::KG, TKI = S::TKI, CPR = S::CPR, THREADS = S::THREADS, NST = S::STAGES;
    constexpr int RB = CPR * 16, A_BYTES = TM * RB, STAGE_BYTES = (TM + TN) * RB;
    constexpr int NWR = TM / WM, NI = WM / MF, NJ = WN / MF, ACC = MF * MF / 64;
    constexpr int LG = 64 / MF, KS = CH * LG;
    constexpr int STEPS = TKI / KS / KG; // matrix-core steps of a group per slice
    constexpr bool CONV = FAM == FAM_CONV;
    using M = Mma<DT, MF>;
    using ARows = AsyncRows<DT, TM, TKI, THREADS>;
    using AGat = AsyncGather<DT, TM, TKI, THREADS>;
    using BRows = AsyncRows<DT, TN, TKI, THREADS>;
    constexpr int LPS = ARows::NL + BRows::NL;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = lds_address(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = wave / S::WAVES, pos = wave % S::WAVES;
    const TileCoord tc = decode_tile(g.map, wg);
    const int k_end = tc.k0 + tc.k_ext; // (whole items only: the gather's walk is the reduction itself)
    const int kt_count = (tc.k_ext + TKI - 1) / TKI;

    const E *a_base = static_cast<const E *>(g.a), *b_base = static_cast<const E *>(g.b);
    if constexpr (!CONV) {
        a_base += (int64_t)tc.hi * g.M * g.K;
        b_base += (int64_t)tc.hi * g.N * g.K;
    }
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(a_base, CONV ? g.a_bytes : (uint32_t)(g.M * g.K * ES));
    const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(b_base, (uint32_t)(g.N * g.K * ES));
    typename ARows::State a_rows;
    typename AGat::State a_gat;
    typename BRows::State b_rows;
    if constexpr (CONV)
        AGat::template init<LISTED>(a_gat, g, tc.m0, tc.k0, tid);
    else
        ARows::init(a_rows, g.K, tc.m0, g.M, tid);
    BRows::init(b_rows, g.K, tc.n0, g.N, tid);
    auto request = [&](int kt, int stage) {
        const int k0 = tc.k0 + kt * TKI;
        uint32_t sa = lds0 + (uint32_t)(stage * STAGE_BYTES);
        if constexpr (LISTED) sa = __builtin_amdgcn_readfirstlane(sa);
        // a slice may reach past the end of this workgroup's split of the reduction: zeros on both sides there
        if constexpr (CONV)
            AGat::issue(a_gat, a_rsrc, sa, g.R, wave, k0 + b_rows.kc < k_end);
        else
            ARows::issue(a_rows, a_rsrc, sa, k0, k_end, wave);
        BRows::issue(b_rows, b_rsrc, sa + A_BYTES, k0, k_end, wave);
    };

    typename M::Acc acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[i][j][v] = 0.0f;
    const int wr = pos % NWR, wc = pos / NWR;
    const int lane_r = lane % MF, lane_g = lane / MF;
    const int swz = chunk_swizzle<CPR>(lane_r);
    const int a_row = (wr * WM + lane_r) * RB, b_row = (wc * WN + lane_r) * RB;

    int requested = 0;
    for (; requested < NST - 1 && requested < kt_count; ++requested) request(requested, requested);

    // The pieces of the output this thread finishes: 8 columns of a row each.  Their bias and residuals are asked for
    // behind the first slices and arrive under the K loop.
    constexpr int CG = TN / 8, PIECES = TM * CG, PPT = (PIECES + THREADS - 1) / THREADS;
    const bool partial = g.map.eff_split_k > 1;
    const bool whole = DT == TT_BF16 ? g.eff_vec_c == 8 : g.eff_vec_c >= 4; // rows are whole 16-byte vectors long
    const int64_t mn = (int64_t)g.M * g.N;
    BiasRegs<DT> bias[PPT];
    u32x4 res[PPT][DT == TT_BF16 ? 1 : 2];
    int64_t at[PPT];
    int first[PPT];
    bool live[PPT];
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        const int e = tid + p * THREADS, row = e / CG;
        first[p] = tc.n0 + (e % CG) * 8;
        live[p] = e < PIECES && tc.m0 + row < g.M && first[p] < g.N;
        at[p] = (int64_t)tc.hi * mn + (int64_t)(tc.m0 + row) * g.N + first[p];
        bias[p] = load_bias_columns<DT>(g, live[p] ? first[p] : g.N);
        if (whole && !partial && g.has_res && live[p]) {
            if constexpr (DT == TT_BF16) {
                res[p][0] = *reinterpret_cast<const u32x4 *>(static_cast<const uint16_t *>(g.res) + at[p]);
            } else {
                res[p][0] = *reinterpret_cast<const u32x4 *>(static_cast<const float *>(g.res) + at[p]);
                if (first[p] + 4 < g.N)
                    res[p][1] = *reinterpret_cast<const u32x4 *>(static_cast<const float *>(g.res) + at[p] + 4);
            }
        }
    }

    int cur = 0, fill = requested == NST - 1 ? NST - 1 : 0; // buffer to compute on / buffer the next request fills
    auto slice = [&](auto requesting) {
        __syncthreads(); // the slice is visible to all waves, and all waves are done with the one before it
        const unsigned char *sa = smem + cur * STAGE_BYTES, *sb = sa + A_BYTES;
        u32x4 rf[STEPS][NI], cf[STEPS][NJ];
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int pos16 = (((group * STEPS + s) * LG + lane_g) ^ swz) * 16;
#pragma unroll
            for (int i = 0; i < NI; ++i) rf[s][i] = *reinterpret_cast<const u32x4 *>(sa + a_row + i * MF * RB + pos16);
#pragma unroll
            for (int j = 0; j < NJ; ++j) cf[s][j] = *reinterpret_cast<const u32x4 *>(sb + b_row + j * MF * RB + pos16);
        }
        __builtin_amdgcn_sched_barrier(0); // the reads go out before the requests' address arithmetic
        if constexpr (decltype(requesting)::value) {
            request(requested, fill);
            ++requested;
            fill = fill + 1 == NST ? 0 : fill + 1;
        }
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) M::run(acc[i][j], rf[s][i], cf[s][j]);
        cur = cur + 1 == NST ? 0 : cur + 1;
    };
    int it = 0;
    for (; requested < kt_count; ++it) {
        wait_loads_outstanding<(NST - 2) * LPS>();
        slice(std::true_type{});
    }
    for (; it < kt_count; ++it) {
        if (kt_count - it - 1 >= 2)
            wait_loads_outstanding<2 * LPS>();
        else if (kt_count - it - 1 == 1)
            wait_loads_outstanding<LPS>();
        else
            wait_loads_outstanding<0>();
        slice(std::false_type{});
    }

    // ---- the groups' sums meet in LDS, as KG row-major tiles ----
    __syncthreads(); // every wave is done reading the operands
    constexpr int SROW = TN + S::PAD;
    float *const sums = reinterpret_cast<float *>(smem);
    float *const mine = sums + (size_t)group * (TM * SROW) + (wr * WM) * SROW + wc * WN + lane_r;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < ACC; ++v) {
                const int row_l = MF == 32 ? (v / 4) * 8 + lane_g * 4 + (v % 4) : lane_g * 4 + v;
                mine[(i * MF + row_l) * SROW + j * MF] = acc[i][j][v];
            }
    __syncthreads();
    float *ws = g.ws + ((int64_t)tc.lo * g.batch) * mn;
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        if (!live[p]) continue;
        const int e = tid + p * THREADS;
        const float *from = sums + (e / CG) * SROW + (e % CG) * 8;
        f32x4 lo = *reinterpret_cast<const f32x4 *>(from), hi = *reinterpret_cast<const f32x4 *>(from + 4);
#pragma unroll
        for (int k = 1; k < KG; ++k) {
            lo += *reinterpret_cast<const f32x4 *>(from + (size_t)k * (TM * SROW));
            hi += *reinterpret_cast<const f32x4 *>(from + (size_t)k * (TM * SROW) + 4);
        }
        if (whole) {
            float biasf[8];
            unpack_bias<DT>(biasf, bias[p]);
            write_row_vector<DT>(g, ws, partial, at[p], first[p], lo, hi, biasf, res[p]);
        } else {
            write_row_in_pieces<DT>(ws, g.out, g.bias, g.res, partial, g.has_bias, g.has_res, g.act, at[p], first[p],
                                    min(8, g.N - first[p]), lo, hi);
        }
    }
}
template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF>
__global__ void __launch_bounds__((GroupShape<DT, TM, TN, WM, WN, MF>::THREADS)) contract_groups_kernel(const ContractArgs args, const PointerSets sets)
{
    contract_groups_tile<DT, FAM, TM, TN, WM, WN, MF, false>(with_set(args, sets, blockIdx.y), (int32_t)blockIdx.x);
}

// Whether a launch is run in groups: whole 16-byte items (what the ring loads), at most one workgroup per CU, and
// a reduction of at least three slices.  With a second workgroup per CU to run, the plain kernel's co-resident
// workgroups do the same and need no exchange of sums (32x32 fp32 tiles at 294 to 448 workgroups: groups take 1.4 times
// as long); below three slices the exchange costs what the shorter loop saves.
// Measured, plain -> groups (us): fp32 32x32 tiles, K = 4608: 32 workgroups 46.1 -> 30.9; K = 2304: 56 workgroups
// 25.2 -> 17.8; K = 1152: 100 workgroups 14.9 -> 11.2; K = 960: 125 workgroups 13.2 -> 9.3; K = 576: 196 workgroups
// 8.9 -> 7.7.  bf16 64x64 tiles: K = 4608: 200 workgroups 23.1 -> 19.7; K = 2048: 16.1 -> 11.8; 64x64 default record
// (register pipeline), K = 1152: 17.4 -> 7.3.
// Larger launches: a record whose ring takes more than half of the LDS (plain_lds; 0: not a ring) runs one workgroup of
// at most four waves per CU whatever its grid, and groups help there too once the reduction has twelve slices.  Plain ->
// groups (us), 64x64 bf16 tiles on 3136 x 1024: K = 384 13.0 -> 14.9, 768 17.9 -> 18.5, 1536 26.9 -> 25.7, 4608
// 67.0 -> 60.2; 64x64 fp32 on 1600 x 800: K = 384 19.4 -> 19.5, 768 32.8 -> 31.8, 4608 169 -> 155; 7x7 3x3 convolutions
// of 512 channels, batch 32, in lists: 21.4 -> 18.8 an entry.
template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF> bool groups_apply(const ContractArgs &a, int grid, int plain_lds)
{
    using S = GroupShape<DT, TM, TN, WM, WN, MF>;
    if constexpr (S::KG == 1) return false;
    const int reduction = a.map.k_iters * a.map.tile_k;
    const bool alone = grid <= compute_units() || (S::WAVES <= 4 && 2 * plain_lds > kLdsBudget && reduction >= 12 * S::TKI);
    return alone && reduction >= 3 * S::TKI && a.eff_vec_a * S::ES == 16 && a.eff_vec_b * S::ES == 16 &&
           (FAM == FAM_CONV || ((int64_t)a.M * a.K * S::ES < (1ll << 31) && (int64_t)a.N * a.K * S::ES < (1ll << 31)));
}

template <int DT, int FAM, int TM, int TN, int WM, int WN, int MF> int launch_groups(const ContractArgs &args, const PointerSets &sets, int grid, void *stream)
{
    using S = GroupShape<DT, TM, TN, WM, WN, MF>;
    if constexpr (S::KG > 1) {
        auto kern = contract_groups_kernel<DT, FAM, TM, TN, WM, WN, MF>;
        static DynamicLdsLimit limit; // per kernel instance
        if (const int rc = limit.raise_to(reinterpret_cast<const void *>(kern), S::LDS); rc != TT_OK) return rc;
        hipLaunchKernelGGL(kern, dim3(grid, sets.count), dim3(S::THREADS), S::LDS, static_cast<hipStream_t>(stream), args, sets);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? TT_OK : note_hip_error((int)e, "contract_groups_kernel launch");
    }
    return TT_ERR_UNSUPPORTED;
}

} // namespace tt
