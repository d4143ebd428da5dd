// Matrix-core contraction in 256 x 256 blocks (bf16), for launches with enough outputs to give every CU one.
//
// A tile kernel brings (TM + TN) rows into a CU's LDS for TM * TN outputs, and a CU takes in some 80 GB/s: 128 x 128
// tiles stop at about 1 PFLOP/s on the whole chip.  A block of 256 x 256 needs half the bytes per product.  Eight waves
// in two teams of four (one wave of each team per SIMD) take turns: while one team multiplies, the other reads its next
// fragments from the LDS and requests global data, and a barrier swaps them, so the matrix cores are fed from one
// team or the other all the time.
//
// The LDS holds two K slices of 64.  Each is four regions: rows 0-127 and 128-255 of the A block, the same of the B
// block.  A wave owns 64 rows of either A region and 32 rows of either B region, i.e. four quadrants of 64 x 32 outputs,
// and a slice is four phases, one quadrant each:
//
//   phase      0            1            2            3
//   multiply   A0 . B0      A0 . B1      A1 . B1      A1 . B0
//   read       A0           B1           A1           B0 of the next slice
//   request    B1 (t + 1)   A1 (t + 1)   A0 (t + 2)   B0 (t + 2)          (slice t, buffer t mod 2)
//
// A region is requested again two phases after it was read (the other team reads one phase later), and is read five or
// six phases after it was requested.  Every phase requests one region, two loads per thread, past the end too
// (zeros nobody multiplies), so all waits are the same constant.
#pragma once

#include "contract.hip.h"

namespace tt {

// Loaders of the 256 rows of a block's operand, one region of 128 rows at a time.  The accumulators and fragments of the
// kernel leave few registers, so their state is smaller than that of the ring's loaders in contract.hip.h.
//
// Rows of a K-contiguous matrix: a thread's rows lie 64 apart, and rows past the matrix are past the end of the buffer
// (the bounds check returns zeros for them), so one offset per thread is enough.
template <int TK, int THREADS> struct BlockRows {
    static constexpr int CPR = TK / 8, STEP = THREADS / CPR, NL = 128 / STEP;
    struct State {
        uint32_t base; // byte offset of this thread's chunk of its first row
        int32_t kc;    // element offset of the chunk inside a slice
    };
    static __device__ __forceinline__ void init(State &st, int K, int row0, int tid)
    {
        const int first = tid / CPR, pos = tid % CPR;
        st.kc = (pos ^ chunk_swizzle<CPR>(first)) * 8;
        st.base = (uint32_t)((row0 + first) * K + st.kc) * 2u;
    }
    static __device__ __forceinline__ void issue(const State &st, __amdgpu_buffer_rsrc_t rsrc, uint32_t lds_region, int region,
                                                 int k0, int K, int wave)
    {
        const bool k_ok = k0 + st.kc < K;
#pragma unroll
        for (int i = 0; i < NL; ++i)
            load16_to_lds(rsrc, k_ok ? st.base + (uint32_t)(((region * 128 + i * STEP) * K + k0) * 2) : kOutOfRange,
                          lds_region + (uint32_t)((i * THREADS + wave * 64) * 16));
    }
};

// The gather of a convolution's activation rows (see AsyncGather).  What it knows of a row stays in an LDS table, 16 bytes a
// row, and is read again for every slice; a thread keeps its position in the reduction only.  Region 0 of a slice is
// requested before region 1 of it, and steps to the slice.
template <int TK, int THREADS> struct BlockGather {
    static constexpr int CPR = TK / 8, STEP = THREADS / CPR, NL = 128 / STEP, TABLE_BYTES = 256 * 16;
    struct State {
        int32_t r, j;
    };
    static __device__ __forceinline__ void init(State &st, const ContractArgs &g, int row0, unsigned char *table, int tid)
    {
        using G = AsyncGather<TT_BF16, 256, CPR * 8, 256 * CPR>; // one row per thread, whatever its chunk
        typename G::State f;
        if (tid < 256) {
            G::init_row(f, 0, g, row0 + tid);
            *reinterpret_cast<u32x4 *>(table + tid * 16) =
                u32x4{(uint32_t)f.origin[0], f.rmask[0], (uint32_t)f.jlo[0], (uint32_t)f.jhi[0]};
        }
        const int kk = (tid % CPR ^ chunk_swizzle<CPR>(tid / CPR)) * 8;
        st.r = kk / g.runp;
        st.j = kk - st.r * g.runp;
    }
    static __device__ __forceinline__ void issue(State &st, const ContractArgs &g, const unsigned char *table,
                                                 __amdgpu_buffer_rsrc_t rsrc, uint32_t lds_region, int region, bool first_slice, int tid)
    {
        u32x4 row[NL]; // origin, filter rows inside the image, first valid position of the run, one past the last
#pragma unroll
        for (int i = 0; i < NL; ++i)
            row[i] = *reinterpret_cast<const u32x4 *>(table + (region * 128 + i * STEP + tid / CPR) * 16);
        if (region == 0 && !first_slice) {
            const int dr = TK / g.runp;
            st.j += TK - dr * g.runp;
            st.r += dr;
            if (st.j >= g.runp) {
                st.j -= g.runp;
                st.r += 1;
            }
        }
        const int kterm = st.r * (g.W * g.C) + st.j;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const bool ok = (st.r < g.R) & (((row[i][1] >> (st.r & 31)) & 1u) != 0) & (st.j >= (int)row[i][2]) & (st.j < (int)row[i][3]);
            load16_to_lds(rsrc, ok ? (uint32_t)((int)row[i][0] + kterm) * 2u : kOutOfRange,
                          lds_region + (uint32_t)((i * THREADS + wave * 64) * 16));
        }
    }
};

template <int FAM> struct BlockShape {
    static constexpr int BM = 256, BN = 256, TK = 64, THREADS = 512, MF = 32;
    static constexpr int ROW_BYTES = TK * 2, REGION_BYTES = 128 * ROW_BYTES, SLICE_BYTES = 4 * REGION_BYTES;
    static constexpr int LDS = 2 * SLICE_BYTES + (FAM == FAM_CONV ? BlockGather<TK, THREADS>::TABLE_BYTES : 0);
    static constexpr int BAND = 4; // block rows walked together (see block_of)
};

// Block `wg` of blocks_m x blocks_n.
template <int FAM> __device__ __forceinline__ void contract_block(const ContractArgs &g, int blocks_m, int blocks_n, int wg)
{
    using S = BlockShape<FAM>;
    constexpr int DT = TT_BF16, MF = S::MF, TK = S::TK, CPR = TK / 8, THREADS = S::THREADS;
    constexpr bool CONV = FAM == FAM_CONV;
    using M = Mma<DT, MF>;
    using Rows = BlockRows<TK, THREADS>;
    using Gather = BlockGather<TK, THREADS>;
    constexpr int NL = Rows::NL; // loads per thread and region

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t lds0 = lds_address(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = wave >> 2;        // waves 0-3 and 4-7: a SIMD has one of either
    const int wm = team, wn = wave & 3; // 64-row and 32-column strip of every region

    // Block of this workgroup: every XCD gets a contiguous run, walked in bands of four block rows, so that the 32
    // blocks an XCD works on at a time form a rectangle (its L2 serves each operand row to 4 or 8 of them).
    TileCoord tc;
    {
        const int total = blocks_m * blocks_n;
        const int per = total / kXcds, rem = total % kXcds, x = wg % kXcds;
        const int L = x * per + min(x, rem) + wg / kXcds;
        const int band = L / (S::BAND * blocks_n), at = L - band * S::BAND * blocks_n;
        const int high = min(S::BAND, blocks_m - band * S::BAND);
        const int im = band * S::BAND + at % high, in = at / high;
        tc.hi = tc.lo = 0;
        tc.m0 = im * S::BM, tc.m_ext = min(S::BM, g.M - tc.m0);
        tc.n0 = in * S::BN, tc.n_ext = min(S::BN, g.N - tc.n0);
        tc.k0 = 0, tc.k_ext = g.K;
    }
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.a, CONV ? g.a_bytes : (uint32_t)(g.M * g.K * 2));
    const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(g.b, (uint32_t)(g.N * g.K * 2));
    typename Rows::State a_rows, b_rows;
    typename Gather::State a_gat;
    unsigned char *const table = smem + 2 * S::SLICE_BYTES;
    if constexpr (CONV) {
        Gather::init(a_gat, g, tc.m0, table, tid);
        __syncthreads();
    } else
        Rows::init(a_rows, g.K, tc.m0, tid);
    Rows::init(b_rows, g.K, tc.n0, tid);
    // regions of a slice buffer: A0, A1, B0, B1
    auto request_a = [&](int h, int t) {
        const uint32_t to = lds0 + (uint32_t)((t & 1) * S::SLICE_BYTES + h * S::REGION_BYTES);
        if constexpr (CONV)
            Gather::issue(a_gat, g, table, a_rsrc, to, h, t == 0, tid);
        else
            Rows::issue(a_rows, a_rsrc, to, h, t * TK, g.K, wave);
    };
    auto request_b = [&](int h, int t) {
        Rows::issue(b_rows, b_rsrc, lds0 + (uint32_t)((t & 1) * S::SLICE_BYTES + (2 + h) * S::REGION_BYTES), h, t * TK, g.K, wave);
    };

    typename M::Acc acc[2][2][2][1]; // [A region][B region][32-row block][.]
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[h][k][i][0][v] = 0.0f;

    const int lane_r = lane % MF, lane_g = lane / MF;
    const int swz = chunk_swizzle<CPR>(lane_r);
    const int a_row = (wm * 64 + lane_r) * S::ROW_BYTES, b_row = (wn * 32 + lane_r) * S::ROW_BYTES;
    constexpr int STEPS = TK / 16;
    u32x4 af[2][STEPS], bf[2][STEPS]; // A region in use; B0 and B1 (B0 of the next slice takes the place of B1)
    auto read_a = [&](int h, int t) {
        const unsigned char *from = smem + (t & 1) * S::SLICE_BYTES + h * S::REGION_BYTES + a_row;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                af[i][s] = *reinterpret_cast<const u32x4 *>(from + i * MF * S::ROW_BYTES + ((s * 2 + lane_g) ^ swz) * 16);
    };
    auto read_b = [&](u32x4 (&to)[STEPS], int h, int t) {
        const unsigned char *from = smem + (t & 1) * S::SLICE_BYTES + (2 + h) * S::REGION_BYTES + b_row;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) to[s] = *reinterpret_cast<const u32x4 *>(from + ((s * 2 + lane_g) ^ swz) * 16);
    };
    auto swap_teams = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    };
    auto multiply = [&](typename M::Acc (&c)[2][1], const u32x4 (&b)[STEPS]) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int i = 0; i < 2; ++i) M::run(c[i][0], af[i][s], b[s]);
        __builtin_amdgcn_s_setprio(0);
    };

    const int slices = (g.K + TK - 1) / TK;
    // slices 0 and 1, in the order the loop would have requested them: all but the last two regions of slice 1
    request_a(0, 0), request_b(0, 0), request_b(1, 0), request_a(1, 0);
    request_a(0, 1), request_b(0, 1);
    wait_loads_outstanding<4 * NL>(); // A0 and B0 of slice 0
    __syncthreads();
    read_b(bf[0], 0, 0);
    if (team == 1) swap_teams(); // team 1 runs one turn behind

    auto slice = [&](int t, u32x4 (&b0)[STEPS], u32x4 (&b1)[STEPS]) {
        // phase 0
        read_a(0, t);
        request_b(1, t + 1);
        wait_loads_outstanding<4 * NL>(); // B1 of this slice has landed (the other team reads it a turn later)
        swap_teams();
        multiply(acc[0][0], b0);
        swap_teams();
        // phase 1
        read_b(b1, 1, t);
        request_a(1, t + 1);
        wait_loads_outstanding<4 * NL>(); // A1 of this slice
        swap_teams();
        multiply(acc[0][1], b1);
        swap_teams();
        // phase 2
        read_a(1, t);
        request_a(0, t + 2);
        wait_loads_outstanding<3 * NL>(); // A0 and B0 of the next slice
        swap_teams();
        multiply(acc[1][1], b1);
        swap_teams();
        // phase 3
        read_b(b1, 0, t + 1);
        request_b(0, t + 2);
        swap_teams();
        multiply(acc[1][0], b0);
        swap_teams();
    };
    for (int t = 0; t < slices; t += 2) {
        slice(t, bf[0], bf[1]);
        if (t + 1 < slices) slice(t + 1, bf[1], bf[0]);
    }
    if (team == 0) swap_teams(); // team 1 is one turn behind
    wait_loads_outstanding<0>();  // the requests past the end: nothing may still write LDS below

    using T = TileOut<128, 64, 32, MF>;
    const int epi_wave = wm + 2 * wn;
    ResRegs<DT, 128, 64, 32, MF, false> no_res;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const BiasRegs<DT> bias = load_bias_columns<DT>(g, tc.n0 + k * 128 + T::col(epi_wave, lane));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            TileCoord q;
            // nothing to write outside the matrix, and no valid address there (the first quadrant is always inside: its
            // barrier separates the operands from the staging of all four)
            if (!block_quadrant(tc, g.M, g.N, h, k, &q)) continue;
            write_tile<DT, 128, 64, 32, MF, typename M::Acc, false, false, false>(acc[h][k], g, q, smem, epi_wave, lane, bias, no_res);
        }
    }
}
template <int FAM>
__global__ void __launch_bounds__(512) contract_block_kernel(const ContractArgs args, int blocks_m, int blocks_n, const PointerSets sets)
{
    contract_block<FAM>(with_set(args, sets, blockIdx.y), blocks_m, blocks_n, (int)blockIdx.x);
}

} // namespace tt
