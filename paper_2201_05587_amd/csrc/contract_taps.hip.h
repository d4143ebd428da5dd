// Matrix-core contraction over rows that are no whole 16-byte items: convolutions whose pixels, and products whose rows of the
// reduction, begin at any element.
//
// The reduction is walked tap by tap (filter row, filter column; a plain product is one tap), each tap's C elements padded up
// to whole 16-byte items.  An item then lies inside one pixel: it is real or padding as a whole, the elements behind a pixel's
// last one are the same for all rows of a slice, and one mask a slice silences them.  A walk along a filter row's run of S * C
// elements (GatherLoader) has items that cross pixels, so each needs bounds, an alignment shift and a mask of its own, some 25
// instructions an item, and registers that leave room for one slice in flight; here an item costs 10, and two are.  The padding
// multiplies the reduction by ceil(C / items) * items / C, which taps_apply bounds.
#pragma once

#include "contract.hip.h"

namespace tt {

// Where a thread is in the walk: it fetches the same chunk of every slice, of all its rows.
template <int DT, int TK> struct TapWalk {
    static constexpr int CH = ElemOf<DT>::CH;
    int32_t r, s, c;
    __device__ __forceinline__ void begin(int k, int padded, int S)
    {
        const int tap = k / padded;
        c = k - tap * padded;
        r = tap / S, s = tap - r * S;
    }
    __device__ __forceinline__ void next(int padded, int S) // TK elements on
    {
        c += TK;
        while (c >= padded) {
            c -= padded;
            if (++s == S) s = 0, ++r;
        }
    }
};

// Rows of an operand: pixels of the activations (CONV), or rows one after the other.  A slice in flight is a Slice, of which
// there may be several.
template <int DT, int ROWS, int TK, int THREADS, bool CONV> struct TapRows {
    using E = typename ElemOf<DT>::type;
    static constexpr int CH = ElemOf<DT>::CH, ES = (int)sizeof(E), CPR = TK / CH, TOTAL = ROWS * CPR;
    static constexpr int NL = (TOTAL + THREADS - 1) / THREADS, STEP = THREADS / CPR;
    static constexpr int ROWB = (TK + CH) * ES;
    static_assert(THREADS % CPR == 0 && NL <= 32, "");
    struct Rows {
        int32_t origin[NL];             // element at which the row's first tap begins (of a convolution: may be negative)
        int32_t h[CONV ? NL : 1], w[CONV ? NL : 1]; // input row and column of the first tap
        int32_t last;                   // last element at which an item can be read
    };
    struct Slice {
        u32x4 raw[NL];
        int32_t at, keep; // element of the walk's position from a row's origin; elements of the item that are real
        uint32_t real;    // bit i: row i's item is inside the image
    };

    static __device__ __forceinline__ void init(Rows &rows, const ContractArgs &g, int row0, int rows_total, int row_elements, int numel, int tid)
    {
        rows.last = numel - CH;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int m = min(row0 + tid / CPR + i * STEP, rows_total - 1); // (rows past the matrix: what they add up to is not stored)
            if constexpr (CONV) {
                const uint32_t img = fast_div((uint32_t)m, g.div_hw), rem = (uint32_t)m - img * (uint32_t)(g.Ho * g.Wo);
                const uint32_t p = fast_div(rem, g.div_wo), q = rem - p * (uint32_t)g.Wo;
                rows.h[i] = (int)p * g.stride_h - g.pad_h, rows.w[i] = (int)q * g.stride_w - g.pad_w;
                rows.origin[i] = (((int)img * g.H + rows.h[i]) * g.W + rows.w[i]) * g.C;
            } else {
                rows.origin[i] = m * row_elements;
            }
        }
    }
    // `pitch`: elements from one filter row to the next
    static __device__ __forceinline__ void load(Slice &sl, const Rows &rows, const ContractArgs &g, const E *base, const TapWalk<DT, TK> &walk, int taps_h,
                                                int pitch, int C)
    {
        const bool live = walk.r < taps_h;
        sl.at = walk.r * pitch + walk.s * C + walk.c;
        sl.keep = live ? C - walk.c : 0;
        sl.real = 0;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            bool ok = live;
            if constexpr (CONV) ok = live & ((uint32_t)(rows.h[i] + walk.r) < (uint32_t)g.H) & ((uint32_t)(rows.w[i] + walk.s) < (uint32_t)g.W);
            if constexpr (CONV) sl.real |= (ok ? 1u : 0u) << i;
            const int from = min(ok ? rows.origin[i] + sl.at : 0, rows.last);
            load16(sl.raw[i], reinterpret_cast<const unsigned char *>(base) + (uint32_t)from * (uint32_t)ES);
        }
    }
    static __device__ __forceinline__ void store(const Slice &sl, const Rows &rows, unsigned char *lds, int tid)
    {
        const int chunk = tid % CPR, first = tid / CPR;
        const u32x4 mask = keep_first<DT>(u32x4{~0u, ~0u, ~0u, ~0u}, sl.keep);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int row = first + i * STEP;
            if (TOTAL % THREADS != 0 && row >= ROWS) continue;
            u32x4 v = sl.raw[i];
            const bool ok = CONV ? ((sl.real >> i) & 1u) != 0 : true;
            // the tensor's last item was read further back, so that the read ends where the tensor does
            const int back = rows.origin[i] + sl.at - rows.last;
            if (__builtin_expect(back > 0 && ok && sl.keep > 0, 0)) v = shift_elems<DT>(v, -min(back, CH - 1));
#pragma unroll
            for (int h = 0; h < 4; ++h) v[h] = ok ? v[h] & mask[h] : 0u;
            *reinterpret_cast<u32x4 *>(lds + row * ROWB + chunk * 16) = v;
        }
    }
};

// Bound by latency where a launch has few workgroups, by the loaders' instructions where it has many: two slices in flight in
// registers, a third in LDS.
template <int DT, int FAM, int TM, int TN, int TK, int WM, int WN, int MF>
__global__ void __launch_bounds__((TM / WM) * (TN / WN) * 64) contract_taps_kernel(const ContractArgs args, const PointerSets sets)
{
    const ContractArgs g = with_set(args, sets, blockIdx.y);
    using E = typename ElemOf<DT>::type;
    using L = StageLayout<DT, FAM_GEMM_TN, TM, TN, TK, MF>;
    constexpr int CH = ElemOf<DT>::CH, ES = (int)sizeof(E);
    constexpr int THREADS = (TM / WM) * (TN / WN) * 64;
    constexpr int ROWB = L::ROWB, A_BYTES = L::A_BYTES, STAGE_BYTES = L::STAGE_BYTES;
    constexpr int NWR = TM / WM, NI = WM / MF, NJ = WN / MF;
    constexpr int LG = 64 / MF, KS = k_granule(DT, MF), NKS = TK / KS, ACC = MF * MF / 64;
    constexpr bool CONV = FAM == FAM_CONV;
    using M = Mma<DT, MF>;
    using ARows = TapRows<DT, TM, TK, THREADS, CONV>;
    using BRows = TapRows<DT, TN, TK, THREADS, false>;

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TileCoord tc = decode_tile(g.map, (int32_t)blockIdx.x);
    const BiasRegs<DT> bias = load_bias_early<DT, TM, WM, WN, MF>(g, tc, wave, lane);
    const int C = CONV ? g.C : g.K, R = CONV ? g.R : 1, S = CONV ? g.S : 1, padded = (C + CH - 1) / CH * CH;
    // Splits share the walk, padding and all, slice by slice: its padding would else be the last one's (34 channels, 5x5, in nine:
    // eight of 3 slices and one of 8, here of 4 and 3).  There are as many slices as the record's reduction has, or more.
    const int slices = (R * S * padded + TK - 1) / TK, share = (int)fast_div((uint32_t)slices, g.map.div_split), longer = slices - share * g.map.eff_split_k;
    const int kt_count = share + (tc.lo < longer ? 1 : 0), first = share * tc.lo + min(tc.lo, longer);
    const E *a_base = static_cast<const E *>(g.a), *b_base = static_cast<const E *>(g.b);
    if constexpr (!CONV) {
        a_base += (int64_t)tc.hi * g.M * g.K;
        b_base += (int64_t)tc.hi * g.N * g.K;
    }
    TapWalk<DT, TK> walk;
    walk.begin(first * TK + tid % (TK / CH) * CH, padded, S);
    typename ARows::Rows a_rows;
    typename BRows::Rows b_rows;
    ARows::init(a_rows, g, tc.m0, g.M, g.K, CONV ? (int)(g.a_bytes / (uint32_t)ES) : g.M * g.K, tid);
    BRows::init(b_rows, g, tc.n0, g.N, g.K, g.N * g.K, tid);

    struct Slices {
        typename ARows::Slice a;
        typename BRows::Slice b;
    };
    auto fetch = [&](Slices &f) { // slices are fetched in order
        ARows::load(f.a, a_rows, g, a_base, walk, R, CONV ? g.W * g.C : 0, C);
        BRows::load(f.b, b_rows, g, b_base, walk, R, S * C, C);
        walk.next(padded, S);
    };
    auto stash = [&](const Slices &f, int stage) {
        ARows::store(f.a, a_rows, smem + stage * STAGE_BYTES, tid);
        BRows::store(f.b, b_rows, smem + stage * STAGE_BYTES + A_BYTES, tid);
    };

    typename M::Acc acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[i][j][v] = 0.0f;
    const int wr = wave % NWR, wc = wave / NWR;
    const int lane_r = lane % MF, lane_g = lane / MF;
    const int r_off = (wr * WM + lane_r) * ROWB + lane_g * 16, c_off = (wc * WN + lane_r) * ROWB + lane_g * 16;
    constexpr int GROUP = steps_per_group(NI + NJ, NKS, THREADS > 512 ? 16 : 48);
    auto multiply = [&](int stage) {
        const unsigned char *sr = smem + stage * STAGE_BYTES + r_off, *sc = smem + stage * STAGE_BYTES + A_BYTES + c_off;
#pragma unroll
        for (int ks0 = 0; ks0 < NKS; ks0 += GROUP) {
            u32x4 rf[GROUP][NI], cf[GROUP][NJ];
#pragma unroll
            for (int s = 0; s < GROUP; ++s) {
#pragma unroll
                for (int i = 0; i < NI; ++i) rf[s][i] = *reinterpret_cast<const u32x4 *>(sr + i * MF * ROWB + (ks0 + s) * KS * ES);
#pragma unroll
                for (int j = 0; j < NJ; ++j) cf[s][j] = *reinterpret_cast<const u32x4 *>(sc + j * MF * ROWB + (ks0 + s) * KS * ES);
            }
            __builtin_amdgcn_sched_barrier(0); // keep the reads ahead of the products
#pragma unroll
            for (int s = 0; s < GROUP; ++s)
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) M::run(acc[i][j], rf[s][i], cf[s][j]);
        }
    };

    // Slices of even and of odd number in flight.  In the loop a step requests one and puts one into LDS without a condition: behind
    // one the compiler moves a slice in flight to other registers, which waits for it.
    Slices even, odd;
    fetch(even);
    fetch(odd); // (of a single slice: zeros, from the tensors' first bytes)
    ResRegs<DT, TM, WM, WN, MF, (THREADS <= 512)> res_early;
    load_res_early(res_early, g, tc, wave, lane);
    stash(even, 0);
    __syncthreads();
    const bool two_stage = g.stages == 2;
    int cur = 0, it = 0;
    const auto publish = [&](const Slices &next) {
        if (!two_stage) __syncthreads();
        if (two_stage) cur ^= 1;
        stash(next, cur);
        __syncthreads();
    };
    for (; it + 3 < kt_count; it += 2) {
        fetch(even);
        multiply(cur);
        publish(odd);
        fetch(odd);
        multiply(cur);
        publish(even);
    }
    // one to three slices are left, `it` of them in LDS and the next in flight
    if (it + 2 < kt_count) fetch(even);
    multiply(cur);
    if (it + 1 < kt_count) {
        publish(odd);
        multiply(cur);
    }
    if (it + 2 < kt_count) {
        publish(even);
        multiply(cur);
    }
    write_tile<DT, TM, WM, WN, MF>(acc, g, tc, smem, wave, lane, bias, res_early);
}

// Whether a launch of the register pipeline walks tap by tap: operands that are no whole items, pixels longer than one (so the
// tensors are), and little padding: up to a seventh in fp32, less than a fifth in bf16, and an eighth where bf16 pixels are odd
// and begin inside words (the other walk fetches whole words and shifts).  20 x 83x83 under the default, run -> taps (us), 3x3
// to 16 channels: bf16 20 channels 13.9 -> 13.4, 21 13.7 -> 15.8, 23 15.2 -> 15.7, 31 18.1 -> 16.3; fp32 7 13.4 -> 12.5, 17 21.8 ->
// 22.6, 19 24.8 -> 22.9.  Others, under the record a search chose: bf16 334 -> 176 channels on 3 x 107x107 160 -> 102, 721 -> 236 on
// 18 x 32x32 222 -> 162, 98 -> 16 on 3 x 10x8 stride 2 21.5 -> 14.8; fp32 842 -> 16 on 10 x 42x55 434 -> 303, 650 -> 384, 5x5, on 2 x
// 19x15 141 -> 113; products of 26 x 1792 x 220 5.4 -> 4.9, 51 x 3040 x 1722 11.4 -> 10.8.
// one_item: fp32 tiles of four 16 x 16 waves over slices of 16 elements, one item a lane and four products a wave and slice.  There
// the second slice in flight costs the eighth wave of a SIMD, which tells from three workgroups a CU on, unless the reduction is short.
// Run -> taps (us): 3x3 over 478 channels, 740 workgroups 209 -> 192; over 445, 798 222 -> 241; over 213, 1362 151 -> 178; over 35,
// 1411 33.0 -> 27.7; products over 107, 4140 workgroups 23.0 -> 22.3; over 151, 12369 78 -> 96.
template <int DT, int FAM> bool taps_apply(const ContractArgs &g, int64_t workgroups, bool one_item)
{
    if (one_item && workgroups >= 768 && std::min<int64_t>((int64_t)g.map.k_iters * g.map.tile_k, g.K) >= (FAM == FAM_CONV ? 512 : 128)) return false;
    constexpr int CH = ElemOf<DT>::CH, ES = 16 / CH;
    const int64_t C = FAM == FAM_CONV ? g.C : g.K, padded = (C + CH - 1) / CH * CH;
    if (FAM != FAM_CONV && ((int64_t)g.M * g.K * ES >= (1ll << 31) || (int64_t)g.N * g.K * ES >= (1ll << 31))) return false;
    if (C % CH == 0 || C <= CH) return false;
    return DT == TT_F32 ? 7 * padded <= 8 * C : C % 2 == 0 ? 5 * padded < 6 * C : 8 * padded <= 9 * C;
}

} // namespace tt
