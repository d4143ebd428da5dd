// Single-precision contractions with a short reduction and many rows (the expanding pointwise layers of a mobile network):
// several entries in one launch.
//
// Such a layer is a stream: 16 to 96 elements in, more out per row, and little to multiply.  A tile kernel spends its
// life on set-up, a round trip of the outputs through LDS and one memory latency per 2 KB of output (2.2 TB/s).  Here a
// workgroup keeps its columns' weights in LDS as matrix-core fragments, and every wave walks down blocks of 16 rows: the
// rows come straight into registers as fragments, those of the next block while this one is multiplied, and with the
// weights as the matrix cores' row operand a lane ends up with four consecutive columns of one row.  Written like that, 64
// bytes a row and store, the stream stays at 3.2 TB/s: memory takes whole lines of 128 (see the exchange below: 4.5 TB/s).
// Tiles of the list rule -> this (us): two entries of 200704 x 96 x 16 56 -> 43, four of 50176 x 144 x 24 57 -> 39 (which
// contractions come here, and what the others lose: thin_pieces in run_list.cpp); a MobileNetV2 pass at batch 16, whose
// reductions of up to 192 all came here before, 250 -> 243.
#pragma once

#include "contract.hip.h"

namespace tt {

// KB: 16-element pieces of the reduction that the instance holds.
template <int KB> __global__ void __launch_bounds__(256) contract_thin_list_kernel(const ThinList list)
{
    using M = Mma<TT_F32, 16>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int at = 0;
#pragma unroll
    for (int i = 1; i < kMaxThin; ++i) at += (int)blockIdx.x >= list.first[i];
    const ThinEntry &g = list.e[at];
    const int wg = (int)blockIdx.x - list.first[at], slab = wg / g.chunks, chunk = wg - slab * g.chunks;
    const int tid = threadIdx.x, lane = tid & 63, lane_r = lane & 15, lane_g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = chunk * g.columns, blocks = (min(g.columns, g.N - n0) + 15) / 16, pieces = (g.K + 15) / 16;

    // weights: fragment (block j, piece s) at j * pieces + s, one item per lane; behind them the bias
    u32x4 *const weights = reinterpret_cast<u32x4 *>(smem);
    float *const bias = reinterpret_cast<float *>(weights + blocks * pieces * 64);
    for (int j = wave; j < blocks; j += 4) {
        const int n = n0 + j * 16 + lane_r;
        u32x4 item[KB];
#pragma unroll
        for (int s = 0; s < KB; ++s) {
            const int k = s * 16 + lane_g * 4;
            item[s] = u32x4{0u, 0u, 0u, 0u};
            if (n < g.N && k < g.K) item[s] = *reinterpret_cast<const u32x4 *>(g.b + (int64_t)n * g.K + k);
        }
#pragma unroll
        for (int s = 0; s < KB; ++s)
            if (s < pieces) weights[(j * pieces + s) * 64 + lane] = item[s];
    }
    for (int i = tid; i < blocks * 16; i += 256) bias[i] = g.bias && n0 + i < g.N ? g.bias[n0 + i] : 0.0f;

    // rows: a wave takes every fourth block of 16
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.a, (uint32_t)(g.M * g.K) * 4u);
    const int row_end = min(g.M, (slab + 1) * g.rows);
    const auto load = [&](u32x4 (&f)[KB], int m0) { // (zeros behind the reduction, and behind the last row)
#pragma unroll
        for (int s = 0; s < KB; ++s) {
            const int k = s * 16 + lane_g * 4;
            f[s] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, k < g.K ? (uint32_t)((m0 + lane_r) * g.K + k) * 4u : kOutOfRange, 0, 0);
        }
    };
    u32x4 rows[KB], ahead[KB];
    int m0 = slab * g.rows + wave * 16;
    if (m0 < row_end) load(rows, m0);
    __syncthreads();
    for (; m0 < row_end; m0 += 64) {
        if (m0 + 64 < row_end) load(ahead, m0 + 64);
        const auto block = [&](int j) {
            f32x4 acc = *reinterpret_cast<const f32x4 *>(bias + j * 16 + lane_g * 4);
#pragma unroll
            for (int s = 0; s < KB; ++s)
                if (s < pieces) M::run(acc, weights[(j * pieces + s) * 64 + lane], rows[s]);
            return acc;
        };
        const auto write = [&](f32x4 v, int m, int n) { // four columns of row m
            if (m >= g.M || n >= g.N) return;
            const int64_t to = (int64_t)m * g.N + n;
            if (g.res) v += *reinterpret_cast<const f32x4 *>(g.res + to);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (g.act != ACT_NONE) v[e] = fmaxf(v[e], 0.0f);
                if (g.act == ACT_RELU6) v[e] = fminf(v[e], 6.0f);
            }
            __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(g.out + to));
        };
        int j = 0;
        // Two blocks of columns at a time: lanes of rows 0-7 hand their second block to those of rows 8-15 and get the first
        // one of these, so that a store writes eight rows of 128 bytes, whole lines, instead of sixteen of 64.
        for (; j + 1 < blocks; j += 2) {
            const f32x4 left = block(j), right = block(j + 1);
            const bool low = lane_r < 8;
            f32x4 got;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                got[e] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(low ? right[e] : left[e]), 0x128, 0xf, 0xf, false)); // row_ror:8
            const int n = n0 + (j + (low ? 0 : 1)) * 16 + lane_g * 4, m = m0 + (lane_r & 7);
            write(low ? left : got, m, n);
            write(low ? got : right, m + 8, n);
        }
        if (j < blocks) write(block(j), m0 + lane_r, n0 + j * 16 + lane_g * 4);
#pragma unroll
        for (int s = 0; s < KB; ++s) rows[s] = ahead[s];
    }
}

} // namespace tt
