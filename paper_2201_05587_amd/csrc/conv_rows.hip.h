// Convolution (bf16) over few channels, whose pixels are not whole 16-byte items (a network's first layer: 7 x 7 over 3 channels).
//
// The gathering register pipeline fetches every item of every filter row of every output pixel from memory, each with its
// own address, border check, alignment shift and mask: that arithmetic, not the matrix products or the memory, was its time.
// Here a workgroup keeps its filters in LDS and walks down the tiles of its columns; the input rows that a tile of pixels
// touches are copied into LDS ONCE, with zeros where the padding is, and those of the next tile are on their way meanwhile
// (asynchronously, straight into LDS).  A fragment is then one LDS read at  pixel + filter row * pitch + chunk: no borders,
// and one mask for the chunk that ends the run of S * C elements.  The record's tile stays, its raster, slices and stages
// have no meaning here; the reduction is walked in one go, so records that split it keep the register pipeline.
#pragma once

#include <algorithm>

#include "contract.hip.h"

namespace tt {

// Waves of a tile: 32 rows each, and 64 columns where that leaves four waves (a wave reads its pixels' fragments once for
// all its columns), else 32.
template <int TM, int TN> struct RowsShape {
    static constexpr int MF = 16, WM = 32, WN = TN % 64 == 0 && (TM / 32) * (TN / 64) >= 4 ? 64 : 32;
    static constexpr int WAVES = (TM / WM) * (TN / WN), THREADS = WAVES * 64;
    static constexpr int CH = 8, ES = 2, LG = 64 / MF;
    static constexpr int EPI_BYTES = WAVES * MF * TileOut<TM, WM, WN, MF>::ESTRIDE * 4;
};

// Layout in LDS, in bytes: the filters (rows of `filter_pitch`, an odd number of items), then two buffers of input rows.  A
// padded row is zeros up to `zone`, the image row, and zeros.  The rows of a tile, once read, give their place to the
// epilogue's staging.
struct RowsLayout {
    int32_t steps, filter_items;         // matrix-core steps of a filter row (whole ones); items of a filter
    int32_t filter_pitch, zone, pitch, rows, buffer; // `rows`: the most input rows that a tile touches
};
// The most input rows that a tile of TM pixels touches: those of its output rows, and the rows between the last of an image
// and the first of the next.  (Int: large enough for what it is asked about.)
template <int TM, typename Int> TT_HD Int rows_of_tile(const ContractArgs &g)
{
    const Int out_rows = (TM - 1 + (Int)g.Wo - 1) / g.Wo + 1;
    const Int turn = (Int)g.H + 2 * (Int)g.pad_h - (Int)g.Ho * g.stride_h;
    return (out_rows - 1) * g.stride_h + g.R + (g.M > g.Ho * g.Wo && turn > 0 ? (out_rows + g.Ho - 1) / g.Ho * turn : 0);
}
// 32 bits are enough for what rows_lds accepts.
template <int TM, int TN> TT_HD RowsLayout rows_layout(const ContractArgs &g)
{
    using S = RowsShape<TM, TN>;
    RowsLayout l;
    l.steps = (g.runp / S::CH + S::LG - 1) / S::LG;
    l.filter_items = g.R * l.steps * S::LG;
    l.filter_pitch = (l.filter_items | 1) * 16;
    l.zone = (g.pad_w * g.C * S::ES + 15) / 16 * 16;
    // (behind the row: padding, and what the last pixel's last step and its alignment word read)
    l.pitch = l.zone + ((g.W + g.pad_w) * g.C * S::ES + S::LG * 16 + 4 + 15) / 16 * 16;
    l.rows = rows_of_tile<TM, int32_t>(g);
    l.buffer = l.rows * l.pitch > S::EPI_BYTES ? l.rows * l.pitch : S::EPI_BYTES;
    const int raw = (TN * g.R * g.run * S::ES + 20 + 15) / 16 * 16; // the filters on their way, and what the last one reads behind it
    l.buffer = l.buffer > raw ? l.buffer : raw;
    return l;
}

// n / d for 0 <= n < 2^20 and d >= 1, given 1 / d: the quotient is at least 1 / (2 d) away from the next integer, and the
// product off by less than 2^-22 of n / d.
__device__ __forceinline__ int divide_small(int n, float inv_d) { return (int)(((float)n + 0.5f) * inv_d); }

// ODD: rows of outputs that are no whole 16-byte vectors.  Two instances: with both epilogues in one, the kernel needs more registers
// than the workgroups that rows_grid counts on leave it (130 for 512 threads, two of which have 128; 114 and 118 apart).
template <int TM, int TN, bool ODD>
__global__ void __launch_bounds__((RowsShape<TM, TN>::THREADS)) conv_rows_kernel(const ContractArgs args, const PointerSets sets)
{
    const ContractArgs g = with_set(args, sets, blockIdx.y);
    using S = RowsShape<TM, TN>;
    using E = uint16_t;
    constexpr int DT = TT_BF16, CH = S::CH, ES = S::ES, MF = S::MF, WM = S::WM, WN = S::WN, NI = WM / MF, NJ = WN / MF, LG = S::LG;
    constexpr int NWR = TM / WM, WAVES = S::WAVES, THREADS = S::THREADS;
    using M = Mma<DT, MF>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const RowsLayout l = rows_layout<TM, TN>(g);
    unsigned char *const filters = smem, *const patches = smem + TN * l.filter_pitch;
    const uint32_t patches0 = lds_address(patches);
    // workgroup -> (column of tiles, first tile and stride along M); the grid is a multiple of the number of columns
    const int columns = g.map.tiles_n, per = (int)gridDim.x / columns;
    TileCoord tc = {};
    tc.n0 = (int)blockIdx.x % columns * TN, tc.n_ext = min(TN, g.N - tc.n0);
    tc.k_ext = g.K;
    const BiasRegs<DT> bias = load_bias_early<DT, TM, WM, WN, MF>(g, tc, wave, lane);

    // Input rows of a tile, in padded rows counted through all images: those of pixel m begin at row base(m).
    const int ph = g.H + 2 * g.pad_h;
    struct Pixel {
        int img, row, col; // image, first padded row, first column
    };
    const auto pixel = [&](int m) {
        const uint32_t um = (uint32_t)min(m, g.M - 1);
        const uint32_t img = fast_div(um, g.div_hw), rem = um - img * (uint32_t)(g.Ho * g.Wo);
        const uint32_t p = fast_div(rem, g.div_wo), q = rem - p * (uint32_t)g.Wo;
        return Pixel{(int)img, (int)img * ph + (int)p * g.stride_h, (int)q * g.stride_w};
    };
    // Request a tile's rows into a buffer: a wave takes every WAVES-th row, 64 items at a time.  An image row is whole items
    // (the host checks), rows of the padding are out of range and arrive as zeros, and the margins of a row, which the
    // staging has overwritten, are written again.
    const int row_items = g.W * g.C / CH, margin = (l.pitch - row_items * 16) / 16;
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.a, g.a_bytes);
    const auto request = [&](int tile, int buffer) {
        if (tile >= g.map.tiles_m) return; // (its first pixel need not be a number of 32 bits)
        const Pixel first = pixel(tile * TM);
        const int rows = pixel(tile * TM + TM - 1).row + g.R - first.row;
        const uint32_t to = __builtin_amdgcn_readfirstlane(patches0 + (uint32_t)(buffer * l.buffer));
        for (int row = wave; row < rows; row += WAVES) {
            int ih = first.row + row - first.img * ph, img = first.img;
            while (ih >= ph) ih -= ph, ++img;
            ih -= g.pad_h;
            const bool real = ih >= 0 && ih < g.H;
            const uint32_t begin = (uint32_t)((img * g.H + ih) * row_items) * 16u;
            for (int i = 0; i < row_items; i += 64)
                if (i + lane < row_items)
                    load16_to_lds(a_rsrc, real ? begin + (uint32_t)(i + lane) * 16u : kOutOfRange,
                                  __builtin_amdgcn_readfirstlane(to + (uint32_t)(row * l.pitch + l.zone + i * 16)));
            for (int i = lane; i < margin; i += 64) {
                const int at = i * 16 < l.zone ? i * 16 : i * 16 + row_items * 16;
                *reinterpret_cast<u32x4 *>(patches + buffer * l.buffer + row * l.pitch + at) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    };
    int tile = (int)blockIdx.x / columns;
    request(tile, 0);

    // The filters, once per workgroup: as they lie in memory into the second buffer of rows (a column's filters are whole
    // items), and from there into rows of whole items, with zeros behind the run of every filter row.
    const int b_row_items = l.steps * LG;
    {
        const int raw_items = TN * g.R * g.run / CH;
        const uint32_t from = (uint32_t)(tc.n0 * g.R * g.run) * (uint32_t)ES, to = __builtin_amdgcn_readfirstlane(patches0 + (uint32_t)l.buffer);
        const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(g.b, g.b_bytes & ~15u);
        for (int i = wave * 64; i < raw_items; i += THREADS)
            if (i + lane < raw_items)
                load16_to_lds(b_rsrc, from + (uint32_t)(i + lane) * 16u, __builtin_amdgcn_readfirstlane(to + (uint32_t)(i * 16)));
        unsigned char *const raw = patches + l.buffer;
        wait_loads_outstanding<0>();
        __syncthreads();
        // (elements of the tensor's last item, where it is not a whole one)
        const int whole = (int)(g.b_bytes / 16u) * CH - tc.n0 * g.R * g.run, left = (g.N - tc.n0) * g.R * g.run - whole;
        if (tid < left && left < CH && whole < raw_items * CH)
            reinterpret_cast<E *>(raw)[whole + tid] = static_cast<const E *>(g.b)[tc.n0 * g.R * g.run + whole + tid];
        if (left > 0 && left < CH) __syncthreads();
        const float inv_filter = 1.0f / (float)l.filter_items, inv_row = 1.0f / (float)b_row_items;
        for (int t = tid; t < TN * l.filter_items; t += THREADS) {
            const int n = divide_small(t, inv_filter), at = t - n * l.filter_items;
            const int r = divide_small(at, inv_row), j = (at - r * b_row_items) * CH;
            const int begin = ((n * g.R + r) * g.run + min(j, g.run)) * ES;
            u32x4 v;
            __builtin_memcpy(&v, __builtin_assume_aligned(raw + (begin & ~3), 4), 16);
            const uint32_t over = *reinterpret_cast<const uint32_t *>(raw + (begin & ~3) + 16), sh = (uint32_t)begin & 2u;
            v = u32x4{__builtin_amdgcn_alignbyte(v[1], v[0], sh), __builtin_amdgcn_alignbyte(v[2], v[1], sh),
                      __builtin_amdgcn_alignbyte(v[3], v[2], sh), __builtin_amdgcn_alignbyte(over, v[3], sh)};
            v = keep_first<DT>(v, tc.n0 + n < g.N ? max(g.run - j, 0) : 0);
            *reinterpret_cast<u32x4 *>(filters + n * l.filter_pitch + at * 16) = v;
        }
    }

    const int lane_r = lane % MF, lane_g = lane / MF;
    const int wr = wave % NWR, wc = wave / NWR;
    const unsigned char *const b_row = filters + (wc * WN + lane_r) * l.filter_pitch + lane_g * 16;
    // What a lane's item of a filter row's last step holds behind the run belongs to other pixels: zeros, whatever it is
    // (a weight of zero would not silence an infinity).
    const u32x4 end_mask = keep_first<DT>(u32x4{~0u, ~0u, ~0u, ~0u}, max(g.run - ((l.steps - 1) * LG + lane_g) * CH, 0));
    const int before = l.zone - g.pad_w * g.C * ES; // of the padding in front of a row
    const bool words = before % 4 == 0 && (g.stride_w * g.C) % 2 == 0;
    wait_loads_outstanding<0>();
    int buffer = 0;
    for (; tile < g.map.tiles_m; tile += per, buffer ^= 1) {
        tc.m0 = tile * TM, tc.m_ext = min(TM, g.M - tc.m0);
        // This wave's rows have landed (the epilogue of the tile before waited for them): now everybody's have, and everybody
        // is done with the staging in the other buffer.
        __syncthreads();
        request(tile + per, buffer ^ 1);
        typename M::Acc acc[NI][NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;
        const unsigned char *const patch = patches + buffer * l.buffer;
        const int row0 = pixel(tc.m0).row;
        int a_words[NI];
        uint32_t a_shift[NI]; // pixels can begin inside a word
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const Pixel px = pixel(tc.m0 + wr * WM + i * MF + lane_r);
            const int a0 = (px.row - row0) * l.pitch + before + px.col * g.C * ES + lane_g * 16;
            a_words[i] = a0 & ~3;
            a_shift[i] = (uint32_t)a0 & 2u;
        }
        const auto k_loop = [&](auto aligned) {
            const auto step = [&](int a_at, int b_at, bool last) {
                u32x4 af[NI], bf[NJ];
                uint32_t over[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const unsigned char *from = patch + a_words[i] + a_at;
                    __builtin_memcpy(&af[i], __builtin_assume_aligned(from, 4), 16);
                    if constexpr (!decltype(aligned)::value) over[i] = *reinterpret_cast<const uint32_t *>(from + 16);
                }
#pragma unroll
                for (int j = 0; j < NJ; ++j) bf[j] = *reinterpret_cast<const u32x4 *>(b_row + j * MF * l.filter_pitch + b_at);
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    u32x4 v = af[i];
                    if constexpr (!decltype(aligned)::value)
                        v = u32x4{__builtin_amdgcn_alignbyte(v[1], v[0], a_shift[i]), __builtin_amdgcn_alignbyte(v[2], v[1], a_shift[i]),
                                  __builtin_amdgcn_alignbyte(v[3], v[2], a_shift[i]), __builtin_amdgcn_alignbyte(over[i], v[3], a_shift[i])};
                    if (last) v &= end_mask;
#pragma unroll
                    for (int j = 0; j < NJ; ++j) M::run(acc[i][j], v, bf[j]);
                }
            };
            int a_at = 0, b_at = 0;
#pragma unroll 2
            for (int r = 0; r < g.R; ++r) {
                int in_row = a_at;
                for (int s = 0; s + 1 < l.steps; ++s, in_row += LG * 16, b_at += LG * 16) step(in_row, b_at, false);
                step(in_row, b_at, true);
                a_at += l.pitch, b_at += LG * 16;
            }
        };
        if (words)
            k_loop(std::true_type{});
        else
            k_loop(std::false_type{});
        // (staged where the rows were, from when all waves have read them; the next rows are waited for before the first store)
        float *const stage = staging<WN, MF>(patches + buffer * l.buffer, wave);
        if constexpr (ODD) {
            write_tile_pieces<DT, TM, WM, WN, MF, typename M::Acc, true>(acc, g, tc, stage, wave, lane);
        } else {
            ResRegs<DT, TM, WM, WN, MF, false> no_res;
            write_tile_whole<DT, TM, WM, WN, MF, typename M::Acc, false, true>(acc, g, tc, stage, wave, lane, bias, no_res);
        }
    }
}

// LDS of a launch, or 0 where the kernel does not apply: filters of one pixel (nothing is read twice: 6.0 -> 6.6 us over 67
// channels on 4 x 56x56), no split of the reduction, image rows of whole items (so that they
// begin at whole items too), and room for two workgroups on a CU.  The layout and the padded rows counted through all images
// are computed in 32 bits, so sizes that cannot fit are turned away first, in 64.
template <int TM, int TN> int rows_lds(const ContractArgs &g)
{
    const int64_t row = ((int64_t)g.W + g.pad_w) * g.C * RowsShape<TM, TN>::ES, rows = rows_of_tile<TM, int64_t>(g);
    if (row > kLdsBudget || rows > kLdsBudget || row * rows > kLdsBudget || (int64_t)TN * g.K * RowsShape<TM, TN>::ES > kLdsBudget) return 0;
    const int64_t images = g.M / ((int64_t)g.Ho * g.Wo), padded_rows = g.H + 2ll * g.pad_h;
    if (images * padded_rows >= 1ll << 30 || g.stride_h >= 1 << 30) return 0;
    const RowsLayout l = rows_layout<TM, TN>(g);
    const int64_t bytes = (int64_t)TN * l.filter_pitch + 2ll * l.buffer;
    if (g.R * g.S == 1 || g.map.eff_split_k != 1 || (int64_t)g.W * g.C * RowsShape<TM, TN>::ES % 16 != 0 || bytes > kLdsBudget / 2) return 0;
    return (int)bytes;
}

// Workgroups of each of `count` pointer sets: as many as the CUs hold (LDS, and 16 waves at these kernels' registers), whole
// columns of tiles.
template <int TM, int TN> int rows_grid(const ContractArgs &args, int count, int lds)
{
    const int fit = std::max(1, std::min(kLdsBudget / lds, 1024 / RowsShape<TM, TN>::THREADS));
    return std::max(1, std::min(args.map.tiles_m, compute_units() * fit / (args.map.tiles_n * count))) * args.map.tiles_n;
}

template <int TM, int TN> int launch_rows(const ContractArgs &args, const PointerSets &sets, void *stream)
{
    using S = RowsShape<TM, TN>;
    const bool odd = !whole_rows<TT_BF16>(args);
    auto kern = odd ? conv_rows_kernel<TM, TN, true> : conv_rows_kernel<TM, TN, false>;
    const int lds = rows_lds<TM, TN>(args);
    static DynamicLdsLimit limits[2]; // per kernel instance
    if (const int rc = limits[odd].raise_to(reinterpret_cast<const void *>(kern), lds); rc != TT_OK) return rc;
    hipLaunchKernelGGL(kern, dim3(rows_grid<TM, TN>(args, sets.count, lds), sets.count), dim3(S::THREADS), lds, static_cast<hipStream_t>(stream), args, sets);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, "conv_rows_kernel launch");
}

} // namespace tt
