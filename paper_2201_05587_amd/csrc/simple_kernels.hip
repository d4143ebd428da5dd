// Kernels that do not use the matrix cores: the "direct"
// sketch (the unscheduled loop nest, always valid), the split-K reduction with
// the fused epilogue, the wave-reduction GEMV sketch for small-M dense kernels,
// the depthwise 3x3 tile kernel, and the index-map dump.
#include <hip/hip_runtime.h>

#include "contract.hip.h"
#include "tt_internal.h"

namespace tt {

namespace {

inline int launched()
{
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? TT_OK : note_hip_error((int)e, "kernel launch");
}

// ---- direct sketch: the unscheduled loop nest, a thread per few outputs ------------------------------------------
// What shapes below the matrix cores' smallest tile run on (a 1x1 convolution over 16 bf16 channels, 20 tokens), so reductions
// are short and the instructions around them count.  A thread forms V neighbouring outputs of a row (4 or 1, see direct_outputs),
// which share its reads of the first operand, and reads both operands in 16-byte PIECES at element alignment, or element by element
// where a run is shorter (a [K][N] operand always: its elements lie next to those of the neighbouring lanes); every sum runs in the
// order of the loop nest.  Rows and columns are counted in 32 bits (I) where they fit.
// A thread per output, element by element and counted in 64 bits -> this (us): bf16 1x1 convolutions, 16 -> 624 channels on 6 x
// 17x17 34.6 -> 10.1, 16 -> 72 on 7 x 25x22 12.0 -> 3.7, 20 -> 128 on 8 x 56x57 59.7 -> 17.9; 3x3 stride 3, 64 -> 33 on 7x7 57.3 -> 12.5;
// 5x5, 4 -> 98 on 3x9 8.6 -> 8.4; 192 products of 31 x 31 x 31 9.1 -> 5.8; fp32 13 -> 64 on 4 x 30x30 6.2 -> 3.8, 3x3 41 -> 29 on 2 x
// 13x13 42.1 -> 16.5; the geometric mean over 750 draws is 1.74 times.
template <int DT, int V, bool PIECES>
__device__ __forceinline__ void add_products(float (&acc)[V], const typename ElemOf<DT>::type *x, const typename ElemOf<DT>::type *const (&w)[V], int count)
{
    constexpr int CH = ElemOf<DT>::CH;
    if constexpr (!PIECES) {
        for (int c = 0; c < count; ++c) {
            const float xv = load_as_float<DT>(x, c);
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = fmaf(xv, load_as_float<DT>(w[v], c), acc[v]);
        }
        return;
    }
    int c = 0;
    for (; c + CH <= count; c += CH) {
        u32x4 xv, wv[V];
        load16(xv, x + c);
#pragma unroll
        for (int v = 0; v < V; ++v) load16(wv[v], w[v] + c);
#pragma unroll
        for (int e = 0; e < CH; ++e)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = fmaf(element_of<DT>(xv, e), element_of<DT>(wv[v], e), acc[v]);
    }
    if (c < count) { // the rest: the last piece, shifted down to where the sum stands (zeros behind it)
        const int back = c + CH - count;
        u32x4 xv, wv[V];
        load16(xv, x + count - CH);
#pragma unroll
        for (int v = 0; v < V; ++v) load16(wv[v], w[v] + count - CH);
        xv = shift_elems<DT>(xv, -back);
#pragma unroll
        for (int v = 0; v < V; ++v) wv[v] = shift_elems<DT>(wv[v], -back);
#pragma unroll
        for (int e = 0; e < CH - 1; ++e)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] = fmaf(element_of<DT>(xv, e), element_of<DT>(wv[v], e), acc[v]);
    }
}
template <int DT, int FAM, int V, bool PIECES, typename I> __global__ void __launch_bounds__(256) direct_kernel(const ContractArgs args, const PointerSets sets)
{
    const ContractArgs g = with_set(args, sets, blockIdx.y);
    using E = typename ElemOf<DT>::type;
    const I columns = (I)((g.N + V - 1) / V);
    const I idx = (I)blockIdx.x * 256 + threadIdx.x;
    const I row = idx / columns; // of all batches
    if (row >= (I)g.batch * (I)g.M) return;
    const int n = (int)(idx - row * columns) * V, count = min(V, g.N - n);
    const E *a = static_cast<const E *>(g.a), *b = static_cast<const E *>(g.b);
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.0f;
    if constexpr (FAM == FAM_CONV) {
        // rows are output pixels (img, p, q); activations NHWC, filters KRSC
        const I img = row / (I)(g.Ho * g.Wo);
        const int rem = (int)(row - img * (I)(g.Ho * g.Wo)), p = rem / g.Wo, q = rem - p * g.Wo;
        for (int r = 0; r < g.R; ++r) {
            const int ih = p * g.stride_h + r - g.pad_h;
            if (ih < 0 || ih >= g.H) continue;
            for (int s = 0; s < g.S; ++s) {
                const int iw = q * g.stride_w + s - g.pad_w;
                if (iw < 0 || iw >= g.W) continue;
                const E *w[V];
#pragma unroll
                for (int v = 0; v < V; ++v) w[v] = b + (((int64_t)min(n + v, g.N - 1) * g.R + r) * g.S + s) * g.C;
                add_products<DT, V, PIECES>(acc, a + (((int64_t)img * g.H + ih) * g.W + iw) * g.C, w, g.C);
            }
        }
    } else {
        const int64_t bi = (int64_t)(row / (I)g.M);
        const E *ar = a + (int64_t)row * g.K, *bb = b + bi * g.N * g.K;
        if constexpr (FAM == FAM_GEMM_TN) {
            const E *w[V];
#pragma unroll
            for (int v = 0; v < V; ++v) w[v] = bb + (int64_t)min(n + v, g.N - 1) * g.K;
            add_products<DT, V, PIECES>(acc, ar, w, g.K);
        } else {
            for (int k = 0; k < g.K; ++k) {
                const float av = load_as_float<DT>(ar, k);
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] = fmaf(av, load_as_float<DT>(bb, (int64_t)k * g.N + min(n + v, g.N - 1)), acc[v]);
            }
        }
    }
    const int64_t at = (int64_t)row * g.N + n;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if (v >= count) break;
        float out = acc[v];
        if (g.has_bias) out += load_as_float<DT>(g.bias, n + v);
        if (g.has_res) out += load_as_float<DT>(g.res, at + v);
        store_from_float<DT>(g.out, at + v, apply_act(out, g.act));
    }
}

// ---- split-K: sum the partial tiles in split order, then the fused epilogue -----------------------
// Bound by latency: a few hundred KB that the contraction has just left in the caches.  A thread takes VEC
// consecutive outputs of one row (N is a multiple of VEC) and asks for the partial sums of two, four or eight splits, as
// many as there are, before it adds the first; workgroups of one wave spread a small output over the CUs.  Both launches
// together, element by element / eight requests whatever the number of splits / this (us): f32 784 x 128, K = 576, two
// splits 8.5 / 9.3 / 8.8; K = 2304, two 13.8 / 12.9 / 12.4, four 12.5 / 12.9 / 12.7, 32 18.4 / 15.5 / 15.1; bf16 4096 x 1024,
// K = 1024, two 35.3 / 35.3 / 33.4.
template <int DT, int VEC> __device__ __forceinline__ void reduce_outputs(const ReduceEntry &g, int64_t idx)
{
    typedef __attribute__((ext_vector_type(VEC))) float vec_t;
    const int64_t total = g.total;
    if (idx >= total) return;
    // (32-bit division where it is enough: the 64-bit one is some hundred instructions)
    const int n = total < (1ll << 31) ? (int)((uint32_t)idx % (uint32_t)g.N) : (int)(idx % g.N), splits = g.splits;
    const float *ws = g.ws + idx;
    float res[VEC] = {}, bias[VEC] = {};
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        if (g.bias) bias[e] = load_as_float<DT>(g.bias, n + e);
        if (g.res) res[e] = load_as_float<DT>(g.res, idx + e);
    }
    vec_t acc = vec_t(0.0f);
    const auto add = [&](int z0, auto width) { // up to `width` splits from z0 on, requested together
        constexpr int P = decltype(width)::value;
        vec_t part[P];
#pragma unroll
        for (int z = 0; z < P; ++z) // (past the last split: the last one again, not added)
            part[z] = *reinterpret_cast<const vec_t *>(ws + (int64_t)min(z0 + z, splits - 1) * total);
#pragma unroll
        for (int z = 0; z < P; ++z)
            if (z0 + z < splits) acc += part[z];
    };
    int z0 = 0;
    for (; splits - z0 > 4; z0 += 8) add(z0, std::integral_constant<int, 8>{});
    if (splits - z0 > 2)
        add(z0, std::integral_constant<int, 4>{});
    else if (splits > z0)
        add(z0, std::integral_constant<int, 2>{});
#pragma unroll
    for (int e = 0; e < VEC; ++e) store_from_float<DT>(g.out, idx + e, apply_act(acc[e] + bias[e] + res[e], g.act));
}
template <int DT, int VEC> __global__ void __launch_bounds__(256) splitk_reduce_kernel(const ContractArgs args, const PointerSets sets)
{
    const ContractArgs g = with_set(args, sets, blockIdx.y);
    const ReduceEntry e = {g.ws, g.has_bias ? g.bias : nullptr, g.has_res ? g.res : nullptr, g.out, (int64_t)g.batch * g.M * g.N,
                           g.N, g.map.eff_split_k, g.act, 0};
    reduce_outputs<DT, VEC>(e, ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * VEC);
}
// The same for entries of different shapes in one launch, workgroups of one wave.
template <int DT, int VEC> __global__ void __launch_bounds__(64) splitk_reduce_list_kernel(const ReduceList list)
{
    int e = 0;
    while (e + 1 < kMaxReduced && (int)blockIdx.x >= list.e[e + 1].first) ++e;
    reduce_outputs<DT, VEC>(list.e[e], ((int64_t)((int)blockIdx.x - list.e[e].first) * 64 + threadIdx.x) * VEC);
}

// ---- GEMV sketch: a wave owns W outputs of R rows; lanes split K ---------------------------------
// Bound by latency (a classifier reads 2 MB): every lane asks for four pieces of EV elements of each row and each
// weight vector before it multiplies the first, so a reduction of 256 EV elements pays the memory once, and the
// lanes' sums are added by data-parallel moves (DPP) instead of six trips through the LDS crossbar.  A first
// version loaded element by element: 1 x 512 x 1000 in f32 took 5.7 us, now 2.8.  A call is then bound by the host's
// launch, which takes 3.1 us with up to 64 bytes of kernel arguments and 4.5 us from 256 bytes on: the arguments are
// this kernel's own, in 64 bytes.
struct GemvArgs {
    const void *x, *w, *bias; // bias may be null
    void *out;
    int32_t M, N, K, tiles_n;
    FastDiv div_n;                          // by tiles_n
    uint8_t tile_m, wave_n, waves, act;     // rows of a workgroup, outputs per wave, waves per workgroup
};
static_assert(sizeof(GemvArgs) <= 64, "");

template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_sum(float v) // the sum of all lanes, in lane 63
{
    v = dpp_add<0x111, 0xf>(v); // row_shr:1
    v = dpp_add<0x112, 0xf>(v); // row_shr:2
    v = dpp_add<0x114, 0xf>(v); // row_shr:4
    v = dpp_add<0x118, 0xf>(v); // row_shr:8: lane 15 of every row of 16 has the row's sum
    v = dpp_add<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
}

template <int DT, int EV> struct GemvPiece { // EV consecutive elements as floats
    using E = typename ElemOf<DT>::type;
    E e[EV];
    __device__ __forceinline__ void load(const E *p) { __builtin_memcpy(e, __builtin_assume_aligned(p, EV * sizeof(E)), sizeof e); }
    __device__ __forceinline__ float at(int i) const
    {
        if constexpr (DT == TT_F32)
            return e[i];
        else
            return bf16_bits_to_float(e[i]);
    }
};

template <int DT, int R, int W, int EV> __global__ void __launch_bounds__(1024) gemv_kernel(const GemvArgs g)
{
    using E = typename ElemOf<DT>::type;
    constexpr int U = R * W >= 64 ? 1 : R * W >= 16 ? 2 : 4; // pieces in flight per vector
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile_m = g.tile_m, wave_n = g.wave_n;
    const int im = (int)fast_div(blockIdx.x, g.div_n), in = (int)blockIdx.x - im * g.tiles_n;
    const int m_first = im * tile_m, n_first = (in * g.waves + wave) * wave_n;
    // rows and outputs beyond tile_m, wave_n or the matrix read the last one again and are not written
    const E *x[R], *w[W];
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = static_cast<const E *>(g.x) + (int64_t)min(m_first + min(i, tile_m - 1), g.M - 1) * g.K;
#pragma unroll
    for (int j = 0; j < W; ++j) w[j] = static_cast<const E *>(g.w) + (int64_t)min(n_first + min(j, wave_n - 1), g.N - 1) * g.K;
    float acc[R][W];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) acc[i][j] = 0.0f;
    for (int kb = lane * EV; kb < g.K; kb += 64 * EV * U) { // K is a multiple of EV: a piece is all in or all out
        GemvPiece<DT, EV> xp[U][R], wp[U][W];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(kb + u * 64 * EV, g.K - EV);
#pragma unroll
            for (int i = 0; i < R; ++i) xp[u][i].load(x[i] + k);
#pragma unroll
            for (int j = 0; j < W; ++j) wp[u][j].load(w[j] + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (kb + u * 64 * EV >= g.K) break;
#pragma unroll
            for (int e = 0; e < EV; ++e)
#pragma unroll
                for (int i = 0; i < R; ++i)
#pragma unroll
                    for (int j = 0; j < W; ++j) acc[i][j] = fmaf(xp[u][i].at(e), wp[u][j].at(e), acc[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) {
            float v = wave_sum(acc[i][j]);
            const int m = m_first + i, n = n_first + j;
            if (lane == 63 && i < tile_m && j < wave_n && m < g.M && n < g.N) {
                if (g.bias) v += load_as_float<DT>(g.bias, n);
                store_from_float<DT>(g.out, (int64_t)m * g.N + n, apply_act(v, g.act));
            }
        }
}

// ---- depthwise 3x3 over NHWC: (rows, cols, planes) tile per workgroup, WM x WN outputs per thread ---
// A plane is one (image, channel) pair, numbered image * C + channel.  Threads are laid out planes
// fastest, then cols, then rows, so the lanes of a wave read and write neighbouring channels of one
// pixel.  With two stages the input patch of the tile is first copied to LDS (planes fastest too).
template <int WM, int WN, int MAXT> __global__ void __launch_bounds__(MAXT) dwconv3x3_kernel(const DwArgs args, const PointerSets sets)
{
    const DwArgs g = with_set(args, sets, blockIdx.y);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    float *patch = reinterpret_cast<float *>(smem_raw);
    const TileCoord tc = decode_tile(g.map, (int32_t)blockIdx.x);
    const int tk = g.map.tile_k;
    const int tcols = g.map.tile_n / WN;
    const int tid = threadIdx.x;
    const int tp = tid % tk, tx = (tid / tk) % tcols, ty = tid / (tk * tcols);
    const int plane = tc.k0 + tp;
    const int p0 = tc.m0 + ty * WM, q0 = tc.n0 + tx * WN;
    const int prow = (g.map.tile_m - 1) * g.stride_h + 3, pcol = (g.map.tile_n - 1) * g.stride_w + 3;
    const int ih_org = tc.m0 * g.stride_h - g.pad_h, iw_org = tc.n0 * g.stride_w - g.pad_w;
    if (g.stages == 2) {
        const int total = prow * pcol * tk;
        for (int e = tid; e < total; e += blockDim.x) {
            const int pl = e % tk, cell = e / tk;
            const int rr = cell / pcol, cc = cell - rr * pcol;
            const int ih = ih_org + rr, iw = iw_org + cc;
            float v = 0.0f;
            if (pl < tc.k_ext && ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) {
                const int pn = (tc.k0 + pl) / g.C, pc = (tc.k0 + pl) - pn * g.C;
                v = g.x[(((int64_t)pn * g.H + ih) * g.W + iw) * g.C + pc];
            }
            patch[e] = v;
        }
        __syncthreads();
    }
    if (tp >= tc.k_ext) return;
    const int img = plane / g.C, ch = plane - img * g.C;
    float wgt[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) wgt[i] = g.w[i * g.C + ch];
    const float bias = g.bias ? g.bias[ch] : 0.0f;
    const float *xp = g.x + (int64_t)img * g.H * g.W * g.C + ch;
    float *yp = g.y + (int64_t)img * g.Ho * g.Wo * g.C + ch;
    auto body = [&](int i) {
        const int p = p0 + i;
        if (p >= g.Ho || p >= tc.m0 + tc.m_ext) return;
        float out[WN];
#pragma unroll
        for (int j = 0; j < WN; ++j) out[j] = bias;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int ih = p * g.stride_h + r - g.pad_h;
#pragma unroll
            for (int j = 0; j < WN; ++j) {
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    const int iw = (q0 + j) * g.stride_w + s - g.pad_w;
                    float v = 0.0f;
                    if (g.stages == 2) {
                        v = patch[((ih - ih_org) * pcol + (iw - iw_org)) * tk + tp];
                    } else if (ih >= 0 && ih < g.H && iw >= 0 && iw < g.W) {
                        v = xp[((int64_t)ih * g.W + iw) * g.C];
                    }
                    out[j] = fmaf(v, wgt[r * 3 + s], out[j]);
                }
            }
        }
        const int qlim = min(g.Wo, tc.n0 + tc.n_ext);
#pragma unroll
        for (int j = 0; j < WN; ++j)
            if (q0 + j < qlim) yp[((int64_t)p * g.Wo + q0 + j) * g.C] = fminf(fmaxf(out[j], 0.0f), 6.0f);
    };
    if (g.unroll >= WM) {
#pragma unroll
        for (int i = 0; i < WM; ++i) body(i);
    } else {
#pragma unroll 1
        for (int i = 0; i < WM; ++i) body(i);
    }
}

// ---- depthwise 3x3 in windows: one entry, or entries of different shapes in one launch ------------------------------
// Bound by memory.  A thread forms WM x WN outputs of VC neighbouring channels and reads every input pixel of its window
// once, all of them before the first product: (WM + 2) (WN + 2) / (WM WN) reads an output at unit stride, 3 for 4 x 2, 4 for
// 2 x 2, where tiles of workgroups with rows of outputs per thread made 9 (1 x 1) to 3.9 (7 columns).  Padding comes from loads
// out of range, which return zero.  The lanes of a wave hold neighbouring channels of one pixel: every access is one run of
// memory.  The sums run in the order of the other kernels.
template <int STR, int VC, int WM, int WN> __device__ __forceinline__ void dw_window(const DwListEntry &g, int wg)
{
    constexpr int ROWS = (WM - 1) * STR + 3, COLS = (WN - 1) * STR + 3;
    typedef __attribute__((ext_vector_type(VC))) float vec_t;
    // every XCD gets a contiguous run of the entry's workgroups: neighbouring windows share rows in its L2
    const int wgs = (g.threads + 255) / 256, per = wgs / kXcds, rem = wgs % kXcds, xcd = wg % kXcds;
    if (wg >= wgs) return;
    const int t = (xcd * per + min(xcd, rem) + wg / kXcds) * 256 + (int)threadIdx.x;
    if (t >= g.threads) return;
    const int lanes = g.C / VC, columns = (g.Wo + WN - 1) / WN, strips = (g.Ho + WM - 1) / WM;
    const int pix = (int)fast_div((uint32_t)t, g.div_c), ch = (t - pix * lanes) * VC;
    const int row = (int)fast_div((uint32_t)pix, g.div_cols), q0 = (pix - row * columns) * WN;
    const int img = (int)fast_div((uint32_t)row, g.div_rows), p0 = (row - img * strips) * WM;

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(g.x, g.x_bytes);
    vec_t in[ROWS][COLS], wgt[9];
    const int ih0 = p0 * STR - g.pad_h, iw0 = q0 * STR - g.pad_w;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            const int ih = ih0 + r, iw = iw0 + c;
            const bool ok = ih >= 0 && ih < g.H && iw >= 0 && iw < g.W;
            const uint32_t off = ok ? (uint32_t)(((img * g.H + ih) * g.W + iw) * g.C + ch) * 4u : kOutOfRange;
            if constexpr (VC == 4)
                in[r][c] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
            else if constexpr (VC == 2)
                in[r][c] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b64(xr, off, 0, 0));
            else
                in[r][c][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xr, off, 0, 0));
        }
#pragma unroll
    for (int i = 0; i < 9; ++i) wgt[i] = *reinterpret_cast<const vec_t *>(g.w + i * g.C + ch);
    vec_t bias = 0.0f;
    if (g.bias) bias = *reinterpret_cast<const vec_t *>(g.bias + ch);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            vec_t out = bias;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int s = 0; s < 3; ++s)
#pragma unroll
                    for (int v = 0; v < VC; ++v) out[v] = fmaf(in[i * STR + r][j * STR + s][v], wgt[r * 3 + s][v], out[v]);
            const int p = p0 + i, q = q0 + j;
            if (p >= g.Ho || q >= g.Wo) continue;
#pragma unroll
            for (int v = 0; v < VC; ++v) out[v] = fminf(fmaxf(out[v], 0.0f), 6.0f);
            __builtin_nontemporal_store(out, reinterpret_cast<vec_t *>(g.y + ((int64_t)(img * g.Ho + p) * g.Wo + q) * g.C + ch)); // streamed
        }
}
// Windows that a list is cut into.
template <int STR> constexpr DwWindow kDwListWindow = {STR == 1 ? 4 : 2, 2};
template <int STR> __global__ void __launch_bounds__(256) dwconv3x3_list_kernel(const DwList list)
{
    int at = 0;
#pragma unroll
    for (int i = 1; i < kMaxDwListed; ++i) at += (int)blockIdx.x >= list.e[i].first;
    const DwListEntry &g = list.e[at];
    dw_window<STR, 4, kDwListWindow<STR>.rows, kDwListWindow<STR>.columns>(g, (int)blockIdx.x - g.first);
}
// (96 bytes of arguments: up to there a launch costs the host 2.9 us, with 704 bytes 3.9)
static_assert(sizeof(DwListEntry) <= 96, "");
template <int STR, int VC, int WM, int WN> __global__ void __launch_bounds__(256) dwconv3x3_window_kernel(const DwListEntry g)
{
    dw_window<STR, VC, WM, WN>(g, (int)blockIdx.x);
}
// Several entries of one plan.
template <int STR, int VC, int WM, int WN> __global__ void __launch_bounds__(256) dwconv3x3_window_sets_kernel(DwListEntry g, const PointerSets sets)
{
    if (blockIdx.y > 0) {
        const PointerSet &p = sets.more[blockIdx.y - 1];
        g.x = static_cast<const float *>(p.a), g.w = static_cast<const float *>(p.b);
        g.bias = static_cast<const float *>(p.bias), g.y = static_cast<float *>(p.out);
    }
    dw_window<STR, VC, WM, WN>(g, (int)blockIdx.x);
}

__global__ void __launch_bounds__(256) dw_direct_kernel(const DwArgs args, const PointerSets sets)
{
    const DwArgs g = with_set(args, sets, blockIdx.y);
    // idx walks the NHWC output: (image, p, q, channel)
    const int64_t total = (int64_t)g.planes * g.Ho * g.Wo;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int ch = (int)(idx % g.C);
        const int64_t pix = idx / g.C;
        const int q = (int)(pix % g.Wo), p = (int)((pix / g.Wo) % g.Ho);
        const int img = (int)(pix / ((int64_t)g.Ho * g.Wo));
        float acc = 0.0f;
        for (int r = 0; r < 3; ++r) {
            const int ih = p * g.stride_h + r - g.pad_h;
            if (ih < 0 || ih >= g.H) continue;
            for (int s = 0; s < 3; ++s) {
                const int iw = q * g.stride_w + s - g.pad_w;
                if (iw < 0 || iw >= g.W) continue;
                acc = fmaf(g.x[(((int64_t)img * g.H + ih) * g.W + iw) * g.C + ch], g.w[(r * 3 + s) * g.C + ch], acc);
            }
        }
        if (g.bias) acc += g.bias[ch];
        g.y[idx] = fminf(fmaxf(acc, 0.0f), 6.0f);
    }
}

__global__ void __launch_bounds__(256) tile_map_dump_kernel(const TileMap map, int32_t *out)
{
    const int wg = blockIdx.x * 256 + threadIdx.x;
    if (wg >= map.grid) return;
    const TileCoord c = decode_tile(map, wg);
    int32_t *o = out + (int64_t)wg * 8;
    o[0] = c.hi;
    o[1] = c.lo;
    o[2] = c.m0;
    o[3] = c.m_ext;
    o[4] = c.n0;
    o[5] = c.n_ext;
    o[6] = c.k0;
    o[7] = c.k_ext;
}

// Whether the direct kernel reads in pieces: reductions (a pixel's channels) of at least one.  Shorter ones are a loop over
// elements, of one output a thread: that loop with four took 1.2 to 1.7 times as long at any size.
bool direct_in_pieces(const ContractArgs &a, int family) { return family != FAM_GEMM_NN && (family == FAM_CONV ? a.C : a.K) >= (a.dtype == TT_F32 ? 4 : 8); }
// Outputs of a thread: four read the first operand a fourth as often, one has four times the threads to wait for memory with.
// One -> four, geometric means over draws (bf16 runs of 8 .. 31 channels, of 32 and more; fp32 of 4 .. 15, of 16 and more): 8 to 30
// thousand outputs 1.57, 1.83, 1.29, 2.05 times as long, 30 to 100 thousand 1.50, 1.63, 1.32, 1.72, 100 to 400 thousand 1.12, 1.13,
// 1.18, 1.08, beyond (to 3 million) 0.83, 0.66, 1.08, 0.98.
int direct_outputs(const ContractArgs &a, int family, int count)
{
    return direct_in_pieces(a, family) && a.N >= 4 && (int64_t)a.batch * a.M * a.N * count >= 400000 ? 4 : 1;
}
template <int DT, int FAM, int V, bool PIECES> int launch_direct_in(int64_t grid, const ContractArgs &a, const PointerSets &sets, hipStream_t s)
{
    const auto kern = grid < 1ll << 23 ? direct_kernel<DT, FAM, V, PIECES, uint32_t> : direct_kernel<DT, FAM, V, PIECES, uint64_t>;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid, sets.count), dim3(256), 0, s, a, sets);
    return launched();
}
template <int DT, int FAM> int launch_direct_of(const ContractArgs &a, const PointerSets &sets, hipStream_t s)
{
    const int64_t grid = direct_workgroups(a, FAM, sets.count);
    if constexpr (FAM != FAM_GEMM_NN)
        if (direct_in_pieces(a, FAM))
            return direct_outputs(a, FAM, sets.count) == 4 ? launch_direct_in<DT, FAM, 4, true>(grid, a, sets, s) : launch_direct_in<DT, FAM, 1, true>(grid, a, sets, s);
    return launch_direct_in<DT, FAM, 1, false>(grid, a, sets, s);
}
template <int DT> int launch_direct_dt(const ContractArgs &a, const PointerSets &sets, int family, hipStream_t s)
{
    switch (family) {
    case FAM_CONV: return launch_direct_of<DT, FAM_CONV>(a, sets, s);
    case FAM_GEMM_TN: return launch_direct_of<DT, FAM_GEMM_TN>(a, sets, s);
    default: return launch_direct_of<DT, FAM_GEMM_NN>(a, sets, s);
    }
}

} // namespace

int64_t direct_workgroups(const ContractArgs &a, int family, int count)
{
    const int v = direct_outputs(a, family, count);
    return ((int64_t)a.batch * a.M * ((a.N + v - 1) / v) + 255) / 256;
}

int launch_direct(const ContractArgs &args, const PointerSets &sets, int family, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    return args.dtype == TT_F32 ? launch_direct_dt<TT_F32>(args, sets, family, s) : launch_direct_dt<TT_BF16>(args, sets, family, s);
}

int launch_splitk_reduce(const ContractArgs &args, const PointerSets &sets, int family, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    (void)family; // every family writes a row-major [M][N] output
    const int vec = args.N % 4 == 0 ? 4 : 1;
    const int64_t threads = (int64_t)args.batch * args.M * args.N / vec;
    const int block = threads <= 256 * 256 ? 64 : 256; // up to a workgroup of one wave for each SIMD of the chip
    const dim3 grid((unsigned)((threads + block - 1) / block), sets.count);
    auto kern = vec == 4 ? splitk_reduce_kernel<TT_F32, 4> : splitk_reduce_kernel<TT_F32, 1>;
    if (args.dtype == TT_BF16) kern = vec == 4 ? splitk_reduce_kernel<TT_BF16, 4> : splitk_reduce_kernel<TT_BF16, 1>;
    hipLaunchKernelGGL(kern, grid, dim3(block), 0, s, args, sets);
    return launched();
}

int launch_reduce_list(ReduceList &list, int count, int dtype, bool fours, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    int grid = 0;
    for (int i = 0; i < kMaxReduced; ++i) {
        list.e[i].first = i < count ? grid : INT32_MAX;
        if (i < count) grid += (int)((list.e[i].total / (fours ? 4 : 1) + 63) / 64);
    }
    auto kern = fours ? splitk_reduce_list_kernel<TT_F32, 4> : splitk_reduce_list_kernel<TT_F32, 1>;
    if (dtype == TT_BF16) kern = fours ? splitk_reduce_list_kernel<TT_BF16, 4> : splitk_reduce_list_kernel<TT_BF16, 1>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64), 0, s, list);
    return launched();
}

namespace {

template <int DT, int R, int W> void launch_gemv_rw(const GemvArgs &g, const tt_plan &plan, hipStream_t s)
{
    auto kern = gemv_kernel<DT, R, W, 1>;
    if (plan.eff_vec_a == 2) kern = gemv_kernel<DT, R, W, 2>;
    if (plan.eff_vec_a == 4) kern = gemv_kernel<DT, R, W, 4>;
    if constexpr (DT == TT_BF16) // (8 x 8 sums leave registers for pieces of 4)
        if (plan.eff_vec_a == 8) kern = gemv_kernel<DT, R, W, R * W < 64 ? 8 : 4>;
    hipLaunchKernelGGL(kern, dim3(plan.grid), dim3(plan.block), 0, s, g);
}
// instances for 1, 2, 4 and 8 rows and outputs per wave; others run on the next larger one
template <int DT, int R> void launch_gemv_r(const GemvArgs &g, const tt_plan &plan, hipStream_t s)
{
    if (plan.wave_n <= 1) return launch_gemv_rw<DT, R, 1>(g, plan, s);
    if (plan.wave_n <= 2) return launch_gemv_rw<DT, R, 2>(g, plan, s);
    if (plan.wave_n <= 4) return launch_gemv_rw<DT, R, 4>(g, plan, s);
    return launch_gemv_rw<DT, R, 8>(g, plan, s);
}
template <int DT> void launch_gemv_dt(const GemvArgs &g, const tt_plan &plan, hipStream_t s)
{
    if (plan.tile_m <= 1) return launch_gemv_r<DT, 1>(g, plan, s);
    if (plan.tile_m <= 2) return launch_gemv_r<DT, 2>(g, plan, s);
    if (plan.tile_m <= 4) return launch_gemv_r<DT, 4>(g, plan, s);
    return launch_gemv_r<DT, 8>(g, plan, s);
}

} // namespace

int launch_gemv(const ContractArgs &args, const PointerSets &sets, const tt_plan &plan, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int i = 0; i < sets.count; ++i) { // (one launch each: the table of sets would not fit the 64 bytes)
        const ContractArgs a = with_set(args, sets, (uint32_t)i);
        const GemvArgs g = {a.a, a.b, a.bias, a.out, a.M, a.N, a.K, plan.tiles_n, a.map.div_n,
                            (uint8_t)plan.tile_m, (uint8_t)plan.wave_n, (uint8_t)(plan.block / 64), (uint8_t)a.act};
        if (args.dtype == TT_F32)
            launch_gemv_dt<TT_F32>(g, plan, s);
        else
            launch_gemv_dt<TT_BF16>(g, plan, s);
        if (const int rc = launched(); rc != TT_OK) return rc;
    }
    return TT_OK;
}

// Workgroups that a depthwise record may name.  The general kernel is compiled for at most 256, 512 and 1024 threads, which leaves
// a lane 512, 256 and 128 registers; of these sizes, by its outputs per row, the compiler keeps everything in registers.  Records
// that ask for neither an LDS patch nor unequal strides (`in_registers`) run in windows of 256 threads whatever they name: their
// bound, input columns of a thread's outputs times planes per access, only says which of them are records at all, so that stored
// pools and the counts of a search stand.
constexpr int dw_block_limit(int wave_m, int wave_n, int planes_per_lane, int stride, bool in_registers)
{
    const auto built = [](int w) { return w == 1 || w == 2 || w == 4 || w == 7; };
    if (!built(wave_m) || !built(wave_n)) return 0; // no instance for other outputs per thread
    if (in_registers) {
        const int in_flight = ((wave_n - 1) * stride + 3) * planes_per_lane;
        return in_flight <= 9 || (in_flight <= 16 && wave_n < 7) ? 1024 : in_flight <= 36 ? 512 : 256;
    }
    return wave_n <= 2 ? 1024 : wave_n <= 4 ? 512 : 256;
}

int dw_max_block(int wave_m, int wave_n, int planes_per_lane, int stride, bool in_registers)
{
    return dw_block_limit(wave_m, wave_n, planes_per_lane, stride, in_registers);
}

namespace {

// The part of an entry that its sizes decide; false: no windows for it.
bool dw_entry(const DwArgs &g, int vc, DwWindow w, DwListEntry *e)
{
    if (g.C % vc != 0 || g.stride_h != g.stride_w || (g.stride_h != 1 && g.stride_h != 2) || g.x_bytes == 0) return false;
    const int64_t columns = (g.Wo + w.columns - 1) / w.columns, strips = (g.Ho + w.rows - 1) / w.rows, threads = g.planes / vc * columns * strips;
    if (threads >= 1ll << 30 || (int64_t)(g.planes / g.C) * g.Ho >= 1ll << 31) return false; // (rows of outputs, too, are counted in 32 bits)
    e->threads = (int32_t)threads;
    e->C = g.C, e->H = g.H, e->W = g.W, e->Ho = g.Ho, e->Wo = g.Wo, e->pad_h = g.pad_h, e->pad_w = g.pad_w, e->x_bytes = g.x_bytes;
    e->div_c = make_fastdiv((uint32_t)(g.C / vc)), e->div_cols = make_fastdiv((uint32_t)columns), e->div_rows = make_fastdiv((uint32_t)strips);
    return true;
}

// The window of a launch of `pieces` outputs of one thread's channels.  A larger one reads less and a smaller one has more threads,
// and less code to fetch before the first load: 1 x 1 up to a workgroup per CU, 1 x 2 up to six, 4 x 2 from 80 on.  Unit stride, 1x1 /
// 1x2 / 2x2 / 4x2 in us, and in rows of the record that a search chose: 57 k pieces 2.7 / 3.0 / 3.6 / 4.8, 3.2; 71 k 3.1 / 3.0 /
// 3.6 / 4.8, 3.7; 100 k 3.2 / 3.1 / 3.7 / 4.9; 202 k 4.4 / 3.8 / 3.8 / 5.0; 306 k 5.1 / 4.7 / 4.8 / 5.3; 368 k 5.6 / 4.5 / 4.5 / 5.1, 5.3; 390 k 5.6 /
// 5.2 / 4.8 / 5.3; 406 k 6.1 / 5.1 / 4.5 / 5.0; 442 k 6.1 / 5.1 / 4.5 / 5.1, -; 609 k 7.8 / 5.8 / 5.4 / 5.8; 1.0 M 10.9 / 7.9 / 6.4 / 6.1, 9.7; 2.1 M
// 20.3 / 14.9 / 12.0 / 12.4; 4.1 M 41.7 / 30.2 / 23.4 / 24.2, 41.6; 5.4 M 56 / 39 / 29.7 / 29.2, 39.5; 6.2 M 67 / 45 / 37.9 / 34.5, 48.3.  So 1x2 and
// 2x2 are level from 200 to 370 thousand, and the last workgroup before the line loses 8 %; between 0.8 and 4 million 2x2 and 4x2 are
// within 5 %, either way.  Stride 2, 1x1 / 1x2 / 2x2: 76 k 3.1 / 3.2 / 4.1, 3.6; 202 k 4.3 / 3.9 / 4.1; 326 k 5.0 / 4.6 / 4.9, 8.7; 390 k 5.6 / 5.5 / 5.2;
// 469 k 6.7 / 5.7 / 5.2, 10.9; 609 k 9.5 / 8.7 / 8.6; 1.4 M 21.0 / 19.4 / 19.0, 22.4; 2.1 M 24.8 / 25.9 / 25.9, where the memory is the bound.
DwWindow dw_window_for(int64_t pieces, int stride)
{
    if (pieces <= 65536) return {1, 1};
    if (pieces <= 6 * 65536) return {1, 2};
    if (stride == 2 || pieces <= 80 * 65536) return {2, 2};
    return {4, 2};
}

template <int STR, int VC, int WM, int WN> int launch_windows(const DwListEntry &e, const PointerSets &sets, hipStream_t s)
{
    const unsigned grid = (unsigned)dw_workgroups(e);
    if (sets.count == 1)
        hipLaunchKernelGGL((dwconv3x3_window_kernel<STR, VC, WM, WN>), dim3(grid), dim3(256), 0, s, e);
    else
        hipLaunchKernelGGL((dwconv3x3_window_sets_kernel<STR, VC, WM, WN>), dim3(grid, sets.count), dim3(256), 0, s, e, sets);
    return launched();
}
template <int STR, int VC> int launch_windows_of(DwWindow w, const DwListEntry &e, const PointerSets &sets, hipStream_t s)
{
    if constexpr (STR == 1)
        if (w.rows == 4) return launch_windows<STR, VC, 4, 2>(e, sets, s);
    if (w.rows == 2) return launch_windows<STR, VC, 2, 2>(e, sets, s);
    if (w.columns == 2) return launch_windows<STR, VC, 1, 2>(e, sets, s);
    return launch_windows<STR, VC, 1, 1>(e, sets, s);
}

} // namespace

// Records of one stage over a tensor within the 2 GiB offset range, strides 1 or 2: in windows, whose size the launch's own
// decides, since a record's outputs per thread cost reads that no tile gets back (see dw_window_for).  An LDS patch (two stages)
// and unequal strides are what the record says.  More windows than they are counted in, which takes padding of many times the
// image, go to the loop nest.
bool dw_in_registers(const DwArgs &g) { return g.stages == 1 && g.stride_h == g.stride_w && (g.stride_h == 1 || g.stride_h == 2) && g.x_bytes != 0; }

bool dw_windows(const DwArgs &g, int count, DwListEntry *e, DwWindow *w, int *vc)
{
    if (!dw_in_registers(g)) return false;
    *vc = g.C % 4 == 0 ? 4 : g.C % 2 == 0 ? 2 : 1;
    *w = dw_window_for((int64_t)g.planes / *vc * g.Ho * g.Wo * count, g.stride_h);
    return dw_entry(g, *vc, *w, e);
}

int launch_dwconv(const DwArgs &a, const PointerSets &sets, const tt_plan &plan, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (plan.variant_id < 0) return TT_ERR_UNSUPPORTED;
    DwListEntry e;
    DwWindow w;
    int vc;
    if (dw_windows(a, sets.count, &e, &w, &vc)) {
        e.x = a.x, e.w = a.w, e.bias = a.bias, e.y = a.y, e.first = 0;
        if (a.stride_h == 1) return vc == 4 ? launch_windows_of<1, 4>(w, e, sets, s) : vc == 2 ? launch_windows_of<1, 2>(w, e, sets, s) : launch_windows_of<1, 1>(w, e, sets, s);
        return vc == 4 ? launch_windows_of<2, 4>(w, e, sets, s) : vc == 2 ? launch_windows_of<2, 2>(w, e, sets, s) : launch_windows_of<2, 1>(w, e, sets, s);
    }
    if (dw_in_registers(a)) return launch_dw_direct(a, sets, kDwLargestDirect, stream);
    const dim3 grid(plan.grid, sets.count), block(plan.block);
    const int lds = plan.lds_bytes;
#define TT_DW_CASE(WM_, WN_)                                                                                         \
    if (a.wave_m == WM_ && a.wave_n == WN_) {                                                                        \
        constexpr int LIMIT = dw_block_limit(WM_, WN_, 1, 1, false);                                                 \
        if ((int)block.x > LIMIT) return TT_ERR_UNSUPPORTED;                                                         \
        const int bc = block.x <= 256 ? 0 : block.x <= 512 ? 1 : 2;                                                  \
        auto kern = dwconv3x3_kernel<WM_, WN_, 256>;                                                                 \
        if constexpr (LIMIT >= 512)                                                                                  \
            if (bc == 1) kern = dwconv3x3_kernel<WM_, WN_, 512>;                                                     \
        if constexpr (LIMIT >= 1024)                                                                                 \
            if (bc == 2) kern = dwconv3x3_kernel<WM_, WN_, 1024>;                                                    \
        static DynamicLdsLimit limits[3]; /* per kernel instance; host threads may launch concurrently */           \
        if (const int rc = limits[bc].raise_to(reinterpret_cast<const void *>(kern), lds); rc != TT_OK) return rc;   \
        hipLaunchKernelGGL(kern, grid, block, lds, s, a, sets);                                                      \
        return launched();                                                                                           \
    }
    TT_DW_CASE(1, 1) TT_DW_CASE(1, 2) TT_DW_CASE(1, 4) TT_DW_CASE(1, 7)
    TT_DW_CASE(2, 1) TT_DW_CASE(2, 2) TT_DW_CASE(2, 4) TT_DW_CASE(2, 7)
    TT_DW_CASE(4, 1) TT_DW_CASE(4, 2) TT_DW_CASE(4, 4) TT_DW_CASE(4, 7)
    TT_DW_CASE(7, 1) TT_DW_CASE(7, 2) TT_DW_CASE(7, 4) TT_DW_CASE(7, 7)
#undef TT_DW_CASE
    return TT_ERR_UNSUPPORTED;
}

DwWindow dw_list_window(int stride) { return stride == 1 ? kDwListWindow<1> : kDwListWindow<2>; }

bool dw_list_entry(const DwArgs &g, DwListEntry *e) { return dw_entry(g, 4, dw_list_window(g.stride_h), e); }

int launch_dw_list(DwList &list, int count, int stride, void *stream)
{
    int grid = 0;
    for (int i = 0; i < kMaxDwListed; ++i) {
        list.e[i].first = i < count ? grid : INT32_MAX;
        if (i < count) grid += (int)dw_workgroups(list.e[i]);
    }
    auto kern = stride == 1 ? dwconv3x3_list_kernel<1> : dwconv3x3_list_kernel<2>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream), list);
    return launched();
}

int launch_dw_direct(const DwArgs &a, const PointerSets &sets, int grid, void *stream)
{
    hipLaunchKernelGGL(dw_direct_kernel, dim3(grid, sets.count), dim3(256), 0, static_cast<hipStream_t>(stream), a, sets);
    return launched();
}

int launch_tile_map_dump(const TileMap &map, int32_t *out_dev, void *stream)
{
    const int grid = (map.grid + 255) / 256;
    hipLaunchKernelGGL(tile_map_dump_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream), map, out_dev);
    return launched();
}

} // namespace tt
