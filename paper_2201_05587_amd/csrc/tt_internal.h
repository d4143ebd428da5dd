// Internal declarations shared by the host code and the HIP kernels of libtt.
#pragma once

#include <stdint.h>

#include "tt.h"

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define TT_HD __host__ __device__ __forceinline__
#else
#define TT_HD inline
#endif

namespace tt {

constexpr int kXcds = 8;           // accelerator complex dies; workgroups are dealt to them round-robin
constexpr int kGroupM = 8;         // band height of raster order 2
constexpr int kLdsBudget = 160 * 1024;

enum Act { ACT_NONE = 0, ACT_RELU = 1, ACT_RELU6 = 2, ACT_GELU = 3 };

// Exact n / d for 0 <= n < 2^31 and 1 <= d < 2^31 by one widening multiply:
// magic = ceil(2^(31+shift) / d) with shift = ceil(log2 d) fits 32 bits, and the
// error n * (magic * d - 2^(31+shift)) / (d * 2^(31+shift)) stays below 1/d.
struct FastDiv {
    uint32_t magic, shift;
};
inline FastDiv make_fastdiv(uint32_t d)
{
    FastDiv f;
    f.shift = 0;
    while ((1ull << f.shift) < d) ++f.shift;
    const uint64_t pw = 1ull << (31 + f.shift);
    f.magic = (uint32_t)((pw + d - 1) / d);
    return f;
}
TT_HD uint32_t fast_div(uint32_t n, const FastDiv &f) { return (uint32_t)((((uint64_t)n * f.magic) >> 31) >> f.shift); }

// What a workgroup needs to find its tile: the integer fields of the plan the index map reads.
struct TileMap {
    int32_t sketch, order, grid;
    int32_t tiles_m, tiles_n, tile_m, tile_n, tile_k;
    int32_t M, N, K;
    int32_t eff_split_k, k_iters, k_tiles;
    // reciprocals of the map's divisors (a workgroup's first instructions; integer division is emulated
    // on the GPU): tiles_m * tiles_n, tiles_m, tiles_n, kGroupM * tiles_n, eff_split_k
    FastDiv div_tiles, div_m, div_n, div_band, div_split;
};

struct TileCoord {
    int32_t hi, lo;        // (batch, k-split); depthwise: (plane tile, 0)
    int32_t m0, m_ext, n0, n_ext, k0, k_ext;
};

// Workgroup id -> tile.  One implementation for the host mirror (tt_plan_tile) and every kernel.
TT_HD TileCoord decode_tile(const TileMap &p, int32_t wg)
{
    int32_t L = wg;
    if (p.order >= 3) {
        // XCD x receives workgroups x, x + 8, ...: give it one contiguous run of logical ids.
        const int32_t per = p.grid / kXcds, rem = p.grid % kXcds;
        const int32_t x = wg % kXcds, j = wg / kXcds;
        L = x * per + (x < rem ? x : rem) + j;
    }
    const int32_t T = p.tiles_m * p.tiles_n;
    const int32_t slab = (int32_t)fast_div((uint32_t)L, p.div_tiles), t = L - slab * T;
    const int32_t base = p.order % 3;
    int32_t im, in;
    if (base == 0) {
        in = (int32_t)fast_div((uint32_t)t, p.div_m);
        im = t - in * p.tiles_m;
    } else if (base == 1) {
        im = (int32_t)fast_div((uint32_t)t, p.div_n);
        in = t - im * p.tiles_n;
    } else {
        const int32_t width = kGroupM * p.tiles_n;
        const int32_t band = (int32_t)fast_div((uint32_t)t, p.div_band);
        const int32_t first = band * kGroupM, at = t - band * width;
        const int32_t left = p.tiles_m - first;
        if (left >= kGroupM) {
            in = at / kGroupM;
            im = first + at % kGroupM;
        } else { // the last, lower band
            in = at / left;
            im = first + at % left;
        }
    }
    TileCoord c;
    c.m0 = im * p.tile_m;
    c.n0 = in * p.tile_n;
    c.m_ext = (p.M - c.m0) < p.tile_m ? (p.M - c.m0) : p.tile_m;
    c.n_ext = (p.N - c.n0) < p.tile_n ? (p.N - c.n0) : p.tile_n;
    if (p.sketch == TT_SK_DWCONV) {
        c.hi = slab;
        c.lo = 0;
        c.k0 = slab * p.tile_k;
        c.k_ext = (p.K - c.k0) < p.tile_k ? (p.K - c.k0) : p.tile_k;
    } else if (p.sketch == TT_SK_GEMV) {
        c.hi = slab;
        c.lo = 0;
        c.k0 = 0;
        c.k_ext = p.K;
    } else {
        c.hi = (int32_t)fast_div((uint32_t)slab, p.div_split);
        c.lo = slab - c.hi * p.eff_split_k;
        const int32_t kt0 = c.lo * p.k_iters;
        int32_t kt1 = kt0 + p.k_iters;
        if (kt1 > p.k_tiles) kt1 = p.k_tiles;
        c.k0 = kt0 * p.tile_k;
        const int32_t kend = kt1 * p.tile_k < p.K ? kt1 * p.tile_k : p.K;
        c.k_ext = kend - c.k0;
    }
    return c;
}

// Element of the residual (and the output) at which a lane fetches its vector of a pass: its own where the lane is
// `live` (row m, columns from `first`, inside the matrix), else the first one of its tile, whose value nobody uses: the
// tile must start inside the matrix.
TT_HD int64_t residual_element(const TileCoord &tc, int32_t M, int32_t N, bool live, int32_t m, int32_t first)
{
    return (int64_t)tc.hi * M * N + (int64_t)(live ? m : tc.m0) * N + (live ? first : tc.n0);
}

// Quadrant (h, k) of a 256 x 256 block, as a tile of its own; false where it lies outside the matrix (a last block of at
// most 128 rows or columns).
TT_HD bool block_quadrant(const TileCoord &block, int32_t M, int32_t N, int32_t h, int32_t k, TileCoord *quadrant)
{
    *quadrant = block;
    quadrant->m0 = block.m0 + h * 128;
    quadrant->n0 = block.n0 + k * 128;
    return quadrant->m0 < M && quadrant->n0 < N;
}

inline TileMap tile_map_of(const tt_plan &pl)
{
    TileMap m;
    m.sketch = pl.sketch;
    m.order = pl.order;
    m.grid = pl.grid;
    m.tiles_m = pl.tiles_m;
    m.tiles_n = pl.tiles_n;
    m.tile_m = pl.tile_m;
    m.tile_n = pl.tile_n;
    m.tile_k = pl.tile_k;
    m.M = pl.M;
    m.N = pl.N;
    m.K = pl.K;
    m.eff_split_k = pl.eff_split_k;
    m.k_iters = pl.k_iters;
    m.k_tiles = pl.k_tiles;
    const auto at_least_one = [](int32_t v) { return (uint32_t)(v > 0 ? v : 1); };
    m.div_tiles = make_fastdiv(at_least_one(pl.tiles_m * pl.tiles_n));
    m.div_m = make_fastdiv(at_least_one(pl.tiles_m));
    m.div_n = make_fastdiv(at_least_one(pl.tiles_n));
    m.div_band = make_fastdiv(at_least_one(kGroupM * pl.tiles_n));
    m.div_split = make_fastdiv(at_least_one(pl.eff_split_k));
    return m;
}

// Operand families of the matrix-core contraction kernel.
enum Family {
    FAM_CONV = 0,    // A = NHWC activations gathered as an implicit GEMM, B = KRSC filters ([N][K])
    FAM_GEMM_TN = 1, // A = [M][K], B = [N][K] (dense; batch matmul with trans_b = 1; unit-stride 1x1 conv)
    FAM_GEMM_NN = 2  // A = [M][K], B = [K][N] (batch matmul with trans_b = 0)
};

// The tensors of one operator call as a kernel sees them, and the sets a launch carries beyond the first: workgroups
// (x, y) work on set y, so that several calls of one plan go out as one launch (see tt_run_kernels).  The first set's
// pointers stay with the other arguments: a lone call reads no further lines of them.
struct PointerSet {
    const void *a, *b, *bias, *res;
    void *out;
    float *ws;
};
constexpr int kMaxSets = TT_MAX_ENTRIES_PER_LAUNCH;
struct PointerSets {
    PointerSet more[kMaxSets - 1];
    int32_t count;
};

// Everything a contraction kernel (matrix-core, direct or split-K reduce) needs, passed by value.
struct ContractArgs {
    const void *a, *b, *bias, *res;
    void *out;
    float *ws;
    TileMap map;
    int32_t batch, M, N, K;
    // FAM_CONV: the extent of the reduction as the gathering loaders walk it, R * runp >= K (see below);
    // the split of the reduction that ends at K runs on to k_walk
    int32_t k_walk;
    // convolution geometry (FAM_CONV).  The reduction index is k = r * runp + j: filter row r and
    // position j inside the run of S * C elements that one filter row covers contiguously in an
    // NHWC image row (and in a KRSC filter); runp is the run rounded up to whole 16-byte items.
    int32_t C, H, W, R, S, stride_h, stride_w, pad_h, pad_w, Ho, Wo;
    int32_t run, runp;
    FastDiv div_hw, div_wo; // output pixel index -> (image, row, column)
    FastDiv div_run;        // position in the walked reduction -> (filter row, position in the run): by runp
    // padded image geometry of the patch kernel: PW = W + 2 pad_w, PHW = (H + 2 pad_h) * PW
    int32_t PW, PHW;
    FastDiv div_phw, div_pw; // flat padded pixel index -> (image, padded row, padded column)
    uint32_t a_bytes, b_bytes; // sizes of the activation and filter tensors (bounds of the gathering loads)
    int32_t eff_vec_a, eff_vec_b, eff_vec_c, stages, unroll, act, has_bias, has_res, dtype;
};

// ---- launches of entries of different shapes (contract_list.hip.h, run_list.cpp) ----------------------
// What a contraction tile needs of its entry; the launch has the tile, the data type and the operand family.
struct ListEntry {
    const void *a, *b, *bias, *res; // bias, res: null where the entry has none
    void *out;
    float *ws;
    int32_t M, N, K, batch;
    int32_t grid, tiles_m, tiles_n, k_iters, k_tiles, splits;
    FastDiv div_tiles, div_n, div_split;
    int32_t C, H, W, R, S, Ho, Wo, stride_h, stride_w, pad_h, pad_w;
    FastDiv div_hw, div_wo;
    uint32_t a_bytes, b_bytes;
    int16_t vec_c, act;
};
constexpr int kMaxListed = 20;  // entries of a launch: the arguments stay within 4 KB
constexpr int kMaxListTiles = 16; // tiles of the list rule
constexpr int kListOrder = 4;   // raster of every entry: columns fastest, a contiguous run of tiles per XCD
struct ContractList {
    int32_t first[kMaxListed]; // first workgroup of every entry, a multiple of the number of XCDs; past the last: INT32_MAX
    ListEntry e[kMaxListed];
};
static_assert(sizeof(ContractList) <= 4096, "");
struct ListTile {
    int32_t dtype, tile_m, tile_n, tile_k;
    float fixed_us, per_k_us, alone_per_k_us; // see list_tiles
    bool blocks;                              // the block kernel, which asks for more (block_tile_fits)
    int (*launch[2])(const ContractList &list, int grid, void *stream); // FAM_CONV, FAM_GEMM_TN
};
const ListTile *list_tiles(int *count);

// Single-precision contractions with a short reduction (contract_thin.hip.h): what the kernel needs of an entry.
struct ThinEntry {
    const float *a, *b, *bias, *res; // bias, res: null where the entry has none
    float *out;
    int32_t M, N, K;
    int32_t rows, columns, chunks; // of a workgroup; workgroups side by side
    int32_t act;
};
constexpr int kMaxThin = 48;
struct ThinList {
    int32_t first[kMaxThin]; // first workgroup; past the last entry: INT32_MAX
    ThinEntry e[kMaxThin];
};
static_assert(sizeof(ThinList) <= 4096, "");
constexpr int kThinPieces[] = {2, 6}; // instances: 16-element pieces of the reduction
// Lays out rows and columns of an entry whose sizes are set, and launches `count` of them on the instance of `pieces`.
void thin_layout(ThinEntry *e);
inline int64_t thin_workgroups(const ThinEntry &e) { return (int64_t)e.chunks * ((e.M + e.rows - 1) / e.rows); }
int launch_thin_list(ThinList &list, int count, int pieces, void *stream);

// What the second step of a split reduction needs of its entry.
struct ReduceEntry {
    const float *ws;
    const void *bias, *res; // null where the entry has none
    void *out;
    int64_t total;          // outputs; also the distance between the partial sums of two splits
    int32_t N, splits, act;
    int32_t first;          // first workgroup of the entry; past the last: INT32_MAX
};
constexpr int kMaxReduced = 64;
struct ReduceList {
    ReduceEntry e[kMaxReduced];
};
static_assert(sizeof(ReduceList) <= 4096, "");
// (`count` entries of one data type; all of rows of whole fours, or all element by element)
int launch_reduce_list(ReduceList &list, int count, int dtype, bool fours, void *stream);

struct DwArgs {
    const float *x, *w, *bias;
    float *y;
    TileMap map;
    int32_t planes, C, H, W, Ho, Wo, stride_h, stride_w, pad_h, pad_w;
    int32_t wave_m, wave_n, stages, unroll;
    int32_t eff_vec;   // channel-contiguous planes per lane (1, 2 or 4)
    uint32_t x_bytes;  // size of the input tensor when it is below 2 GiB, else 0
};

// A depthwise entry in windows of outputs, alone or beside others of different shapes (simple_kernels.hip).
struct DwWindow {
    int32_t rows, columns;
};
struct DwListEntry {
    const float *x, *w, *bias; // bias may be null
    float *y;
    int32_t first;             // first workgroup, a multiple of the number of XCDs; past the last entry: INT32_MAX
    int32_t threads, C, H, W, Ho, Wo, pad_h, pad_w;
    uint32_t x_bytes;
    FastDiv div_c, div_cols, div_rows; // by the threads along C, the columns and the rows of a plane
};
constexpr int kMaxDwListed = 36;
struct DwList {
    DwListEntry e[kMaxDwListed];
};
static_assert(sizeof(DwList) <= 4096, "");
// Depthwise plans that windows are for, and workgroups of the loop nest for those of them that have too many (2^31 threads: the
// runtime takes less than 2^32).
bool dw_in_registers(const DwArgs &g);
constexpr int kDwLargestDirect = 1 << 23;
// Whether a launch of `count` entries runs in windows: the entry without its pointers, the window and the channels of a thread.
bool dw_windows(const DwArgs &g, int count, DwListEntry *e, DwWindow *w, int *vc);
// Fills in the part of an entry that the launch decides on; false: the entry is not one for a list (C not a multiple of four).
bool dw_list_entry(const DwArgs &g, DwListEntry *e);
inline int64_t dw_workgroups(const DwListEntry &e) { return ((e.threads + 255ll) / 256 + kXcds - 1) / kXcds * kXcds; }
// The outputs that a thread of a list forms (of four channels).
DwWindow dw_list_window(int stride);
int launch_dw_list(DwList &list, int count, int stride, void *stream);

TT_HD ContractArgs with_set(ContractArgs g, const PointerSets &sets, uint32_t set)
{
    if (set == 0) return g;
    const PointerSet &p = sets.more[set - 1];
    g.a = p.a;
    g.b = p.b;
    g.bias = p.bias;
    g.res = p.res;
    g.out = p.out;
    g.ws = p.ws;
    return g;
}
TT_HD DwArgs with_set(DwArgs g, const PointerSets &sets, uint32_t set)
{
    if (set == 0) return g;
    const PointerSet &p = sets.more[set - 1];
    g.x = static_cast<const float *>(p.a);
    g.w = static_cast<const float *>(p.b);
    g.bias = static_cast<const float *>(p.bias);
    g.y = static_cast<float *>(p.out);
    return g;
}

// The device tensors of one operator call (conv: x, w, bias, residual, y; dense and depthwise without a residual;
// batch matmul without bias and residual) and the split-K workspace.
struct OpPointers {
    const void *a, *b, *bias, *res;
    void *out, *ws;
    size_t ws_bytes;
};

// A kernel under a record, laid out once: the plan and the launch arguments without the pointers.
struct PreparedOp {
    tt_plan plan;   // of the record
    tt_plan launch; // what is launched for it (ops.hip, launch_plan_of)
    int32_t cls, family;
    bool supported; // false: a valid plan that the entry point refuses (TT_ERR_UNSUPPORTED)
    int64_t a_bytes, b_bytes, bias_bytes, out_bytes; // sizes of the tensors (a residual is as large as the output)
    ContractArgs g; // every class but the depthwise one
    DwArgs d;
};

// The operator entry points in three steps (ops.hip): argument check, plan and launch arguments (record NULL = the
// default), launch of 1..kMaxSets calls (all with a bias or all without).  A caller that launches a kernel
// repeatedly, or needs the plan's workspace size, does the second step once.
int check_op_pointers(int cls, const OpPointers &p);
int prepare_op(const tt_schedule *sched, int cls, const void *shape, PreparedOp *op);
int launch_op(PreparedOp &op, const OpPointers *calls, int count, void *stream);
bool workspace_fits(const PreparedOp &op, const OpPointers &p);

// The tensors of a kernel description, set `turn` of those it has (run_list.cpp).
OpPointers pointers_of(const tt_kernel_desc &k, int64_t turn = 0);
// Same knobs: the thirteen that lead the record.
bool same_knobs(const tt_schedule &x, const tt_schedule &y);

// What runs a launch (tt_launch_kernel), and the grid (of one pointer set), workgroup and LDS it has.
struct LaunchShape {
    int32_t kernel, grid, block, lds_bytes;
};

struct Variant {
    int32_t dtype, family, tile_m, tile_n, tile_k, wave_m, wave_n, mfma;
    int32_t amode; // conv family: bytes per gathered load (16 or the element size); 0 otherwise
    int32_t pipe;  // 0: register-staged loads, 1 or 2 LDS stages; 1: asynchronous loads into a ring of 3 or 4;
                   // 2: 3x3 conv with the padded input patch in LDS and a filter ring of 3 or 4 (stages 5 or 6)
                   // 3: persistent dense kernel, the B panel resident in LDS and two A buffers (stages 7)
    int32_t stride; // pipe 2: the convolution stride the kernel is compiled for; 0 otherwise
    int (*launch)(const ContractArgs &args, const PointerSets &sets, int grid, int lds_bytes, void *stream);
    LaunchShape (*shape)(const ContractArgs &args, int count, int grid, int lds_bytes); // of a launch of `count` sets; pipes
                                                                                        // 2 and 3: null, the plan's own
    int (*stage_bytes)();        // pipes 0, 1: LDS bytes of one pipeline stage; pipe 2: pixels a patch buffer holds;
                                 // pipe 3: request instructions per lane and K slice
    int (*lds_bytes)(int stages); // LDS bytes for a plan's number of stages (pipe 3: for its number of K slices), as
                                  // the compiled kernel lays LDS out
};

// Reduction elements one 16-byte operand fragment per lane feeds to the matrix cores: a block of MF rows
// leaves 64 / MF lane groups along K, each holding 16 bytes.  tile_k must be a multiple of it.
constexpr int k_granule(int dtype, int mfma) { return (dtype == TT_F32 ? 4 : 8) * (64 / mfma); }

// variant table (generated) and lookups
extern const Variant kVariants[];
extern const int kNumVariants;
int find_variant(int dtype, int family, int tm, int tn, int tk, int wm, int wn, int mf, int amode, int pipe,
                 int stride = 0);
int family_of(int cls, int trans_b);

// launchers of the non-matrix-core kernels (simple_kernels.hip)
int64_t direct_workgroups(const ContractArgs &args, int family, int count); // of one of `count` pointer sets
int launch_direct(const ContractArgs &args, const PointerSets &sets, int family, void *stream);
int launch_splitk_reduce(const ContractArgs &args, const PointerSets &sets, int family, void *stream);
int launch_gemv(const ContractArgs &args, const PointerSets &sets, const tt_plan &plan, void *stream);
// the 256 x 256 block kernel (contract_block.hip): whether a launch of `count` sets runs on it, and its launch
bool block_applies(const ContractArgs &args, int family, int count, int tile_outputs);
int launch_blocks(const ContractArgs &args, const PointerSets &sets, int family, void *stream);
LaunchShape blocks_shape(const ContractArgs &args, int family);
// the convolution kernel with the input rows of a tile in LDS (conv_rows.hip): its launch of `count` sets for element-wise
// gathers (a grid of 0: it does not apply)
LaunchShape rows_shape(const ContractArgs &args, int count);
int launch_conv_rows(const ContractArgs &args, const PointerSets &sets, void *stream);
int dw_max_block(int wave_m, int wave_n, int planes_per_lane, int stride, bool in_registers);
int launch_dwconv(const DwArgs &args, const PointerSets &sets, const tt_plan &plan, void *stream);
int launch_dw_direct(const DwArgs &args, const PointerSets &sets, int grid, void *stream);
int launch_tile_map_dump(const TileMap &map, int32_t *out_dev, void *stream);

// Compute units of the current device (asked once; one device per process).
int compute_units();

// Remember the text of a failed HIP call for tt_last_error(); returns TT_ERR_HIP.
int note_hip_error(int hip_error_code, const char *where);

inline int act_of_class(int cls)
{
    switch (cls) {
    case TT_CONV2D_BIAS_RELU:
    case TT_CONV2D_BIAS_ADD_RELU:
    case TT_DENSE_BIAS_RELU:
        return ACT_RELU;
    case TT_CONV2D_BIAS_RELU6:
    case TT_DWCONV_BIAS_RELU6:
        return ACT_RELU6;
    case TT_DENSE_BIAS_GELU:
        return ACT_GELU;
    default:
        return ACT_NONE;
    }
}

inline bool is_conv_class(int cls) { return cls >= TT_CONV2D_ADD && cls <= TT_CONV2D_BIAS_RELU6; }
inline bool is_dense_class(int cls) { return cls >= TT_DENSE_ADD && cls <= TT_DENSE_BIAS_GELU; }

} // namespace tt
