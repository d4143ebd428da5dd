// C-ABI operator entry points, standalone pair timing and the transfer-tuning sweep.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "tt_internal.h"

using namespace tt;

namespace tt {
static thread_local char g_last_error[256] = "";
int note_hip_error(int code, const char *where)
{
    snprintf(g_last_error, sizeof g_last_error, "%s: %s (%d)", where, hipGetErrorString((hipError_t)code), code);
    return TT_ERR_HIP;
}
} // namespace tt

namespace tt {
// Compute units of the current device (asked once; one device per process).
int compute_units()
{
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return n;
    }();
    return cus;
}
} // namespace tt

extern "C" const char *tt_last_error(void) { return tt::g_last_error; }

namespace {

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int conv_out(int in, int f, int stride, int pad) { return (in + 2 * pad - f) / stride + 1; }

// Estimated time (us) of a launch in tiles of tm x tn: a CU takes in 80 GB/s of operand rows and multiplies at 1/256 of
// the rate a large product reaches (bf16 1450, f32 147 TFLOP/s); workgroups beyond one per CU share both.  Tiles of 32 x 32
// take a quarter longer than that (16 x 16 wave tiles read two LDS fragments per product).
double tile_estimate(const tt_plan &p, int dtype, int tm, int tn)
{
    const double tiles = (double)p.batch * ((p.M + tm - 1) / tm) * ((p.N + tn - 1) / tn);
    const double rows = (tm + tn) * (dtype == TT_F32 ? 4.0 : 2.0) / 80e3;
    const double products = 2.0 * tm * tn / (dtype == TT_F32 ? 0.57e6 : 5.65e6);
    return std::ceil(tiles / compute_units()) * p.K * std::max(rows, products) * (tm * tn <= 1024 ? 1.25 : 1.0);
}

// The plan that is launched for a record's plan.  The default schedule of a kernel stands for "as the library sees fit": its
// record names a register-pipeline tile, and where the asynchronous ring can load the operands it is run on the ring
// instance that the estimate above likes best for this shape, whether the caller passed no record or the default's own.
// Any other record runs in the tile, raster and pipeline that it names, so that a search times what it will store.
// Splits of the reduction keep their own kernel: their partial sums are cut where the record says.
// The register pipeline holds one slice in flight, in registers.  Default records, before -> after (us): bf16 dense
// 73x168x3152 46.9 -> 7.1, f32 dense 77x40x1040 42.7 -> 9.4, f32 3x3 392 -> 104 channels on 2 x 15x15 133 -> 25.7, bf16 1x1
// 152 -> 440 on 13x13 5.4 -> 3.5; the geometric mean over 60 shapes drawn between 2 MFLOP and 60 GFLOP is 2.1 times.
tt_plan launch_plan_of(const tt_plan &plan, const tt_schedule &rec, int cls, const void *shape, int dtype)
{
    if (plan.sketch != TT_SK_MFMA || plan.variant_id < 0 || plan.stages > 2 || plan.eff_split_k != 1) return plan;
    tt_schedule def;
    if (tt_schedule_default(cls, shape, &def) != TT_OK || !same_knobs(rec, def)) return plan;
    static const int tiles[2][6][6] = {
        // tile_m, tile_n, tile_k, wave_m, wave_n, mfma
        {{32, 32, 32, 16, 16, 16}, {64, 64, 32, 32, 32, 16}, {128, 64, 32, 32, 32, 16}, {64, 128, 32, 32, 32, 16}, {128, 128, 32, 32, 64, 16}, {}},
        {{32, 32, 64, 16, 16, 16}, {64, 64, 64, 32, 32, 16}, {128, 64, 64, 32, 32, 16}, {64, 128, 128, 32, 32, 16}, {128, 128, 64, 32, 64, 32}, {128, 256, 64, 32, 64, 16}},
    };
    tt_plan best = plan;
    double best_us = 1e30;
    for (const auto &t : tiles[dtype == TT_F32 ? 0 : 1]) {
        if (!t[0]) continue;
        const double us = tile_estimate(plan, dtype, t[0], t[1]);
        if (us >= best_us) continue;
        tt_schedule r;
        std::memset(&r, 0, sizeof r);
        r.cls = cls, r.sketch = TT_SK_MFMA;
        r.tile_m = t[0], r.tile_n = t[1], r.tile_k = t[2], r.wave_m = t[3], r.wave_n = t[4], r.mfma = t[5];
        r.split_k = 1, r.order = 4, r.vec = dtype == TT_F32 ? 4 : 8, r.unroll = 8, r.stages = 3;
        tt_plan p;
        if (tt_schedule_apply(&r, cls, shape, 0, &p) != TT_OK || p.stages != 3 || p.variant_id < 0) continue;
        best = p;
        best_us = us;
    }
    return best;
}

void fill_common(ContractArgs &g, const tt_plan &plan, int cls, int dtype)
{
    g.map = tile_map_of(plan);
    g.batch = plan.batch;
    g.M = plan.M;
    g.N = plan.N;
    g.K = plan.K;
    g.eff_vec_a = plan.eff_vec_a;
    g.eff_vec_b = plan.eff_vec_b;
    g.eff_vec_c = plan.eff_vec_c;
    g.stages = plan.stages;
    g.unroll = plan.eff_unroll;
    g.act = act_of_class(cls);
    g.dtype = dtype;
}

int run_contraction(const ContractArgs &g, const PointerSets &sets, const tt_plan &plan, int family, void *stream)
{
    switch (plan.sketch) {
    case TT_SK_DIRECT:
        return launch_direct(g, sets, family, stream);
    case TT_SK_GEMV:
        return launch_gemv(g, sets, plan, stream);
    case TT_SK_MFMA: {
        if (plan.variant_id < 0 || plan.variant_id >= kNumVariants) return TT_ERR_UNSUPPORTED;
        const int rc = kVariants[plan.variant_id].launch(g, sets, plan.grid, plan.lds_bytes, stream);
        if (rc != TT_OK) return rc;
        if (plan.eff_split_k > 1) return launch_splitk_reduce(g, sets, family, stream);
        return TT_OK;
    }
    default:
        return TT_ERR_UNSUPPORTED;
    }
}

void prepare_conv(const tt_conv_shape &s, PreparedOp *op)
{
    const tt_plan &plan = op->launch;
    // the matrix-core kernels address both tensors with 32-bit byte offsets below 2^31 and keep one
    // bit per filter row
    const int elem = s.dtype == TT_F32 ? 4 : 2;
    const int64_t x_bytes = op->a_bytes, w_bytes = op->b_bytes;
    op->supported = !(plan.sketch == TT_SK_MFMA && (x_bytes >= (1ll << 31) || w_bytes >= (1ll << 31) || s.r > 32));
    ContractArgs &g = op->g;
    fill_common(g, plan, op->cls, s.dtype);
    g.C = s.c;
    g.H = s.h;
    g.W = s.w;
    g.R = s.r;
    g.S = s.s;
    g.stride_h = s.stride_h;
    g.stride_w = s.stride_w;
    g.pad_h = s.pad_h;
    g.pad_w = s.pad_w;
    g.Ho = conv_out(s.h, s.r, s.stride_h, s.pad_h);
    g.Wo = conv_out(s.w, s.s, s.stride_w, s.pad_w);
    const int per_item = 16 / elem;
    g.run = s.s * s.c;
    g.runp = (g.run + per_item - 1) / per_item * per_item;
    g.k_walk = s.r * g.runp;
    g.div_hw = make_fastdiv((uint32_t)(g.Ho * g.Wo));
    g.div_wo = make_fastdiv((uint32_t)g.Wo);
    g.div_run = make_fastdiv((uint32_t)g.runp);
    g.PW = s.w + 2 * s.pad_w;
    g.PHW = (s.h + 2 * s.pad_h) * g.PW;
    g.div_phw = make_fastdiv((uint32_t)g.PHW);
    g.div_pw = make_fastdiv((uint32_t)g.PW);
    g.a_bytes = (uint32_t)x_bytes;
    g.b_bytes = (uint32_t)w_bytes;
    op->family = FAM_CONV;
    if (plan.sketch == TT_SK_MFMA && plan.variant_id >= 0 && plan.variant_id < kNumVariants)
        op->family = kVariants[plan.variant_id].family; // the dense family for unit-stride 1x1 filters
}

void prepare_dw(const tt_conv_shape &s, PreparedOp *op)
{
    const tt_plan &plan = op->plan;
    op->supported = s.dtype == TT_F32 && s.r == 3 && s.s == 3;
    DwArgs &g = op->d;
    g.map = tile_map_of(plan);
    g.planes = s.n * s.c;
    g.C = s.c;
    g.H = s.h;
    g.W = s.w;
    g.Ho = plan.M;
    g.Wo = plan.N;
    g.stride_h = s.stride_h;
    g.stride_w = s.stride_w;
    g.pad_h = s.pad_h;
    g.pad_w = s.pad_w;
    g.wave_m = plan.wave_m;
    g.wave_n = plan.wave_n;
    g.stages = plan.stages;
    g.unroll = plan.eff_unroll;
    g.eff_vec = plan.eff_vec_a;
    g.x_bytes = op->supported && op->a_bytes < (1ll << 31) ? (uint32_t)op->a_bytes : 0u;
}

} // namespace

namespace tt {

int prepare_op(const tt_schedule *sched, int cls, const void *shape, PreparedOp *op)
{
    tt_schedule def;
    if (!sched) {
        const int rc = tt_schedule_default(cls, shape, &def);
        if (rc != TT_OK) return rc;
        sched = &def;
    }
    const int rc = tt_schedule_apply(sched, cls, shape, 0, &op->plan);
    if (rc != TT_OK) return rc;
    op->cls = cls;
    op->supported = true;
    op->launch = op->plan;
    const bool image = is_conv_class(cls) || cls == TT_DWCONV_BIAS_RELU6;
    const tt_conv_shape *cs = static_cast<const tt_conv_shape *>(shape);
    const tt_gemm_shape *gs = static_cast<const tt_gemm_shape *>(shape);
    const int64_t elem = (image ? cs->dtype : gs->dtype) == TT_F32 ? 4 : 2;
    if (image) {
        const int64_t pixels = (int64_t)cs->n * conv_out(cs->h, cs->r, cs->stride_h, cs->pad_h) *
                               conv_out(cs->w, cs->s, cs->stride_w, cs->pad_w);
        op->a_bytes = (int64_t)cs->n * cs->h * cs->w * cs->c * elem;
        op->b_bytes = (int64_t)cs->k * cs->r * cs->s * (cls == TT_DWCONV_BIAS_RELU6 ? 1 : cs->c) * elem;
        op->bias_bytes = cs->k * elem;
        op->out_bytes = pixels * cs->k * elem;
    } else {
        op->a_bytes = (int64_t)gs->batch * gs->m * gs->k * elem;
        op->b_bytes = (int64_t)gs->batch * gs->n * gs->k * elem;
        op->bias_bytes = gs->n * elem;
        op->out_bytes = (int64_t)gs->batch * gs->m * gs->n * elem;
    }
    std::memset(&op->g, 0, sizeof op->g);
    if (cls == TT_DWCONV_BIAS_RELU6) {
        std::memset(&op->d, 0, sizeof op->d);
        prepare_dw(*cs, op);
    } else if (is_conv_class(cls)) {
        op->launch = launch_plan_of(op->plan, *sched, cls, shape, cs->dtype);
        prepare_conv(*cs, op);
    } else {
        op->launch = launch_plan_of(op->plan, *sched, cls, shape, gs->dtype);
        fill_common(op->g, op->launch, cls, gs->dtype);
        op->g.Ho = op->g.Wo = 1;
        op->family = family_of(cls, gs->trans_b);
    }
    return TT_OK;
}

int check_op_pointers(int cls, const OpPointers &p)
{
    if (!p.a || !p.b || !p.out) return TT_ERR_BAD_ARG;
    if (!aligned16(p.a) || !aligned16(p.b) || !aligned16(p.out) || !aligned16(p.bias) || !aligned16(p.res))
        return TT_ERR_BAD_ARG;
    if (is_conv_class(cls) && (cls == TT_CONV2D_BIAS_ADD_RELU) != (p.res != nullptr)) return TT_ERR_BAD_ARG;
    return TT_OK;
}

bool workspace_fits(const PreparedOp &op, const OpPointers &p)
{
    return op.plan.workspace_bytes == 0 || (p.ws && (int64_t)p.ws_bytes >= op.plan.workspace_bytes && aligned16(p.ws));
}

int launch_op(PreparedOp &op, const OpPointers *calls, int count, void *stream)
{
    PointerSets sets;
    sets.count = count;
    for (int i = 0; i < count; ++i) {
        const OpPointers &p = calls[i];
        if (!workspace_fits(op, p)) return TT_ERR_WORKSPACE;
        if (i > 0) sets.more[i - 1] = {p.a, p.b, p.bias, p.res, p.out, static_cast<float *>(p.ws)};
    }
    if (!op.supported) return TT_ERR_UNSUPPORTED;
    const OpPointers &first = calls[0];
    if (op.cls == TT_DWCONV_BIAS_RELU6) {
        DwArgs &d = op.d;
        d.x = static_cast<const float *>(first.a);
        d.w = static_cast<const float *>(first.b);
        d.bias = static_cast<const float *>(first.bias);
        d.y = static_cast<float *>(first.out);
        if (op.plan.sketch == TT_SK_DIRECT) return launch_dw_direct(d, sets, op.plan.grid, stream);
        return launch_dwconv(d, sets, op.plan, stream);
    }
    ContractArgs &g = op.g;
    g.a = first.a;
    g.b = first.b;
    g.bias = first.bias;
    g.res = first.res;
    g.out = first.out;
    g.ws = static_cast<float *>(first.ws);
    g.has_bias = first.bias != nullptr;
    g.has_res = first.res != nullptr;
    return run_contraction(g, sets, op.launch, op.family, stream);
}

} // namespace tt

namespace {

int run_op(const tt_schedule *sched, int cls, const void *shape, const OpPointers &p, void *stream)
{
    if (const int rc = check_op_pointers(cls, p); rc != TT_OK) return rc;
    PreparedOp op;
    if (const int rc = prepare_op(sched, cls, shape, &op); rc != TT_OK) return rc;
    return launch_op(op, &p, 1, stream);
}

} // namespace

// ---- what a launch runs on -----------------------------------------------------------------------------

namespace {

// Whether a launch of `count` sets is a depthwise one in windows: its record's stages and strides allow them, and the operator
// takes the record.
bool in_windows(const PreparedOp &op, int count, DwListEntry *e, DwWindow *w, int *vc)
{
    return op.launch.sketch == TT_SK_DWCONV && op.launch.variant_id >= 0 && dw_windows(op.d, count, e, w, vc);
}

// The kernel of a launch of `count` sets, and the plan as it is launched there.
int launched_plan(const PreparedOp &op, int count, tt_plan *plan)
{
    *plan = op.launch;
    DwListEntry windows;
    DwWindow w;
    int vc;
    if (in_windows(op, count, &windows, &w, &vc)) {
        plan->grid = (int32_t)dw_workgroups(windows), plan->block = 256;
        plan->wave_m = w.rows, plan->wave_n = w.columns, plan->eff_vec_a = plan->eff_vec_c = vc;
        return TT_LAUNCH_RECORD;
    }
    if (plan->sketch == TT_SK_DWCONV && plan->variant_id >= 0 && dw_in_registers(op.d))
        plan->sketch = TT_SK_DIRECT, plan->grid = kDwLargestDirect, plan->block = 256;
    if (plan->sketch == TT_SK_DIRECT && op.cls != TT_DWCONV_BIAS_RELU6) plan->grid = (int32_t)direct_workgroups(op.g, op.family, count);
    if (plan->sketch != TT_SK_MFMA || plan->variant_id < 0 || plan->variant_id >= kNumVariants) return TT_LAUNCH_RECORD;
    const Variant &v = kVariants[plan->variant_id];
    if (!v.shape) return TT_LAUNCH_RECORD;
    const LaunchShape s = v.shape(op.g, count, plan->grid, plan->lds_bytes);
    plan->grid = s.grid;
    plan->block = s.block;
    plan->lds_bytes = s.lds_bytes;
    return s.kernel;
}

} // namespace

extern "C" int tt_debug_launch(const tt_schedule *sched, int cls, const void *shape, int count, tt_plan *launched, int32_t *kernel)
{
    if (!shape || !launched || !kernel || count < 1 || count > kMaxSets) return TT_ERR_BAD_ARG;
    if (cls < 0 || cls >= TT_NUM_CLASSES) return TT_ERR_BAD_ARG;
    PreparedOp op;
    if (const int rc = prepare_op(sched, cls, shape, &op); rc != TT_OK) return rc;
    if (!op.supported || (op.launch.sketch != TT_SK_DIRECT && op.launch.variant_id < 0)) return TT_ERR_UNSUPPORTED;
    *kernel = launched_plan(op, count, launched);
    return TT_OK;
}

// ---- split-K partial sums without a caller's workspace ----------------------------------------------
// One array per GPU, part of the library's code object: it exists from the moment the library is loaded
// on a device until the process ends.  In host code the array's name is only a handle; the address the
// kernels get comes from hipGetSymbolAddress, asked for once per device with that device current.
static __device__ __align__(256) unsigned char scratch[TT_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kMaxDevices = 64;

int static_workspace(void **ptr)
{
    static std::mutex guard;
    static void *per_device[kMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return note_hip_error((int)e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return TT_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(guard);
    if (!per_device[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return note_hip_error((int)e, "hipGetSymbolAddress(scratch)");
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    return TT_OK;
}

} // namespace

extern "C" int tt_conv2d_bias_relu_noalloc(const void *x, const void *w, const void *bias, const void *residual,
                                           void *y, const tt_conv_shape *shape, int cls, const tt_schedule *sched,
                                           void *stream)
{
    void *ws = nullptr;
    if (const int rc = static_workspace(&ws); rc != TT_OK) return rc;
    const int rc = tt_conv2d_bias_relu(x, w, bias, residual, y, shape, cls, sched, ws, TT_STATIC_WORKSPACE_BYTES, stream);
    if (rc == TT_ERR_WORKSPACE)
        snprintf(tt::g_last_error, sizeof tt::g_last_error,
                 "tt_conv2d_bias_relu_noalloc: the split-K partial sums of this (schedule, shape) exceed the "
                 "library's static workspace of %d bytes", (int)TT_STATIC_WORKSPACE_BYTES);
    return rc;
}

extern "C" int tt_conv2d_bias_relu(const void *x, const void *w, const void *bias, const void *residual, void *y,
                                   const tt_conv_shape *shape, int cls, const tt_schedule *sched, void *ws,
                                   size_t ws_bytes, void *stream)
{
    if (!shape || !is_conv_class(cls)) return TT_ERR_BAD_ARG;
    return run_op(sched, cls, shape, {x, w, bias, residual, y, ws, ws_bytes}, stream);
}

extern "C" int tt_dense_bias_relu(const void *x, const void *w, const void *bias, void *y,
                                  const tt_gemm_shape *shape, int cls, const tt_schedule *sched, void *ws,
                                  size_t ws_bytes, void *stream)
{
    if (!shape || !is_dense_class(cls)) return TT_ERR_BAD_ARG;
    return run_op(sched, cls, shape, {x, w, bias, nullptr, y, ws, ws_bytes}, stream);
}

extern "C" int tt_batch_matmul(const void *a, const void *b, void *c, const tt_gemm_shape *shape,
                               const tt_schedule *sched, void *ws, size_t ws_bytes, void *stream)
{
    if (!shape) return TT_ERR_BAD_ARG;
    return run_op(sched, TT_BATCH_MATMUL, shape, {a, b, nullptr, nullptr, c, ws, ws_bytes}, stream);
}

extern "C" int tt_dwconv(const void *x, const void *w, const void *bias, void *y, const tt_conv_shape *shape,
                         const tt_schedule *sched, void *stream)
{
    if (!shape) return TT_ERR_BAD_ARG;
    return run_op(sched, TT_DWCONV_BIAS_RELU6, shape, {x, w, bias, nullptr, y, nullptr, 0}, stream);
}

extern "C" int tt_debug_tile_map(const tt_plan *plan, int32_t *out_dev, void *stream)
{
    if (!plan || !out_dev || plan->status != TT_OK || plan->sketch == TT_SK_DIRECT || plan->grid < 1)
        return TT_ERR_BAD_ARG;
    return launch_tile_map_dump(tile_map_of(*plan), out_dev, stream);
}

// ---- standalone timing of one (kernel, schedule) pair (Section 4.3: pairs run as distinct programs) ----------

namespace {

// A kernel's plan and launch arguments are laid out once (prepare_op) and launched as often as needed.
int launch_desc(PreparedOp &op, const tt_kernel_desc &k, void *stream, int64_t turn = 0)
{
    const OpPointers p = pointers_of(k, turn);
    if (const int rc = check_op_pointers(k.cls, p); rc != TT_OK) return rc;
    return launch_op(op, &p, 1, stream);
}

// Events of the timing functions, created as they are first asked for and kept while the sweep lasts.
class Timer {
public:
    Timer() = default;
    Timer(const Timer &) = delete;
    Timer &operator=(const Timer &) = delete;
    ~Timer()
    {
        for (hipEvent_t e : events_) (void)hipEventDestroy(e);
    }
    bool record(size_t i, hipStream_t s)
    {
        while (events_.size() <= i) {
            hipEvent_t e = nullptr;
            if (hipEventCreate(&e) != hipSuccess) return false;
            events_.push_back(e);
        }
        return hipEventRecord(events_[i], s) == hipSuccess;
    }
    bool wait(size_t i) { return hipEventSynchronize(events_[i]) == hipSuccess; }
    bool elapsed_ms(size_t from, size_t to, float *ms) { return hipEventElapsedTime(ms, events_[from], events_[to]) == hipSuccess; }

private:
    std::vector<hipEvent_t> events_;
};

tt_sweep_opts resolve(const tt_sweep_opts *o)
{
    tt_sweep_opts r;
    r.warmup = 3;
    r.samples = 10;
    r.min_sample_us = 200;
    r.max_launches = 64;
    r.flags = 0;
    r.allow_slower_than_default = 0;
    r.pair_budget = 0;
    r.prioritise = 0;
    r.seed = 0;
    if (o) {
        r.pair_budget = o->pair_budget;
        r.prioritise = o->prioritise;
        r.seed = o->seed;
        if (o->warmup >= 0) r.warmup = o->warmup;
        if (o->samples > 0) r.samples = o->samples;
        if (o->min_sample_us > 0) r.min_sample_us = o->min_sample_us;
        if (o->max_launches > 0) r.max_launches = o->max_launches;
        r.flags = o->flags;
        r.allow_slower_than_default = o->allow_slower_than_default;
    }
    return r;
}

// Times of one kernel's launches under one protocol, for as long as a sweep lasts.  Records that differ only in knobs the
// kernel they run on does not have (stages, tile_k and unroll of a launch in groups, vec and unroll of a walk by taps, everything of
// one in blocks or windows) come to the same launch: they share the time of the first, and the rule for ties decides among them instead of noise.
class LaunchTimes {
public:
    struct Time {
        double median_us, min_us;
    };
    using Key = std::array<int32_t, 20>;
    static Key key_of(const PreparedOp &op)
    {
        tt_plan p;
        const int kernel = launched_plan(op, 1, &p);
        DwListEntry windows;
        DwWindow w;
        int vc;
        if (in_windows(op, 1, &windows, &w, &vc)) return Key{-1}; // (a record that the operator refuses has a key of its own)
        if (kernel == TT_LAUNCH_BLOCKS) return Key{kernel};
        if (kernel == TT_LAUNCH_ROWS) return Key{kernel, p.tile_m, p.tile_n, p.eff_vec_c, p.order};
        if (kernel == TT_LAUNCH_GROUPS)
            return Key{kernel, p.tile_m, p.tile_n, p.wave_m, p.wave_n, p.mfma, p.eff_split_k,
                       (int32_t)std::min<int64_t>((int64_t)p.k_iters * p.tile_k, p.K), p.eff_vec_c, p.order};
        if (kernel == TT_LAUNCH_TAPS) p.eff_vec_a = p.eff_vec_b = p.eff_unroll = 0;
        return Key{kernel, p.sketch, p.variant_id, p.tile_m, p.tile_n, p.tile_k, p.wave_m, p.wave_n, p.mfma, p.eff_split_k,
                   p.k_iters, p.eff_vec_a, p.eff_vec_b, p.eff_vec_c, p.eff_unroll, p.stages, p.order, p.grid, p.block, p.lds_bytes};
    }
    const Time *find(const Key &key) const
    {
        const auto it = times_.find(key);
        return it == times_.end() ? nullptr : &it->second;
    }
    void add(const Key &key, double median_us, double min_us) { times_[key] = {median_us, min_us}; }

private:
    std::map<Key, Time> times_;
};

int time_pair(const tt_kernel_desc &k, const tt_schedule *sched, const tt_sweep_opts &o, hipStream_t s, Timer &t,
              double *median_us, double *min_us, LaunchTimes *times = nullptr)
{
    // Validity first: nothing is launched for a record that does not apply.
    tt_schedule def;
    const tt_schedule *rec = sched;
    if (!rec) {
        const int rc = tt_schedule_default(k.cls, k.shape, &def);
        if (rc != TT_OK) return rc;
        rec = &def;
    }
    if (k.n_alt < 0 || (k.n_alt > 0 && !k.alt_bufs)) return TT_ERR_BAD_ARG;
    tt_plan plan;
    int rc = tt_schedule_apply(rec, k.cls, k.shape, o.flags, &plan);
    if (rc != TT_OK) return rc;
    // Launches so far, over all timed pairs of the process: every launch moves on to the next tensor set, and
    // the next pair carries on where this one stops (a pair that started over at the first set would find it,
    // and the few sets a short measurement touches, still in the memory-side cache from the pair before).
    static std::atomic<int64_t> turns{0};
    auto next_turn = [&]() { return turns.fetch_add(1, std::memory_order_relaxed); };
    // The plan is laid out once for all launches of the pair: planning a launch took longer than a small kernel
    // runs, so such a pair was timed, and the search waited for, at the host's pace.
    PreparedOp op;
    rc = prepare_op(rec, k.cls, k.shape, &op);
    if (rc != TT_OK) return rc;
    LaunchTimes::Key key{};
    if (times) {
        key = LaunchTimes::key_of(op);
        if (const LaunchTimes::Time *known = times->find(key)) {
            if (median_us) *median_us = known->median_us;
            if (min_us) *min_us = known->min_us;
            return TT_OK;
        }
    }
    for (int i = 0; i < std::max(1, o.warmup); ++i) {
        rc = launch_desc(op, k, s, next_turn());
        if (rc != TT_OK) return rc;
    }
    // Size a sample: time one launch, then batch enough launches to fill min_sample_us.
    float ms = 0.0f;
    if (!t.record(0, s)) return TT_ERR_HIP;
    rc = launch_desc(op, k, s, next_turn());
    if (rc != TT_OK) return rc;
    if (!t.record(1, s) || !t.wait(1) || !t.elapsed_ms(0, 1, &ms)) return TT_ERR_HIP;
    const double one_us = std::max(1.0, (double)ms * 1000.0);
    const int launches = (int)std::min<double>(o.max_launches, std::max(1.0, o.min_sample_us / one_us + 0.999));
    // All samples are enqueued back to back with one event between two of them, and waited for once: a wait per
    // sample drained the stream each time and added its latency to the search.
    if (!t.record(0, s)) return TT_ERR_HIP;
    for (int smp = 0; smp < o.samples; ++smp) {
        for (int l = 0; l < launches; ++l) {
            rc = launch_desc(op, k, s, next_turn());
            if (rc != TT_OK) return rc;
        }
        if (!t.record(smp + 1, s)) return TT_ERR_HIP;
    }
    if (!t.wait(o.samples)) return TT_ERR_HIP;
    std::vector<double> us(o.samples);
    for (int smp = 0; smp < o.samples; ++smp) {
        if (!t.elapsed_ms(smp, smp + 1, &ms)) return TT_ERR_HIP;
        us[smp] = (double)ms * 1000.0 / launches;
    }
    std::sort(us.begin(), us.end());
    const int n = (int)us.size();
    const double median = n % 2 ? us[n / 2] : 0.5 * (us[n / 2 - 1] + us[n / 2]);
    if (times) times->add(key, median, us[0]);
    if (median_us) *median_us = median;
    if (min_us) *min_us = us[0];
    return TT_OK;
}

} // namespace

extern "C" int tt_time_pair(const tt_kernel_desc *kernel, const tt_schedule *sched, const tt_sweep_opts *opts,
                            void *stream, double *median_us, double *min_us)
{
    if (!kernel || !kernel->shape) return TT_ERR_BAD_ARG;
    Timer t;
    return time_pair(*kernel, sched, resolve(opts), static_cast<hipStream_t>(stream), t, median_us, min_us);
}

extern "C" int tt_transfer_sweep(const tt_kernel_desc *kernels, int nk, const tt_schedule *pool, int np,
                                 const tt_sweep_opts *opts, void *stream, tt_sweep_row *rows, double *pair_us,
                                 int64_t *evaluations, double *wall_seconds)
{
    if (nk < 0 || np < 0 || (nk && (!kernels || !rows)) || (np && !pool)) return TT_ERR_BAD_ARG;
    const auto t0 = std::chrono::steady_clock::now();
    const tt_sweep_opts o = resolve(opts);
    hipStream_t s = static_cast<hipStream_t>(stream);
    Timer timer;
    std::vector<double> local((size_t)nk * np, -2.0), defaults(nk, 0.0), weight(nk, 0.0);
    std::vector<int32_t> kcls(nk), pcls(np);
    std::vector<LaunchTimes> times(nk);
    for (int p = 0; p < np; ++p) pcls[p] = pool[p].cls;
    int64_t evals = 0;
    // the default ("untuned") schedule is always evaluated: it is the baseline and the fallback
    for (int k = 0; k < nk; ++k) {
        if (!kernels[k].shape) return TT_ERR_BAD_ARG;
        kcls[k] = kernels[k].cls;
        const int rc = time_pair(kernels[k], nullptr, o, s, timer, &defaults[k], nullptr, &times[k]);
        if (rc != TT_OK) return rc;
        weight[k] = defaults[k] * std::max(1, kernels[k].use_count);
        ++evals;
    }
    // which same-class pairs are tried: all of them, or the budgeted subset
    std::vector<uint8_t> mask((size_t)nk * np + 1, 0);
    if (const int rc = tt_sweep_plan(kcls.data(), weight.data(), nk, pcls.data(), np, o.pair_budget, o.prioritise, o.seed,
                                     mask.data(), nullptr);
        rc != TT_OK)
        return rc;
    for (int k = 0; k < nk; ++k)
        for (int p = 0; p < np; ++p) {
            if (pool[p].cls != kernels[k].cls) continue; // other classes are never tried (Section 4.2)
            if (!mask[(size_t)k * np + p]) {
                local[(size_t)k * np + p] = -3.0;
                continue;
            }
            ++evals;
            double us = -1.0;
            const int rc = time_pair(kernels[k], &pool[p], o, s, timer, &us, nullptr, &times[k]);
            if (rc == TT_ERR_HIP) return rc;
            // every other failure means "this record does not fit this kernel": the paper's -1
            local[(size_t)k * np + p] = rc == TT_OK ? us : -1.0;
        }
    if (hipStreamSynchronize(s) != hipSuccess) return TT_ERR_HIP;
    const int rc = tt_sweep_select(kcls.data(), nk, pcls.data(), np, local.data(), defaults.data(),
                                   o.allow_slower_than_default, rows);
    if (rc != TT_OK) return rc;
    if (pair_us) std::copy(local.begin(), local.end(), pair_us);
    if (evaluations) *evaluations = evals;
    if (wall_seconds) *wall_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return TT_OK;
}

// ---- local refinement of a record (Section 6's outlook) and the native sweep of one kernel -----------------

extern "C" int tt_refine(const tt_kernel_desc *kernel, const tt_schedule *base, int rounds, const tt_sweep_opts *opts,
                         void *stream, tt_schedule *best, double *best_us, double *base_us, int32_t *tried)
{
    if (!kernel || !kernel->shape || !base || !best || rounds < 0) return TT_ERR_BAD_ARG;
    const tt_sweep_opts o = resolve(opts);
    hipStream_t s = static_cast<hipStream_t>(stream);
    Timer timer;
    LaunchTimes times;
    double cur_us = 0.0;
    int rc = time_pair(*kernel, base, o, s, timer, &cur_us, nullptr, &times);
    if (rc != TT_OK) return rc;
    int32_t n = 1;
    tt_schedule cur = *base;
    if (base_us) *base_us = cur_us;
    for (int r = 0; r < rounds; ++r) {
        const int count = tt_refine_space(&cur, nullptr, 0);
        if (count <= 0) break;
        std::vector<tt_schedule> near(count);
        tt_refine_space(&cur, near.data(), count);
        int win = -1;
        double win_us = cur_us;
        for (int i = 0; i < count; ++i) {
            double us = 0.0;
            rc = time_pair(*kernel, &near[i], o, s, timer, &us, nullptr, &times);
            if (rc == TT_ERR_HIP) return rc;
            if (rc != TT_OK) continue; // does not apply to this kernel, or no kernel implements it
            ++n;
            if (us < win_us) { // strict: the current record, then the lowest index, win ties
                win_us = us;
                win = i;
            }
        }
        if (win < 0) break;
        const int32_t keep_id = cur.id;
        cur = near[win];
        cur.id = keep_id;
        cur_us = win_us;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return TT_ERR_HIP;
    *best = cur;
    if (best_us) *best_us = cur_us;
    if (tried) *tried = n;
    return TT_OK;
}

extern "C" int tt_native_sweep(const tt_kernel_desc *kernel, int level, int finalists, const tt_sweep_opts *explore,
                               const tt_sweep_opts *full, void *stream, tt_schedule *best, double *best_us,
                               double *default_us, int32_t *n_valid, int32_t *n_records)
{
    if (!kernel || !kernel->shape || !best || finalists < 1) return TT_ERR_BAD_ARG;
    tt_sweep_opts quick;
    std::memset(&quick, 0, sizeof quick);
    quick.warmup = 1;
    quick.samples = 3;
    quick.min_sample_us = 60;
    quick.max_launches = 16;
    const tt_sweep_opts ex = explore ? resolve(explore) : quick, fu = resolve(full);
    const bool conv = is_conv_class(kernel->cls) || kernel->cls == TT_DWCONV_BIAS_RELU6;
    const int dtype = conv ? static_cast<const tt_conv_shape *>(kernel->shape)->dtype
                           : static_cast<const tt_gemm_shape *>(kernel->shape)->dtype;
    const int count = tt_schedule_space(kernel->cls, dtype, level, nullptr, 0);
    if (count < 0) return count;
    std::vector<tt_schedule> space(std::max(count, 1));
    tt_schedule_space(kernel->cls, dtype, level, space.data(), count);
    hipStream_t s = static_cast<hipStream_t>(stream);
    Timer timer;

    // the `keep` fastest records of a list under one protocol, fastest first (ties: list order)
    struct Timed {
        double us;
        int index;
    };
    int valid = 0;
    LaunchTimes ex_times, fu_times;
    const auto fastest = [&](const std::vector<tt_schedule> &list, int n, const tt_sweep_opts &o, LaunchTimes &times, size_t keep, bool count_valid,
                             std::vector<tt_schedule> *out, std::vector<double> *out_us) -> int {
        std::vector<Timed> t;
        for (int i = 0; i < n; ++i) {
            double us = 0.0;
            const int rc = time_pair(*kernel, &list[i], o, s, timer, &us, nullptr, &times);
            if (rc == TT_ERR_HIP) return rc;
            if (rc != TT_OK) continue;
            if (count_valid) ++valid;
            t.push_back({us, i});
        }
        std::stable_sort(t.begin(), t.end(), [](const Timed &a, const Timed &b) { return a.us < b.us; });
        out->clear();
        if (out_us) out_us->clear();
        for (size_t i = 0; i < t.size() && i < keep; ++i) {
            out->push_back(list[t[i].index]);
            if (out_us) out_us->push_back(t[i].us);
        }
        return TT_OK;
    };
    std::vector<tt_schedule> top;
    int rc = fastest(space, count, ex, ex_times, (size_t)finalists, true, &top, nullptr);
    if (rc != TT_OK) return rc;
    if (!top.empty() && top[0].sketch == TT_SK_MFMA) {
        // the enumerated space carries one unroll setting and (below level 2) two workgroup orders: the
        // finalists are re-tried under all of them
        std::vector<tt_schedule> wide;
        for (const tt_schedule &f : top)
            for (int order = 0; order < 6; ++order)
                for (int unroll : {8, 1}) {
                    tt_schedule r = f;
                    r.order = order;
                    r.unroll = unroll;
                    bool seen = false;
                    for (const tt_schedule &w : wide) seen = seen || std::memcmp(&w, &r, sizeof(int32_t) * 13) == 0;
                    if (!seen) wide.push_back(r);
                }
        rc = fastest(wide, (int)wide.size(), ex, ex_times, (size_t)finalists, false, &top, nullptr);
        if (rc != TT_OK) return rc;
    }
    std::vector<double> top_us;
    rc = fastest(top, (int)top.size(), fu, fu_times, 1, false, &top, &top_us);
    if (rc != TT_OK) return rc;
    double def_us = 0.0;
    rc = time_pair(*kernel, nullptr, fu, s, timer, &def_us, nullptr, &fu_times);
    if (rc != TT_OK) return rc;
    if (hipStreamSynchronize(s) != hipSuccess) return TT_ERR_HIP;
    if (!top.empty() && top_us[0] < def_us) { // the default wins ties
        *best = top[0];
        if (best_us) *best_us = top_us[0];
    } else {
        rc = tt_schedule_default(kernel->cls, kernel->shape, best);
        if (rc != TT_OK) return rc;
        if (best_us) *best_us = def_us;
    }
    if (default_us) *default_us = def_us;
    if (n_valid) *n_valid = valid;
    if (n_records) *n_records = count;
    return TT_OK;
}
