// Lists of kernels: which entries may run at the same time, and which launches they go out in.
//
// The entries of a list run in order as far as they depend on each other: an entry that touches what an earlier one writes
// (or writes what an earlier one touches) comes behind it.  A stretch of entries that are all independent of each other is a
// window, and a window is sent out in as few launches as its kernels allow.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <exception>
#include <vector>

#include "tt_internal.h"

namespace tt {

// The pointers of tensor set `turn`: 0 = bufs, then the alternatives in order, round and round.
OpPointers pointers_of(const tt_kernel_desc &k, int64_t turn)
{
    void *const *b = k.bufs;
    if (k.n_alt > 0) {
        const int set = (int)(turn % (k.n_alt + 1));
        if (set > 0) b = k.alt_bufs + (size_t)(set - 1) * 5;
    }
    if (is_conv_class(k.cls)) return {b[0], b[1], b[2], b[3], b[4], k.ws, k.ws_bytes};
    if (k.cls == TT_BATCH_MATMUL) return {b[0], b[1], nullptr, nullptr, b[2], k.ws, k.ws_bytes};
    return {b[0], b[1], b[2], nullptr, b[3], k.ws, k.ws_bytes}; // dense, depthwise
}

bool same_knobs(const tt_schedule &x, const tt_schedule &y) { return std::memcmp(&x, &y, sizeof(int32_t) * 13) == 0; }

namespace {

struct Range {
    const char *at, *end;
};
inline bool overlap(const Range &x, const Range &y) { return x.at && y.at && x.at < y.end && y.at < x.end; }

// An entry of a window.
struct Entry {
    int op;       // index of its plan
    int index;    // place in the caller's list
    OpPointers p;
    Range writes[2], reads[4];
};

Entry entry_at(int index, int op_index, const PreparedOp &op, const OpPointers &p)
{
    const auto range = [](const void *at, int64_t bytes) {
        const char *c = static_cast<const char *>(at);
        return Range{c, c + bytes};
    };
    Entry e{op_index, index, p, {}, {}};
    e.writes[0] = range(p.out, op.out_bytes);
    e.writes[1] = range(op.plan.workspace_bytes > 0 ? p.ws : nullptr, op.plan.workspace_bytes);
    e.reads[0] = range(p.a, op.a_bytes);
    e.reads[1] = range(p.b, op.b_bytes);
    e.reads[2] = range(p.bias, op.bias_bytes);
    e.reads[3] = range(p.res, op.out_bytes);
    return e;
}

// Whether two entries may run at the same time: neither writes what the other reads or writes.
bool independent(const Entry &p, const Entry &q)
{
    for (const Range &w : p.writes)
        for (const Range &v : q.writes)
            if (overlap(w, v)) return false;
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 4; ++j)
            if (overlap(p.writes[i], q.reads[j]) || overlap(p.reads[j], q.writes[i])) return false;
    return true;
}

// Same class, shape and record: one plan.
bool same_plan(const tt_kernel_desc &x, const tt_schedule *sx, const tt_kernel_desc &y, const tt_schedule *sy)
{
    if (x.cls != y.cls || (sx == nullptr) != (sy == nullptr)) return false;
    if (sx && sx != sy && !same_knobs(*sx, *sy)) return false;
    const bool image = is_conv_class(x.cls) || x.cls == TT_DWCONV_BIAS_RELU6;
    return x.shape == y.shape || std::memcmp(x.shape, y.shape, image ? sizeof(tt_conv_shape) : sizeof(tt_gemm_shape)) == 0;
}

// Whether the operator would refuse the plan.
bool refused(const PreparedOp &op)
{
    return !op.supported || ((op.launch.sketch == TT_SK_MFMA || op.launch.sketch == TT_SK_DWCONV) && op.launch.variant_id < 0);
}

// Whether a contraction can share a launch with others of its data type and operand family: what the ring loads (whole
// 16-byte items, operands within the offset range), whatever tile its record names.
bool listable(const PreparedOp &op)
{
    const tt_plan &pl = op.launch;
    if (pl.sketch != TT_SK_MFMA || (op.family != FAM_CONV && op.family != FAM_GEMM_TN)) return false;
    if (kVariants[pl.variant_id].pipe > 1) return false; // the patch and the persistent kernel are a choice of their own
    const int64_t elem = op.g.dtype == TT_F32 ? 4 : 2;
    if (pl.eff_vec_a * elem != 16 || pl.eff_vec_b * elem != 16) return false;
    if (op.family == FAM_GEMM_TN && ((int64_t)pl.M * pl.K * elem >= (1ll << 31) || (int64_t)pl.N * pl.K * elem >= (1ll << 31))) return false;
    return (int64_t)pl.batch * pl.M * pl.N < (1ll << 31);
}

// What the block kernel asks for beyond that.
bool block_tile_fits(const PreparedOp &op)
{
    const tt_plan &pl = op.launch;
    return pl.eff_vec_c == 8 && pl.eff_split_k == 1 && pl.batch == 1 && pl.K >= 512 &&
           (op.family == FAM_CONV || ((int64_t)pl.M * pl.K < (1ll << 30) && (int64_t)pl.N * pl.K < (1ll << 30)));
}

// Tiles of a plan in a tile of the list rule: how many, the split of the reduction, and what one costs a compute unit.
struct Cut {
    int64_t tiles;
    int k_tiles, k_iters, splits;
    double us, alone_us;
};
Cut cut_into(const PreparedOp &op, const ListTile &t)
{
    const tt_plan &pl = op.launch;
    Cut c;
    c.k_tiles = (pl.K + t.tile_k - 1) / t.tile_k;
    c.k_iters = (c.k_tiles + pl.eff_split_k - 1) / pl.eff_split_k;
    c.splits = (c.k_tiles + c.k_iters - 1) / c.k_iters;
    c.tiles = (int64_t)((pl.M + t.tile_m - 1) / t.tile_m) * ((pl.N + t.tile_n - 1) / t.tile_n) * pl.batch * c.splits;
    const double k = std::min<double>((double)c.k_iters * t.tile_k, pl.K);
    c.us = t.fixed_us + t.per_k_us * k;
    c.alone_us = t.fixed_us + t.alone_per_k_us * k;
    if (op.cls == TT_CONV2D_BIAS_ADD_RELU) // the residual: as many bytes as the output
        c.us += (double)t.tile_m * t.tile_n * (op.g.dtype == TT_F32 ? 4 : 2) * compute_units() / 5.0e6;
    return c;
}

// Estimated time (us) of the launches of a set of contractions when each takes the cheaper of two tiles.  A launch costs
// 2.5 us; its workgroups, the longest first, are dealt to the CUs, so its end is ragged by the shortest of them; nothing is
// faster than the longest alone, or than memory.
double estimate(const std::vector<const PreparedOp *> &ops, const std::vector<std::vector<Cut>> &cuts, int t0, int t1, std::vector<int> *chosen)
{
    double sum[2] = {}, least[2] = {1e30, 1e30}, longest[2] = {}, bytes[2] = {};
    for (size_t i = 0; i < ops.size(); ++i) {
        const Cut &x = cuts[i][t0], &y = cuts[i][t1];
        const double cost[2] = {x.tiles * x.us, y.tiles * y.us};
        const int pick = cost[1] < cost[0];
        if (cost[pick] >= 1e30) return 1e30;
        const Cut &c = pick ? y : x;
        sum[pick] += cost[pick];
        least[pick] = std::min(least[pick], c.us);
        longest[pick] = std::max(longest[pick], c.alone_us);
        const PreparedOp &op = *ops[i];
        bytes[pick] += (double)op.a_bytes + op.b_bytes + op.out_bytes * (op.cls == TT_CONV2D_BIAS_ADD_RELU ? 2 : 1);
        if (chosen) (*chosen)[i] = pick ? t1 : t0;
    }
    double us = 0;
    for (int h = 0; h < 2; ++h)
        if (sum[h] > 0) us += 2.5 + std::max({std::ceil(sum[h] / compute_units() / least[h]) * least[h], longest[h], bytes[h] / 5.0e6});
    return us;
}

ListEntry list_entry(const PreparedOp &op, const OpPointers &p, const ListTile &t, const Cut &c)
{
    const ContractArgs &g = op.g;
    const tt_plan &pl = op.launch;
    ListEntry e;
    std::memset(&e, 0, sizeof e);
    e.a = p.a, e.b = p.b, e.bias = p.bias, e.res = p.res, e.out = p.out, e.ws = static_cast<float *>(p.ws);
    e.M = pl.M, e.N = pl.N, e.K = pl.K, e.batch = pl.batch;
    e.grid = (int32_t)c.tiles;
    e.tiles_m = (pl.M + t.tile_m - 1) / t.tile_m, e.tiles_n = (pl.N + t.tile_n - 1) / t.tile_n;
    e.k_iters = c.k_iters, e.k_tiles = c.k_tiles, e.splits = c.splits;
    e.div_tiles = make_fastdiv((uint32_t)(e.tiles_m * e.tiles_n));
    e.div_n = make_fastdiv((uint32_t)e.tiles_n);
    e.div_split = make_fastdiv((uint32_t)e.splits);
    e.C = g.C, e.H = g.H, e.W = g.W, e.R = g.R, e.S = g.S, e.Ho = g.Ho, e.Wo = g.Wo;
    e.stride_h = g.stride_h, e.stride_w = g.stride_w, e.pad_h = g.pad_h, e.pad_w = g.pad_w;
    e.div_hw = g.div_hw, e.div_wo = g.div_wo;
    e.a_bytes = g.a_bytes, e.b_bytes = g.b_bytes;
    e.vec_c = (int16_t)pl.eff_vec_c, e.act = (int16_t)g.act;
    return e;
}

// A launch of a window: entries of one plan on pointer sets (tile -1), or listed contractions in a tile of the list rule.
struct Launch {
    int tile, family;
    std::vector<int> entries; // of the window
};

class Window {
public:
    explicit Window(std::vector<PreparedOp> &ops) : ops_(ops) {}
    bool admits(const Entry &e) const
    {
        for (const Entry &f : entries_)
            if (!independent(e, f)) return false;
        return true;
    }
    void add(const Entry &e) { entries_.push_back(e); }
    bool empty() const { return entries_.empty(); }
    const std::vector<Entry> &entries() const { return entries_; }
    void clear() { entries_.clear(); }

    std::vector<Launch> launches() const
    {
        std::vector<Launch> out;
        int tiles = 0;
        list_tiles(&tiles);
        const int n = (int)entries_.size();
        std::vector<char> done(n, 0);
        for (int dt = 0; dt < 2; ++dt)
            for (int family : {FAM_CONV, FAM_GEMM_TN}) {
                std::vector<int> members;
                for (int i = 0; i < n; ++i) {
                    const PreparedOp &op = ops_[entries_[i].op];
                    if (op.cls != TT_DWCONV_BIAS_RELU6 && op.g.dtype == dt && op.family == family && listable(op)) members.push_back(i);
                }
                if (members.size() < 2) continue;
                // (splits of one plan alone: nothing to share that their own launches would not)
                const PreparedOp &first = ops_[entries_[members[0]].op];
                const bool one_plan = std::all_of(members.begin(), members.end(), [&](int i) { return entries_[i].op == entries_[members[0]].op; });
                if (one_plan && first.launch.eff_split_k > 1) continue;
                for (int i : members) done[i] = 1;
                list(members, dt, family, &out);
            }
        // the rest: entries of one plan, all with a bias or all without, share a launch
        std::vector<Launch> plain;
        for (int i = 0; i < n; ++i) {
            if (done[i]) continue;
            Launch l{-1, 0, {i}};
            for (int j = i + 1; j < n && (int)l.entries.size() < kMaxSets; ++j)
                if (!done[j] && entries_[j].op == entries_[i].op && (entries_[j].p.bias == nullptr) == (entries_[i].p.bias == nullptr)) {
                    l.entries.push_back(j);
                    done[j] = 1;
                }
            plain.push_back(std::move(l));
        }
        out.insert(out.begin(), plain.begin(), plain.end());
        return out;
    }

    int run(const Launch &l, void *stream) const
    {
        if (l.tile < 0) {
            OpPointers calls[kMaxSets];
            for (size_t i = 0; i < l.entries.size(); ++i) calls[i] = entries_[l.entries[i]].p;
            return launch_op(ops_[entries_[l.entries[0]].op], calls, (int)l.entries.size(), stream);
        }
        int tiles = 0;
        const ListTile &t = list_tiles(&tiles)[l.tile];
        ContractList list;
        int grid = 0;
        for (int i = 0; i < kMaxListed; ++i) {
            list.first[i] = i < (int)l.entries.size() ? grid : INT32_MAX;
            if (i >= (int)l.entries.size()) continue;
            const Entry &e = entries_[l.entries[i]];
            const PreparedOp &op = ops_[e.op];
            list.e[i] = list_entry(op, e.p, t, cut_into(op, t));
            grid += (list.e[i].grid + kXcds - 1) / kXcds * kXcds;
        }
        return t.launch[l.family == FAM_CONV ? 0 : 1](list, grid, stream);
    }

    // The second step of the split reductions among listed entries.
    int reduce(const std::vector<Launch> &launches, void *stream) const
    {
        int tiles = 0;
        const ListTile *table = list_tiles(&tiles);
        for (int dt = 0; dt < 2; ++dt)
            for (bool fours : {true, false}) {
                ReduceList list;
                int count = 0;
                const auto send = [&]() {
                    const int rc = count ? launch_reduce_list(list, count, dt, fours, stream) : TT_OK;
                    count = 0;
                    return rc;
                };
                for (const Launch &l : launches) {
                    if (l.tile < 0) continue;
                    for (int i : l.entries) {
                        const Entry &e = entries_[i];
                        const PreparedOp &op = ops_[e.op];
                        const tt_plan &pl = op.launch;
                        const Cut c = cut_into(op, table[l.tile]);
                        if (c.splits == 1 || op.g.dtype != dt || (pl.N % 4 == 0) != fours) continue;
                        list.e[count++] = {static_cast<float *>(e.p.ws), e.p.bias, e.p.res, e.p.out, (int64_t)pl.batch * pl.M * pl.N,
                                           pl.N, c.splits, op.g.act, 0};
                        if (count == kMaxReduced)
                            if (const int rc = send(); rc != TT_OK) return rc;
                    }
                }
                if (const int rc = send(); rc != TT_OK) return rc;
            }
        return TT_OK;
    }

private:
    void list(const std::vector<int> &members, int dt, int family, std::vector<Launch> *out) const
    {
        int n_tiles = 0;
        const ListTile *tiles = list_tiles(&n_tiles);
        std::vector<const PreparedOp *> ops;
        std::vector<std::vector<Cut>> cuts;
        for (int i : members) {
            const PreparedOp &op = ops_[entries_[i].op];
            ops.push_back(&op);
            std::vector<Cut> c;
            for (int t = 0; t < n_tiles; ++t) {
                c.push_back(cut_into(op, tiles[t]));
                if (tiles[t].dtype != dt || (tiles[t].tile_m == 256 && !block_tile_fits(op))) c.back().us = 1e30;
            }
            cuts.push_back(std::move(c));
        }
        int b0 = -1, b1 = -1;
        double best = 1e30;
        for (int t0 = 0; t0 < n_tiles; ++t0) {
            if (tiles[t0].dtype != dt) continue;
            for (int t1 = t0; t1 < n_tiles; ++t1) {
                if (tiles[t1].dtype != dt) continue;
                const double us = estimate(ops, cuts, t0, t1, nullptr);
                if (us < best) best = us, b0 = t0, b1 = t1;
            }
        }
        std::vector<int> chosen(members.size());
        estimate(ops, cuts, b0, b1, &chosen);
        for (int t : {b0, b1}) {
            std::vector<int> at;
            for (size_t i = 0; i < members.size(); ++i)
                if (chosen[i] == t) at.push_back((int)i);
            // the longest first, so that the end of the launch is not one long tile
            std::stable_sort(at.begin(), at.end(), [&](int x, int y) { return cuts[x][t].us > cuts[y][t].us; });
            for (size_t i = 0; i < at.size(); i += kMaxListed) {
                Launch l{t, family, {}};
                for (size_t j = i; j < std::min(at.size(), i + kMaxListed); ++j) l.entries.push_back(members[at[j]]);
                out->push_back(std::move(l));
            }
            if (b0 == b1) break;
        }
    }

    std::vector<PreparedOp> &ops_;
    std::vector<Entry> entries_;
};

int send(Window &w, void *stream)
{
    if (w.empty()) return TT_OK;
    const std::vector<Launch> launches = w.launches();
    for (const Launch &l : launches)
        if (const int rc = w.run(l, stream); rc != TT_OK) return rc;
    const int rc = w.reduce(launches, stream);
    w.clear();
    return rc;
}

constexpr size_t kMaxWindow = 128; // the check for independence looks at every pair

// Walks the list and hands every window to `emit` (window, whether its one entry runs `use_count` times).
template <typename Emit>
int walk(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, std::vector<PreparedOp> &ops, Emit &&emit)
{
    Window w(ops);
    int last = -1; // the entry whose plan is ops.back()
    for (int k = 0; k < nk; ++k) {
        const tt_kernel_desc &d = kernels[k];
        const tt_schedule *rec = scheds ? scheds[k] : nullptr;
        const auto fail = [&](int rc) { // what stands before the entry that fails is enqueued
            const int before = emit(w, 1);
            return before != TT_OK ? before : rc;
        };
        if (!d.shape) return fail(TT_ERR_BAD_ARG);
        if (d.use_count <= 0) continue; // nothing to launch: neither record nor tensors are looked at
        if (d.cls < 0 || d.cls >= TT_NUM_CLASSES) return fail(TT_ERR_BAD_ARG);
        const OpPointers p = pointers_of(d, 0);
        if (const int rc = check_op_pointers(d.cls, p); rc != TT_OK) return fail(rc);
        if (last < 0 || !same_plan(kernels[last], scheds ? scheds[last] : nullptr, d, rec)) {
            ops.emplace_back();
            if (const int rc = prepare_op(rec, d.cls, d.shape, &ops.back()); rc != TT_OK) {
                ops.pop_back();
                return fail(rc);
            }
            last = k;
        }
        const PreparedOp &op = ops.back();
        if (!workspace_fits(op, p)) return fail(TT_ERR_WORKSPACE);
        if (refused(op)) return fail(TT_ERR_UNSUPPORTED);
        const Entry e = entry_at(k, (int)ops.size() - 1, op, p);
        const bool again = d.use_count != 1;
        if (again || w.entries().size() >= kMaxWindow || !w.admits(e))
            if (const int rc = emit(w, 1); rc != TT_OK) return rc;
        w.add(e);
        if (again)
            if (const int rc = emit(w, d.use_count); rc != TT_OK) return rc;
    }
    return emit(w, 1);
}

} // namespace
} // namespace tt

using namespace tt;

// (the bookkeeping allocates, and nothing may be thrown through the C interface)
template <typename F> static int without_exceptions(F &&f)
{
    try {
        return f();
    } catch (const std::exception &) {
        return note_hip_error(2 /* hipErrorOutOfMemory */, "list of kernels");
    }
}

extern "C" int tt_run_kernels(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, int repeat, void *stream)
{
    if (nk < 0 || repeat < 0 || (nk && !kernels)) return TT_ERR_BAD_ARG;
    return without_exceptions([&]() {
        std::vector<PreparedOp> ops;
        for (int r = 0; r < repeat; ++r) {
            ops.clear();
            const int rc = walk(kernels, scheds, nk, ops, [&](Window &w, int times) {
                for (int u = 1; u < times; ++u) {
                    Window again = w;
                    if (const int rc = send(again, stream); rc != TT_OK) return rc;
                }
                return send(w, stream);
            });
            if (rc != TT_OK) return rc;
        }
        return (int)TT_OK;
    });
}

extern "C" int tt_debug_list(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, tt_listed *out)
{
    if (nk < 0 || (nk && (!kernels || !out))) return TT_ERR_BAD_ARG;
    return without_exceptions([&]() {
        std::vector<PreparedOp> ops;
        for (int k = 0; k < nk; ++k) out[k] = {-1, 0, 0, 0, 0, 0};
        int launch = 0, tiles = 0;
        const ListTile *table = list_tiles(&tiles);
        return walk(kernels, scheds, nk, ops, [&](Window &w, int) {
            for (const Launch &l : w.launches()) {
                for (int i : l.entries) {
                    const Entry &e = w.entries()[i];
                    const tt_plan &pl = ops[e.op].launch;
                    out[e.index] = {launch, l.tile >= 0, l.tile >= 0 ? table[l.tile].tile_m : pl.tile_m,
                                    l.tile >= 0 ? table[l.tile].tile_n : pl.tile_n, l.tile >= 0 ? table[l.tile].tile_k : pl.tile_k,
                                    (int32_t)l.entries.size()};
                }
                ++launch;
            }
            w.clear();
            return (int)TT_OK;
        });
    });
}
