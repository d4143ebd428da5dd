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
    const char *at, *end; // empty where at is null
};

// Address ranges, for the question whether another one touches any of them.
class Ranges {
public:
    bool touches(const Range &r) const
    {
        if (!r.at || r.at == r.end) return false;
        const auto it = std::lower_bound(sorted_.begin(), sorted_.end(), r.end, [](const Item &x, const char *end) { return x.at < end; });
        return it != sorted_.begin() && (it - 1)->reach > r.at; // of those that begin before its end, the furthest end
    }
    void add(const Range &r)
    {
        if (!r.at || r.at == r.end) return;
        auto it = std::upper_bound(sorted_.begin(), sorted_.end(), r.at, [](const char *at, const Item &x) { return at < x.at; });
        const char *reach = it == sorted_.begin() ? r.end : std::max((it - 1)->reach, r.end);
        it = sorted_.insert(it, {r.at, reach});
        for (++it; it != sorted_.end() && it->reach < reach; ++it) it->reach = reach;
    }
    void clear() { sorted_.clear(); }

private:
    struct Item {
        const char *at, *reach; // `reach`: the largest end up to here
    };
    std::vector<Item> sorted_; // by `at`
};

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

// The sizes of a stream, laid out for the thin kernel.
ThinEntry thin_entry(const PreparedOp &op)
{
    ThinEntry e = {};
    e.M = op.launch.M, e.N = op.launch.N, e.K = op.launch.K, e.act = op.g.act;
    thin_layout(&e);
    return e;
}

// Whether a listed contraction is a stream for the thin kernel, and the instance that holds its reduction (0: none): single
// precision, rows of whole fours, no split of the reduction, and rows enough that a workgroup's weights, which it loads into
// LDS first, are less than half of what it reads and writes.  Of those, the ones that the tiles of the rule do not stream as
// fast; two entries of M x N x K in tiles -> as streams (us):
//   reductions of up to 32 that read less than twice what they write: 200704 x 24 x 16 23 -> 20, x 96 x 24 67 -> 48, 50176 x 144
//   x 24 31 -> 21, 12544 x 192 x 24 12 -> 11, but 50176 x 16 x 32 7.6 -> 8.1
//   reductions of up to 96 over more than 32 columns that tiles of 64 do not divide: 200704 x 144 x 64 171 -> 112, 50176 x 48 x
//   96 29 -> 24, x 96 x 64 29 -> 26, but x 192 x 64 40 -> 50, x 64 x 96 22 -> 26, x 32 x 96 15 -> 17
//   with workgroups for half of the CUs, or little for each of them to multiply: 3136 x 64 x 16 4.9 -> 4.7, but x 64 x 32 4.7 ->
//   5.4, x 48 x 96 4.7 -> 6.7, x 192 x 24 5.7 -> 8.9
//   longer ones: 50176 x 24 x 144 19 -> 24, x 32 x 192 23 -> 31, x 64 x 144 30 -> 37, x 144 x 192 77 -> 72
int thin_pieces(const PreparedOp &op)
{
    const tt_plan &pl = op.launch;
    if (op.g.dtype != TT_F32 || op.family != FAM_GEMM_TN || pl.eff_split_k != 1 || pl.batch != 1 || op.g.act == ACT_GELU) return 0;
    if (pl.N % 4 != 0 || pl.K % 4 != 0) return 0;
    const ThinEntry e = thin_entry(op);
    if ((int64_t)std::min(e.rows, e.M) * (e.K + e.columns) < 2ll * e.K * e.columns) return 0;
    if (e.K <= 32 ? e.K >= 2 * (int64_t)e.N : e.N <= 32 || e.N % 64 == 0) return 0;
    if (thin_workgroups(e) < compute_units() / 2 && (int64_t)e.K * e.columns > 1024) return 0;
    for (int p : kThinPieces)
        if (pl.K <= p * 16) return p;
    return 0;
}

// What the block kernel asks for beyond that.
bool block_tile_fits(const PreparedOp &op)
{
    const tt_plan &pl = op.launch;
    return pl.eff_vec_c == 8 && pl.eff_split_k == 1 && pl.batch == 1 && pl.K >= 512 &&
           (op.family == FAM_CONV || ((int64_t)pl.M * pl.K < (1ll << 30) && (int64_t)pl.N * pl.K < (1ll << 30)));
}

constexpr double kUnfit = 1e30; // the cost of a tile that a plan cannot run in

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

// A plan of a window's contractions, how many entries have it, and what their tiles cost in every tile of the rule.
struct Kind {
    const PreparedOp *op;
    int count, own_tile; // entries; the tile of the rule that is its record's (-1: none)
    double bytes; // of all its entries
    struct {
        double all_us, us, alone_us; // of all its entries' tiles on one CU; of one; of one with the CU to itself
    } in[kMaxListTiles];
};

// Estimated time (us) of the launches of a set of contractions when each takes the cheapest of some tiles (-1: none).  A
// launch costs 2.5 us; its workgroups, the longest first, are dealt to the CUs, so its end is ragged by the shortest of them;
// nothing is faster than the longest alone, or than memory.  An entry with a launch to itself runs under its record, so sets
// that leave a tile to one entry count only where its record names that tile (a transformer layer of 2079 tokens, whose one
// batched product would have a tile to itself: under its record, of another tile, 84 us, beside the others 75; a MobileNetV2
// pass at batch 16 with a layer that has one, 16 x 16 x 16, in its record too: 243.5 us, with that layer beside others 248).
constexpr int kTilesAtOnce = 3;
double estimate(const std::vector<Kind> &kinds, const int (&tiles)[kTilesAtOnce], int *chosen)
{
    int count[kTilesAtOnce] = {}, own[kTilesAtOnce] = {};
    double sum[kTilesAtOnce] = {}, longest[kTilesAtOnce] = {}, bytes[kTilesAtOnce] = {}, least[kTilesAtOnce] = {1e30, 1e30, 1e30};
    for (size_t i = 0; i < kinds.size(); ++i) {
        const Kind &k = kinds[i];
        int pick = -1;
        for (int h = 0; h < kTilesAtOnce; ++h)
            if (tiles[h] >= 0 && (pick < 0 || k.in[tiles[h]].all_us < k.in[tiles[pick]].all_us)) pick = h;
        if (pick < 0 || k.in[tiles[pick]].us >= kUnfit) return kUnfit;
        const auto &c = k.in[tiles[pick]];
        count[pick] += k.count, own[pick] = k.own_tile;
        sum[pick] += c.all_us;
        least[pick] = std::min(least[pick], c.us);
        longest[pick] = std::max(longest[pick], c.alone_us);
        bytes[pick] += k.bytes;
        if (chosen) chosen[i] = tiles[pick];
    }
    double us = 0;
    for (int h = 0; h < kTilesAtOnce; ++h)
        if (count[h] == 1 && own[h] != tiles[h]) return kUnfit;
    for (int h = 0; h < kTilesAtOnce; ++h)
        if (sum[h] > 0) us += 2.5 + std::max({std::ceil(sum[h] / compute_units() / least[h]) * least[h], longest[h], bytes[h] / 5.0e6});
    return us;
}

// The tiles that suit a set of contractions: the best pair of all, and a third beside it if that helps.
void best_tiles(const std::vector<Kind> &kinds, const ListTile *tiles, int n_tiles, int dt, int (&best)[kTilesAtOnce])
{
    double best_us = kUnfit;
    const auto try_set = [&](int x, int y, int z) {
        const int set[kTilesAtOnce] = {x, y, z};
        const double us = estimate(kinds, set, nullptr);
        if (us < best_us) best_us = us, std::copy(set, set + kTilesAtOnce, best);
    };
    for (int x = 0; x < n_tiles; ++x)
        if (tiles[x].dtype == dt) try_set(x, -1, -1);
    for (int x = 0; x < n_tiles; ++x)
        for (int y = x + 1; y < n_tiles; ++y)
            if (tiles[x].dtype == dt && tiles[y].dtype == dt) try_set(x, y, -1);
    const int x = best[0], y = best[1];
    for (int z = 0; z < n_tiles && y >= 0; ++z)
        if (tiles[z].dtype == dt && z != x && z != y) try_set(x, y, z);
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

// A launch of a window: entries of one plan on pointer sets, listed contractions in a tile of the list rule (`tile`),
// listed depthwise kernels of one stride, or listed streams of one instance.
constexpr int kOnePlan = -1, kDepthwise = -2, kThin = -3;
// Workgroups that entries of different shapes share: a launch holds less than 2^32 threads, of workgroups of at most 1024.
constexpr int64_t kMaxSharedGrid = 1 << 21;
struct Launch {
    int tile, family; // (depthwise: the stride; streams: the pieces of the reduction)
    std::vector<int> entries; // of the window
};

class Window {
public:
    Window(std::vector<PreparedOp> &ops, bool as_recorded) : ops_(ops), as_recorded_(as_recorded) {}
    // Whether an entry may run at the same time as all others: neither writes what the other reads or writes.
    bool admits(const Entry &e) const
    {
        for (const Range &w : e.writes)
            if (written_.touches(w) || read_.touches(w)) return false;
        for (const Range &r : e.reads)
            if (written_.touches(r)) return false;
        return true;
    }
    void add(const Entry &e)
    {
        for (const Range &w : e.writes) written_.add(w);
        for (const Range &r : e.reads) read_.add(r);
        entries_.push_back(e);
    }
    bool empty() const { return entries_.empty(); }
    const std::vector<Entry> &entries() const { return entries_; }
    void clear() { entries_.clear(), written_.clear(), read_.clear(); }

    std::vector<Launch> launches() const
    {
        std::vector<Launch> out;
        int tiles = 0;
        list_tiles(&tiles);
        const int n = (int)entries_.size();
        std::vector<char> done(n, 0);
        for (int dt = 0; dt < 2 && !as_recorded_; ++dt)
            for (int family : {FAM_CONV, FAM_GEMM_TN}) {
                std::vector<int> members;
                for (int i = 0; i < n; ++i) {
                    const PreparedOp &op = ops_[entries_[i].op];
                    if (op.cls != TT_DWCONV_BIAS_RELU6 && op.g.dtype == dt && op.family == family && listable(op)) members.push_back(i);
                }
                if (dt == TT_F32 && family == FAM_GEMM_TN) stream(&members, &done, &out);
                if (members.size() < 2) continue;
                // (splits of one plan alone: nothing to share that their own launches would not)
                const PreparedOp &first = ops_[entries_[members[0]].op];
                const bool one_plan = std::all_of(members.begin(), members.end(), [&](int i) { return entries_[i].op == entries_[members[0]].op; });
                if (one_plan && first.launch.eff_split_k > 1) continue;
                list(members, dt, family, &done, &out);
            }
        for (int stride : {1, 2}) {
            if (as_recorded_) break;
            std::vector<int> members;
            DwListEntry e;
            for (int i = 0; i < n; ++i) {
                const PreparedOp &op = ops_[entries_[i].op];
                if (op.cls == TT_DWCONV_BIAS_RELU6 && op.d.stride_h == stride && dw_list_entry(op.d, &e)) members.push_back(i);
            }
            share(largest_first(members), kDepthwise, stride, kMaxDwListed,
                  [&](int i) { return dw_list_entry(ops_[entries_[i].op].d, &e) ? dw_workgroups(e) : 0; }, &done, &out);
        }
        // the rest: entries of one plan, all with a bias or all without, share a launch
        std::vector<Launch> plain;
        for (int i = 0; i < n; ++i) {
            if (done[i]) continue;
            Launch l{kOnePlan, 0, {i}};
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
        if (l.tile == kThin) {
            ThinList list;
            std::memset(&list, 0, sizeof list);
            for (size_t i = 0; i < l.entries.size(); ++i) {
                const Entry &e = entries_[l.entries[i]];
                const PreparedOp &op = ops_[e.op];
                ThinEntry &t = list.e[i];
                t = thin_entry(op);
                t.a = static_cast<const float *>(e.p.a), t.b = static_cast<const float *>(e.p.b), t.bias = static_cast<const float *>(e.p.bias);
                t.res = static_cast<const float *>(e.p.res), t.out = static_cast<float *>(e.p.out);
            }
            return launch_thin_list(list, (int)l.entries.size(), l.family, stream);
        }
        if (l.tile == kDepthwise) {
            DwList list;
            std::memset(&list, 0, sizeof list);
            for (size_t i = 0; i < l.entries.size(); ++i) {
                const Entry &e = entries_[l.entries[i]];
                (void)dw_list_entry(ops_[e.op].d, &list.e[i]);
                list.e[i].x = static_cast<const float *>(e.p.a), list.e[i].w = static_cast<const float *>(e.p.b);
                list.e[i].bias = static_cast<const float *>(e.p.bias), list.e[i].y = static_cast<float *>(e.p.out);
            }
            return launch_dw_list(list, (int)l.entries.size(), l.family, stream);
        }
        if (l.tile == kOnePlan) {
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
                int64_t grid = 0;
                const auto send = [&]() {
                    const int rc = count ? launch_reduce_list(list, count, dt, fours, stream) : TT_OK;
                    count = 0, grid = 0;
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
                        const int64_t outputs = (int64_t)pl.batch * pl.M * pl.N, wgs = (outputs / (fours ? 4 : 1) + 63) / 64;
                        if (count && grid + wgs > kMaxSharedGrid)
                            if (const int rc = send(); rc != TT_OK) return rc;
                        grid += wgs;
                        list.e[count++] = {static_cast<float *>(e.p.ws), e.p.bias, e.p.res, e.p.out, outputs,
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
    // Cuts entries into launches of at most `most`, and of no more workgroups than a shared launch holds.  An entry that
    // would be left with a launch to itself shares nothing: it is not done, and runs under its own record.
    template <typename Workgroups>
    static void share(const std::vector<int> &entries, int tile, int family, int most, Workgroups &&workgroups, std::vector<char> *done, std::vector<Launch> *out)
    {
        std::vector<int> launch;
        int64_t grid = 0;
        const auto close = [&]() {
            if (launch.size() > 1) {
                for (int i : launch) (*done)[i] = 1;
                out->push_back({tile, family, launch});
            }
            launch.clear(), grid = 0;
        };
        for (size_t i = 0; i < entries.size(); ++i) {
            const int64_t more = workgroups(entries[i]);
            const bool leaves_one = (int)launch.size() == most - 1 && entries.size() - i == 2; // the last two share one
            if ((int)launch.size() == most || leaves_one || grid + more > kMaxSharedGrid) close();
            launch.push_back(entries[i]), grid += more;
        }
        close();
    }
    std::vector<int> largest_first(std::vector<int> entries) const
    {
        std::stable_sort(entries.begin(), entries.end(), [&](int x, int y) { return ops_[entries_[x].op].out_bytes > ops_[entries_[y].op].out_bytes; });
        return entries;
    }
    // Takes the streams out of the members.
    void stream(std::vector<int> *members, std::vector<char> *done, std::vector<Launch> *out) const
    {
        for (int pieces : kThinPieces) {
            std::vector<int> streams;
            for (int i : *members)
                if (thin_pieces(ops_[entries_[i].op]) == pieces) streams.push_back(i);
            share(largest_first(streams), kThin, pieces, kMaxThin, [&](int i) { return thin_workgroups(thin_entry(ops_[entries_[i].op])); }, done, out);
        }
        members->erase(std::remove_if(members->begin(), members->end(), [&](int i) { return (*done)[i]; }), members->end());
    }
    void list(const std::vector<int> &members, int dt, int family, std::vector<char> *done, std::vector<Launch> *out) const
    {
        int n_tiles = 0;
        const ListTile *tiles = list_tiles(&n_tiles);
        std::vector<Kind> kinds;
        std::vector<int> kind_of(members.size());
        for (size_t m = 0; m < members.size(); ++m) {
            const PreparedOp &op = ops_[entries_[members[m]].op];
            size_t at = 0;
            while (at < kinds.size() && kinds[at].op != &op) ++at;
            kind_of[m] = (int)at;
            if (at == kinds.size()) {
                kinds.emplace_back();
                kinds[at].op = &op, kinds[at].count = 0;
            }
            ++kinds[at].count;
        }
        for (Kind &k : kinds) {
            k.bytes = k.count * ((double)k.op->a_bytes + k.op->b_bytes + k.op->out_bytes * (k.op->cls == TT_CONV2D_BIAS_ADD_RELU ? 2.0 : 1.0));
            const tt_plan &pl = k.op->launch;
            k.own_tile = -1;
            for (int t = 0; t < n_tiles; ++t) {
                if (tiles[t].dtype == dt && tiles[t].tile_m == pl.tile_m && tiles[t].tile_n == pl.tile_n && tiles[t].tile_k == pl.tile_k) k.own_tile = t;
                if (tiles[t].dtype != dt || (tiles[t].blocks && !block_tile_fits(*k.op))) {
                    k.in[t] = {kUnfit, kUnfit, kUnfit};
                    continue;
                }
                const Cut c = cut_into(*k.op, tiles[t]);
                k.in[t] = {c.tiles * c.us * k.count, c.us, c.alone_us};
            }
        }
        int best[kTilesAtOnce] = {-1, -1, -1};
        best_tiles(kinds, tiles, n_tiles, dt, best);
        std::vector<int> chosen(kinds.size());
        estimate(kinds, best, chosen.data());
        for (int t : best) {
            std::vector<int> at;
            for (size_t m = 0; m < members.size(); ++m)
                if (t >= 0 && chosen[kind_of[m]] == t) at.push_back((int)m);
            // the longest first, so that the end of the launch is not one long tile
            std::stable_sort(at.begin(), at.end(), [&](int x, int y) { return kinds[kind_of[x]].in[t].us > kinds[kind_of[y]].in[t].us; });
            for (int &m : at) m = members[m];
            share(at, t, family, kMaxListed, [&](int i) { return cut_into(ops_[entries_[i].op], tiles[t]).tiles; }, done, out);
        }
    }

    std::vector<PreparedOp> &ops_;
    const bool as_recorded_; // entries share launches of their own plan only
    std::vector<Entry> entries_;
    Ranges written_, read_;
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

constexpr size_t kMaxWindow = 128; // bounds what is planned before the first launch goes out

// Walks the list and hands every window to `emit` (window, whether its one entry runs `use_count` times).
template <typename Emit>
int walk(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, bool as_recorded, std::vector<PreparedOp> &ops, Emit &&emit)
{
    Window w(ops, as_recorded);
    std::vector<int> first; // of every plan, the entry it was laid out for
    int last = 0;           // the plan of the entry before
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
        const auto planned = [&](int plan) { return same_plan(kernels[first[plan]], scheds ? scheds[first[plan]] : nullptr, d, rec); };
        if (last >= (int)first.size() || !planned(last)) {
            for (last = 0; last < (int)first.size() && !planned(last);) ++last;
            if (last == (int)first.size()) {
                ops.emplace_back();
                if (const int rc = prepare_op(rec, d.cls, d.shape, &ops.back()); rc != TT_OK) {
                    ops.pop_back();
                    return fail(rc);
                }
                first.push_back(k);
            }
        }
        const PreparedOp &op = ops[last];
        if (!workspace_fits(op, p)) return fail(TT_ERR_WORKSPACE);
        if (refused(op)) return fail(TT_ERR_UNSUPPORTED);
        const Entry e = entry_at(k, last, op, p);
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

static int run_kernels(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, int repeat, bool as_recorded, void *stream)
{
    if (nk < 0 || repeat < 0 || (nk && !kernels)) return TT_ERR_BAD_ARG;
    return without_exceptions([&]() {
        std::vector<PreparedOp> ops;
        for (int r = 0; r < repeat; ++r) {
            ops.clear();
            const int rc = walk(kernels, scheds, nk, as_recorded, ops, [&](Window &w, int times) {
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

extern "C" int tt_run_kernels(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, int repeat, void *stream)
{
    return run_kernels(kernels, scheds, nk, repeat, false, stream);
}

extern "C" int tt_run_kernels_as_recorded(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, int repeat, void *stream)
{
    return run_kernels(kernels, scheds, nk, repeat, true, stream);
}

extern "C" int tt_debug_list(const tt_kernel_desc *kernels, const tt_schedule *const *scheds, int nk, tt_listed *out)
{
    if (nk < 0 || (nk && (!kernels || !out))) return TT_ERR_BAD_ARG;
    return without_exceptions([&]() {
        std::vector<PreparedOp> ops;
        for (int k = 0; k < nk; ++k) out[k] = {-1, 0, 0, 0, 0, 0, 0};
        int launch = 0, tiles = 0;
        const ListTile *table = list_tiles(&tiles);
        return walk(kernels, scheds, nk, false, ops, [&](Window &w, int) {
            for (const Launch &l : w.launches()) {
                tt_listed as = {launch, l.tile != kOnePlan, 16, 16, l.family * 16, (int32_t)l.entries.size(), TT_LISTED_STREAM};
                if (l.tile >= 0) {
                    const ListTile &t = table[l.tile];
                    as.tile_m = t.tile_m, as.tile_n = t.tile_n, as.tile_k = t.tile_k, as.kernel = TT_LISTED_TILES;
                } else if (l.tile == kDepthwise) {
                    const DwWindow w = dw_list_window(l.family);
                    as.tile_m = w.rows, as.tile_n = w.columns, as.tile_k = 4, as.kernel = TT_LISTED_DEPTHWISE;
                } else if (l.tile == kOnePlan) { // (one plan for all of its entries)
                    const tt_plan &pl = ops[w.entries()[l.entries[0]].op].launch;
                    as.tile_m = pl.tile_m, as.tile_n = pl.tile_n, as.tile_k = pl.tile_k, as.kernel = TT_LISTED_RECORD;
                }
                for (int i : l.entries) out[w.entries()[i].index] = as;
                ++launch;
            }
            w.clear();
            return (int)TT_OK;
        });
    });
}
