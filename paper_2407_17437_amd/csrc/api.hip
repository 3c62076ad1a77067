// C ABI of the sparse MLP training step: argument checking, layer / MLP handles, the
// one-off mirror build, and the kernel sequence of a training step.
#include "../../include/nerva_sparse.h"
#include "../../include/nerva_sparse_bench.h"

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <algorithm>
#include <climits>
#include <atomic>
#include <functional>
#include <mutex>
#include <vector>

#include "kernels.h"

using namespace nerva;

// Workspace of mlp_train_step_static: one array per GPU, part of the library's code object, held
// from the moment the library is loaded on a device until the process ends.  In host code the
// name is only a handle for hipGetSymbolAddress; the device address it yields (one per device) is
// what kernels, copies and fills are given.
constexpr size_t kStaticScratchBytes = NERVA_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each device, once resolved
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (resolved once per device, with that device current).
hipError_t static_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

thread_local std::string g_last_error;
std::atomic<int> g_partition_mode{0};  // see nerva_set_partition_mode

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    (void)hipGetLastError();   // reported here: the runtime keeps it, and the next launch that asks must not find it
    return fail(NERVA_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(expr)                                        \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);    \
    } while (0)

inline hipStream_t as_stream(void *s) { return static_cast<hipStream_t>(s); }
inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

}  // namespace

// What a bound pattern owns on the device besides scratch: the mirror and the partition tables.  A
// layer keeps two sets: sparse_linear_rebind builds the new pattern's structures in the spare set while
// the current one stays valid, and swaps on success; buffers are reused when large enough, so
// repeated topology updates do not allocate.
struct PatternBuffers {
    int32_t *indptr_t = nullptr;    // [cols + 1]
    int32_t *mirror_mem = nullptr;  // indices_t | perm | pos_t | values_t, round_up(nnz, 64) elements each
    size_t mirror_ints = 0;
    int32_t *plan_mem = nullptr;    // tables of both orientations
    size_t plan_ints = 0;
    int32_t *table = nullptr;       // pattern table, 2 ints per row and 32 columns
    size_t table_ints = 0;
    bool has_table = false;         // it holds the pattern (else the layer is too sparse for it)
    int32_t *row_table = nullptr;   // the same of the dense rows alone (DenseRows)
    size_t row_table_ints = 0;
    float *row_partial = nullptr;   // sliced results of their product, and its operand's parts
    size_t row_partial_floats = 0;
    int32_t *whole_staged = nullptr;   // staged plan of all rows beside that of the rows that are not dense
    size_t whole_staged_ints = 0;
    int32_t *hot = nullptr;         // entry | at | perm of HotRows | mirror values in that order | sets | scratch of launch_hot_order
    size_t hot_ints = 0;
    DenseSplit split{};             // views into plan_mem and row_table
};

enum HotState { kHotUnordered, kHotOnItsWay, kHotOrdered };   // the entries in the order of HotRows

struct nerva_layer {
    int32_t rows = 0, cols = 0, nnz = 0, activation = 0, max_batch = 0;
    // caller-owned
    const int32_t *indptr = nullptr;
    const int32_t *indices = nullptr;
    float *values = nullptr;
    float *bias = nullptr;
    // owned: CSR of W^T and the position maps (views into cur.mirror_mem / cur.indptr_t)
    PatternBuffers cur, spare;
    int32_t *indptr_t = nullptr;   // [cols+1]
    int32_t *indices_t = nullptr;  // [nnz] row index of each mirror entry
    float *values_t = nullptr;     // [nnz]
    int32_t *perm = nullptr;       // [nnz] mirror position -> CSR position
    int32_t *pos_t = nullptr;      // [nnz] CSR position -> mirror position
    // static work partitions of W (by rows) and of the mirror (by W's columns): views into cur.plan_mem
    RowBlocks plan{}, plan_t{};
    Strips strips;                  // segs nullptr: none
    HotRows hot;                    // entry nullptr: none
    HotState hot_state = kHotUnordered;
    hipEvent_t hot_event = nullptr; // after the launches that put the entries in that order (order_hot_rows)
    bool hot_at_bind = true;        // made as a pattern is bound: the first one, and the next after a call that has taken it
    // owned scratch of the set-up kernels, and what they report (pinned host memory)
    int32_t *build_work = nullptr;
    size_t build_work_ints = 0;
    BindResult *bind_result = nullptr;
    // owned: partial rows of huge-row work-groups, shared by the forward and the transposed product
    float *scratch = nullptr;
    size_t scratch_floats = 0;
    int64_t scratch_ld = 0;
    // owned: tickets of the huge rows (SpmmArgs::tickets), 0 but while a product runs
    int32_t *tickets = nullptr;
    size_t ticket_ints = 0;
    // owned: stream of a forward product in strips (SpmmCall::strip_stream), or nullptr
    float *strip_stream = nullptr;
    size_t strip_floats = 0;
    // owned: per-tile partial products of the SDDMM and of the backward pass on one gather stream, as many tiles as
    // they take at any batch up to max_batch; fewer or none where there was no room for them
    float *partial = nullptr;
    size_t partial_floats = 0;
    int64_t partial_stride = 0, partial_db_at = 0;
    int32_t partial_tiles = 0;
    // owned, only for a ReLU layer with entries enough: dZ of a stand-alone backward pass, (rows, dz_ld); nullptr: too large to be
    // worth it, or no room
    float *dz = nullptr;
    size_t dz_floats = 0;
    int64_t dz_ld = 0;
    // owned, only on the dense route (sparse_linear_enable_dense, or chosen when the pattern was bound): a
    // zero-filled dense copy of W (rows x dense_ld, dense_ld = cols rounded up to kDenseLdAlign)
    bool dense_on = false;
    float *dense = nullptr;
    int64_t dense_ld = 0;
    float *dense_shares = nullptr;   // behind it, scratch of its forward product (DenseArgs::tickets, then ::partial), or nullptr
    // owned, only for a matrix that stores every entry and has at most kFullMaxRows rows
    bool full = false;               // the bound pattern is such a matrix
    float *full_scratch = nullptr;   // slice partials of the streaming product, (slices * rows, full_scratch_ld); kept once allocated, nullptr: no room
    size_t full_scratch_floats = 0;
    int64_t full_scratch_ld = 0;
    // values_t lags behind values[]: a training step updated this layer as the first layer of an MLP,
    // whose mirror no product reads, and left the mirror's values alone.  Whoever reads values_t next
    // (a step that has the layer further up, sparse_linear_backward, sparse_linear_sync_values)
    // refreshes it first.
    bool mirror_stale = false;
};

// Optional per-kernel timing of mlp_train_step: one HIP event before every launch and one after
// the last launch of each of the first `max_steps` steps after mlp_profile_enable.  A launch's
// time is the span to the next event: kernels of a step run back to back on one stream, so the
// spans add up to the step and each carries the cost of one event, not two.
struct StepProfiler {
    bool on = false;
    int32_t max_steps = 0, step = 0, slot = 0;
    std::vector<std::string> names;    // one per launch of a step, in launch order
    std::vector<hipEvent_t> events;    // [step][slot 0 .. n, end of step], grown while recording
    void release()
    {
        for (hipEvent_t e : events) (void)hipEventDestroy(e);
        events.clear();
        names.clear();
        on = false;
        step = slot = 0;
    }
};

struct nerva_mlp {
    std::vector<nerva_layer *> layers;
    std::vector<float *> vel;
    std::vector<float *> bias_vel;
    int32_t max_batch = 0;
    int32_t flags = 0;
    // fused head of a small output layer: per-column losses [max_batch]
    bool head = false;
    float *head_scratch = nullptr;
    StepProfiler prof;
};

namespace {

// Offsets of a step's intermediates.  Filled on every call, so it takes no heap memory for networks of up to
// kInlineLayers layers (four vectors cost 0.7 us per call, next to steps of 20 us).
constexpr int kInlineLayers = 16;
struct Layout {
    struct Offsets { int64_t A, dZ, g, db; };
    int64_t ld = 0, bytes = 0;
    Offsets inline_[kInlineLayers];
    std::vector<Offsets> more_;
    Offsets &operator[](size_t l) { return l < kInlineLayers ? inline_[l] : more_[l - kInlineLayers]; }
    const Offsets &operator[](size_t l) const { return l < kInlineLayers ? inline_[l] : more_[l - kInlineLayers]; }
};

void make_layout(const nerva_mlp *m, int32_t batch, Layout &L)
{
    if (m->layers.size() > kInlineLayers) L.more_.resize(m->layers.size() - kInlineLayers);
    L.ld = round_up(batch, 32);  // rows start on 128-byte boundaries
    int64_t off = 0;
    auto take = [&](int64_t floats) {
        int64_t o = off;
        off += round_up(floats * 4, 256);
        return o;
    };
    for (size_t k = 0; k < m->layers.size(); ++k) {
        const nerva_layer *l = m->layers[k];
        L[k].A = take(static_cast<int64_t>(l->rows) * L.ld);
        L[k].dZ = take(static_cast<int64_t>(l->rows) * L.ld);
        L[k].g = take(l->nnz);
        L[k].db = take(l->rows);
    }
    L.bytes = off;
}

// Rows by stored entries descending, ties by row id: one counting sort, O(rows + longest row), that
// every partition of a pattern is then read off from.
struct RowsByLength {
    std::vector<int32_t> order;
    int32_t longest = 0;
};

RowsByLength rows_by_length(int32_t rows, const int32_t *indptr)
{
    RowsByLength R;
    for (int32_t i = 0; i < rows; ++i) R.longest = std::max(R.longest, indptr[i + 1] - indptr[i]);
    std::vector<int32_t> start(static_cast<size_t>(R.longest) + 2, 0);
    for (int32_t i = 0; i < rows; ++i) ++start[R.longest - (indptr[i + 1] - indptr[i]) + 1];
    for (size_t k = 1; k < start.size(); ++k) start[k] += start[k - 1];
    R.order.resize(rows);
    for (int32_t i = 0; i < rows; ++i) R.order[start[R.longest - (indptr[i + 1] - indptr[i])]++] = i;
    return R;
}

// Rows are grouped by the number of waves that share one row: 2^lg, the smallest power of two
// that leaves each wave at most `target` stored entries, target = nnz / 4096 kept within 8..64
// (measured: with every gather of a pass in flight, fewer and longer shares beat more waves).  A
// row of more than 4 * kWavesPerBlock * huge_target entries is huge: it is cut into work-groups
// of at most 2 * kWavesPerBlock * huge_target entries each, huge_target = nnz / 16384 within
// 8..64 -- finer than `target`, because the few huge rows decide the run time and need many
// work-groups (a dense 10 x 8192 layer: 320 work-groups instead of 130).
struct RowPlan {
    std::vector<int32_t> row_order;  // ordinary rows
    std::vector<int32_t> blocks;     // 4 ints per work-group, huge ones first
    std::vector<int32_t> huge_rows;  // 4 ints per huge row
    std::vector<int32_t> waves;      // 4 ints per wave, kWavesPerBlock waves per work-group
    int32_t n_huge_blocks = 0;
    int32_t n_blocks() const { return static_cast<int32_t>(blocks.size() / 4); }
    int32_t n_huge_rows() const { return static_cast<int32_t>(huge_rows.size() / 4); }
};

// skip_upto >= 0: rows with at most that many entries are left out (they go to the packed path);
// only_upto: rows with more entries than that are left out (they go to the staged kernels).
RowPlan plan_rows(int32_t rows, const int32_t *indptr, const RowsByLength &by_len, int32_t skip_upto = -1, int32_t only_upto = INT32_MAX)
{
    RowPlan P;
    const int64_t nnz = indptr[rows];
    // entries per wave aimed at: ordinary rows, and (finer, for more work-groups on the few rows
    // that decide the run time) the shares of huge rows
    int64_t target = nnz / 4096;
    if (target < 8) target = 8;
    if (target > 64) target = 64;
    int64_t huge_target = nnz / 16384;
    if (huge_target < 8) huge_target = 8;
    if (huge_target > 64) huge_target = 64;
    const int64_t block_cap = huge_target * kWavesPerBlock;
    int max_lg = 0;
    while ((1 << max_lg) < kWavesPerBlock) ++max_lg;
    std::vector<int8_t> ordinary(rows);
    std::vector<int32_t> count(max_lg + 1, 0);
    const bool row_split_only = g_partition_mode.load() == NERVA_PARTITION_ROW_SPLIT;
    int32_t n_ordinary = 0;
    for (int32_t i = 0; i < rows; ++i) {   // huge rows keep row order: their work-groups are also their scratch slots
        const int64_t n = indptr[i + 1] - indptr[i];
        ordinary[i] = 0;
        if (n <= skip_upto || n > only_upto) continue;
        if (!row_split_only && n > 4 * block_cap) {
            const int32_t parts = static_cast<int32_t>((n + 2 * block_cap - 1) / (2 * block_cap));
            const int64_t share = (n + parts - 1) / parts;
            const int32_t first = P.n_blocks();
            for (int32_t q = 0; q < parts; ++q) {
                const int64_t b = indptr[i] + q * share;
                const int64_t e = b + share < indptr[i + 1] ? b + share : indptr[i + 1];
                P.blocks.insert(P.blocks.end(), {NERVA_HUGE_FLAG | q, i, static_cast<int32_t>(b), static_cast<int32_t>(e)});
            }
            P.huge_rows.insert(P.huge_rows.end(), {i, first, parts, 0});
            continue;
        }
        int lg = 0;
        if (!row_split_only)   // (plain row splitting: one wave per row whatever its length)
            while (lg < max_lg && (n + (1 << lg) - 1) / (1 << lg) > target) ++lg;
        ordinary[i] = 1;
        ++count[lg];
        ++n_ordinary;
    }
    P.n_huge_blocks = P.n_blocks();
    // A class whose rows do not fill its last work-group hands that work-group's rows (its longest)
    // to the next class, twice the waves per row, if that class's own last work-group has room for
    // them: one work-group fewer to schedule.  (The 1024 x 3072
    // layer of the paper's MLP at 90 % sparsity has 1023 rows of one class and 1 of the next: 513
    // work-groups on a chip that holds 512 at a time.)  The class is monotone in the row's length, so
    // in the order "longest first" every class is one run of rows and the rows handed up are the
    // first of their class's run: only the counts move.
    if (!row_split_only && skip_upto < 0 && only_upto == INT32_MAX) {
        for (int lg = 0; lg < max_lg; ++lg) {
            const int32_t left_over = count[lg] % (kWavesPerBlock >> lg), above = kWavesPerBlock >> (lg + 1);
            // ... where the next class has room for them in a work-group it needs anyway
            if (!left_over || (count[lg + 1] + left_over + above - 1) / above != (count[lg + 1] + above - 1) / above) continue;
            count[lg] -= left_over;
            count[lg + 1] += left_over;
        }
    }
    // ordinary rows longest first, ties in row order: the classes follow each other, heaviest first, and
    // inside a class the rows of a work-group are alike and the work-groups that take longest start first
    P.row_order.reserve(n_ordinary);
    for (int32_t r : by_len.order)
        if (ordinary[r]) P.row_order.push_back(r);
    {
        int32_t f = 0;
        for (int lg = max_lg; lg >= 0; --lg) {
            const int32_t end = f + count[lg], per_block = kWavesPerBlock >> lg;
            for (; f < end; f += per_block) {
                const int32_t n_rows = end - f < per_block ? end - f : per_block;
                P.blocks.insert(P.blocks.end(), {lg | (n_rows << 8), f, 0, 0});
            }
            f = end;
        }
    }
    // The same partition per wave: each of the 2^lg waves of a row takes a contiguous share of
    // its entries, a multiple of 4 entries long (the kernels work on 1, 2 or 4 entries at a time).
    P.waves.resize(P.blocks.size() * kWavesPerBlock);
    int32_t *out = P.waves.data();
    for (int32_t b = 0; b < P.n_blocks(); ++b) {
        const int32_t info = P.blocks[4 * b], y = P.blocks[4 * b + 1];
        const bool huge = (info & NERVA_HUGE_FLAG) != 0;
        const int lg = huge ? max_lg : (info & 0xff);
        for (int w = 0; w < kWavesPerBlock; ++w) {
            const int part = w & ((1 << lg) - 1);
            int32_t row = -1;
            int64_t p0 = 0, p1 = 0;
            bool lead = false;
            if (huge) {
                row = y; p0 = P.blocks[4 * b + 2]; p1 = P.blocks[4 * b + 3];
                lead = w == 0 && (info & ~NERVA_HUGE_FLAG) == 0;
            } else if ((w >> lg) < (info >> 8)) {
                row = P.row_order[y + (w >> lg)];
                p0 = indptr[row]; p1 = indptr[row + 1];
                lead = part == 0;
            }
            int64_t per = ((p1 - p0) + (1 << lg) - 1) >> lg;
            per = (per + 3) / 4 * 4;
            const int64_t s0 = p0 + part * per < p1 ? p0 + part * per : p1;
            const int64_t s1 = s0 + per < p1 ? s0 + per : p1;
            *out++ = row;
            *out++ = static_cast<int32_t>(s0);
            *out++ = static_cast<int32_t>(s1);
            *out++ = part | (lg << 4) | (lead ? 256 : 0) | (huge ? 512 : 0);
        }
    }
    return P;
}

// Rows of at most kPackMaxLen entries, longest first (ties in row order), 4 ints per row
// {row, first entry, entries, 0}, padded with {-1, 0, 0, 0} to a multiple of 64 rows.  Empty when
// there are fewer than kPackMinRows of them: the packed path pays off on large matrices only.
std::vector<int32_t> short_row_table(int32_t rows, const int32_t *indptr, const RowsByLength &by_len, int32_t *n_short)
{
    int32_t n = 0;
    for (int32_t i = 0; i < rows; ++i) n += indptr[i + 1] - indptr[i] <= kPackMaxLen;
    *n_short = 0;
    std::vector<int32_t> t;
    if (n < kPackMinRows || indptr[rows] == 0 || g_partition_mode.load() == NERVA_PARTITION_ROW_SPLIT) return t;
    t.assign(static_cast<size_t>(round_up(n, 64)) * 4, 0);
    for (int64_t k = n; k < round_up(n, 64); ++k) t[4 * k] = -1;
    int32_t k = 0;
    for (int32_t i : by_len.order) {
        const int32_t len = indptr[i + 1] - indptr[i];
        if (len > kPackMaxLen) continue;
        t[4 * k] = i; t[4 * k + 1] = indptr[i]; t[4 * k + 2] = len;
        ++k;
    }
    *n_short = n;
    return t;
}

// Row ranges and slot order of the staged product (RowBlocks::staged_*) for a matrix whose products
// run at up to max_batch columns; empty when that product would never be chosen.  The segment
// bounds (`ends`) depend on the column indices: the host API fills them here, a layer on the device.
struct StagedPlan {
    std::vector<int32_t> rows;    // [ranges * kStageRangeRows]
    std::vector<int32_t> ends;    // [ranges * (cblocks + 1) * kStageRangeRows] (host API only)
    std::vector<int32_t> groups;  // [ranges]
    int32_t ranges = 0, cblocks = 0;
    int32_t longest_share = 0;    // most entries any one slot serves
    int32_t n_rows = 0;           // rows the plan covers
    int64_t nnz = 0;              // and their stored entries
    size_t ends_ints() const { return static_cast<size_t>(ranges) * (cblocks + 1) * kStageRangeRows; }
};

StagedPlan plan_staged(int32_t all_rows, int32_t cols, const int32_t *indptr, const RowsByLength &by_len, int32_t max_batch,
                       int32_t min_len = 0)
{
    StagedPlan H;
    // the rows the plan covers: all of them, or those of at least min_len stored entries
    std::vector<int32_t> covered;
    int64_t nnz = 0;
    for (int32_t r = 0; r < all_rows; ++r)
        if (indptr[r + 1] - indptr[r] >= min_len) {
            covered.push_back(r);
            nnz += indptr[r + 1] - indptr[r];
        }
    const int32_t rows = static_cast<int32_t>(covered.size());  // from here on: rows of the plan, covered[k] their ids
    const int32_t want = staged_ranges_wanted(rows, nnz, cols, max_batch, g_partition_mode.load(), staged_range_bound(all_rows, cols, max_batch));
    if (want == 0) return H;
    const int32_t cblocks = (cols + kStageRows - 1) / kStageRows;
    // ranges of about equal cost: a stored entry costs one gather, a segment about two more
    auto cost = [&](int32_t r) {
        const int64_t len = indptr[r + 1] - indptr[r];
        return len + 2 * (len < cblocks ? len : cblocks) + 1;
    };
    int64_t total = 0;
    for (int32_t k = 0; k < rows; ++k) total += cost(covered[k]);
    // A row of 16 lanes serves a row alone.  A row much longer than a wave's fair share of its range
    // would make that wave the range's critical path: it gets the four lane rows of a wave instead, each a
    // quarter of every segment ("quad": four slots, group-aligned).
    const int64_t quad_len = std::max<int64_t>(256, total / want / 32);
    auto slots_of = [&](int32_t r) { return indptr[r + 1] - indptr[r] >= quad_len ? 4 : 1; };
    // a range begins where the row's share of the total cost does, and after every kStageRangeFill slots of a share
    std::vector<int32_t> range_of(all_rows, -1);
    int32_t ranges = 0;
    {
        int32_t last_cut = -1, last_part = 0, slots = 0;
        int64_t done = 0;
        for (int32_t k = 0; k < rows; ++k) {
            const int32_t r = covered[k], cut = staged_cut(done, want, total);
            if (cut != last_cut) slots = 0;
            const int32_t part = slots / kStageRangeFill;
            if (cut != last_cut || part != last_part) ++ranges;
            last_cut = cut;
            last_part = part;
            done += cost(r);
            slots += slots_of(r);
            range_of[r] = ranges - 1;
        }
    }
    H.ranges = ranges;
    H.cblocks = cblocks;
    H.n_rows = rows;
    H.nnz = nnz;
    H.rows.assign(static_cast<size_t>(ranges) * kStageRangeRows, -1);
    H.groups.assign(ranges, 0);
    // inside a range: longest first, ties in row order -- the global order, read range by range;
    // quads come first (the longest rows), so they start at multiples of 4
    std::vector<int32_t> slot(ranges, 0);
    for (int32_t r : by_len.order) {
        const int32_t q = range_of[r];
        if (q < 0) continue;
        const int32_t copies = slots_of(r), len = indptr[r + 1] - indptr[r];
        const int32_t share = copies == 4 ? (len + 3) / 4 : len;
        if (share > H.longest_share) H.longest_share = share;
        for (int32_t c = 0; c < copies; ++c)
            H.rows[static_cast<size_t>(q) * kStageRangeRows + slot[q] + c] = copies == 4 ? (r | kStageQuad) : r;
        slot[q] += copies;
    }
    for (int32_t q = 0; q < ranges; ++q) H.groups[q] = (slot[q] + 63) / 64;
    return H;
}

// the segment bounds of a plan from host copies of the pattern (what plan_cuts_kernel computes for a layer)
void fill_staged_ends_host(StagedPlan &H, const int32_t *indptr, const int32_t *indices)
{
    H.ends.assign(H.ends_ints(), 0);
    for (int32_t q = 0; q < H.ranges; ++q) {
        int32_t *e = H.ends.data() + static_cast<size_t>(q) * (H.cblocks + 1) * kStageRangeRows;
        for (int32_t slot = 0; slot < kStageRangeRows; ++slot) {
            int32_t r = H.rows[static_cast<size_t>(q) * kStageRangeRows + slot];
            if (r < 0) continue;
            r &= ~kStageQuad;
            const int32_t *lo = indices + indptr[r], *hi = indices + indptr[r + 1];
            for (int32_t b = 0; b <= H.cblocks; ++b) {
                if (b > 0) lo = std::lower_bound(lo, hi, b * kStageRows);
                e[static_cast<size_t>(b) * kStageRangeRows + slot] = static_cast<int32_t>(lo - indices);
            }
        }
    }
}

// Sizes of the tables of one orientation, from bounds that hold for every pattern with these row and entry counts:
// the tables are laid out before the planner, which runs on the device, has counted anything.
struct PlanRoom {
    int64_t blocks, long_blocks, rest_blocks, huge_rows, rows_by_length, dense_rows = 0, dense_flags = 0, strip_sets = 0;
    int32_t ranges, cblocks, strip_blocks = 0;
    PlanRoom(int32_t rows, int32_t other, int64_t nnz, int32_t max_batch, bool strips = false, int32_t dense_len = INT32_MAX)
    {
        if (strips) {
            strip_blocks = strip_blocks_of(other);
            strip_sets = (static_cast<int64_t>(rows) + kStripSet - 1) / kStripSet;
        }
        if (dense_len < INT32_MAX) {
            dense_rows = round_up(std::min<int64_t>(rows, nnz / dense_len), 4);
            dense_flags = round_up(rows, 16) / 4;
        }
        const int64_t target = std::min<int64_t>(std::max<int64_t>(nnz / 4096, 8), 64);
        const int64_t cap = std::min<int64_t>(std::max<int64_t>(nnz / 16384, 8), 64) * kWavesPerBlock;
        // a row's waves number 1 or fewer than 2 * entries / target; a class ends in a work-group that may not be full
        auto room = [&](int64_t n_rows, int64_t n) { return n_rows / kWavesPerBlock + n / (8 * target) + 8; };
        huge_rows = nnz / (4 * cap) + 1;
        const int64_t huge_blocks = nnz / (2 * cap) + huge_rows;
        blocks = room(rows, nnz) + huge_blocks;
        const bool packed = rows >= kPackMinRows;
        long_blocks = packed ? room(std::min<int64_t>(rows, nnz / kPackMaxLen), nnz) + huge_blocks : 0;
        rest_blocks = packed ? room(rows, std::min<int64_t>(nnz, static_cast<int64_t>(rows) * kPackMaxLen)) : 0;
        rows_by_length = rows_table_size(rows);
        ranges = staged_range_bound(rows, other, max_batch);
        cblocks = (other + kStageRows - 1) / kStageRows;
    }
    size_t staged_ints() const { return static_cast<size_t>(ranges) * (kStageRangeRows * (cblocks + 2) + 4); }
    size_t ints() const
    {
        return static_cast<size_t>(4 * (kWavesPerBlock * (blocks + long_blocks + rest_blocks) + huge_rows + rows_by_length)) +
               static_cast<size_t>(strip_sets * (2 * strip_blocks + kStripSet * (strip_blocks + 2))) + staged_ints() + static_cast<size_t>(dense_rows + dense_flags) +
               (dense_flags ? static_cast<size_t>(4 * kWavesPerBlock * (blocks + long_blocks)) : 0);
    }
    // the tables at `mem` (16-byte records first)
    PlanTables at(int32_t *mem) const
    {
        PlanTables t;
        int4 *r = reinterpret_cast<int4 *>(mem);
        t.waves = r; r += kWavesPerBlock * blocks;
        t.long_waves = r; r += kWavesPerBlock * long_blocks;
        t.rest_waves = r; r += kWavesPerBlock * rest_blocks;
        t.huge_rows = r; r += huge_rows;
        t.rows_by_length = r; r += rows_by_length;
        t.other_waves = t.other_long_waves = nullptr;
        if (dense_flags) {
            t.other_waves = r; r += kWavesPerBlock * blocks;
            t.other_long_waves = r; r += kWavesPerBlock * long_blocks;
        }
        int32_t *i = reinterpret_cast<int32_t *>(r);
        t.strip_segs = reinterpret_cast<int2 *>(i); i += 2 * strip_sets * strip_blocks;
        t.strip_cuts = i; i += strip_sets * kStripSet * (strip_blocks + 1);
        t.strip_rows = i; i += strip_sets * kStripSet;
        t.dense_rows = i; i += dense_rows;
        t.dense_flag = reinterpret_cast<uint8_t *>(i); i += dense_flags;
        staged_at(t, i);
        return t;
    }
    void staged_at(PlanTables &t, int32_t *i) const
    {
        t.staged_rows = i; i += static_cast<size_t>(ranges) * kStageRangeRows;
        t.staged_ends = i; i += static_cast<size_t>(ranges) * kStageRangeRows * (cblocks + 1);
        t.staged_groups = i;
    }
};

// RowBlocks of one orientation from what the planner reports of it; hot_nnz: entries of the most referenced operand rows
RowBlocks plan_view(const PlanTables &t, const PlanCounts &c, int32_t other, int32_t nnz, int32_t other_hot_nnz, int32_t mode)
{
    RowBlocks v{};
    v.huge_rows = t.huge_rows; v.waves = t.waves; v.long_waves = t.long_waves; v.rest_waves = t.rest_waves;
    v.n_blocks = c.n_blocks; v.n_huge_rows = c.n_huge_rows; v.n_huge_blocks = c.n_huge_blocks;
    v.n_short = c.n_short; v.n_long_blocks = c.n_long_blocks; v.n_rest_blocks = c.n_rest_blocks; v.long_nnz = c.long_nnz;
    v.hot_share = nnz == 0 ? 0.f : other <= kHotRows ? 1.f : static_cast<float>(static_cast<double>(other_hot_nnz) / static_cast<double>(nnz));
    v.staged_ranges = c.staged_ranges;
    v.staged_cblocks = c.staged_ranges ? (other + kStageRows - 1) / kStageRows : 0;
    v.staged_rows = c.staged_ranges ? t.staged_rows : nullptr;
    v.staged_ends = c.staged_ranges ? t.staged_ends : nullptr;
    v.staged_groups = c.staged_ranges ? t.staged_groups : nullptr;
    v.staged_longest_share = c.staged_longest_share;
    v.staged_longest_row = c.longest_row;
    v.staged_partial = c.staged_partial;
    v.staged_row_count = c.staged_rows;
    v.staged_nnz = c.staged_nnz;
    v.rows_by_length = t.rows_by_length;
    v.short_rows = t.rows_by_length + (c.n_short > 0 ? c.n_long_rows : 0);
    v.staged_preferred = mode == NERVA_PARTITION_PREFER_STAGED;
    return v;
}

void free_pattern_buffers(PatternBuffers &b)
{
    (void)hipFree(b.indptr_t);
    (void)hipFree(b.mirror_mem);
    (void)hipFree(b.plan_mem);
    (void)hipFree(b.table);
    (void)hipFree(b.row_table);
    (void)hipFree(b.row_partial);
    (void)hipFree(b.whole_staged);
    (void)hipFree(b.hot);
    b = PatternBuffers{};
}

void free_layer_buffers(nerva_layer *l)
{
    free_pattern_buffers(l->cur);
    free_pattern_buffers(l->spare);
    (void)hipFree(l->build_work);
    if (l->bind_result) (void)hipHostFree(l->bind_result);
    if (l->hot_event) (void)hipEventDestroy(l->hot_event);
    (void)hipFree(l->scratch);
    (void)hipFree(l->tickets);
    (void)hipFree(l->strip_stream);
    (void)hipFree(l->partial);
    (void)hipFree(l->dz);
    (void)hipFree(l->dense);
    (void)hipFree(l->full_scratch);
}

// Room for `need` elements of 4 bytes in *ptr, whose capacity is *have: kept if large enough, else
// replaced by a larger allocation (the old contents are not kept; the new ones are 0 if `zeroed`; an eighth more than asked for if
// `spare`, for the patterns to come).  On failure nothing changes.
template <typename T>
hipError_t reserve(T **ptr, size_t *have, size_t need, bool zeroed = false, hipStream_t s = nullptr, bool spare = true)
{
    if (need <= *have && *ptr) return hipSuccess;
    if (need == 0) need = 1;
    const size_t want = need + (spare ? need / 8 : 0);
    void *fresh = nullptr;
    hipError_t e = hipMalloc(&fresh, want * 4);
    if (e != hipSuccess) return e;
    if (zeroed) {
        e = hipMemsetAsync(fresh, 0, want * 4, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            (void)hipFree(fresh);
            return e;
        }
    }
    (void)hipFree(*ptr);
    *ptr = static_cast<T *>(fresh);
    *have = want;
    return hipSuccess;
}

// The same for a buffer that the layer can do without: whether there was room for it.
template <typename T>
bool reserve_optional(T **ptr, size_t *have, size_t need, bool spare = true)
{
    if (reserve(ptr, have, need, false, nullptr, spare) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}

// Marks the start of one launch with an event while profiling is on; costs one branch otherwise.
struct Timed {
    StepProfiler &P;
    hipStream_t s;
    bool live;
    Timed(StepProfiler &p, hipStream_t st, const char *kind, int layer) : P(p), s(st), live(p.on && p.step < p.max_steps)
    {
        if (!live) return;
        if (P.step == 0) {
            char buf[64];
            snprintf(buf, sizeof buf, "%s[%d]", kind, layer);
            P.names.push_back(buf);
        }
        hipEvent_t b = nullptr;
        if (hipEventCreate(&b) != hipSuccess) { live = false; return; }
        P.events.push_back(b);
        (void)hipEventRecord(b, s);
    }
};

int check_batch(int32_t batch, int32_t ld, const char *name)
{
    if (batch <= 0) return fail(NERVA_ERR_ARGUMENT, "batch must be positive (got %d)", batch);
    if (ld < batch) return fail(NERVA_ERR_SHAPE, "%s = %d is smaller than batch = %d", name, ld, batch);
    if (ld >= (1 << 30)) return fail(NERVA_ERR_SHAPE, "%s = %d: rows of 4 GiB or more are not supported", name, ld);
    return NERVA_OK;
}

}  // namespace

extern "C" {

const char *nerva_last_error(void) { return g_last_error.c_str(); }

const char *nerva_build_info(void) { return "nerva_sparse 0.1 gfx950 fp32/int32"; }

int nerva_validate_csr_host(int32_t rows, int32_t cols, int64_t nnz, const int32_t *indptr,
                            const int32_t *indices)
{
    if (rows < 0 || cols < 0 || nnz < 0) return fail(NERVA_ERR_ARGUMENT, "negative size");
    if (!indptr || (nnz > 0 && !indices)) return fail(NERVA_ERR_ARGUMENT, "null pattern array");
    if (nnz > INT32_MAX) return fail(NERVA_ERR_ARGUMENT, "nnz does not fit int32 indices");
    if (indptr[0] != 0) return fail(NERVA_ERR_CSR, "indptr[0] = %d, expected 0", indptr[0]);
    for (int32_t i = 0; i < rows; ++i) {
        const int64_t b = indptr[i], e = indptr[i + 1];
        if (e < b) return fail(NERVA_ERR_CSR, "indptr decreases at row %d", i);
        if (e > nnz) return fail(NERVA_ERR_CSR, "indptr[%d] = %lld exceeds nnz = %lld", i + 1, (long long)e, (long long)nnz);
        for (int64_t p = b; p < e; ++p) {
            const int32_t j = indices[p];
            if (j < 0 || j >= cols) return fail(NERVA_ERR_CSR, "column index %d out of range at position %lld", j, (long long)p);
            if (p > b && indices[p - 1] >= j)
                return fail(NERVA_ERR_CSR, "column indices not strictly ascending in row %d", i);
        }
    }
    if (indptr[rows] != nnz) return fail(NERVA_ERR_CSR, "indptr[rows] = %d, expected nnz = %lld", indptr[rows], (long long)nnz);
    return NERVA_OK;
}

int nerva_set_partition_mode(int32_t mode)
{
    if (mode < NERVA_PARTITION_BALANCED || mode > NERVA_PARTITION_PREFER_STRIPS) return fail(NERVA_ERR_ARGUMENT, "unknown partition mode %d", mode);
    g_partition_mode.store(mode);
    return NERVA_OK;
}

int nerva_plan_rows_host(int32_t rows, const int32_t *indptr_host, int32_t *row_order_host,
                         int32_t *blocks_host, int32_t *huge_rows_host, int32_t *waves_host, int32_t *counts_host)
{
    if (rows <= 0 || !indptr_host || !counts_host) return fail(NERVA_ERR_ARGUMENT, "bad argument");
    const RowPlan P = plan_rows(rows, indptr_host, rows_by_length(rows, indptr_host));
    counts_host[0] = static_cast<int32_t>(P.row_order.size());
    counts_host[1] = P.n_blocks();
    counts_host[2] = P.n_huge_rows();
    counts_host[3] = P.n_huge_blocks;
    if (row_order_host && !P.row_order.empty()) memcpy(row_order_host, P.row_order.data(), P.row_order.size() * 4);
    if (blocks_host && !P.blocks.empty()) memcpy(blocks_host, P.blocks.data(), P.blocks.size() * 4);
    if (huge_rows_host && !P.huge_rows.empty()) memcpy(huge_rows_host, P.huge_rows.data(), P.huge_rows.size() * 4);
    if (waves_host && !P.waves.empty()) memcpy(waves_host, P.waves.data(), P.waves.size() * 4);
    return NERVA_OK;
}

int nerva_plan_short_rows_host(int32_t rows, const int32_t *indptr_host, int32_t *short_rows_host,
                               int32_t *long_waves_host, int32_t *counts_host)
{
    if (rows <= 0 || !indptr_host || !counts_host) return fail(NERVA_ERR_ARGUMENT, "bad argument");
    int32_t n_short = 0;
    const RowsByLength by_len = rows_by_length(rows, indptr_host);
    const std::vector<int32_t> t = short_row_table(rows, indptr_host, by_len, &n_short);
    RowPlan Q;
    if (n_short > 0) Q = plan_rows(rows, indptr_host, by_len, kPackMaxLen);
    counts_host[0] = n_short;
    counts_host[1] = Q.n_blocks();
    counts_host[2] = Q.n_huge_blocks;
    if (short_rows_host && !t.empty()) memcpy(short_rows_host, t.data(), t.size() * 4);
    if (long_waves_host && !Q.waves.empty()) memcpy(long_waves_host, Q.waves.data(), Q.waves.size() * 4);
    return NERVA_OK;
}

int nerva_plan_staged_host(int32_t rows, int32_t cols, const int32_t *indptr_host, const int32_t *indices_host,
                           int32_t max_batch, int32_t min_entries, int32_t *slot_rows_host, int32_t *ends_host,
                           int32_t *counts_host)
{
    if (rows <= 0 || cols <= 0 || min_entries < 0 || !indptr_host || !counts_host || (indptr_host[rows] > 0 && !indices_host))
        return fail(NERVA_ERR_ARGUMENT, "bad argument");
    static_assert(NERVA_STAGE_ROWS == kStageRows && NERVA_STAGE_COLS == kStageCols && NERVA_STAGE_MIN_BATCH == kStageMinBatch &&
                  NERVA_STAGE_RANGE_ROWS == kStageRangeRows && NERVA_STAGE_QUAD == kStageQuad, "header and kernels disagree");
    StagedPlan H = plan_staged(rows, cols, indptr_host, rows_by_length(rows, indptr_host), max_batch, min_entries);
    if (ends_host && H.ranges) fill_staged_ends_host(H, indptr_host, indices_host);
    counts_host[0] = H.ranges;
    counts_host[1] = H.cblocks;
    if (slot_rows_host && !H.rows.empty()) memcpy(slot_rows_host, H.rows.data(), H.rows.size() * 4);
    if (ends_host && !H.ends.empty()) memcpy(ends_host, H.ends.data(), H.ends.size() * 4);
    return NERVA_OK;
}

// Density from which a layer bound by sparse_linear_create / sparse_linear_rebind takes the dense route by
// itself (process-wide; nerva_set_dense_threshold).  The default is the measured cut-over on the paper's MLP.
std::atomic<float> g_dense_threshold{kDenseFromDensity};

static bool dense_shape_ok(int32_t rows, int32_t cols)
{
    // (a thin full matrix has its own streaming kernels; the copy stays below 2 GiB)
    return rows >= 64 && cols >= 64 && static_cast<int64_t>(rows) * round_up(cols, kDenseLdAlign) < (1ll << 29);
}

static int32_t table_words(const nerva_layer *l) { return (l->cols + 31) / 32; }

// The dense copy for the dense route: allocated zero, then filled from the stored entries; and the pattern table, where
// the layer has none yet.
static hipError_t build_dense_copies(nerva_layer *l, hipStream_t s)
{
    l->dense_ld = round_up(l->cols, kDenseLdAlign);
    const size_t bytes = static_cast<size_t>(l->rows) * l->dense_ld * 4;
    // behind the copy: tickets and shares of tiles that several work-groups form (one allocation: each costs a create a quarter of a millisecond)
    size_t tickets = dense_shares_possible(l->rows, l->cols, l->max_batch) ? kNnTickets * 4 : 0;
    hipError_t e = hipMalloc(&l->dense, bytes + tickets + (tickets ? static_cast<size_t>(kNnShareFloats) * 4 : 0));
    if (e != hipSuccess && tickets) {
        (void)hipGetLastError();
        tickets = 0;
        e = hipMalloc(&l->dense, bytes);
    }
    l->dense_shares = e == hipSuccess && tickets ? l->dense + bytes / 4 : nullptr;
    if (e == hipSuccess && !l->cur.has_table && reserve_optional(&l->cur.table, &l->cur.table_ints, static_cast<size_t>(l->rows) * table_words(l) * 2)) {
        e = launch_pattern_table(l->indptr, l->indices, nullptr, l->rows, table_words(l), reinterpret_cast<uint2 *>(l->cur.table), nullptr, s);
        if (e == hipSuccess) l->cur.has_table = true;
    }
    if (e == hipSuccess) e = hipMemsetAsync(l->dense, 0, bytes + tickets, s);
    if (e == hipSuccess) e = launch_dense_refresh(l->indptr, l->indices, l->values, l->rows, l->dense, l->dense_ld, s);
    return e;
}

static hipError_t refresh_dense_copies(const nerva_layer *l, hipStream_t s)
{
    return launch_dense_refresh(l->indptr, l->indices, l->values, l->rows, l->dense, l->dense_ld, s);
}

// Y = act(W X + b) through the dense copy
static hipError_t dense_forward(const nerva_layer *l, const float *X, int64_t ldx, float *Y, int64_t ldy, int32_t batch,
                                hipStream_t s)
{
    DenseArgs d{};
    d.W = l->dense; d.ldw = l->dense_ld; d.trans = 0; d.X = X; d.ldx = ldx; d.Y = Y; d.ldy = ldy; d.bias = l->bias;
    d.rows = l->rows; d.cols = l->cols; d.batch = batch; d.relu = l->activation == NERVA_ACT_RELU;
    if (l->dense_shares) { d.tickets = reinterpret_cast<int32_t *>(l->dense_shares); d.partial = l->dense_shares + kNnTickets; }
    return launch_dense_product(d, s);
}

// dX = (W^T dZ) * [mask > 0] through the same copy
static hipError_t dense_transposed(const nerva_layer *l, const float *dZ, int64_t lddz, float *dX, int64_t lddx,
                                   const float *mask, int64_t ldmask, int32_t batch, hipStream_t s)
{
    DenseArgs d{};
    d.W = l->dense; d.ldw = l->dense_ld; d.trans = 1; d.X = dZ; d.ldx = lddz; d.Y = dX; d.ldy = lddx;
    d.YM = mask; d.ldym = ldmask; d.rows = l->rows; d.cols = l->cols; d.batch = batch;
    return launch_dense_product(d, s);
}

static int enable_dense(nerva_layer *layer, hipStream_t s);

// whether a layer is, or with `nnz` entries is going to be, on the dense route
static bool takes_dense_route(const nerva_layer *l, int32_t nnz)
{
    return l->dense_on || (dense_shape_ok(l->rows, l->cols) &&
                           static_cast<double>(nnz) >= static_cast<double>(g_dense_threshold.load()) * l->rows * l->cols);
}

// the dense route needs a batch wide enough to fill its 16-column tiles
static bool use_dense(const nerva_layer *l, int32_t batch) { return l->dense_on && batch >= 16; }

// tickets of the huge rows of W (side 0) or of its mirror (side 1): rows of the two alternate
static int32_t *tickets_of(const nerva_layer *l, int side) { return l->tickets ? l->tickets + side * huge_row_tickets(l->scratch_ld) : nullptr; }

// The mirror's entries in the order of `v`, in b.hot (views of b's own arrays).
static hipError_t make_hot_order(const PatternBuffers &b, const HotRows &v, int32_t rows, int32_t cols, int32_t nnz, const RowBlocks &plan_t, hipStream_t s)
{
    const size_t n64 = static_cast<size_t>(round_up(nnz, 64));
    int32_t *sets = b.hot + 4 * n64;
    return launch_hot_order(v.rows, rows, b.indptr_t, b.mirror_mem, cols, b.mirror_mem + n64, sets + 4 * hot_sets_size(cols), b.hot, b.hot + n64, b.hot + 2 * n64,
                            plan_t.rows_by_length, reinterpret_cast<int4 *>(sets), s);
}
// For a call that takes it: where it is not made yet by the first, which the others, on whatever stream, wait for.  (One that is recorded into a graph has not run: it makes the order in
// the graph, the same again.)
static hipError_t order_hot_rows(nerva_layer *l, hipStream_t s)
{
    l->hot_at_bind = true;
    if (l->hot_state == kHotOrdered) return hipSuccess;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
        (void)hipGetLastError();
        capture = hipStreamCaptureStatusActive;
    }
    if (capture == hipStreamCaptureStatusNone && l->hot_state == kHotOnItsWay) {
        if (hipEventQuery(l->hot_event) == hipSuccess) {
            l->hot_state = kHotOrdered;
            return hipSuccess;
        }
        (void)hipGetLastError();   // (not ready)
        return hipStreamWaitEvent(s, l->hot_event, 0);
    }
    hipError_t e = make_hot_order(l->cur, l->hot, l->rows, l->cols, l->nnz, l->plan_t, s);
    if (e != hipSuccess || capture != hipStreamCaptureStatusNone) return e;
    e = hipEventRecord(l->hot_event, s);
    if (e == hipSuccess) l->hot_state = kHotOnItsWay;
    return e;
}

static float *hot_values_of(const nerva_layer *l) { return l->hot.entry ? reinterpret_cast<float *>(l->cur.hot) + 3 * static_cast<size_t>(round_up(l->nnz, 64)) : nullptr; }

static const DenseSplit *split_of(const nerva_layer *l) { return l->cur.split.rows.n > 0 ? &l->cur.split : nullptr; }

// Message for the status word of the device-side CSR check (bind_check_kernel).
static int csr_status_error(const int32_t *st)
{
    const int f = st[0];
    if (f & kCsrBadFirst) return fail(NERVA_ERR_CSR, "indptr[0] is not 0");
    if (f & kCsrDecreasing) return fail(NERVA_ERR_CSR, "indptr decreases at row %d", st[1]);
    if (f & kCsrBeyondNnz) return fail(NERVA_ERR_CSR, "indptr[%d] lies outside [0, nnz]", st[1]);
    if (f & kCsrBadLast) return fail(NERVA_ERR_CSR, "indptr[rows] differs from nnz");
    if (f & kCsrColumnRange) return fail(NERVA_ERR_CSR, "column index out of range at position %d", st[2]);
    if (f & kCsrNotAscending) return fail(NERVA_ERR_CSR, "column indices not strictly ascending at position %d", st[2]);
    return fail(NERVA_ERR_CSR, "pattern is not canonical CSR (status 0x%x)", f);
}

// Everything a pattern allows to be precomputed, for a layer `l` that describes the NEW pattern (sizes,
// caller-owned arrays, max_batch) and owns the buffers to build into: l->spare receives the mirror and the
// partition tables (l->cur, if any, is not touched), the scratch buffers grow as needed.  All of it -- the CSR check,
// the mirror with its position maps, the partitions of both orientations -- runs on the device in one chain of
// launches (structure.hip); the host waits once, for the check's verdict and the partitions' sizes.  On failure
// (NERVA_ERR_CSR, NERVA_ERR_HIP) nothing that a product reads has been changed.  On success the caller swaps
// l->spare into l->cur and adopts `plan`, `plan_t`.
constexpr size_t kPartialMaxBytes = 4ull << 30, kDzMaxBytes = 1ull << 30, kStripMaxBytes = 1ull << 30;
struct BuiltPattern {
    RowBlocks plan{}, plan_t{};
    Strips strips;                  // segs nullptr: none
    HotRows hot;                    // entry nullptr: none
    int64_t partial_stride = 0, partial_db_at = 0;
    int32_t partial_tiles = 0;
    int64_t scratch_ld = 0, full_scratch_ld = 0;
    bool full = false;
};

// room for the product of the dense rows of the pattern in `B`: whether there was
static bool reserve_dense_rows(PatternBuffers &B, const DenseRowsRoom &want)
{
    DenseRows &D = B.split.rows;
    const int64_t partial = round_up(want.partial_floats, 64);
    D.partial_floats = D.parts_ints = 0;
    if (partial + want.parts_ints == 0 || !reserve_optional(&B.row_partial, &B.row_partial_floats, static_cast<size_t>(partial + want.parts_ints))) return false;
    D.partial = B.row_partial;
    D.partial_floats = want.partial_floats;
    D.parts = reinterpret_cast<uint32_t *>(B.row_partial + partial);
    D.parts_ints = want.parts_ints;
    return true;
}

static int build_structures(nerva_layer *l, int32_t nnz, const int32_t *indptr, const int32_t *indices, const float *values,
                            BuiltPattern *out, hipStream_t s)
{
    const int32_t rows = l->rows, cols = l->cols, max_batch = l->max_batch, asked = g_partition_mode.load();
    const int32_t mode = asked == NERVA_PARTITION_PREFER_DENSE_ROWS || asked == NERVA_PARTITION_PREFER_STRIPS ? NERVA_PARTITION_BALANCED : asked;
    static_assert(kPlanBalanced == NERVA_PARTITION_BALANCED && kPlanRowSplit == NERVA_PARTITION_ROW_SPLIT &&
                  kPlanPreferStaged == NERVA_PARTITION_PREFER_STAGED, "header and kernels disagree");
    PatternBuffers &B = l->spare;
    const size_t n64 = static_cast<size_t>(round_up(nnz > 0 ? nnz : 1, 64));
    size_t indptr_t_have = B.indptr_t ? static_cast<size_t>(cols) + 1 : 0;
    HIP_TRY(reserve(&B.indptr_t, &indptr_t_have, static_cast<size_t>(cols) + 1));
    HIP_TRY(reserve(&B.mirror_mem, &B.mirror_ints, 4 * n64));
    // rows long enough for matrix instructions are looked for unless the layer takes the dense route as a whole
    const bool seek_dense = mode == NERVA_PARTITION_BALANCED && asked != NERVA_PARTITION_PREFER_STRIPS && cols >= kDenseRowsMinCols && max_batch >= kDenseRowsMinBatch && nnz < (1 << 30) &&
                            !takes_dense_route(l, nnz);
    const int32_t dense_len = seek_dense ? dense_row_length(cols) : INT32_MAX;
    const bool strips = !takes_dense_route(l, nnz) &&
                        (asked == NERVA_PARTITION_PREFER_STRIPS
                             ? strip_possible(rows, cols, nnz, max_batch)
                             : mode == NERVA_PARTITION_BALANCED &&
                                   strip_wanted(rows, cols, nnz, max_batch, staged_ranges_wanted(rows, nnz, cols, max_batch, mode, staged_range_bound(rows, cols, max_batch))));
    const PlanRoom room(rows, cols, nnz, max_batch, strips, dense_len), room_t(cols, rows, nnz, max_batch);
    const size_t plan_ints = static_cast<size_t>(round_up(static_cast<int64_t>(room.ints()), 64));
    HIP_TRY(reserve(&B.plan_mem, &B.plan_ints, plan_ints + room_t.ints()));
    if (!l->bind_result) HIP_TRY(hipHostMalloc(&l->bind_result, sizeof(BindResult), hipHostMallocDefault));

    // scratch of the set-up kernels: carved out of one buffer
    const MirrorGeometry geo = mirror_geometry(rows, cols, nnz);
    const int64_t col_blocks = (static_cast<int64_t>(cols) + geo.block_cols - 1) / geo.block_cols;
    size_t ints = 0;
    auto carve = [&](size_t n) { const size_t at = ints; ints += (n + 63) / 64 * 64; return at; };
    const size_t status_at = carve(4), base_at = carve(static_cast<size_t>(col_blocks) + 1), total_at = carve(geo.bins),
                 counts_at = carve(static_cast<size_t>(geo.bins) * geo.tiles), bucket_at = carve(2 * n64), bucket_col_at = carve(n64);
    size_t work_at[2];
    const int32_t side_rows[2] = {rows, cols}, side_ranges[2] = {room.ranges, room_t.ranges};
    constexpr size_t kCountInts = sizeof(PlanCounts) / 4;
    for (int k = 0; k < 2; ++k) work_at[k] = carve(6 * static_cast<size_t>(side_rows[k]) + static_cast<size_t>(side_ranges[k]) + 1 + kCountInts);
    const size_t strip_at = carve(8);
    HIP_TRY(reserve(&l->build_work, &l->build_work_ints, ints));
    int32_t *W = l->build_work;

    MirrorArgs m{};
    static_cast<MirrorGeometry &>(m) = geo;
    m.rows = rows; m.cols = cols; m.nnz = nnz; m.indptr = indptr; m.indices = indices; m.values = values;
    m.status = W + status_at; m.block_base = W + base_at; m.bin_total = W + total_at; m.counts = W + counts_at;
    m.bucket = reinterpret_cast<int2 *>(W + bucket_at); m.bucket_col = W + bucket_col_at;
    m.indptr_t = B.indptr_t; m.indices_t = B.mirror_mem; m.perm = B.mirror_mem + n64; m.pos_t = B.mirror_mem + 2 * n64;
    m.values_t = reinterpret_cast<float *>(B.mirror_mem + 3 * n64);
    PlanArgs p{};
    p.nnz = nnz; p.max_batch = max_batch; p.mode = mode; p.status = m.status; p.result = l->bind_result;
    p.result->strip = 0; p.prefer_strips = asked == NERVA_PARTITION_PREFER_STRIPS;
    for (int k = 0; k < 2; ++k) {
        PlanSide &side = p.side[k];
        side.rows = side_rows[k]; side.other = side_rows[1 - k]; side.range_bound = side_ranges[k];
        side.strip_blocks = k == 0 ? room.strip_blocks : 0;
        side.dense_len = k == 0 ? dense_len : INT32_MAX;
        side.indptr = k == 0 ? indptr : B.indptr_t; side.indices = k == 0 ? indices : m.indices_t;
        side.tables = k == 0 ? room.at(B.plan_mem) : room_t.at(B.plan_mem + plan_ints);
        int32_t *w = W + work_at[k];
        const size_t r = static_cast<size_t>(side.rows);
        side.work = PlanWork{w, w + r, w + 2 * r, w + 3 * r, w + 4 * r, w + 5 * r, w + 6 * r,
                             reinterpret_cast<PlanCounts *>(w + 6 * r + static_cast<size_t>(side.range_bound) + 1),
                             reinterpret_cast<unsigned long long *>(W + strip_at)};
    }
    HIP_TRY(launch_bind(m, p, s));
    B.has_table = (l->dense_on || static_cast<double>(nnz) >= static_cast<double>(kTableFromDensity) * rows * cols) &&
                  reserve_optional(&B.table, &B.table_ints, static_cast<size_t>(rows) * table_words(l) * 2);
    if (B.has_table) {
        HIP_TRY(launch_pattern_table(indptr, indices, nullptr, rows, table_words(l), reinterpret_cast<uint2 *>(B.table), m.status, s));
    }
    HIP_TRY(hipStreamSynchronize(s));
    const BindResult R = *l->bind_result;
    if (R.status[0] != 0) return csr_status_error(R.status);
    out->plan = plan_view(p.side[0].tables, R.plan[0], cols, nnz, R.plan[1].hot_nnz, mode);
    bool more_work = false;   // launches after the wait
    B.split = DenseSplit{};
    const int32_t n_dense = R.plan[0].n_dense;
    if (n_dense > 0 && !reserve_optional(&B.row_table, &B.row_table_ints, static_cast<size_t>(n_dense) * table_words(l) * 2)) {
        out->plan.staged_rows = nullptr;   // (it covers the other rows only: the dense ones stay with them, unstaged)
    } else if (n_dense > 0) {
        const PlanTables &t = p.side[0].tables;
        DenseRows &D = B.split.rows;
        D.list = t.dense_rows; D.n = n_dense; D.words = table_words(l);
        D.table = reinterpret_cast<const uint2 *>(B.row_table);
        const DenseRowsRoom want = dense_rows_room(D.n, cols, max_batch, false);
        if (!reserve_dense_rows(B, want) && want.parts_ints > 0) (void)reserve_dense_rows(B, DenseRowsRoom{want.partial_floats, 0});
        B.split.from_batch = asked == NERVA_PARTITION_PREFER_DENSE_ROWS ? kDenseRowsMinBatch : dense_rows_from(R.plan[0].dense_nnz);
        B.split.dense_nnz = R.plan[0].dense_nnz;
        B.split.flag = t.dense_flag;
        B.split.others = out->plan;
        B.split.others.waves = t.other_waves;
        B.split.others.long_waves = t.other_long_waves;
        // The staged plan covers the other rows only.  Narrower batches, at which the dense rows are rows like any other, get one of
        // all rows where the widest of them that fills its tiles (staged_pays) has work-groups enough for it.
        out->plan.staged_rows = nullptr;
        const int32_t tiles = static_cast<int32_t>(std::min<int64_t>(5ll * (B.split.from_batch - 1), 5ll * max_batch) / (4 * kStageCols));
        if (B.split.from_batch > kStageMinBatch && room.ranges > 0 && tiles * staged_ranges_aim(rows, max_batch) >= kStageTargetGroups / 2 &&
            reserve_optional(&B.whole_staged, &B.whole_staged_ints, room.staged_ints())) {
            PlanArgs whole = p;
            whole.side[0].dense_len = INT32_MAX;
            room.staged_at(whole.side[0].tables, B.whole_staged);
            HIP_TRY(launch_plan(whole, 1, s));   // (the other tables come out as they are)
            HIP_TRY(hipStreamSynchronize(s));
            out->plan = plan_view(whole.side[0].tables, l->bind_result->plan[0], cols, nnz, R.plan[1].hot_nnz, mode);
        }
        HIP_TRY(launch_pattern_table(indptr, indices, D.list, D.n, D.words, reinterpret_cast<uint2 *>(B.row_table), nullptr, s));
        more_work = true;
    } else if (asked == NERVA_PARTITION_BALANCED && seek_dense && B.has_table && rows >= kThinRows && cols >= kThinCols && max_batch >= kThinBatch &&
               static_cast<double>(nnz) >= static_cast<double>(kThinDensity) * rows * cols) {
        DenseRows &D = B.split.rows;
        D.n = rows; D.words = table_words(l);
        D.table = reinterpret_cast<const uint2 *>(B.table);
        B.split.thin_nnz = nnz; B.split.max_batch = max_batch;
        const DenseRowsRoom want = dense_rows_room(rows, cols, max_batch, true);
        D.partial_floats = want.partial_floats; D.parts_ints = want.parts_ints;
        if (!thin_rows_pay_somewhere(B.split, cols) || !reserve_dense_rows(B, want)) B.split = DenseSplit{};
    }
    out->plan_t = plan_view(p.side[1].tables, R.plan[1], rows, nnz, R.plan[0].hot_nnz, mode);
    const float in_lds = nnz > 0 ? static_cast<float>(static_cast<double>(R.plan[0].hot_lds_nnz) / nnz) : 0.f;
    auto takes_hot_rows = [&] {
        HotRows order;
        order.share = in_lds;
        SpmmCall t{};
        t.blocks = out->plan_t; t.hot = &order; t.rows = cols; t.x_rows = rows; t.nnz = nnz;
        SddmmCall g{};
        g.blocks = out->plan; g.perm = m.perm; g.rows = rows; g.x_rows = cols; g.nnz = nnz;
        g.partial_stride = round_up(nnz, 64) + round_up(rows, 64);
        g.partial_tiles = static_cast<int32_t>(std::min<int64_t>(INT32_MAX, static_cast<int64_t>(kPartialMaxBytes / 4) / g.partial_stride));
        if (B.has_table) g.table = reinterpret_cast<const uint2 *>(B.table);
        g.split = B.split.rows.n > 0 ? &B.split : nullptr;
        return hot_rows_pay_somewhere(t, g, max_batch);
    };
    auto has_event = [&] {
        if (l->hot_event || hipEventCreateWithFlags(&l->hot_event, hipEventDisableTiming) == hipSuccess) return true;
        (void)hipGetLastError();
        l->hot_event = nullptr;
        return false;
    };
    // (The dense route has no use for it.  A new pattern of a layer whose calls have not taken it, as the first one of a network, waits for a call that does: making it
    // takes 28 us of the 117 that binding 1100 x 2600 at 10 % does; a step of 2667-1317-8 at 6.7 %, batch 1016, with new patterns for both layers 217 -> 179.)
    if (asked == NERVA_PARTITION_BALANCED && nnz > 0 && !takes_dense_route(l, nnz) && takes_hot_rows() &&
        has_event() &&
        reserve_optional(&B.hot, &B.hot_ints, 4 * n64 + 4 * static_cast<size_t>(hot_sets_size(cols)) + static_cast<size_t>(rows) + cols)) {
        HotRows &v = out->hot;
        v.entry = B.hot; v.at = B.hot + n64; v.perm = B.hot + 2 * n64; v.sets = reinterpret_cast<const int4 *>(B.hot + 4 * n64); v.rows = out->plan.rows_by_length; v.share = in_lds;
        if (l->hot_at_bind) {
            HIP_TRY(make_hot_order(B, v, rows, cols, nnz, out->plan_t, s));
            more_work = true;
        }
    }

    // scratch buffers of the products (they hold nothing between calls, the tickets zeros: grown in place, so that the old
    // pattern's products find them whatever fails from here on)
    {
        // per-tile partial products: room for the tiles of every batch, or what there is room for (kPartialMaxBytes: beyond
        // that they are not worth it), below which the kernels without them stay
        int32_t tiles = partial_tiles_wanted(out->plan, out->plan_t, rows, cols, nnz, max_batch);
        if ((out->plan.staged_rows || B.split.others.staged_rows) && (max_batch + kStageCols - 1) / kStageCols > tiles) tiles = (max_batch + kStageCols - 1) / kStageCols;
        if (out->hot.entry) tiles = std::max(tiles, (max_batch + 63) / 64);
        out->partial_db_at = round_up(nnz, 64);
        out->partial_stride = out->partial_db_at + round_up(rows, 64);
        const size_t slice = static_cast<size_t>(out->partial_stride);
        tiles = static_cast<int32_t>(std::min<size_t>(tiles, kPartialMaxBytes / 4 / slice));
        out->partial_tiles = tiles;
        if (tiles > 0 && !reserve_optional(&l->partial, &l->partial_floats, tiles * slice))
            out->partial_tiles = static_cast<int32_t>(std::min<size_t>(tiles, l->partial_floats / slice));
        l->dz_ld = round_up(max_batch, 32);
        const size_t dz = static_cast<size_t>(rows) * l->dz_ld;
        if (l->activation == NERVA_ACT_RELU && max_batch > 4 && nnz >= 4 * static_cast<int64_t>(rows) && dz * 4 <= kDzMaxBytes)
            (void)reserve_optional(&l->dz, &l->dz_floats, dz, false);
        const int64_t slots = out->plan.n_huge_blocks > out->plan_t.n_huge_blocks ? out->plan.n_huge_blocks : out->plan_t.n_huge_blocks;
        const size_t chunks = static_cast<uint32_t>(R.strip), need = (chunks + 2) * kStripChunk * kStripSet * 2;
        const int32_t steps = static_cast<int32_t>(R.strip >> 32);
        if (chunks > 0 && need * 4 <= kStripMaxBytes && (p.prefer_strips || strips_pay_somewhere(out->plan, rows, cols, nnz, max_batch, steps, static_cast<double>(chunks))) &&
            reserve_optional(&l->strip_stream, &l->strip_floats, need)) {
            Strips &v = out->strips;
            v.rows = p.side[0].tables.strip_rows; v.segs = p.side[0].tables.strip_segs; v.cuts = p.side[0].tables.strip_cuts;
            v.blocks = room.strip_blocks; v.block_rows = strip_block_rows_of(cols);
            v.chunks = static_cast<int32_t>(chunks); v.steps = steps;
            v.preferred = p.prefer_strips;
        }
        out->scratch_ld = round_up(max_batch, 64);
        if (slots > 0) {
            const int64_t huge = std::max(out->plan.n_huge_rows, out->plan_t.n_huge_rows);
            HIP_TRY(reserve(&l->tickets, &l->ticket_ints, static_cast<size_t>(2 * huge * huge_row_tickets(out->scratch_ld)), true, s));
            HIP_TRY(reserve(&l->scratch, &l->scratch_floats, static_cast<size_t>(slots * out->scratch_ld)));
        }
        out->full = rows <= kFullMaxRows && static_cast<int64_t>(nnz) == static_cast<int64_t>(rows) * cols;
        out->full_scratch_ld = round_up(max_batch, 64);
        if (out->full) {
            const int64_t slices = (cols + kFullSlice - 1) / kFullSlice;
            (void)reserve_optional(&l->full_scratch, &l->full_scratch_floats, static_cast<size_t>(slices) * rows * out->full_scratch_ld, false);
        }
    }
    if (more_work) HIP_TRY(hipStreamSynchronize(s));   // (a product on another stream may follow)
    return NERVA_OK;
}

// The spare set, just built, becomes the layer's pattern; the set it replaces becomes the spare one.
static void adopt_pattern(nerva_layer *l, int32_t nnz, const int32_t *indptr, const int32_t *indices, float *values, const BuiltPattern &bp)
{
    std::swap(l->cur, l->spare);
    const size_t n64 = static_cast<size_t>(round_up(nnz > 0 ? nnz : 1, 64));
    l->nnz = nnz; l->indptr = indptr; l->indices = indices; l->values = values;
    l->indptr_t = l->cur.indptr_t;
    l->indices_t = l->cur.mirror_mem;
    l->perm = l->cur.mirror_mem + n64;
    l->pos_t = l->cur.mirror_mem + 2 * n64;
    l->values_t = reinterpret_cast<float *>(l->cur.mirror_mem + 3 * n64);
    l->plan = bp.plan; l->plan_t = bp.plan_t; l->strips = bp.strips; l->hot = bp.hot; l->hot_state = l->hot_at_bind ? kHotOrdered : kHotUnordered; l->hot_at_bind = false;
    l->partial_stride = bp.partial_stride; l->partial_db_at = bp.partial_db_at; l->partial_tiles = bp.partial_tiles;
    l->scratch_ld = bp.scratch_ld;
    l->full_scratch_ld = bp.full_scratch_ld;
    l->full = bp.full;
    l->mirror_stale = false;
}

int sparse_linear_create(nerva_layer **out, int32_t rows, int32_t cols, int32_t nnz, const int32_t *indptr,
                         const int32_t *indices, float *values, float *bias, int32_t activation, int32_t max_batch,
                         void *stream)
{
    if (!out) return fail(NERVA_ERR_ARGUMENT, "out is null");
    *out = nullptr;
    if (rows <= 0 || cols <= 0 || nnz < 0) return fail(NERVA_ERR_ARGUMENT, "bad layer size %d x %d, nnz %d", rows, cols, nnz);
    if (!indptr || (nnz > 0 && (!indices || !values))) return fail(NERVA_ERR_ARGUMENT, "null pattern or values pointer");
    if (activation != NERVA_ACT_NONE && activation != NERVA_ACT_RELU) return fail(NERVA_ERR_ARGUMENT, "unknown activation %d", activation);
    if (max_batch <= 0 || max_batch >= (1 << 30)) return fail(NERVA_ERR_ARGUMENT, "max_batch must be positive (got %d)", max_batch);
    nerva_layer *l = new (std::nothrow) nerva_layer;
    if (!l) return fail(NERVA_ERR_ARGUMENT, "out of host memory");
    l->rows = rows; l->cols = cols; l->activation = activation; l->max_batch = max_batch; l->bias = bias;
    BuiltPattern bp;
    const int rc = build_structures(l, nnz, indptr, indices, values, &bp, as_stream(stream));
    if (rc != NERVA_OK) {
        free_layer_buffers(l);
        delete l;
        return rc;
    }
    adopt_pattern(l, nnz, indptr, indices, values, bp);
    // the density-adaptive choice: dense products where the pattern is dense enough for them to be the faster ones
    if (takes_dense_route(l, nnz)) {
        const int rd = enable_dense(l, as_stream(stream));
        if (rd != NERVA_OK) {
            free_layer_buffers(l);
            delete l;
            return rd;
        }
    }
    *out = l;
    return NERVA_OK;
}

int sparse_linear_rebind(nerva_layer *layer, int32_t nnz, const int32_t *indptr, const int32_t *indices, float *values,
                         void *stream)
{
    if (!layer) return fail(NERVA_ERR_ARGUMENT, "layer is null");
    if (nnz < 0 || !indptr || (nnz > 0 && (!indices || !values))) return fail(NERVA_ERR_ARGUMENT, "null pattern or values pointer");
    hipStream_t s = as_stream(stream);
    // (launches already queued on this stream use the old structures, which the new ones do not overwrite)
    BuiltPattern bp;
    const int rc = build_structures(layer, nnz, indptr, indices, values, &bp, s);
    if (rc != NERVA_OK) return rc;  // the layer keeps its old pattern: only the spare set and scratch buffers were written
    adopt_pattern(layer, nnz, indptr, indices, values, bp);
    if (!layer->dense_on && takes_dense_route(layer, nnz))
        return enable_dense(layer, s);   // (a pattern that has grown dense; a route once taken is kept)
    if (layer->dense_on) {
        // the dense copies hold the old pattern's entries: cleared and filled again
        const size_t bytes = static_cast<size_t>(layer->rows) * layer->dense_ld * 4;
        HIP_TRY(hipMemsetAsync(layer->dense, 0, bytes, s));
        HIP_TRY(refresh_dense_copies(layer, s));
        HIP_TRY(hipStreamSynchronize(s));
    }
    return NERVA_OK;
}

static int enable_dense(nerva_layer *layer, hipStream_t s)
{
    if (layer->dense_on) return NERVA_OK;
    if (static_cast<int64_t>(layer->rows) * round_up(layer->cols, kDenseLdAlign) >= (1ll << 31))
        return fail(NERVA_ERR_SHAPE, "a %d x %d layer is too large for the dense route", layer->rows, layer->cols);
    hipError_t e = build_dense_copies(layer, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(layer->dense);
        layer->dense = layer->dense_shares = nullptr;
        return hip_fail(e, "sparse_linear_enable_dense");
    }
    layer->dense_on = true;
    return NERVA_OK;
}

int sparse_linear_enable_dense(nerva_layer *layer, void *stream)
{
    if (!layer) return fail(NERVA_ERR_ARGUMENT, "layer is null");
    return enable_dense(layer, as_stream(stream));
}

int nerva_set_dense_threshold(float density)
{
    if (!(density >= 0.f)) return fail(NERVA_ERR_ARGUMENT, "the density threshold must not be negative");
    g_dense_threshold.store(density);
    return NERVA_OK;
}

int sparse_linear_sync_values(nerva_layer *layer, void *stream)
{
    if (!layer) return fail(NERVA_ERR_ARGUMENT, "layer is null");
    hipStream_t s = as_stream(stream);
    HIP_TRY(launch_gather(layer->values_t, layer->values, layer->perm, layer->nnz, s));
    layer->mirror_stale = false;
    if (layer->dense_on) HIP_TRY(refresh_dense_copies(layer, s));
    return NERVA_OK;
}

void sparse_linear_destroy(nerva_layer *layer)
{
    if (!layer) return;
    free_layer_buffers(layer);
    delete layer;
}

int sparse_linear_mirror(const nerva_layer *layer, const int32_t **indptr_t, const int32_t **indices_t,
                         const float **values_t, const int32_t **perm)
{
    if (!layer) return fail(NERVA_ERR_ARGUMENT, "layer is null");
    if (indptr_t) *indptr_t = layer->indptr_t;
    if (indices_t) *indices_t = layer->indices_t;
    if (values_t) *values_t = layer->values_t;
    if (perm) *perm = layer->perm;
    return NERVA_OK;
}

int sparse_linear_partition(const nerva_layer *layer, int32_t side, int32_t table, const int32_t **table_out, int64_t *ints_out)
{
    if (!layer || !table_out || !ints_out || side < 0 || side > 1) return fail(NERVA_ERR_ARGUMENT, "bad argument");
    const RowBlocks &b = side ? layer->plan_t : layer->plan;
    const void *p = nullptr;
    int64_t n = 0;
    switch (table) {
        case NERVA_TABLE_WAVES: p = b.waves; n = 4ll * kWavesPerBlock * b.n_blocks; break;
        case NERVA_TABLE_HUGE_ROWS: p = b.huge_rows; n = 4ll * b.n_huge_rows; break;
        case NERVA_TABLE_SHORT_ROWS: p = b.short_rows; n = 4 * round_up(b.n_short, 64); break;
        case NERVA_TABLE_LONG_WAVES: p = b.long_waves; n = 4ll * kWavesPerBlock * b.n_long_blocks; break;
        case NERVA_TABLE_STAGED_ROWS: p = b.staged_rows; n = b.staged_rows ? static_cast<int64_t>(b.staged_ranges) * kStageRangeRows : 0; break;
        case NERVA_TABLE_STAGED_ENDS: p = b.staged_ends; n = b.staged_rows ? static_cast<int64_t>(b.staged_ranges) * kStageRangeRows * (b.staged_cblocks + 1) : 0; break;
        default: return fail(NERVA_ERR_ARGUMENT, "unknown table %d", table);
    }
    *table_out = n > 0 ? static_cast<const int32_t *>(p) : nullptr;
    *ints_out = n;
    return NERVA_OK;
}

// Y = act(W X + b)
static SpmmCall forward_args(const nerva_layer *ly, const float *in, int64_t ldin, float *out, int64_t ldout, int32_t batch)
{
    SpmmCall a{};
    a.blocks = ly->plan; a.nnz = ly->nnz; a.scratch = ly->scratch; a.tickets = tickets_of(ly, 0); a.scratch_ld = ly->scratch_ld;
    a.strips = ly->strips.segs ? &ly->strips : nullptr; a.strip_stream = reinterpret_cast<float4 *>(ly->strip_stream);
    a.indptr = ly->indptr; a.indices = ly->indices; a.values = ly->values; a.bias = ly->bias;
    a.X = in; a.ldx = ldin; a.Y = out; a.ldy = ldout;
    a.rows = ly->rows; a.x_rows = ly->cols; a.batch = batch; a.relu = ly->activation == NERVA_ACT_RELU;
    a.full_scratch = ly->full ? ly->full_scratch : nullptr; a.full_scratch_ld = ly->full_scratch_ld;
    a.split = split_of(ly);
    return a;
}

int sparse_linear_forward(const nerva_layer *layer, const float *X, int32_t ldx, float *Y, int32_t ldy,
                          int32_t batch, void *stream)
{
    if (!layer || !X || !Y) return fail(NERVA_ERR_ARGUMENT, "null argument");
    int rc = check_batch(batch, ldx, "ldx");
    if (rc == NERVA_OK) rc = check_batch(batch, ldy, "ldy");
    if (rc == NERVA_OK && batch > layer->max_batch) rc = fail(NERVA_ERR_SHAPE, "batch %d exceeds the layer's max_batch %d", batch, layer->max_batch);
    if (rc != NERVA_OK) return rc;
    if (use_dense(layer, batch)) {
        // a stand-alone call cannot know whether the caller has changed values[] since the last one
        HIP_TRY(refresh_dense_copies(layer, as_stream(stream)));
        HIP_TRY(dense_forward(layer, X, ldx, Y, ldy, batch, as_stream(stream)));
        return NERVA_OK;
    }
    HIP_TRY(launch_spmm(forward_args(layer, X, ldx, Y, ldy, batch), as_stream(stream)));
    return NERVA_OK;
}

// A call of sparse_linear_backward as its launches see it.
struct BackwardCall {
    const nerva_layer *layer;
    const float *X, *Y, *dY;
    int32_t ldx, ldy, lddy;
    float *dX;
    int32_t lddx;
    float *dvalues, *dbias;
    int32_t batch;
    bool form_dz, mask;   // dY is dZ, which a launch of this call has formed; dY still is the gradient of a ReLU's output
};
static SpmmCall transposed_args(const BackwardCall &c)
{
    const nerva_layer *layer = c.layer;
    SpmmCall a{};
    a.blocks = layer->plan_t; a.hot = layer->hot.entry ? &layer->hot : nullptr; a.nnz = layer->nnz; a.scratch = layer->scratch; a.tickets = tickets_of(layer, 1); a.scratch_ld = layer->scratch_ld;
    a.indptr = layer->indptr_t; a.indices = layer->indices_t; a.values = layer->values_t;
    a.X = c.dY; a.ldx = c.lddy;
    if (c.mask) { a.XM = c.Y; a.ldxm = c.ldy; }
    a.Y = c.dX; a.ldy = c.lddx; a.rows = layer->cols; a.x_rows = layer->rows; a.batch = c.batch;
    return a;
}
static SddmmCall gradient_args(const BackwardCall &c)
{
    const nerva_layer *layer = c.layer;
    SddmmCall a{};
    a.blocks = layer->plan;
    a.indptr = layer->indptr; a.indices = layer->indices; a.perm = layer->perm;
    a.dZ = c.dY; a.lddz = c.lddy;
    if (c.mask) { a.ZM = c.Y; a.ldzm = c.ldy; }
    a.X = c.X; a.ldx = c.ldx; a.g = c.dvalues; a.db = c.dbias;
    a.rows = layer->rows; a.x_rows = layer->cols; a.batch = c.batch; a.nnz = layer->nnz;
    a.partial = layer->partial; a.partial_stride = layer->partial_stride;
    a.partial_db_at = layer->partial_db_at; a.partial_tiles = layer->partial_tiles;
    a.skip_products = c.dvalues ? 0 : 1;  // only the bias gradient is wanted
    if (!c.form_dz) { a.values = layer->values; a.values_t = layer->values_t; }   // (where the mirror values are not up to date yet)
    if (layer->cur.has_table) { a.table = reinterpret_cast<const uint2 *>(layer->cur.table); a.table_words = table_words(layer); }
    a.split = split_of(layer);
    a.hot_values = hot_values_of(layer);
    return a;
}
// (a small layer takes both gradients, and the mask, in one launch)
static bool backward_in_one(const BackwardCall &c)
{
    return c.mask && c.dX && c.dvalues && !use_dense(c.layer, c.batch) && backward_fused_ok(transposed_args(c), gradient_args(c), true);
}
// dZ of a ReLU layer: formed once where a transposed product would gather its rows from two operands, unless the
// matrix is so sparse that the pass over dY and Y costs more than the gathers it saves
static bool backward_forms_dz(const BackwardCall &c)
{
    return c.mask && c.dX && c.layer->dz && c.batch > 4 && c.layer->nnz >= 4 * static_cast<int64_t>(c.layer->rows);
}
static void take_formed_dz(BackwardCall &c)
{
    c.form_dz = true; c.mask = false;
    c.dY = c.layer->dz; c.lddy = static_cast<int32_t>(c.layer->dz_ld);
}

int sparse_linear_backward(nerva_layer *layer, const float *X, int32_t ldx, const float *Y, int32_t ldy,
                           const float *dY, int32_t lddy, float *dX, int32_t lddx, float *dvalues, float *dbias,
                           int32_t batch, void *stream)
{
    if (!layer || !dY) return fail(NERVA_ERR_ARGUMENT, "null argument");
    const bool relu = layer->activation == NERVA_ACT_RELU;
    if (relu && !Y) return fail(NERVA_ERR_ARGUMENT, "a ReLU layer needs its output Y for the backward pass");
    if (dvalues && !X) return fail(NERVA_ERR_ARGUMENT, "dvalues needs the layer input X");
    int rc = check_batch(batch, lddy, "lddy");
    if (rc == NERVA_OK && relu) rc = check_batch(batch, ldy, "ldy");
    if (rc == NERVA_OK && dvalues) rc = check_batch(batch, ldx, "ldx");
    if (rc == NERVA_OK && dX) rc = check_batch(batch, lddx, "lddx");
    if (rc == NERVA_OK && batch > layer->max_batch) rc = fail(NERVA_ERR_SHAPE, "batch %d exceeds the layer's max_batch %d", batch, layer->max_batch);
    if (rc != NERVA_OK) return rc;
    hipStream_t s = as_stream(stream);
    BackwardCall c{layer, X, Y, dY, ldx, ldy, lddy, dX, lddx, dvalues, dbias, batch, false, relu};
    const bool in_one = backward_in_one(c);
    if (!in_one && backward_forms_dz(c)) {
        HIP_TRY(launch_backward_prep(layer->values_t, layer->values, layer->perm, layer->nnz, dY, lddy, Y, ldy, layer->dz, layer->dz_ld,
                                     layer->rows, batch, s));
        layer->mirror_stale = false;
        take_formed_dz(c);
    }
    if (dX && use_dense(layer, batch) && !c.mask) {
        HIP_TRY(refresh_dense_copies(layer, s));
        HIP_TRY(dense_transposed(layer, c.dY, c.lddy, dX, lddx, nullptr, 0, batch, s));
    } else if (dX && dvalues && (in_one || (!c.mask && backward_fused_ok(transposed_args(c), gradient_args(c), true)))) {
        if (!c.form_dz && !backward_fused_refreshes(transposed_args(c), gradient_args(c))) HIP_TRY(launch_gather(layer->values_t, layer->values, layer->perm, layer->nnz, s));
        layer->mirror_stale = false;
        if (backward_hot_ok(transposed_args(c), gradient_args(c))) HIP_TRY(order_hot_rows(layer, s));
        HIP_TRY(launch_backward_fused(transposed_args(c), gradient_args(c), true, s));
        return NERVA_OK;
    } else if (dX) {
        if (!c.form_dz) HIP_TRY(launch_gather(layer->values_t, layer->values, layer->perm, layer->nnz, s));
        layer->mirror_stale = false;
        HIP_TRY(launch_spmm(transposed_args(c), s));
    }
    if (dvalues || dbias) {
        HIP_TRY(launch_sddmm(gradient_args(c), s));
    }
    return NERVA_OK;
}

int sparse_linear_routes(const nerva_layer *layer, int32_t batch, int32_t *routes_out)
{
    if (!layer || !routes_out) return fail(NERVA_ERR_ARGUMENT, "null argument");
    int rc = check_batch(batch, batch, "ld");
    if (rc == NERVA_OK && batch > layer->max_batch) rc = fail(NERVA_ERR_SHAPE, "batch %d exceeds the layer's max_batch %d", batch, layer->max_batch);
    if (rc != NERVA_OK) return rc;
    *routes_out = 0;
    if (use_dense(layer, batch)) return NERVA_OK;
    float *any = layer->values;   // (nothing is launched)
    if (spmm_takes_strip(forward_args(layer, any, batch, any, batch, batch))) *routes_out |= NERVA_ROUTE_FORWARD_STRIPS;
    BackwardCall c{layer, any, any, any, batch, batch, batch, any, batch, any, any, batch, false, layer->activation == NERVA_ACT_RELU};
    if (backward_in_one(c)) return NERVA_OK;
    if (backward_forms_dz(c)) take_formed_dz(c);
    if (!c.mask && backward_fused_ok(transposed_args(c), gradient_args(c), true) && backward_hot_ok(transposed_args(c), gradient_args(c))) *routes_out |= NERVA_ROUTE_BACKWARD_HOT_ROWS;
    return NERVA_OK;
}

int sgd_update_values(float *values, float *velocity, const float *grad, int64_t n, float lr, float momentum,
                      void *stream)
{
    if (n < 0) return fail(NERVA_ERR_ARGUMENT, "n is negative");
    if (n > 0 && (!values || !velocity || !grad)) return fail(NERVA_ERR_ARGUMENT, "null argument");
    HIP_TRY(launch_momentum(values, velocity, grad, n, lr, momentum, 0, as_stream(stream)));
    return NERVA_OK;
}

int sgd_update_values_nesterov(float *values, float *velocity, const float *grad, int64_t n, float lr, float momentum,
                               void *stream)
{
    if (n < 0) return fail(NERVA_ERR_ARGUMENT, "n is negative");
    if (n > 0 && (!values || !velocity || !grad)) return fail(NERVA_ERR_ARGUMENT, "null argument");
    HIP_TRY(launch_momentum(values, velocity, grad, n, lr, momentum, 1, as_stream(stream)));
    return NERVA_OK;
}

int softmax_cross_entropy(const float *Z, int32_t ldz, const int32_t *labels, int32_t classes, int32_t batch,
                          float *dZ, int32_t lddz, float *loss_out, void *stream)
{
    if (!Z || !labels || !dZ) return fail(NERVA_ERR_ARGUMENT, "null argument");
    if (classes <= 0) return fail(NERVA_ERR_ARGUMENT, "classes must be positive");
    int rc = check_batch(batch, ldz, "ldz");
    if (rc == NERVA_OK) rc = check_batch(batch, lddz, "lddz");
    if (rc != NERVA_OK) return rc;
    HIP_TRY(launch_softmax_ce(Z, ldz, labels, classes, batch, dZ, lddz, loss_out, as_stream(stream)));
    return NERVA_OK;
}

int mlp_create(nerva_mlp **out, int32_t n_layers, nerva_layer *const *layers, float *const *velocities,
               float *const *bias_velocities, int32_t max_batch, int32_t flags)
{
    if (!out) return fail(NERVA_ERR_ARGUMENT, "out is null");
    *out = nullptr;
    if (n_layers <= 0 || !layers || !velocities || !bias_velocities) return fail(NERVA_ERR_ARGUMENT, "null or empty layer list");
    if (max_batch <= 0) return fail(NERVA_ERR_ARGUMENT, "max_batch must be positive");
    if (flags & ~(NERVA_MLP_UNFUSED | NERVA_MLP_NESTEROV | NERVA_MLP_SEPARATE_HEAD)) return fail(NERVA_ERR_ARGUMENT, "unknown flags 0x%x", flags);
    for (int32_t l = 0; l < n_layers; ++l) {
        if (!layers[l]) return fail(NERVA_ERR_ARGUMENT, "layer %d is null", l);
        if (layers[l]->nnz > 0 && !velocities[l]) return fail(NERVA_ERR_ARGUMENT, "velocity of layer %d is null", l);
        if (layers[l]->bias && !bias_velocities[l]) return fail(NERVA_ERR_ARGUMENT, "bias velocity of layer %d is null", l);
        if (layers[l]->max_batch < max_batch)
            return fail(NERVA_ERR_SHAPE, "layer %d was created for batches up to %d, the MLP asks for %d", l, layers[l]->max_batch, max_batch);
        if (l > 0 && layers[l]->cols != layers[l - 1]->rows)
            return fail(NERVA_ERR_SHAPE, "layer %d has %d inputs but layer %d has %d outputs", l, layers[l]->cols, l - 1, layers[l - 1]->rows);
        const int32_t want = l + 1 < n_layers ? NERVA_ACT_RELU : NERVA_ACT_NONE;
        if (layers[l]->activation != want)
            return fail(NERVA_ERR_ARGUMENT, "layer %d: hidden layers must be ReLU and the last layer linear", l);
    }
    nerva_mlp *m = new (std::nothrow) nerva_mlp;
    if (!m) return fail(NERVA_ERR_ARGUMENT, "out of host memory");
    {
        // set-up time: the address of the static workspace on this device, so that
        // mlp_train_step_static has nothing left to look up
        void *ptr = nullptr;
        const hipError_t e = static_scratch(&ptr);
        if (e != hipSuccess) {
            delete m;
            return hip_fail(e, "address of the static workspace");
        }
    }
    m->layers.assign(layers, layers + n_layers);
    m->vel.assign(velocities, velocities + n_layers);
    m->bias_vel.assign(bias_velocities, bias_velocities + n_layers);
    m->max_batch = max_batch;
    m->flags = flags;
    const nerva_layer *last = layers[n_layers - 1];
    m->head = n_layers >= 2 && !(flags & NERVA_MLP_SEPARATE_HEAD) && head_ok(last->rows, last->cols, last->nnz, 1);
    if (m->head || (n_layers >= 2 && last->full && last->rows <= kFullMaxRows)) {   // per-column losses between two launches of a step
        const size_t bytes = static_cast<size_t>(max_batch) * 4;
        hipError_t e = hipMalloc(&m->head_scratch, bytes);
        if (e == hipSuccess) e = hipMemset(m->head_scratch, 0, bytes);
        if (e != hipSuccess) {
            if (m->head_scratch) (void)hipFree(m->head_scratch);
            delete m;
            return hip_fail(e, "head work space");
        }
    }
    *out = m;
    return NERVA_OK;
}

int mlp_rebind_velocity(nerva_mlp *mlp, int32_t layer_index, float *velocity)
{
    if (!mlp) return fail(NERVA_ERR_ARGUMENT, "mlp is null");
    if (layer_index < 0 || layer_index >= static_cast<int32_t>(mlp->layers.size()))
        return fail(NERVA_ERR_ARGUMENT, "layer index %d out of range", layer_index);
    if (!velocity && mlp->layers[layer_index]->nnz > 0) return fail(NERVA_ERR_ARGUMENT, "velocity is null");
    mlp->vel[layer_index] = velocity;
    return NERVA_OK;
}

void mlp_destroy(nerva_mlp *mlp)
{
    if (!mlp) return;
    mlp->prof.release();
    if (mlp->head_scratch) (void)hipFree(mlp->head_scratch);
    delete mlp;
}

int mlp_profile_enable(nerva_mlp *mlp, int32_t max_steps)
{
    if (!mlp || max_steps < 0) return fail(NERVA_ERR_ARGUMENT, "bad argument");
    mlp->prof.release();
    mlp->prof.on = max_steps > 0;
    mlp->prof.max_steps = max_steps;
    return NERVA_OK;
}

int mlp_profile_read(nerva_mlp *mlp, int32_t max_slots, int32_t *n_slots_host, double *ms_sum_host,
                     int32_t *steps_host)
{
    if (!mlp || !n_slots_host || !ms_sum_host || !steps_host) return fail(NERVA_ERR_ARGUMENT, "null argument");
    StepProfiler &P = mlp->prof;
    const int32_t n = static_cast<int32_t>(P.names.size());
    if (n > max_slots) return fail(NERVA_ERR_ARGUMENT, "%d slots, room for %d", n, max_slots);
    *n_slots_host = n;
    *steps_host = P.step;
    for (int32_t k = 0; k < n; ++k) ms_sum_host[k] = 0.0;
    if (P.events.size() != static_cast<size_t>(P.step) * (n + 1)) return fail(NERVA_ERR_HIP, "event bookkeeping is inconsistent");
    for (int32_t t = 0; t < P.step; ++t)
        for (int32_t k = 0; k < n; ++k) {
            const size_t i = static_cast<size_t>(t) * (n + 1) + k;
            HIP_TRY(hipEventSynchronize(P.events[i + 1]));
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, P.events[i], P.events[i + 1]));
            ms_sum_host[k] += ms;
        }
    return NERVA_OK;
}

const char *mlp_profile_slot_name(const nerva_mlp *mlp, int32_t slot)
{
    if (!mlp || slot < 0 || slot >= static_cast<int32_t>(mlp->prof.names.size())) return "";
    return mlp->prof.names[slot].c_str();
}

size_t mlp_workspace_bytes(const nerva_mlp *mlp, int32_t batch)
{
    if (!mlp || batch <= 0) return 0;
    Layout L;
    make_layout(mlp, batch, L);
    return static_cast<size_t>(L.bytes);
}

int mlp_workspace_layout(const nerva_mlp *mlp, int32_t batch, int64_t *layout_host)
{
    if (!mlp || !layout_host) return fail(NERVA_ERR_ARGUMENT, "null argument");
    if (batch <= 0) return fail(NERVA_ERR_ARGUMENT, "batch must be positive");
    Layout L;
    make_layout(mlp, batch, L);
    layout_host[0] = L.ld;
    for (size_t l = 0; l < mlp->layers.size(); ++l) {
        layout_host[1 + 4 * l + 0] = L[l].A;
        layout_host[1 + 4 * l + 1] = L[l].dZ;
        layout_host[1 + 4 * l + 2] = L[l].g;
        layout_host[1 + 4 * l + 3] = L[l].db;
    }
    return NERVA_OK;
}

static int check_step_args(const nerva_mlp *mlp, const float *X, int32_t ldx, int32_t batch, void *workspace,
                           size_t workspace_bytes, Layout &L)
{
    if (!mlp || !X || !workspace) return fail(NERVA_ERR_ARGUMENT, "null argument");
    int rc = check_batch(batch, ldx, "ldx");
    if (rc != NERVA_OK) return rc;
    if (batch > mlp->max_batch) return fail(NERVA_ERR_SHAPE, "batch %d exceeds max_batch %d", batch, mlp->max_batch);
    make_layout(mlp, batch, L);
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(NERVA_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    if (workspace_bytes < static_cast<size_t>(L.bytes))
        return fail(NERVA_ERR_WORKSPACE, "workspace has %zu bytes, %lld needed", workspace_bytes, (long long)L.bytes);
    return NERVA_OK;
}

static int forward_chain(nerva_mlp *mlp, const float *X, int32_t ldx, int32_t batch, char *ws, const Layout &L,
                         hipStream_t s, size_t n_layers)
{
    auto A_of = [&](size_t l) { return reinterpret_cast<float *>(ws + L[l].A); };
    auto args_of = [&](size_t l) { return forward_args(mlp->layers[l], l > 0 ? A_of(l - 1) : X, l > 0 ? L.ld : ldx, A_of(l), L.ld, batch); };
    // the streams of products in strips, which depend on the weights alone, in one launch at the start
    size_t ready = 0;   // layers below this one have theirs
    if (batch > kStripFromBatch) {
        SpmmCall strips[kStripStreams];
        int n = 0;
        for (; ready < n_layers && n < kStripStreams; ++ready)
            if (!use_dense(mlp->layers[ready], batch)) {
                strips[n] = args_of(ready);
                n += spmm_takes_strip(strips[n]);
            }
        if (n > 0) {
            Timed tm(mlp->prof, s, "strip_streams", 0);
            HIP_TRY(launch_strip_streams(strips, n, s));
        }
    }
    const float *in = X;
    int64_t ldin = ldx;
    for (size_t l = 0; l < n_layers; ++l) {
        const nerva_layer *ly = mlp->layers[l];
        float *A = A_of(l);
        SpmmCall a = args_of(l);
        a.strip_ready = l < ready;
        if (use_dense(ly, batch)) {
            Timed tm(mlp->prof, s, "dense_forward", static_cast<int>(l));
            HIP_TRY(dense_forward(ly, in, ldin, A, L.ld, batch, s));
        } else {
            Timed tm(mlp->prof, s, "spmm_forward", static_cast<int>(l));
            HIP_TRY(launch_spmm(a, s));
        }
        in = A;
        ldin = L.ld;
    }
    return NERVA_OK;
}

int mlp_forward(nerva_mlp *mlp, const float *X, int32_t ldx, int32_t batch, void *workspace, size_t workspace_bytes,
                void *stream)
{
    Layout L;
    int rc = check_step_args(mlp, X, ldx, batch, workspace, workspace_bytes, L);
    if (rc != NERVA_OK) return rc;
    return forward_chain(mlp, X, ldx, batch, static_cast<char *>(workspace), L, as_stream(stream), mlp->layers.size());
}

static int train_step(nerva_mlp *mlp, const float *X, int32_t ldx, const int32_t *labels, int32_t batch, float lr,
                      float momentum, void *workspace, const Layout &L, float *loss_out, void *stream);

int mlp_train_step(nerva_mlp *mlp, const float *X, int32_t ldx, const int32_t *labels, int32_t batch, float lr,
                   float momentum, void *workspace, size_t workspace_bytes, float *loss_out, void *stream)
{
    Layout L;
    int rc = check_step_args(mlp, X, ldx, batch, workspace, workspace_bytes, L);
    if (rc != NERVA_OK) return rc;
    if (!labels) return fail(NERVA_ERR_ARGUMENT, "labels is null");
    return train_step(mlp, X, ldx, labels, batch, lr, momentum, workspace, L, loss_out, stream);
}

int mlp_train_step_static(nerva_mlp *mlp, const float *X, int32_t ldx, const int32_t *labels, int32_t batch, float lr,
                          float momentum, float *loss_out, void *stream)
{
    if (!mlp || !X || !labels) return fail(NERVA_ERR_ARGUMENT, "null argument");
    if (mlp->prof.on) return fail(NERVA_ERR_ARGUMENT, "per-launch timing creates events: not available in mlp_train_step_static");
    int rc = check_batch(batch, ldx, "ldx");
    if (rc != NERVA_OK) return rc;
    if (batch > mlp->max_batch) return fail(NERVA_ERR_SHAPE, "batch %d exceeds max_batch %d", batch, mlp->max_batch);
    Layout L;
    make_layout(mlp, batch, L);
    if (static_cast<size_t>(L.bytes) > kStaticScratchBytes)
        return fail(NERVA_ERR_WORKSPACE, "this MLP at batch %d needs a workspace of %lld bytes, the static one has %zu: use mlp_train_step with a workspace of your own",
                    batch, (long long)L.bytes, kStaticScratchBytes);
    void *ws = nullptr;
    const hipError_t e = static_scratch(&ws);  // a table look-up once mlp_create has run on this device
    if (e != hipSuccess) return hip_fail(e, "address of the static workspace");
    // nothing in the workspace has to start at zero: every stage writes what the next one reads
    return train_step(mlp, X, ldx, labels, batch, lr, momentum, ws, L, loss_out, stream);
}

static int train_step(nerva_mlp *mlp, const float *X, int32_t ldx, const int32_t *labels, int32_t batch, float lr,
                      float momentum, void *workspace, const Layout &L, float *loss_out, void *stream)
{
    int rc = NERVA_OK;
    hipStream_t s = as_stream(stream);
    char *ws = static_cast<char *>(workspace);
    const int n = static_cast<int>(mlp->layers.size());
    const bool fused = !(mlp->flags & NERVA_MLP_UNFUSED);
    const int nesterov = (mlp->flags & NERVA_MLP_NESTEROV) ? 1 : 0;
    auto A = [&](int l) { return reinterpret_cast<float *>(ws + L[l].A); };
    auto dZ = [&](int l) { return reinterpret_cast<float *>(ws + L[l].dZ); };

    // a layer that was last trained as the first layer of another MLP: its mirror's values are behind
    for (int l = 1; l < n; ++l) {
        nerva_layer *ly = mlp->layers[l];
        if (!ly->mirror_stale) continue;
        HIP_TRY(launch_gather(ly->values_t, ly->values, ly->perm, ly->nnz, s));
        ly->mirror_stale = false;
    }
    if (mlp->layers[0]->nnz > 0) mlp->layers[0]->mirror_stale = true;  // neither pipeline below writes layer 0's mirror

    // feedforward, then the loss gradient / batch size
    const nerva_layer *last = mlp->layers[n - 1];
    const bool head = mlp->head && head_ok(last->rows, last->cols, last->nnz, batch);  // (a rebind may have grown the layer)
    bool ce_fused = false;  // softmax cross-entropy in the finish pass of the output layer's forward product
    int bias_done = -1;     // a layer whose biases the launch that formed its dZ has already updated
    // backpropagate and optimize, last layer first.  Layer l's transposed product T_l runs before
    // anything updates layer l's weights, so every gradient sees the weights of the step's start.
    auto make_T = [&](int l) {
        // dZ_{l-1} = (W_l^T dZ_l) * [A_{l-1} > 0]: the ReLU derivative of the layer below is
        // applied as the transposed product is stored
        nerva_layer *ly = mlp->layers[l];
        SpmmCall t{};
        t.blocks = ly->plan_t; t.hot = ly->hot.entry ? &ly->hot : nullptr; t.nnz = ly->nnz; t.scratch = ly->scratch; t.tickets = tickets_of(ly, 1); t.scratch_ld = ly->scratch_ld;
        t.indptr = ly->indptr_t; t.indices = ly->indices_t; t.values = ly->values_t;
        t.X = dZ(l); t.ldx = L.ld; t.Y = dZ(l - 1); t.ldy = L.ld;
        t.YM = A(l - 1); t.ldym = L.ld;
        t.rows = ly->cols; t.x_rows = ly->rows; t.batch = batch;
        return t;
    };
    auto make_S = [&](int l) {
        nerva_layer *ly = mlp->layers[l];
        SddmmCall g{};
        g.blocks = ly->plan;
        g.indptr = ly->indptr; g.indices = ly->indices;
        g.dZ = dZ(l); g.lddz = L.ld;
        g.X = l > 0 ? A(l - 1) : X; g.ldx = l > 0 ? L.ld : ldx;
        g.rows = ly->rows; g.x_rows = ly->cols; g.batch = batch; g.nnz = ly->nnz;
        g.partial = ly->partial; g.partial_stride = ly->partial_stride;
        g.partial_db_at = ly->partial_db_at; g.partial_tiles = ly->partial_tiles;
        if (ly->cur.has_table) { g.table = reinterpret_cast<const uint2 *>(ly->cur.table); g.table_words = table_words(ly); }
        g.split = split_of(ly);
        g.hot_values = hot_values_of(ly);
        if ((head || ce_fused) && l == n - 1 && loss_out) { g.loss_cols = mlp->head_scratch; g.loss_out = loss_out; g.loss_n = batch; }
        if (fused) {
            g.fused = 1; g.nesterov = nesterov; g.lr = lr; g.momentum = momentum;
            g.values = ly->values; g.velocity = mlp->vel[l];
            if (l > 0) { g.values_t = ly->values_t; g.pos_t = ly->pos_t; g.perm = ly->perm; }  // the first layer's mirror is never read
            if (ly->dense_on) { g.dense = ly->dense; g.dense_ld = ly->dense_ld; }
            if (l != bias_done) { g.bias = ly->bias; g.bias_velocity = mlp->bias_vel[l]; }
        } else {
            g.g = reinterpret_cast<float *>(ws + L[l].g);
            g.db = reinterpret_cast<float *>(ws + L[l].db);
        }
        return g;
    };

    // A saturated output layer too large for the head: its forward product streams the operand, and the finish pass of
    // that product can form the loss gradient as it stores the logits, when the layer's backward pass (one streaming
    // launch as well) is there to take the mean of the per-column losses.
    SpmmCall last_F{};
    if (!head && fused && n >= 2 && mlp->head_scratch && !use_dense(last, batch)) {
        last_F = forward_args(last, A(n - 2), L.ld, A(n - 1), L.ld, batch);
        last_F.ce_labels = labels; last_F.ce_dZ = dZ(n - 1); last_F.ce_lddz = L.ld; last_F.ce_loss_cols = mlp->head_scratch;
        ce_fused = true;  // (make_S then asks for the mean of the losses)
        ce_fused = spmm_softmax_epilogue_ok(last_F) && full_backward_ok(make_T(n - 1), make_S(n - 1));
    }
    rc = forward_chain(mlp, X, ldx, batch, ws, L, s, head || ce_fused ? n - 1 : n);
    if (rc != NERVA_OK) return rc;
    if (ce_fused) {
        Timed tm(mlp->prof, s, "spmm_forward+softmax_ce", n - 1);
        HIP_TRY(launch_spmm(last_F, s));
    } else if (head) {
        // output layer, loss and the gradient handed to layer n-2 in one launch
        HeadArgs h{};
        h.indptr = last->indptr; h.indices = last->indices; h.values = last->values; h.bias = last->bias;
        h.indptr_t = last->indptr_t; h.indices_t = last->indices_t; h.values_t = last->values_t;
        h.rows = last->rows; h.cols = last->cols; h.batch = batch; h.nnz = last->nnz;
        h.X = A(n - 2); h.ldx = L.ld; h.Z = A(n - 1); h.ldz = L.ld; h.labels = labels;
        h.dZ = dZ(n - 1); h.lddz = L.ld; h.dX = dZ(n - 2); h.lddx = L.ld;
        h.loss_cols = mlp->head_scratch;  // their mean is taken by the launch that runs S_{n-1}
        Timed tm(mlp->prof, s, "spmm_forward+softmax_ce+spmm_transposed", n - 1);
        HIP_TRY(launch_head(h, s));
    } else {
        Timed tm(mlp->prof, s, "softmax_ce", n - 1);
        HIP_TRY(launch_softmax_ce(A(n - 1), L.ld, labels, last->rows, batch, dZ(n - 1), L.ld, loss_out, s));
    }

    if (fused) {
        // Launch order T_{n-1} | T_{n-2} + S_{n-1} | ... | T_1 + S_2 | S_1 + S_0 (the last two as one where chain_ok): the fused
        // SDDMM+update S_l of a layer shares a grid with the transposed product of the layer
        // below, which no longer depends on it (S_l only needs dZ_l and must follow T_l).
        // dZ_{l-1} through the dense copy of layer l's weights
        auto dense_T = [&](int l) {
            return dense_transposed(mlp->layers[l], dZ(l), L.ld, dZ(l - 1), L.ld, A(l - 1), L.ld, batch, s);
        };
        // `pending`: a layer whose transposed product has run and whose S has not.  Where a layer's T and S
        // can share their gathers (backward_fused_ok) they run as one launch and nothing stays pending.
        int pending = -1;
        // Layers whose S runs as MFMA tiles sampled on the pattern (sddmm_sampled_ok) wait for the end of the step and
        // share one grid; nothing in the step depends on them.
        SampledArgs sampled{};
        int last_sampled = 0;
        auto flush_sampled = [&]() -> int {
            if (sampled.n == 0) return NERVA_OK;
            const bool dense_alone = sampled.n == 1 && mlp->layers[last_sampled]->dense_on;
            Timed tm(mlp->prof, s, dense_alone ? "dense_sddmm_update" : sampled.n == 1 ? "sddmm_update" : "sddmm_update+sddmm_update", last_sampled);
            HIP_TRY(launch_sampled(sampled, s));
            sampled = SampledArgs{};
            return NERVA_OK;
        };
        auto defer_S = [&](int l) -> int {
            // (timed launch by launch, every layer on the dense route gets a slot of its own)
            const bool apart = mlp->prof.on && mlp->layers[l]->dense_on;
            if (sampled.n == kSampledLayers || (apart && sampled.n > 0))
                if (const int e = flush_sampled(); e != NERVA_OK) return e;
            add_sampled(sampled, make_S(l));
            last_sampled = l;
            return apart ? flush_sampled() : static_cast<int>(NERVA_OK);
        };
        BackwardFinish finish{};   // layer 1's, which S_0 does not wait for
        auto run_S_alone = [&](int l) -> int {
            const SddmmCall g = make_S(l);
            if (sddmm_sampled_ok(g)) {
                HIP_TRY(launch_backward_finish(finish, s));
                return defer_S(l);
            }
            Timed tm(mlp->prof, s, "sddmm_update", l);
            HIP_TRY(launch_sddmm(g, s, &finish));
            return NERVA_OK;
        };
        if (head) pending = n - 1;  // the head launch has run T_{n-1}
        bool chained = false;       // S_0 has run
        for (int l = head ? n - 2 : n - 1; l >= 1; --l) {
            // dZ_l is ready: T_l (which hands dZ_{l-1} down) and S_l
            const SpmmCall t = make_T(l);
            if (use_dense(mlp->layers[l], batch)) {
                // (no grid to share with a dense product: a small output layer joins the sampled ones where it has a table)
                if (pending >= 0 && (rc = sddmm_sampled_possible(make_S(pending)) ? defer_S(pending) : run_S_alone(pending)) != NERVA_OK) return rc;
                { Timed tm(mlp->prof, s, "dense_transposed", l); HIP_TRY(dense_T(l)); }
                pending = l;
                continue;
            }
            const SddmmCall g_same = make_S(l);
            if (l == 1 && !use_dense(mlp->layers[0], batch) && chain_ok(t, g_same, make_S(0))) {
                // the rest of the step in one launch
                const SddmmCall g0 = make_S(0);
                SddmmCall waiting{};
                if (pending >= 0) waiting = make_S(pending);
                const bool along = pending >= 0 && can_pair(g0, waiting);
                if (pending >= 0 && !along && (rc = run_S_alone(pending)) != NERVA_OK) return rc;
                Timed tm(mlp->prof, s, "backward_chain", 1);
                HIP_TRY(launch_chain(t, g_same, g0, along ? &waiting : nullptr, s));
                pending = -1;
                chained = true;
                continue;
            }
            if (full_backward_ok(t, g_same)) {
                if (pending >= 0 && (rc = run_S_alone(pending)) != NERVA_OK) return rc;
                pending = -1;
                SddmmCall g_full = g_same;
                if (bias_done < 0 && mlp->layers[l - 1]->bias) {
                    // dZ_{l-1} is formed a whole row per wave: the bias gradient of layer l-1 is that row's sum
                    g_full.below_bias = mlp->layers[l - 1]->bias; g_full.below_bias_velocity = mlp->bias_vel[l - 1];
                    bias_done = l - 1;
                }
                Timed tm(mlp->prof, s, "backward_full", l);
                HIP_TRY(launch_full_backward(t, g_full, s));
                continue;
            }
            if (backward_fused_ok(t, g_same, false)) {
                if (pending >= 0 && (rc = run_S_alone(pending)) != NERVA_OK) return rc;
                pending = -1;
                Timed tm(mlp->prof, s, "backward_fused", l);
                if (backward_hot_ok(t, g_same)) HIP_TRY(order_hot_rows(mlp->layers[l], s));
                // (not while a profile is on, whose slots hold what their names say, nor where both layers are one handle: S_0 would write the partial products that the finish pass reads)
                HIP_TRY(launch_backward_fused(t, g_same, false, s, l == 1 && !mlp->prof.on && mlp->layers[0] != mlp->layers[1] ? &finish : nullptr));
                continue;
            }
            if (pending >= 0) {
                const SddmmCall g = make_S(pending);
                if (can_pair(t, g)) {
                    Timed tm(mlp->prof, s, "spmm_transposed+sddmm_update", l);
                    HIP_TRY(launch_pair(t, g, s));
                } else {
                    { Timed tm(mlp->prof, s, "spmm_transposed", l); HIP_TRY(launch_spmm(t, s)); }
                    if ((rc = run_S_alone(pending)) != NERVA_OK) return rc;
                }
            } else {
                Timed tm(mlp->prof, s, "spmm_transposed", l);
                HIP_TRY(launch_spmm(t, s));
            }
            pending = l;
        }
        // the first layer has no transposed product: its S, with the one still pending if any
        if (!chained && pending >= 0) {
            const SddmmCall gp = make_S(pending), g0 = make_S(0);
            if (pending == 1 && can_pair(g0, gp)) {
                Timed tm(mlp->prof, s, "sddmm_update+sddmm_update", 0);
                HIP_TRY(launch_pair(g0, gp, s));  // the larger layer's work-groups start first
            } else {
                if ((rc = run_S_alone(pending)) != NERVA_OK) return rc;
                if (pending != 0 && (rc = run_S_alone(0)) != NERVA_OK) return rc;
            }
        } else if (!chained && (rc = run_S_alone(0)) != NERVA_OK) {
            return rc;
        }
        if ((rc = flush_sampled()) != NERVA_OK) return rc;
    } else {
        const bool as_chain = n > (head ? 2 : 1) && !use_dense(mlp->layers[1], batch) && !use_dense(mlp->layers[0], batch) && chain_shape_ok(make_T(1), make_S(1), make_S(0));
        for (int l = n - 1; l >= 0; --l) {
            nerva_layer *ly = mlp->layers[l];
            if (l > 0 && !(head && l == n - 1)) {
                if (use_dense(ly, batch)) {
                    Timed tm(mlp->prof, s, "dense_transposed", l);
                    HIP_TRY(dense_transposed(ly, dZ(l), L.ld, dZ(l - 1), L.ld, A(l - 1), L.ld, batch, s));
                } else {
                    Timed tm(mlp->prof, s, "spmm_transposed", l);
                    if (l == 1 && as_chain)
                        HIP_TRY(launch_chain_transposed(make_T(1), make_S(1), make_S(0), s));
                    else
                        HIP_TRY(launch_spmm(make_T(l), s));
                }
            }
            SddmmCall g = make_S(l);
            g.chain_lanes = as_chain && l <= 1;
            {
                Timed tm(mlp->prof, s, "sddmm", l);
                HIP_TRY(launch_sddmm(g, s));
            }
            {
                Timed tm(mlp->prof, s, "momentum_values", l);
                HIP_TRY(launch_momentum(ly->values, mlp->vel[l], g.g, ly->nnz, lr, momentum, nesterov, s));
            }
            if (ly->bias) {
                Timed tm(mlp->prof, s, "momentum_bias", l);
                HIP_TRY(launch_momentum(ly->bias, mlp->bias_vel[l], g.db, ly->rows, lr, momentum, nesterov, s));
            }
            if (l > 0) {
                Timed tm(mlp->prof, s, "mirror_refresh", l);
                HIP_TRY(launch_gather(ly->values_t, ly->values, ly->perm, ly->nnz, s));
            }
            if (ly->dense_on) {
                Timed tm(mlp->prof, s, "dense_refresh", l);
                HIP_TRY(refresh_dense_copies(ly, s));
            }
        }
    }
    if (mlp->prof.on && mlp->prof.step < mlp->prof.max_steps) {
        hipEvent_t e = nullptr;  // closes the last launch of the step
        HIP_TRY(hipEventCreate(&e));
        mlp->prof.events.push_back(e);
        HIP_TRY(hipEventRecord(e, s));
        ++mlp->prof.step;
    }
    return NERVA_OK;
}

int nerva_copy_f32(float *dst, const float *src, int64_t n, void *stream)
{
    if (n < 0 || (n > 0 && (!dst || !src))) return fail(NERVA_ERR_ARGUMENT, "bad argument");
    HIP_TRY(launch_copy(dst, src, n, as_stream(stream)));
    return NERVA_OK;
}

}  // extern "C"
