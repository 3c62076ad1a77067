// Internal launch interface between the C ABI (api.hip) and the gfx950 kernels (kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nerva {

constexpr int kWavesPerBlock = 16;   // 1024 threads

// Static partition of the rows of a CSR matrix over work-groups, built once per pattern.
// A work-group has kWavesPerBlock waves.  Ordinary rows: the work-group serves
// (kWavesPerBlock >> lg) rows, 2^lg waves per row, each wave taking a contiguous share of the
// row's stored entries.  Huge rows (more entries than a whole work-group should take) are cut
// into several work-groups; each leaves a partial result, and the last of them to do so adds them
// up in share order.  Huge work-groups come first, so blockIdx.x is also their scratch slot.
struct RowBlocks {
    const int4 *huge_rows;     // [n_huge_rows] {row, first work-group, number of work-groups, 0}
    const int4 *waves;         // [n_blocks * kWavesPerBlock] the partition, spelled out per wave:
                               // {row or -1, first entry, end entry, part | lg << 4 | lead << 8 | huge << 9 | index in huge_rows << 10}
    int32_t n_blocks;
    int32_t n_huge_rows;
    int32_t n_huge_blocks;
    // Optional second partition, built for matrices with many short rows (n_short > 0): rows of
    // at most kPackMaxLen entries are listed longest first and served one row per lane group,
    // 64/GS rows per wave (spmm_packed_kernel); the remaining rows keep a partition of their
    // own, huge work-groups first exactly as in `waves` (same scratch slots, same huge_rows).
    const int4 *short_rows;    // [n_short rounded up to a multiple of 64] {row or -1, first entry, entries, 0}
    const int4 *long_waves;    // [n_long_blocks * kWavesPerBlock], records as in `waves`
    int32_t n_short;
    int32_t n_long_blocks;
    // Share of the stored entries whose gathered operand row is one of the kHotRows most
    // referenced ones: when it is large the gathers hit in cache without any column tiling.
    float hot_share;
    // Optional third form, for the staged product (spmm_staged_kernel; staged_rows != nullptr).
    // The rows are cut into staged_ranges ranges of at most kStageRangeRows rows and about equal
    // work; inside a range the rows are listed longest first (slot 0, 1, ...; unused slots hold
    // -1).  A row much longer than its range's mean takes four slots, a multiple of 4 onwards, marked
    // kStageQuad: the four lane rows of one wave then serve a quarter of each of its segments each
    // and their results are added at the end.  Every row is cut into segments at the multiples of kStageRows in its column indices:
    // staged_ends[(range * (staged_cblocks + 1) + b) * kStageRangeRows + slot] is the position of
    // the slot's first stored entry with column >= b * kStageRows (b = 0: the row's first entry,
    // b = staged_cblocks: one past its last; unused slots: 0 throughout).
    const int32_t *staged_rows;    // [staged_ranges * kStageRangeRows]
    const int32_t *staged_ends;
    const int32_t *staged_groups;  // [staged_ranges] rows of the range / 64, rounded up
    int32_t staged_ranges;
    int32_t staged_cblocks;
    int32_t staged_longest_share;  // most stored entries any one lane row serves
    int32_t staged_longest_row;    // stored entries of the longest row
    int32_t staged_partial;        // the plan covers the rows of more than kPackMaxLen entries only: the others are
                                   // short_rows and take the packed kernel
    int32_t staged_row_count;      // rows the plan covers
    const int4 *rest_waves;        // where there are both short and longer rows: partition of the rows of at most kPackMaxLen
    int32_t n_rest_blocks;         //   entries alone, records as in `waves` (no huge rows among them)
    int32_t long_nnz;              // stored entries of the rows beyond kPackMaxLen (those of long_waves)
    int32_t staged_nnz;            // and their stored entries
    int32_t staged_preferred;      // measurement aid: take the staged kernels wherever they can run
    const int4 *rows_by_length;    // every row, as in short_rows (which is the end of this table)
};

// What few kernels read of a pattern, apart from RowBlocks, which every launch carries (with these and the strips' in it calls of 4 to 12 us took 1 to 4 % longer).
// The product in strips (spmm_strip_kernel): sets of kStripSet rows, longer ones first, cut into segments at the multiples of block_rows in the column indices.
struct Strips {
    const int32_t *rows = nullptr;    // [sets * kStripSet] row or -1
    const int2 *segs = nullptr;       // [sets * blocks] {first chunk of the stream, entries of the longest of the set's segments in that block}
    const int32_t *cuts = nullptr;    // [sets * (blocks + 1) * kStripSet] position of a row's first entry of a block, and one past its last
    int32_t blocks = 0, block_rows = 0;
    int32_t chunks = 0, steps = 0;    // of the stream; the sum of the longest segments
    int32_t preferred = 0;            // measurement aid: take it wherever it can run
};
// Of a mirror, where a few rows of the matrix hold most of its entries (backward_hot_kernel): the entries of a mirror row in another order, those of the
// kHotRowsLds longest rows of the matrix first.
struct HotRows {
    const int32_t *entry = nullptr;   // [nnz] 256 times the row's place among the longest, for the hot ones of a mirror row; the row itself for the others
    const int32_t *at = nullptr;      // [nnz] the entry's position in the mirror
    const int4 *sets = nullptr;       // [mirror rows, padded as rows_by_length] {row or -1, first entry, entries, hot ones}: longest first, those of about one length by their hot entries
    const int32_t *perm = nullptr;    // [nnz] CSR position
    const int4 *rows = nullptr;       // the matrix's rows_by_length
    float share = 0.f;                // of the entries, those of the kHotRowsLds longest rows
};

// Strips: kStripRows operand rows of kStripCols columns lie in LDS at a time; the operand's blocks are of equal size, a multiple of 256 rows.
constexpr int32_t kStripRows = 2048, kStripCols = 16, kStripSet = 16;
constexpr int32_t kStripChunk = 8;       // entries of each of a set's rows in a chunk of the stream, kStripChunk * kStripSet * 8 bytes
constexpr int32_t kStripFromBatch = 192; // wider ones only
constexpr int32_t kStripMaxBlocks = 32;
__host__ __device__ inline int32_t strip_blocks_of(int32_t x_rows) { return (x_rows + kStripRows - 1) / kStripRows; }
__host__ __device__ inline int32_t strip_block_rows_of(int32_t x_rows)
{
    const int32_t n = strip_blocks_of(x_rows);
    return ((x_rows + n - 1) / n + 255) / 256 * 256;
}
// first operand row that LDS holds in block b: the last block starts early enough to be whole
__host__ __device__ inline int32_t strip_block_base(int32_t b, int32_t block_rows, int32_t x_rows)
{
    const int32_t last = x_rows > block_rows ? x_rows - block_rows : 0;
    return b * block_rows < last ? b * block_rows : last;
}

constexpr int32_t kHotRowsLds = 512;
constexpr int32_t kStageRows = 512;      // operand rows held in LDS at a time
constexpr int32_t kStageCols = 64;       // columns of the operand (examples) per work-group
constexpr int32_t kStageJ = 8;           // rows per row of 16 lanes
constexpr int32_t kStageQuad = 1 << 30;  // flag in staged_rows: the slot is one of the four of a split row
constexpr int32_t kStageRangeRows = 512; // rows per work-group: 16 waves x 4 lane rows x kStageJ
constexpr int32_t kStageRangeFill = kStageRangeRows - 4;  // slots after which a range is cut (a split row takes four at once)
constexpr int32_t kStageMinBatch = 128;  // narrower batches never take the staged product
constexpr int32_t kStageTargetGroups = 256;  // work-groups wanted at max_batch (one per compute unit)
constexpr float kStageMinReuse = 2.f;    // stored entries per staged operand row and work-group, at least
// Mean entries per segment from which staging pays whatever the operand's size.  Products: kStageLongSegment, kStageSegmentSomeWork from so much work
// (the plan's entries times columns) on: 8.7 and 10 entries, in column tiles / staged, us: 8192^2 at 1.7 / 1.95 %, batch 256 / 512 / 1024 77 / 76, 136 / 99,
// 267 / 192 and 84 / 77, 152 / 104, 295 / 198; 4500^2 and 6000^2 at 1.75 %, batch 512 43 / 47, 61 / 64, batch 1024 65 / 59, 119 / 92; of 44 more staged takes 0.59
// to 1.01 of the time above the line and 0.81 to 1.52 below it, by shape and not by work; below 8 no plan is made but for operands of 48 MiB.
constexpr int32_t kStageLongSegment = 10;
constexpr int32_t kStageSegmentSomeWork = 8;
constexpr int64_t kStageSomeWork = 324 << 20;
// The SDDMM, which has its second pass to pay for as well, and from so much work on: 8192^2 at 1.95 / 2.5 / 3.5 %, batch 256 76 / 91 / 135 -> 86 / 97 / 116, batch
// 512 143 / 173 / 254 -> 128 / 147 / 177, batch 1024 271 / 328 / 477 -> 251 / 288 / 338; 5000^2, batch 512 54 / 69 / 90 -> 61 / 68 / 81; 12000^2 at 2.5 %, batch 256 /
// 1024 233 / 853 -> 177 / 529; of 58 more 0.67 to 1.04 above the line, 0.81 to 1.53 below.
constexpr int32_t kStageLongSegmentSddmm = 20;
constexpr int32_t kStageSegmentMuchWork = 10;
constexpr int64_t kStageMuchWork = 420 << 20;
constexpr int32_t kStageSegmentBesideDense = 8;   // ... and the SDDMM of the rows beside dense ones (DenseSplit), from batch 512 on: power-law 16384^2 at 3 / 10 %,
                                                  // batch 1024: 1249 -> 932 and 3405 -> 2265 us; at batch 256 4096^2 loses (55 -> 84)
constexpr int64_t kStageBigOperand = 48ll << 20;  // operand bytes no set of L2s holds: staging pays for shorter segments,
constexpr int32_t kStageSegmentBigOperand = 4;    // ... from this many entries per segment on
constexpr int32_t kHotRows = 1024;
constexpr int32_t kPackMaxLen = 128;     // longest row served by the packed path
constexpr int32_t kPackMinRows = 2048;   // fewer short rows than this: no packed path
constexpr int32_t kPackSets = 1;         // row sets (64/GS rows each) per wave; measured on the wide MLP: 1 / 2 / 4 / 8 sets give 500 / 504 / 527 / 548 us per step

// Rows of a matrix that are dense enough for matrix instructions (dense_rows_kernel in dense.hip), and their pattern table.
struct DenseRows {
    const int32_t *list;           // [n] ascending, or nullptr: all rows
    const uint2 *table;            // [n * words] {bits of 32 columns, CSR position of the first of them}
    int32_t n, words;
    float *partial;                // results of the slices of K, partial_floats long
    int64_t partial_floats;
    uint32_t *parts;               // parts of the operand for the product on the bf16 units, parts_ints long (operand_parts_ints)
    int64_t parts_ints;
};
// A matrix some of whose rows are served that way, from `from_batch` columns on: those, and the partition without them that the
// others then run on.  Host memory.
struct DenseSplit {
    DenseRows rows;                // n = 0: there are none, or too few
    int32_t from_batch;
    int64_t dense_nnz;             // the listed rows' stored entries
    int64_t thin_nnz;              // all rows of a matrix of kThinDensity: its stored entries, or 0; then also
    int32_t max_batch;             // what it is bound for
    const uint8_t *flag;           // [rows of the matrix] 1: a dense row
    RowBlocks others;
};
constexpr int32_t kDenseRowsMinCols = 1024;    // (so that a dense row is longer than kPackMaxLen)
constexpr int32_t kDenseRowsMin = 17;          // fewer rows than this stay with the others
constexpr int64_t kDenseRowsMinWork = 192 << 20;  // entries times columns of the batch from which the extra launch pays
constexpr int32_t kDenseRowsMinBatch = 128;    // (narrower ones leave much of a tile of 64 or 128 columns idle)
// the batch from which the listed rows have that much work
__host__ __device__ inline int32_t dense_rows_from(int64_t dense_nnz)
{
    const int64_t b = (kDenseRowsMinWork + dense_nnz - 1) / dense_nnz;
    return b > kDenseRowsMinBatch ? static_cast<int32_t>(b) : kDenseRowsMinBatch;
}
// A matrix of at least kThinDensity that has no such rows (dense_rows_pay) pays on the bf16 units alone (split.hip), with all its rows, and there at batches that
// fill their tiles of 256 columns and that gathering is slow at (dense_rows_product_ok): many rows of many columns, wide batches.  Its partitions stay
// those of a sparse one, so that binding it takes no launch more.
constexpr int32_t kThinRows = 512, kThinCols = 2048, kThinBatch = 192;
constexpr int64_t kThinWork = 384 << 20;
constexpr float kThinDensity = 0.17f;          // (has a pattern table: kTableFromDensity)
// Stored entries from which a row counts as dense: an eighth of its columns.  At batch 1024 such a row costs the matrix units
// 0.30 us per 16384 columns and the staged kernel 2.0 us times its density among power-law rows.  On the bf16 units it costs 0.20, but the staged kernel
// gains less from what is taken out of it: forward products of 16384^2 at batch 1024 with an 8th / 10th / 12th / 16th: 10 % 1590 / 1621 / 1635 / 1708 us,
// 6 % 1204 / 1242 / 1233 / 1671, 3 % 703 / 709 / 711 / 722.
__host__ __device__ inline int32_t dense_row_length(int32_t cols) { return cols / 8 > 128 ? cols / 8 : 129; }

// Y = epilogue( W * gather(X) ) for a CSR matrix W (rows x cols); also used on the CSC
// mirror, where "rows" are W's columns.
struct SpmmArgs {
    RowBlocks blocks;
    const int32_t *indptr;   // [rows+1]
    const int32_t *indices;  // [nnz]
    const float *values;     // [nnz]
    const float *bias;       // [rows] or nullptr
    const float *X;          // gathered operand, (cols, ldx)
    int64_t ldx;
    const float *XM;         // optional (cols, ldxm): operand row j is X[j,c] * [XM[j,c] > 0]
    int64_t ldxm;
    float *Y;                // (rows, ldy)
    int64_t ldy;
    const float *YM;         // optional (rows, ldym): result is multiplied by [YM[i,c] > 0]
    int64_t ldym;
    int32_t rows;
    int32_t x_rows;          // rows of the gathered operand (columns of the sparse matrix)
    int32_t batch;
    int32_t relu;            // clamp the result at zero
    int32_t wide_offsets;    // an operand spans 4 GiB or more (set by the launch)
    int32_t nnz;             // length of indices/values
    float *scratch;          // partial rows of huge-row work-groups, (n_huge_blocks, scratch_ld)
    int64_t scratch_ld;
    int32_t *tickets;        // huge row k's: huge_row_tickets(scratch_ld) of them from tickets + 2 * k * huge_row_tickets(scratch_ld) on (the
                             // other orientation's lie between); all 0 between launches
    // Only for a matrix that stores every entry and has at most kFullMaxRows rows (a saturated
    // output layer): values[] is then the row-major dense matrix, and the product streams the
    // operand once for all rows instead of gathering it once per row.  Partial results of the
    // kFullSlice-column slices of W: full_scratch[(slice * rows + row) * full_scratch_ld + column].
    float *full_scratch;     // or nullptr: the matrix is not full, or has too many rows
    int64_t full_scratch_ld;
    // Optional epilogue for an output layer served that way (spmm_softmax_epilogue_ok): the softmax
    // cross-entropy of the logits Y against ce_labels -- ce_dZ = (softmax(Y) - onehot) / batch, one
    // loss per column into ce_loss_cols (their mean is taken by a later launch, SddmmArgs::loss_cols).
    const int32_t *ce_labels;  // [batch] or nullptr: no epilogue
    float *ce_dZ;              // (rows, ce_lddz)
    int64_t ce_lddz;
    float *ce_loss_cols;       // [batch]
};
// A call: what its kernels are given, and what chooses among them and is no kernel's of the others (in host memory).  Every launch carries all of its
// kernel's arguments, so that what one kernel reads is handed to that one: with 88 bytes more in them calls of 4 to 12 us take 1 to 4 % longer.
struct SpmmCall : SpmmArgs {
    const DenseSplit *split;   // or nullptr
    const Strips *strips;      // the pattern's, or nullptr
    const HotRows *hot;        // of a mirror, or nullptr
    float4 *strip_stream;      // (device memory) room for the plan's chunks and two more, or nullptr
    int32_t strip_ready;       // launch_strip_streams has filled it
};
static_assert(sizeof(SpmmArgs) <= 336, "every product's launch carries them");
// What the product in strips is given in place of the matrix, for up to kStripStreams products in one launch.
constexpr int kStripStreams = 4;
struct StripStream {
    const int2 *segs;
    const int32_t *cuts, *indices;
    const float *values;
    float4 *out;
    int32_t sets, blocks, block_rows, x_rows, nnz;
};
struct StripStreams {
    StripStream of[kStripStreams];
};
bool spmm_takes_strip(const SpmmCall &a);
hipError_t launch_strip_streams(const SpmmCall *list, int n, hipStream_t s);
// tickets per huge row, one per 32 columns
__host__ __device__ inline int64_t huge_row_tickets(int64_t scratch_ld) { return scratch_ld / 32; }
bool spmm_softmax_epilogue_ok(const SpmmCall &a);
constexpr int32_t kFullMaxRows = 16;
constexpr int32_t kFullSlice = 128;   // columns of W (rows of the operand) per work-group
hipError_t launch_spmm(const SpmmCall &a, hipStream_t s);

// g[p] = <dZ[row(p),:], X[indices[p],:]>, db[i] = sum_c dZ[i,c]; optionally followed, inside
// the same kernel, by the momentum step on values/velocity (and bias/bias_velocity).
struct SddmmArgs {
    RowBlocks blocks;
    const int32_t *indptr;
    const int32_t *indices;
    const float *dZ;         // (rows, lddz)
    int64_t lddz;
    const float *ZM;         // optional (rows, ldzm): dZ is multiplied by [ZM > 0]
    int64_t ldzm;
    const float *X;          // (cols, ldx)
    int64_t ldx;
    float *g;                // [nnz] or nullptr
    float *db;               // [rows] or nullptr
    int32_t rows;
    int32_t x_rows;          // rows of X (columns of the sparse matrix)
    int32_t batch;
    int32_t skip_products;   // only db is wanted: do not touch indptr/indices/X
    // fused momentum step (fused != 0): g/db are not stored unless non-null
    int32_t fused;
    int32_t nesterov;
    float lr, momentum;
    float *values;           // [nnz]
    float *velocity;         // [nnz]
    float *values_t;         // mirror values or nullptr
    const int32_t *pos_t;    // CSR position -> mirror position (needed iff values_t)
    const int32_t *perm;     // mirror position -> CSR position (only the fused backward pass needs it)
    float *bias;             // [rows] or nullptr
    float *bias_velocity;    // [rows] or nullptr
    // launch_full_backward only: the biases of the layer BELOW and their momentum buffer, or nullptr.  That layer's
    // bias gradient is the row sum of the dX this launch forms, a wave per row, so its update can ride along
    // (the caller then leaves the biases out of that layer's own update).
    float *below_bias;
    float *below_bias_velocity;
    // by-product, unrelated to the layer: *loss_out = mean(loss_cols[0..loss_n)), summed in one fixed
    // order by the first wave of the launch.  The head kernel leaves one loss per batch column; a
    // grid-wide sum inside it would need device-scope fences, which write back and invalidate the L2s.
    const float *loss_cols;  // or nullptr
    float *loss_out;
    int32_t loss_n;
    // column-tiled route for operands X that no L2 holds: per-tile partial products
    // [tile][partial_stride] (values first, then the per-row sums of dZ at partial_db_at), added in
    // tile order by a second kernel that also applies the update.  nullptr: route not available.
    float *partial;
    int64_t partial_stride;   // floats per tile, >= partial_db_at + rows
    int64_t partial_db_at;    // >= nnz
    int32_t partial_tiles;    // tiles the buffer has room for
    int32_t nnz;
    // dense copy of a layer on the dense route (or nullptr): the fused update stores every new
    // weight there too, dense[row * dense_ld + col]
    float *dense;
    int64_t dense_ld;
    // pattern table of a layer dense enough for the sampled gradient (or nullptr): [rows * table_words]
    const uint2 *table;
    int32_t table_words;
    int32_t chain_lanes;            // 1: the sums of chain_kernel, for a step whose launches are kept apart
};
struct SddmmCall : SddmmArgs {      // (see SpmmCall)
    const DenseSplit *split;        // or nullptr
    const DenseSplit *split_done;   // (set by the launch) the dense rows are served already
    float *hot_values;              // (device memory) scratch [nnz] of backward_hot_kernel, or nullptr
};
static_assert(sizeof(SddmmArgs) <= 424, "every launch of a gradient carries them");
// Column-tile width (in columns) the products use when their gathered operand has x_rows rows and
// does not fit an L2; 0: no tiling.  Shared by the kernels' dispatch and by the sizing of the
// SDDMM partial buffer when a layer is created.
int tile_columns(int32_t x_rows, int32_t batch, int64_t nnz, int32_t rows, int32_t longest_row, float hot_share, bool masked, bool for_sddmm = false);
struct BackwardFinish;
// first: a finish pass of the layer above that waits, which runs before or in this launch
hipError_t launch_sddmm(const SddmmCall &a, hipStream_t s, BackwardFinish *first = nullptr);
// Slices of partial products (SddmmArgs::partial) that the column-tiled SDDMM and the fused backward pass take at any batch up to max_batch
int32_t partial_tiles_wanted(const RowBlocks &plan, const RowBlocks &plan_t, int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch);

// Transposed product and SDDMM of one layer on one gather stream (backward_fused_kernel).
struct BackwardArgs {
    RowBlocks blocks;            // the mirror's partition (its table of short rows)
    const int32_t *indices;      // mirror: row of W of each entry
    const float *values;         // mirror values
    const float *dZ;             // (rows of W, lddz): gathered
    int64_t lddz;
    const float *ZM;             // optional: dZ is multiplied by [ZM > 0]
    int64_t ldzm;
    const float *X;              // (cols of W, ldx): the layer's input; second operand of the products and mask of dX
    int64_t ldx;
    float *dX;                   // (cols of W, lddx)
    int64_t lddx;
    int32_t mask;                // multiply dX by [X > 0]
    int32_t rows, x_rows, batch, nnz;   // rows = mirror rows = columns of W; x_rows = rows of W
    float *partial;              // [tile][partial_stride]: products in mirror order
    int64_t partial_stride;
    const int32_t *perm;         // mirror position -> CSR position
    const float *refresh;        // values[] (CSR order), from which the launch brings the mirror values up to date (w_t), or nullptr
    // what the second pass does with the sums: store them (g, db: CSR order) and / or the momentum step
    float *g, *db;
    int32_t fused, nesterov;
    float lr, momentum;
    float *w, *velocity, *w_t;   // values[], velocity[] (CSR order), mirror values
    float *bias, *bias_velocity;
};
static_assert(sizeof(BackwardArgs) <= 352, "every launch of a backward pass carries them");
// alone: a single call, not part of a training step, where the two may share their launches with other layers' instead
bool backward_fused_ok(const SpmmCall &t, const SddmmCall &g, bool alone);
// whether such a call also brings the mirror values (g.values_t) up to date with g.values, so that the caller need not
bool backward_fused_refreshes(const SpmmCall &t, const SddmmCall &g);
// whether it takes the hot rows of dZ out of LDS
bool backward_hot_ok(const SpmmCall &t, const SddmmCall &g);
// The second pass over the partial products, where it is left to a launch that follows (later, which launch_sddmm or launch_backward_finish take).
struct BackwardFinish {
    BackwardArgs a;
    const int32_t *hot_at;       // of an order of HotRows, in which the products are then: the entries' positions in the mirror; else nullptr
    int32_t n_tiles, n_entry_blocks, n_row_blocks;
    bool waiting;
};
hipError_t launch_backward_finish(BackwardFinish &f, hipStream_t s);
hipError_t launch_backward_fused(const SpmmCall &t, const SddmmCall &g, bool alone, hipStream_t s, BackwardFinish *later = nullptr);
bool full_backward_ok(const SpmmCall &t, const SddmmCall &g);
hipError_t launch_full_backward(const SpmmCall &t, const SddmmCall &g, hipStream_t s);

// Two independent launches in one grid (both on the 16-byte path, batch <= 1024, one column tile).
bool can_pair(const SpmmCall &a, const SddmmCall &b);
bool can_pair(const SddmmCall &a, const SddmmCall &b);
hipError_t launch_pair(const SpmmCall &a, const SddmmCall &b, hipStream_t s);
// The end of a training step in one launch (chain_kernel): T_1, S_1 and S_0, and the SDDMM of a layer above that waits for its update (or nullptr;
// can_pair(g0, it)).
struct ChainArgs {
    const int32_t *indptr_t, *indices_t, *perm;   // W_1's mirror
    float *values_t, *w, *velocity;               // its values, W_1's values[] and velocity[]
    float *bias, *bias_velocity;                  // of W_1
    const float *dZ, *A;                          // dZ_1 and A_0
    float *dZ_below;                              // dZ_0
    int64_t lddz, lda, lddz_below;
    int32_t rows;                                 // of dZ_1
};
constexpr int32_t kChainMinRows = 256, kChainMaxBatch = 192;
// chain_shape_ok: the part that does not depend on whether the updates are fused; then a step that keeps its launches apart forms dZ_0 in the same order.
bool chain_ok(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0);
bool chain_shape_ok(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0);
hipError_t launch_chain_transposed(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0, hipStream_t s);
hipError_t launch_chain(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0, const SddmmCall *waiting, hipStream_t s);
hipError_t launch_pair(const SddmmCall &a, const SddmmCall &b, hipStream_t s);

hipError_t launch_momentum(float *w, float *v, const float *g, int64_t n, float lr, float mu, int nesterov,
                           hipStream_t s);
// values_t[q] = values[perm[q]]
hipError_t launch_gather(float *values_t, const float *values, const int32_t *perm, int64_t n,
                         hipStream_t s);
// the same, and dZ = dY * [Y > 0] (rows x batch, batch >= 4) in one launch
hipError_t launch_backward_prep(float *values_t, const float *values, const int32_t *perm, int64_t nnz, const float *dY, int64_t lddy,
                                const float *Y, int64_t ldy, float *dZ, int64_t lddz, int32_t rows, int32_t batch, hipStream_t s);
hipError_t launch_softmax_ce(const float *Z, int64_t ldz, const int32_t *labels, int32_t classes,
                             int32_t batch, float *dZ, int64_t lddz, float *loss, hipStream_t s);
hipError_t launch_copy(float *dst, const float *src, int64_t n, hipStream_t s);

// Dense route of a layer whose density is high (the density-adaptive layer the paper plans in
// "Discussion and Conclusion" and Appendix C.3).  One zero-filled dense copy of the weights, row-major
// W[i * ldw + j] with ldw = cols rounded up to kDenseLdAlign (zero off the pattern and in the padding), serves
// the forward product and the transposed product (the same copy read down its columns); the update of the stored
// entries is sampled from tiles of G = dZ X^T (SampledLayer below), which is never stored.
constexpr int32_t kDenseLdAlign = 64;
constexpr float kTableFromDensity = 0.15f;  // layers at least this dense get a pattern table when they are bound
// Layers at least this dense take the dense route by themselves.  Steps of 3072-1024-512-10 at batch 100, dense / sparse route: 53.2 / 78.6 us at
// 50 % density, 51.2 / 80.6 at 40 %, 48.4 / 56.5 at 20 %; 2048-4096-2048-10 at batch 64 127 / 268, 121 / 229, 105 / 138, at 1024 854 / 856, 844 / 785, 830 / 683:
// below the line the dense route would be the faster one for narrow batches too, but an infinity in an operand reaches every row on it.
constexpr float kDenseFromDensity = 0.4f;
struct DenseArgs {
    const float *W;      // the dense copy, (rows, ldw)
    int64_t ldw;
    int32_t trans;       // 0: Y (rows x batch) = act(W X + b);  1: Y (cols x batch) = (W^T X) * [YM > 0]
    const float *X;      // (cols, ldx) or, transposed, (rows, ldx)
    int64_t ldx;
    float *Y;
    int64_t ldy;
    const float *bias;   // [rows] or nullptr (forward only)
    const float *YM;     // optional: result is multiplied by [YM > 0]
    int64_t ldym;
    int32_t rows, cols, batch;
    int32_t relu;
    float *partial;      // forward: kNnShareFloats floats and kNnTickets zeros (as the product leaves them), for tiles that several work-groups
    int32_t *tickets;    //   share; or nullptr: none is shared
};
constexpr int32_t kNnShareTiles = 256, kNnShareFloats = 2 * kNnShareTiles * 1024;   // (less than 2 * kNnShareTiles work-groups, 16 x 64 sums each)
// A ticket always counts up to the same number: with one set for tiles in two and in four slices, calls of different batches that overlap
// would leave it between the two, and calls after them would find it there.
constexpr int32_t kNnTickets = kNnShareTiles + kNnShareTiles / 2;                   // of tiles in two slices, then in four (nn_cut)
constexpr int32_t kNnShareCols = 1536, kNnShareFourCols = 1792;   // length of the sum, for two and for four slices
// whether some batch of up to max_batch columns has tiles shared (nn_cut)
inline bool dense_shares_possible(int32_t rows, int32_t cols, int32_t max_batch)
{
    const int64_t across = (static_cast<int64_t>(rows) + 15) / 16;
    return cols >= kNnShareCols && max_batch > 32 && across < kNnShareTiles && across * ((static_cast<int64_t>(max_batch) + 63) / 64) >= kNnShareTiles / 4;
}
hipError_t launch_dense_product(const DenseArgs &a, hipStream_t s);
// Gradient and update of up to kSampledLayers layers in one grid: G = dZ X^T in MFMA tiles, of which the entries on the
// pattern are stored or take the momentum step (sampled_update_kernel in dense.hip).
constexpr int kSampledLayers = 4;
constexpr int32_t kSampledMinBatch = 16;
struct SampledLayer {
    const int32_t *list; // the rows, or nullptr: 0 .. rows - 1
    const uint2 *table;  // [rows * words] {bits of 32 columns of the row's pattern, CSR position of the first of them}
    int32_t words, rows, cols, nnz, fused;
    int32_t tiles_i, tiles_j, first_block; // set by launch_sampled
    const float *dZ, *X;
    int64_t lddz, ldx;
    float *g, *db;                         // stored unless nullptr
    float *values, *velocity, *values_t;   // fused: values_t may be nullptr
    const int32_t *pos_t;
    float *dense;                          // fused: dense copy or nullptr
    int64_t dense_ld;
    float *bias, *bias_velocity;           // fused: may be nullptr
};
struct SampledArgs {
    SampledLayer layer[kSampledLayers];
    int32_t n, batch, nesterov;
    float lr, momentum;
    const float *loss_cols;                // by-product as in SddmmArgs
    float *loss_out;
    int32_t loss_n;
};
// whether launch_sddmm takes that route for `a`, and whether it could be served by it beside layers that do
bool sddmm_sampled_ok(const SddmmCall &a);
bool sddmm_sampled_possible(const SddmmCall &a);
void add_sampled(SampledArgs &list, const SddmmCall &a);
hipError_t launch_sampled(SampledArgs &a, hipStream_t s);
// Y = act(W X + b) of a matrix's dense rows, and the room in DenseRows that takes at up to max_batch columns
bool dense_rows_product_ok(const DenseSplit *d, int32_t cols, int32_t batch);
bool dense_rows_sddmm_ok(const DenseSplit *d, int32_t batch);
bool thin_rows_pay_somewhere(const DenseSplit &d, int32_t cols);
bool sampled_operands_ok(const SddmmCall &a);
hipError_t launch_dense_rows(const SpmmCall &a, hipStream_t s);
__host__ __device__ inline int64_t dense_rows_ld(int32_t batch) { return (batch + 31) / 32 * 32; }
// The same on the bf16 matrix units, every fp32 number as three bf16 ones (split.hip): work-groups, most chunks of 32 columns of the matrix in one
// of them, and the operand's parts: 12 ints per 8 rows and column, columns rounded up to whole work-groups, and a flag per 32 rows
// and work-group's columns.
int64_t split_dense_rows_tiles(int32_t n, int32_t batch);
void launch_split_dense_rows(const SpmmArgs &a, const DenseRows &D, int slices, hipStream_t s);
constexpr int32_t kSplitMaxChunks = 2048, kSplitCols = 256;
__host__ __device__ inline int64_t operand_parts_ld(int32_t batch) { return (batch + kSplitCols - 1) / kSplitCols * kSplitCols; }
__host__ __device__ inline int64_t operand_parts_ints(int32_t rows, int32_t batch)
{
    const int64_t groups = (static_cast<int64_t>(rows) + 31) / 32;
    return groups * 48 * operand_parts_ld(batch) + groups * (operand_parts_ld(batch) / kSplitCols);
}
struct DenseRowsRoom {
    int64_t partial_floats, parts_ints;
};
DenseRowsRoom dense_rows_room(int32_t n, int32_t cols, int32_t max_batch, bool thin);
void add_sampled_rows(SampledArgs &list, const SddmmCall &a);
// status: result of the pattern check (the launch does nothing where it is not 0), or nullptr
// list: the rows (or nullptr: 0 .. rows - 1)
hipError_t launch_pattern_table(const int32_t *indptr, const int32_t *indices, const int32_t *list, int32_t rows, int32_t words, uint2 *table,
                                const int32_t *status, hipStream_t s);
// D[i * ld + j] = values[p] for every stored entry p = (i, j); the rest of D is not touched (zero since allocation)
hipError_t launch_dense_refresh(const int32_t *indptr, const int32_t *indices, const float *values, int32_t rows, float *D, int64_t ld,
                                hipStream_t s);

// ---- binding a pattern: one chain of launches on the device (structure.hip) ----
// Flags of the check that device arrays hold a canonical CSR pattern: status (device, 4 ints) receives {OR of the
// flags found, first row with wrong row pointers, first entry with a wrong column index, 0}.
enum : int32_t { kCsrBadFirst = 1, kCsrDecreasing = 2, kCsrBeyondNnz = 4, kCsrBadLast = 8, kCsrColumnRange = 16, kCsrNotAscending = 32 };

// How the mirror build cuts a matrix: tiles of entries, bins of 2^bin_shift columns, a bin's bitmap over seg_words * 32
// rows at a time, launches of block_cols columns.
struct MirrorGeometry {
    int32_t bin_shift, bins, seg_words, tiles, tile_entries, block_cols;
};
MirrorGeometry mirror_geometry(int32_t rows, int32_t cols, int32_t nnz);
struct MirrorArgs : MirrorGeometry {
    int32_t rows, cols, nnz;
    int32_t col_lo, cols_here;       // columns of the launch (set by launch_bind)
    const int32_t *indptr, *indices;
    const float *values;
    int32_t *status;
    int32_t *counts;                 // [bins * tiles]
    int32_t *bin_total;              // [bins]
    int32_t *block_base;             // [blocks of columns + 1] mirror position of a block's first entry
    int2 *bucket;                    // [nnz] {row, entry}, bin by bin
    int32_t *bucket_col;             // [nnz]
    // CSR of W^T: row pointers, row of each mirror entry, mirror position -> CSR position and back, values
    int32_t *indptr_t, *indices_t, *perm, *pos_t;
    float *values_t;
};

// What the planner reports of one orientation; RowBlocks holds the meanings.
struct PlanCounts {
    int32_t n_blocks, n_huge_rows, n_huge_blocks, n_short, n_long_blocks, n_rest_blocks, long_nnz, longest_row;
    int32_t n_long_rows;             // rows of more than kPackMaxLen entries
    int32_t hot_nnz, hot_lds_nnz;    // stored entries of the kHotRows, the kHotRowsLds longest rows
    int32_t n_dense, dense_nnz;      // rows of PlanSide::dense_len entries or more, and their entries
    int32_t staged_ranges, staged_partial, staged_rows, staged_nnz, staged_quad_len, staged_longest_share;
    int32_t cls[3][5];               // rows per class of the partitions waves / long_waves / rest_waves
};
struct PlanTables {
    int4 *waves, *huge_rows, *long_waves, *rest_waves, *rows_by_length;
    int32_t *staged_rows, *staged_groups, *staged_ends;
    int2 *strip_segs;
    int32_t *strip_rows, *strip_cuts;
    int32_t *dense_rows;             // [room for the rows of dense_len entries or more] ascending
    uint8_t *dense_flag;             // [rows]
    int4 *other_waves, *other_long_waves;   // copies of the tables above with row -1 in the place of dense rows
};
// Records of PlanTables::rows_by_length: padded, so that sets of up to 64 rows from any row on can be read.
__host__ __device__ inline int64_t rows_table_size(int32_t rows) { return (static_cast<int64_t>(rows) + 63) / 64 * 64 + 64; }
struct PlanWork {                    // scratch, [rows] ints each but for the last two
    int32_t *order, *tmp, *lens, *covered, *cut, *slots;
    int32_t *range_first;            // [range_bound + 1]
    PlanCounts *counts;
    unsigned long long *strip_count; // {chunks, steps in the upper half, dealt out so far; work-groups done}
};
struct PlanSide {
    int32_t rows, other;             // of this orientation
    int32_t range_bound;             // ranges the staged tables have room for, 0: no staged plan
    int32_t strip_blocks;            // of W alone, 0: no plan for strips
    int32_t dense_len;               // rows this long are listed, and left out of the staged plan where they are many (INT32_MAX: none)
    const int32_t *indptr, *indices;
    PlanTables tables;
    PlanWork work;
};
struct BindResult {                  // pinned host memory
    int32_t status[4];
    PlanCounts plan[2];
    unsigned long long strip;        // chunks, steps in the upper half; zeroed by the host, 0 without a plan for strips
};
enum : int32_t { kPlanBalanced = 0, kPlanRowSplit = 1, kPlanPreferStaged = 2 };
struct PlanArgs {
    PlanSide side[2];                // W, its mirror
    int32_t nnz, max_batch, mode;
    int32_t prefer_strips;
    const int32_t *status;
    BindResult *result;
};
hipError_t launch_bind(const MirrorArgs &m, const PlanArgs &p, hipStream_t s);
// place: scratch, [x_rows + rows]; sets: room for hot_sets_size(rows)
hipError_t launch_hot_order(const int4 *rows_by_length, int32_t x_rows, const int32_t *indptr_t, const int32_t *indices_t, int32_t rows, const int32_t *perm,
                            int32_t *place, int32_t *entry, int32_t *at, int32_t *hot_perm, const int4 *mirror_rows, int4 *sets, hipStream_t s);
hipError_t launch_plan(const PlanArgs &p, int sides, hipStream_t s);   // its last part alone: the partitions of W, or of W and its mirror

// Whether the product in strips can run (256 operand rows travel at a time), and whether a matrix is looked at for a plan: some work, segments
// neither so short that a set's differ too much nor so long that the staged product, whose gathers are wider, is as fast; and by the estimates that
// calls ask (spmm_strip_ok) strips may be the shorter way at a batch up to max_batch.  Before the plan is made these are of the best that it can come
// to (strips_may_pay), and of what has come out before its stream gets room.  Rows of different lengths have no use for it: a wave would run as long
// as the longest.
__host__ __device__ inline bool strip_possible(int32_t rows, int32_t cols, int64_t nnz, int32_t max_batch)
{
    return max_batch > kStripFromBatch && cols >= 256 && strip_blocks_of(cols) <= kStripMaxBlocks && nnz > 0 && nnz < (1 << 30) && static_cast<int64_t>(rows) * strip_blocks_of(cols) <= (1 << 28);
}
bool strips_pay_somewhere(const RowBlocks &plan, int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch, double steps, double chunks);
bool strips_may_pay(int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch, int32_t staged_ranges);   // staged_ranges: that a staged plan would aim at, 0: none
inline bool strip_wanted(int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch, int32_t staged_ranges)
{
    const int64_t segments = static_cast<int64_t>(rows) * strip_blocks_of(cols);
    return strip_possible(rows, cols, nnz, max_batch) && rows >= 256 && cols >= 1024 && static_cast<int64_t>(nnz) * max_batch >= (96 << 20) && nnz >= 4 * segments && nnz <= 160 * segments &&
           strips_may_pay(rows, cols, nnz, max_batch, staged_ranges);
}
__host__ __device__ inline bool strip_even(int32_t longest_row, int32_t rows, int64_t nnz) { return static_cast<int64_t>(longest_row) * rows <= 3 * nnz; }
// Whether a call or a training step on up to max_batch columns takes the hot rows of dZ out of LDS (backward_hot_ok): the
// mirror then gets the order of HotRows.  t, g: as these have them, but for batch, operands and room, with HotRows' share.
constexpr int32_t kHotFromBatch = 192;
inline int64_t hot_sets_size(int32_t rows) { return (static_cast<int64_t>(rows) + 255) / 256 * 256; }
bool hot_rows_pay_somewhere(SpmmCall t, SddmmCall g, int32_t max_batch);
// Ranges a staged plan over `rows` rows with `nnz` entries aims at, 0: such a plan would never be chosen.  (Host and
// device; `cols`: operand rows.)
__host__ __device__ inline int32_t staged_ranges_aim(int32_t rows, int32_t max_batch)
{
    const int32_t n_tiles = (max_batch + kStageCols - 1) / kStageCols;
    int32_t want = kStageTargetGroups / n_tiles;
    if (want > rows / 64) want = rows / 64;
    // (ranges cut by cost are not equally long: leave an eighth of the slots as slack)
    const int32_t at_least = (rows + kStageRangeRows * 7 / 8 - 1) / (kStageRangeRows * 7 / 8);
    if (want < at_least) want = at_least;
    // one work-group fits a compute unit at a time: fill the last round of the grid as well
    if (static_cast<int64_t>(want) * n_tiles > kStageTargetGroups) {
        const int64_t rounds = (static_cast<int64_t>(want) * n_tiles + kStageTargetGroups - 1) / kStageTargetGroups;
        want = static_cast<int32_t>(rounds * kStageTargetGroups / n_tiles);
    }
    return want;
}
__host__ __device__ inline int32_t staged_ranges_wanted(int32_t rows, int64_t nnz, int32_t cols, int32_t max_batch, int32_t mode,
                                                        int32_t range_bound)
{
    if (range_bound == 0 || mode == kPlanRowSplit || max_batch < kStageMinBatch || nnz == 0) return 0;
    const int32_t want = staged_ranges_aim(rows, max_batch);
    if (mode != kPlanPreferStaged && static_cast<double>(nnz) < static_cast<double>(kStageMinReuse) * want * cols) return 0;
    // segments shorter than at any batch pay (staged_pays) on an operand that stays small: binding 8192 x 3072 at 1.7 %, whose plan nothing took, took 31 us more (plan, tables and
    // segment bounds 39 + 14 + 9 -> 22 + 5 + 4)
    if (mode != kPlanPreferStaged && static_cast<int64_t>(cols) * max_batch * 4 < kStageBigOperand &&
        nnz < static_cast<int64_t>(kStageSegmentBesideDense) * rows * ((cols + kStageRows - 1) / kStageRows)) return 0;
    return want;
}
// Most ranges any staged plan of a matrix with that many rows can have; 0 where its tables would pass 1 GiB.  A plan over
// some of the rows aims at no more ranges than one over all of them, but for the rounding to whole rounds of the grid;
// the ranges that overflow add one per kStageRangeFill slots, of which split rows take three more each
// (at most 32 split rows per range aimed at).
__host__ __device__ inline int32_t staged_range_bound(int32_t rows, int32_t cols, int32_t max_batch)
{
    if (max_batch < kStageMinBatch) return 0;
    const int32_t n_tiles = (max_batch + kStageCols - 1) / kStageCols;
    const int64_t want = (static_cast<int64_t>(rows) + kStageRangeRows * 7 / 8 - 1) / (kStageRangeRows * 7 / 8) + 2 * (kStageTargetGroups / n_tiles) + 2;
    const int64_t bound = want + (rows + 96 * want) / kStageRangeFill + 2;
    return bound * ((cols + kStageRows - 1) / kStageRows + 1) * kStageRangeRows > (1ll << 28) ? 0 : static_cast<int32_t>(bound);
}
// Whether the listed rows are worth a route of their own at max_batch columns (calls ask again: dense_rows_product_ok).  Without -> with it on the
// fp32 units, forward product: power-law 4096^2 at 5 % (297 rows, 0.53 M entries) at batch 256 / 512 / 1024: 48 -> 50, 81 -> 77, 129 -> 120 us; 8192
// x 1024 at 10 %: 35 -> 36, 87 -> 51, 109 -> 82.  Rows of like length are cheaper to gather for: uniform 4096^2 at batch 1024 breaks even with the
// fp32 units at 30 % (324 us; 20 %: 235 -> 326).
__host__ __device__ inline bool dense_rows_pay(int32_t n_dense, int64_t dense_nnz, int64_t nnz, int32_t cols, int32_t max_batch)
{
    return n_dense >= kDenseRowsMin && dense_nnz * 8 >= nnz && dense_nnz * 10 >= static_cast<int64_t>(n_dense) * cols * 3 &&
           max_batch >= dense_rows_from(dense_nnz);
}
// which of `want` equal shares of the total cost a row falls into that has `done` of it before it
__host__ __device__ inline int32_t staged_cut(int64_t done, int32_t want, int64_t total)
{
    const int32_t cut = static_cast<int32_t>(static_cast<double>(done) * want / static_cast<double>(total));
    return cut < want ? cut : want - 1;
}

// The end of the forward pass and the start of the backward pass for a small output layer, in
// one launch: logits Z = W X + b, softmax cross-entropy (loss and dZ = (softmax - onehot) / batch),
// and the gradient handed to the layer below, dX = (W^T dZ) * [X > 0] (X is that layer's ReLU
// output).  Every step is local to a column of the batch, so a work-group owns 4 columns.
constexpr int kHeadMaxRows = 32;
struct HeadArgs {
    const int32_t *indptr, *indices;      // W in CSR (rows x cols)
    const float *values, *bias;           // bias may be null
    const int32_t *indptr_t, *indices_t;  // its mirror: CSR of W^T
    const float *values_t;
    int32_t rows, cols, batch, nnz;
    const float *X;                       // (cols, ldx)
    int64_t ldx;
    float *Z;                             // (rows, ldz)
    int64_t ldz;
    const int32_t *labels;                // [batch]
    float *dZ;                            // (rows, lddz)
    int64_t lddz;
    float *dX;                            // (cols, lddx)
    int64_t lddx;
    float *loss_cols;                     // [batch]: per-column losses; a later launch takes their mean (SddmmArgs)
};
bool head_ok(int32_t rows, int32_t cols, int32_t nnz, int32_t batch);
hipError_t launch_head(const HeadArgs &a, hipStream_t s);

}  // namespace nerva
