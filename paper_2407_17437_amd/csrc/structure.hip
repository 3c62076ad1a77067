// Device side of binding a pattern to a layer (sparse_linear_create / sparse_linear_rebind): the check that
// the caller's arrays hold canonical CSR, the CSC mirror with the two position maps, and the work partitions
// of both orientations.  One chain of launches and one synchronisation: every kernel behind the check looks
// at its status word first and leaves if the pattern is not valid, and what the host needs (how many
// work-groups each partition has) comes back in one small pinned struct at the end.
//
// The mirror is the stable sort of the stored entries by column, without a sort of single entries:
//   1. tiles of consecutive entries count their entries per bin of consecutive columns
//   2. per bin, a scan over the tiles gives each tile's first slot inside the bin
//   3. every tile appends its entries to the bins, in any order
//   4. a work-group per bin marks its entries in a bitmap (column x row) in LDS; an entry's position inside its
//      column is the number of marked rows before it.  The result does not depend on the order of the entries
//      inside a bin: it is the canonical CSR of W^T, bit for bit the same on every run.
// What bounds it is the chain of launches; the passes move about 60 bytes per stored entry.  (Before, one wave per
// row tile walked its rows with an atomic per entry whose result it waited for: 104 us of kernels for the 8192 x 8192
// layer of the wide MLP, 499 k entries, now 47.)
//
// The partitions depend on the row lengths only.  plan_kernel, a work-group per orientation, orders the rows by
// length (a stable radix sort), counts the classes and cuts the staged plan's ranges; plan_fill_kernel and
// plan_cuts_kernel write the tables.  They are those of the host planner (nerva_plan_*_host, api.hip), entry for
// entry.  (On the host, with the row pointers copied there and the tables copied back, a rebind of that layer
// took 0.38 ms, now 0.09 ms.)
#include "kernels.h"

#include <climits>

namespace nerva {
namespace {

constexpr int kWave = 64;
constexpr int kBig = 1024;    // work-group of the entry passes and of the planner
constexpr int kWaves = kBig / kWave;
constexpr int kSetupBlock = 256;
constexpr int kTileRows = 2048;   // rows of a tile whose row pointers fit in LDS
constexpr int kBinWords = 8192;   // bitmap words of a bin in LDS: 32 KiB, and as much for their prefix sums

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)); }
__device__ __forceinline__ int lanes_below(uint64_t mask) { return __popcll(mask & ((1ull << lane_id()) - 1)); }

// Sums, prefix sums and maxima over a wave, all lanes active.  Those of 32 bits by moves between lanes (DPP): a prefix sum through the LDS crossbar
// is six round trips of some 100 cycles, and the set-up kernels are chains of them (8192^2 at 0.74 %: bin_place_kernel 20.7 -> 16.1 us, plan_kernel,
// whose first thread no longer writes all it reports alone either, 22.2 -> 18.1).
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int32_t lanes_moved(int32_t v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false); }   // (0 where no lane is named)
template <typename F>
__device__ __forceinline__ int32_t wave_scan(int32_t v, F &&f)   // f(0, v) = v
{
    v = f(lanes_moved<0x111>(v), v);        // row_shr 1, 2, 4, 8: within rows of 16
    v = f(lanes_moved<0x112>(v), v);
    v = f(lanes_moved<0x114>(v), v);
    v = f(lanes_moved<0x118>(v), v);
    v = f(lanes_moved<0x142, 0xA>(v), v);   // the last lane of rows 0 and 2 into rows 1 and 3
    return f(lanes_moved<0x143, 0xC>(v), v);   // that of row 1 into rows 2 and 3
}
__device__ __forceinline__ int32_t last_lane(int32_t v) { return __builtin_amdgcn_readlane(v, kWave - 1); }
__device__ __forceinline__ int32_t wave_inclusive(int32_t v)
{
    return wave_scan(v, [](int32_t a, int32_t b) { return a + b; });
}
__device__ __forceinline__ int32_t wave_sum(int32_t v) { return last_lane(wave_inclusive(v)); }
__device__ __forceinline__ int32_t wave_max(int32_t v)   // v >= 0
{
    return last_lane(wave_scan(v, [](int32_t a, int32_t b) { return max(a, b); }));
}
__device__ __forceinline__ int64_t wave_sum(int64_t v)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) v += __shfl_xor(v, d, kWave);
    return v;
}
__device__ __forceinline__ int64_t wave_inclusive(int64_t v)
{
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int64_t y = __shfl_up(v, d, kWave);
        if (lane_id() >= d) v += y;
    }
    return v;
}

__global__ void status_init_kernel(int32_t *status, int32_t *block_base)
{
    if (threadIdx.x == 0) {
        block_base[0] = 0;
        status[0] = 0;
        status[1] = INT_MAX;  // first row whose row pointers are wrong
        status[2] = INT_MAX;  // first stored entry whose column index is wrong
        status[3] = 0;
    }
}

// first i in [0, n] with v[i] >= target (i = n: none below n); v ascending on valid patterns, any contents are safe
__device__ __forceinline__ int32_t lower_bound(const int32_t *v, int32_t lo, int32_t hi, int32_t target)
{
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (v[mid] >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// The same for two targets, t0 <= t1, by the whole work-group: 1024 positions are probed at a time, so that a search over
// a million rows is two round trips and not twenty.
__device__ __forceinline__ void block_lower_bounds(const int32_t *v, int32_t n, int32_t t0, int32_t t1, int32_t &r0, int32_t &r1)
{
    __shared__ int32_t below[2];
    int32_t lo[2] = {0, 0}, len[2] = {n, n};
    const int32_t target[2] = {t0, t1};
    while (len[0] > 0 || len[1] > 0) {   // uniform
        if (threadIdx.x < 2) below[threadIdx.x] = 0;
        __syncthreads();
        int32_t step[2];
        bool hit[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            // probe the last element of the i-th run of `step` elements
            step[k] = (len[k] + kBig - 1) / kBig;
            const int64_t at = (static_cast<int64_t>(threadIdx.x) + 1) * step[k];
            hit[k] = step[k] > 0 && at <= len[k] && v[lo[k] + at - 1] < target[k];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint64_t mask = __ballot(hit[k]);
            if (lane_id() == 0 && mask) atomicAdd(&below[k], __popcll(mask));
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int32_t skip = below[k] * step[k];   // (step 0: the search is over)
            lo[k] += skip;
            len[k] = step[k] > 1 ? min(step[k] - 1, len[k] - skip) : 0;
        }
        __syncthreads();
    }
    r0 = lo[0];
    r1 = lo[1];
}

// Check, and entries per (bin, tile).  Tile t covers the entries [t * E, (t + 1) * E); the entries that start a row
// are marked in LDS, so that a row of any length is checked entry by entry.  Nothing outside indices[0 .. nnz) and
// indptr[0 .. rows] is read, whatever they hold.
__global__ __launch_bounds__(kBig) void bind_check_kernel(const MirrorArgs m)
{
    extern __shared__ int32_t lds[];
    int32_t *hist = lds;
    uint32_t *starts = reinterpret_cast<uint32_t *>(lds + m.bins);
    const int32_t t = blockIdx.x, tid = threadIdx.x;
    for (int64_t i = static_cast<int64_t>(t) * kBig + tid; i <= m.rows; i += static_cast<int64_t>(gridDim.x) * kBig) {
        const int32_t v = m.indptr[i];
        int flags = 0;
        if (i == 0 && v != 0) flags |= kCsrBadFirst;
        if (v < 0 || v > m.nnz) flags |= kCsrBeyondNnz;
        if (i < m.rows && m.indptr[i + 1] < v) flags |= kCsrDecreasing;
        if (i == m.rows && v != m.nnz) flags |= kCsrBadLast;
        if (flags) {
            atomicOr(&m.status[0], flags);
            atomicMin(&m.status[1], static_cast<int32_t>(i));
        }
    }
    const int32_t p0 = min(static_cast<int64_t>(t) * m.tile_entries, static_cast<int64_t>(m.nnz));
    const int32_t p1 = min(static_cast<int64_t>(p0) + m.tile_entries, static_cast<int64_t>(m.nnz));
    for (int b = tid; b < m.bins; b += kBig) hist[b] = 0;
    for (int b = tid; b < (m.tile_entries + 31) / 32; b += kBig) starts[b] = 0;
    __syncthreads();
    int32_t r_lo, r_hi;
    block_lower_bounds(m.indptr, m.rows, p0, p1, r_lo, r_hi);
    for (int32_t r = r_lo + tid; r < r_hi; r += kBig) {
        const int32_t v = m.indptr[r];
        if (v >= p0 && v < p1) atomicOr(&starts[(v - p0) >> 5], 1u << ((v - p0) & 31));
    }
    __syncthreads();
    for (int32_t p = p0 + tid; p < p1; p += kBig) {
        const int32_t j = m.indices[p], before = p > 0 ? m.indices[p - 1] : -1;
        const bool first = (starts[(p - p0) >> 5] >> ((p - p0) & 31)) & 1u;
        int flags = 0;
        if (j < 0 || j >= m.cols)
            flags = kCsrColumnRange;
        else if (!first && before >= j)
            flags = kCsrNotAscending;
        if (flags) {
            atomicOr(&m.status[0], flags);
            atomicMin(&m.status[2], p);
        } else if (j >= m.col_lo && j - m.col_lo < m.cols_here) {
            atomicAdd(&hist[(j - m.col_lo) >> m.bin_shift], 1);
        }
    }
    __syncthreads();
    for (int b = tid; b < m.bins; b += kBig) m.counts[static_cast<int64_t>(b) * m.tiles + t] = hist[b];
}

// A wave per bin: counts of the tiles -> each tile's first slot inside the bin; the bin's entries.
__global__ __launch_bounds__(kSetupBlock) void bin_scan_kernel(const MirrorArgs m)
{
    const int bin = blockIdx.x * (kSetupBlock / kWave) + wave_id();
    if (bin >= m.bins || m.status[0] != 0) return;
    int32_t *c = m.counts + static_cast<int64_t>(bin) * m.tiles;
    int32_t run = 0;
    for (int t0 = 0; t0 < m.tiles; t0 += kWave) {
        const int t = t0 + lane_id();
        const int32_t v = t < m.tiles ? c[t] : 0;
        const int32_t incl = wave_inclusive(v);
        if (t < m.tiles) c[t] = run + incl - v;
        run += last_lane(incl);
    }
    if (lane_id() == 0) m.bin_total[bin] = run;
}

// The entries of tile t go to their bins: {row, entry} and the column, at the tile's slots, in any order.
__global__ __launch_bounds__(kBig) void bin_scatter_kernel(const MirrorArgs m)
{
    extern __shared__ int32_t cursor[];   // [bins]
    __shared__ int32_t wave_total[kWaves];
    __shared__ int32_t first[kTileRows];  // row pointers of the tile's rows, where they fit
    if (m.status[0] != 0) return;
    const int32_t t = blockIdx.x, tid = threadIdx.x;
    // bins' first slots: exclusive scan of their totals, `per` consecutive bins per thread
    const int per = (m.bins + kBig - 1) / kBig;
    int32_t mine = 0;
    for (int k = 0; k < per; ++k) {
        const int b = tid * per + k;
        if (b < m.bins) mine += m.bin_total[b];
    }
    const int32_t incl = wave_inclusive(mine);
    if (lane_id() == kWave - 1) wave_total[wave_id()] = incl;
    __syncthreads();
    int32_t run = incl - mine;
    for (int w = 0; w < wave_id(); ++w) run += wave_total[w];
    for (int k = 0; k < per; ++k) {
        const int b = tid * per + k;
        if (b < m.bins) {
            cursor[b] = run + m.counts[static_cast<int64_t>(b) * m.tiles + t];
            run += m.bin_total[b];
        }
    }
    __syncthreads();
    const int32_t p0 = min(static_cast<int64_t>(t) * m.tile_entries, static_cast<int64_t>(m.nnz));
    const int32_t p1 = min(static_cast<int64_t>(p0) + m.tile_entries, static_cast<int64_t>(m.nnz));
    if (p0 >= p1) return;
    // rows of the tile's first and last entry: the last row that starts at or before them
    int32_t r_lo, r_hi;
    block_lower_bounds(m.indptr, m.rows, p0 + 1, p1, r_lo, r_hi);
    --r_lo;
    --r_hi;
    const bool in_lds = r_hi - r_lo <= kTileRows;   // uniform
    if (in_lds)
        for (int32_t r = r_lo + 1 + tid; r <= r_hi; r += kBig) first[r - r_lo - 1] = m.indptr[r];
    __syncthreads();
    for (int32_t p = p0 + tid; p < p1; p += kBig) {
        const int32_t j = m.indices[p];
        if (j < m.col_lo || j - m.col_lo >= m.cols_here) continue;
        const int32_t row = in_lds ? r_lo + lower_bound(first, 0, r_hi - r_lo, p + 1) : lower_bound(m.indptr, r_lo + 1, r_hi + 1, p + 1) - 1;
        const int32_t at = atomicAdd(&cursor[(j - m.col_lo) >> m.bin_shift], 1);
        m.bucket[at] = make_int2(row, p);
        m.bucket_col[at] = j;
    }
}

// A work-group per bin: the mirror of the bin's columns.
constexpr int kPlaceBlock = 512;
constexpr int kPlaceHeld = 8;   // entries per thread held in registers over the three passes (bins of up to 4096 entries)
__global__ __launch_bounds__(kPlaceBlock) void bin_place_kernel(const MirrorArgs m)
{
    extern __shared__ int32_t lds[];
    const int width = 1 << m.bin_shift;            // columns of a bin
    const int words = m.seg_words;                 // bitmap words per column and segment of rows
    int32_t *col_count = lds, *col_first = lds + width, *col_run = lds + 2 * width;
    uint32_t *bits = reinterpret_cast<uint32_t *>(lds + 3 * width);
    int32_t *before = lds + 3 * width + width * words;
    __shared__ int32_t part[kPlaceBlock / kWave];
    if (m.status[0] != 0) return;
    const int bin = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int32_t c0 = m.col_lo + (bin << m.bin_shift), c_end = m.col_lo + m.cols_here;
    int32_t sum = 0;
    for (int b = tid; b < bin; b += kPlaceBlock) sum += m.bin_total[b];
    sum = wave_sum(sum);
    if (lane == 0) part[wv] = sum;
    for (int c = tid; c < width; c += kPlaceBlock) col_count[c] = col_run[c] = 0;
    __syncthreads();
    int32_t first = 0;       // of the bin's entries among those of the launch's columns
    for (int w = 0; w < kPlaceBlock / kWave; ++w) first += part[w];
    const int32_t base = *m.block_base + first;   // ... and in the mirror
    const int32_t n = m.bin_total[bin];
    int2 held[kPlaceHeld];
    int32_t held_col[kPlaceHeld];
    const int32_t n_held = min(n, kPlaceHeld * kPlaceBlock);
    if (n > 0)
#pragma unroll
        for (int k = 0; k < kPlaceHeld; ++k)
            if (k * kPlaceBlock < n) {   // uniform
                const int e = min(k * kPlaceBlock + tid, n - 1);
                held[k] = m.bucket[first + e];
                held_col[k] = m.bucket_col[first + e] - c0;
            }
    // f(row and entry, column inside the bin) for every entry of the bin
    auto every = [&](auto &&f) {
#pragma unroll
        for (int k = 0; k < kPlaceHeld; ++k)
            if (k * kPlaceBlock + tid < n_held) f(held[k], held_col[k]);
        for (int e = n_held + tid; e < n; e += kPlaceBlock) f(m.bucket[first + e], m.bucket_col[first + e] - c0);
    };
    every([&](int2, int c) { atomicAdd(&col_count[c], 1); });
    __syncthreads();
    if (wv == 0) {
        int32_t run = 0;
        for (int cb = 0; cb < width; cb += kWave) {
            const int c = cb + lane;
            const int32_t v = c < width ? col_count[c] : 0;
            const int32_t incl = wave_inclusive(v);
            if (c < width) {
                col_first[c] = base + run + incl - v;
                if (c0 + c < c_end) m.indptr_t[c0 + c] = base + run + incl - v;
            }
            run += last_lane(incl);
        }
        if (lane == 0 && bin == m.bins - 1) {
            m.indptr_t[c_end] = base + n;
            m.block_base[1] = base + n;
        }
    }
    const int32_t seg_rows = words * 32;
    for (int64_t at = 0; at < m.rows; at += seg_rows) {   // one segment up to kBinWords / width * 32 rows
        const int32_t s0 = static_cast<int32_t>(at);
        for (int k = tid; k < width * words; k += kPlaceBlock) bits[k] = 0;
        __syncthreads();
        every([&](int2 rp, int c) {
            const int32_t r = rp.x - s0;
            if (r >= 0 && r < seg_rows) atomicOr(&bits[c * words + (r >> 5)], 1u << (r & 31));
        });
        __syncthreads();
        for (int c = wv; c < width; c += kPlaceBlock / kWave) {
            int32_t run = col_run[c];
            for (int w0 = 0; w0 < words; w0 += kWave) {
                const int w = w0 + lane;
                const int32_t v = w < words ? __popc(bits[c * words + w]) : 0;
                const int32_t incl = wave_inclusive(v);
                if (w < words) before[c * words + w] = run + incl - v;
                run += last_lane(incl);
            }
            if (lane == 0) col_run[c] = run;
        }
        __syncthreads();
        every([&](int2 rp, int c) {
            const int32_t r = rp.x - s0;
            if (r < 0 || r >= seg_rows) return;
            const int w = c * words + (r >> 5);
            const int32_t q = col_first[c] + before[w] + __popc(bits[w] & ((1u << (r & 31)) - 1u));
            m.indices_t[q] = rp.x;
            m.perm[q] = rp.y;
            m.pos_t[rp.y] = q;
            m.values_t[q] = m.values[rp.y];
        });
        __syncthreads();
    }
}

constexpr int64_t kPlanLds = 128 << 10;

// ---- work partitions ---------------------------------------------------------------------------

// log2 of the waves that share a row of n entries: the smallest that leaves each at most `target`, 16 waves at most
__device__ __forceinline__ int row_class(int32_t n, int32_t target)
{
    int lg = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) lg += n > (target << k);
    return lg;
}
__device__ __forceinline__ int32_t blocks_of(const int32_t (&cls)[5])
{
    int32_t nb = 0;
#pragma unroll
    for (int k = 0; k < 5; ++k) nb += (cls[k] + (kWavesPerBlock >> k) - 1) / (kWavesPerBlock >> k);
    return nb;
}

// One orientation per work-group.  The rows are dealt to the 16 waves in contiguous chunks; a wave walks its chunk
// 64 rows at a time, so that prefix sums in row order need one exchange of the waves' totals.  What the walks read --
// the row lengths, then the cuts and slots of the staged plan -- lies in LDS as far as it fits (kPlanLds): from memory
// every step of every walk was a round trip (59 us for 8192 rows of 60 entries, 22 us from LDS, 18 with the waves' totals by DPP and LDS atomics).
__global__ __launch_bounds__(kBig) __attribute__((amdgpu_waves_per_eu(4, 4))) void plan_kernel(const PlanArgs A)
{
    __shared__ int32_t hist[kWaves][256];
    __shared__ int32_t tot[256];
    __shared__ int64_t wtot[kWaves][8];
    extern __shared__ int32_t plan_lds[];
    __shared__ int32_t cnt[16], hot_cnt[2];
    __shared__ PlanCounts C;   // (written by the first thread)
    __shared__ int32_t dense_cnt[3];   // rows, their entries, and the length from which the staged plan leaves rows out
    const PlanSide &S = A.side[blockIdx.x];
    const int32_t n = S.rows, nnz = A.nnz, tid = threadIdx.x;
    const int lane = lane_id(), wv = wave_id();
    if (blockIdx.x == 0 && tid < 4) A.result->status[tid] = A.status[tid];
    if (A.status[0] != 0) return;
    const int32_t *indptr = S.indptr;
    const bool row_split = A.mode == kPlanRowSplit;
    const int32_t target = min(max(nnz / 4096, 8), 64), cap = min(max(nnz / 16384, 8), 64) * kWavesPerBlock;
    const int32_t chunk = (n + kBig - 1) / kBig * kWave, k_lo = min(wv * chunk, n), k_hi = min(k_lo + chunk, n);
    const int64_t lds_arrays = kPlanLds / 4 / max(n, 1);
    int32_t *lens = lds_arrays >= 1 ? plan_lds : S.work.lens;
    int32_t *cut = lds_arrays >= 2 ? plan_lds + n : S.work.cut, *sl = lds_arrays >= 3 ? plan_lds + 2 * n : S.work.slots;
    if (tid < 16) cnt[tid] = 0;
    if (tid < 2) hot_cnt[tid] = 0;
    for (int32_t i = tid; i < n; i += kBig) lens[i] = indptr[i + 1] - indptr[i];
    __syncthreads();

    // classes, huge rows, totals
    int32_t long_cls[5] = {0, 0, 0, 0, 0}, rest_cls[5] = {0, 0, 0, 0, 0}, longest = 0, n_le = 0, n_huge = 0, parts = 0;
    int32_t long_nnz = 0;
    for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
        const int32_t i = i0 + lane;
        const bool ok = i < k_hi;
        const int32_t len = ok ? lens[i] : 0;
        const bool is_long = len > kPackMaxLen, huge = !row_split && len > 4 * cap;
        const int lg = row_split ? 0 : row_class(len, target);
        longest = max(longest, len);
        if (is_long) long_nnz += len;
        if (huge) parts += (len + 2 * cap - 1) / (2 * cap);
        n_huge += __popcll(__ballot(huge));
        n_le += __popcll(__ballot(ok && !is_long));
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            long_cls[k] += __popcll(__ballot(ok && !huge && is_long && lg == k));
            rest_cls[k] += __popcll(__ballot(ok && !is_long && lg == k));
        }
    }
    longest = wave_max(longest);
    long_nnz = wave_sum(long_nnz);
    parts = wave_sum(parts);
    {
        // lane k of a wave adds its k-th total
        int32_t v = lane == 1 ? n_le : lane == 2 ? n_huge : lane == 3 ? parts : long_nnz;
#pragma unroll
        for (int k = 0; k < 5; ++k) v = lane == 4 + k ? long_cls[k] : lane == 9 + k ? rest_cls[k] : v;
        if (lane == 0) atomicMax(&cnt[0], longest);
        else if (lane < 15) atomicAdd(&cnt[lane], v);
        if (lane == 2 || lane == 3) hist[wv][lane] = v;
    }
    __syncthreads();
    auto total_of = [&](int k) { return __builtin_amdgcn_readfirstlane(cnt[k]); };
    longest = total_of(0);
    n_le = total_of(1);
    n_huge = total_of(2);
    parts = total_of(3);
    long_nnz = total_of(14);
    int32_t huge_before = 0, parts_before = 0;
    if (n_huge > 0)
        for (int w = 0; w < wv; ++w) {
            huge_before += hist[w][2];
            parts_before += hist[w][3];
        }
    __syncthreads();

    // huge rows keep row order: their work-groups are also their scratch slots
    if (n_huge > 0)
        for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
            const int32_t i = i0 + lane;
            const int32_t len = i < k_hi ? lens[i] : 0;
            const bool huge = len > 4 * cap;
            const int32_t mine = huge ? (len + 2 * cap - 1) / (2 * cap) : 0, incl = wave_inclusive(mine);
            const uint64_t mask = __ballot(huge);
            if (huge) S.tables.huge_rows[huge_before + lanes_below(mask)] = make_int4(i, parts_before + incl - mine, mine, 0);
            huge_before += __popcll(mask);
            parts_before += last_lane(incl);
        }

    // rows long enough for the matrix instructions: listed where they hold enough of the entries
    if (tid == 0) { dense_cnt[0] = 0; dense_cnt[1] = 0; dense_cnt[2] = INT_MAX; }
    if (S.dense_len < INT_MAX && longest >= S.dense_len) {   // uniform
        int32_t mine = 0;
        int64_t entries = 0;
        for (int32_t i = k_lo + lane; i < k_hi; i += kWave)
            if (lens[i] >= S.dense_len) {
                ++mine;
                entries += lens[i];
            }
        mine = wave_sum(mine);
        entries = wave_sum(entries);
        if (lane == 0) { wtot[wv][1] = entries; hist[wv][0] = mine; }
        __syncthreads();
        if (tid == 0) {
            int32_t rows = 0;
            entries = 0;
            for (int w = 0; w < kWaves; ++w) {
                const int32_t here = hist[w][0];
                hist[w][0] = rows;
                rows += here;
                entries += wtot[w][1];
            }
            if (dense_rows_pay(rows, entries, nnz, S.other, A.max_batch)) {
                dense_cnt[0] = rows;
                dense_cnt[1] = static_cast<int32_t>(entries);
                dense_cnt[2] = S.dense_len;
            }
        }
        __syncthreads();
        if (dense_cnt[0] > 0) {
            int32_t at = hist[wv][0];
            for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
                const int32_t i = i0 + lane;
                const bool dense = i < k_hi && lens[i] >= S.dense_len;
                const uint64_t mask = __ballot(dense);
                if (dense) S.tables.dense_rows[at + lanes_below(mask)] = i;
                if (i < k_hi) S.tables.dense_flag[i] = dense;
                at += __popcll(mask);
            }
        }
    }
    __syncthreads();

    // rows by length, longest first, ties in row order: radix sort of longest - length, 8 bits a pass, stable because
    // every wave ranks its chunk in order
    int32_t *from = S.work.tmp, *to = S.work.order;
    int passes = 1;
    while (passes < 4 && (longest >> (8 * passes)) != 0) ++passes;
    if (passes % 2 == 0) { int32_t *x = from; from = to; to = x; }   // the last pass writes `order`
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = 8 * pass;
        for (int d = lane; d < 256; d += kWave) hist[wv][d] = 0;
        auto item = [&](int32_t k) { return pass == 0 ? k : from[k]; };
        auto digit = [&](int32_t r) { return ((longest - lens[r]) >> shift) & 255; };
        for (int32_t k = k_lo + lane; k < k_hi; k += kWave) atomicAdd(&hist[wv][digit(item(k))], 1);
        __syncthreads();
        if (tid < 256) {
            int32_t run = 0, v[kWaves];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v[w] = hist[w][tid];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                hist[w][tid] = run;
                run += v[w];
            }
            tot[tid] = run;
        }
        __syncthreads();
        if (wv == 0) {
            int32_t run = 0;
            for (int d0 = 0; d0 < 256; d0 += kWave) {
                const int32_t v = tot[d0 + lane], incl = wave_inclusive(v);
                tot[d0 + lane] = run + incl - v;
                run += last_lane(incl);
            }
        }
        __syncthreads();
        // (in the last pass the entries of the first rows, the most referenced ones of the other orientation's gathers, are counted as well, and those of the ones that HotRows keeps in LDS)
        const bool last_pass = pass + 1 == passes;
        int32_t hot = 0, hot_lds = 0;
        for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
            const bool ok = i0 + lane < k_hi;
            const int32_t r = ok ? item(i0 + lane) : 0, len = ok ? lens[r] : 0;
            const int d = ok ? ((longest - len) >> shift) & 255 : 0;
            uint64_t same = __ballot(ok);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t set = __ballot((d >> b) & 1);
                same &= (d >> b) & 1 ? set : ~set;
            }
            if (ok) {
                const int32_t at = hist[wv][d], rank = lanes_below(same);
                const int32_t place = tot[d] + at + rank;
                to[place] = r;
                hot += place < kHotRows ? len : 0;
                hot_lds += place < kHotRowsLds ? len : 0;
                if (rank == 0) hist[wv][d] = at + __popcll(same);   // (after every lane of the wave has read it)
            }
        }
        if (last_pass) {
            hot = wave_sum(hot);
            hot_lds = wave_sum(hot_lds);
            if (lane < 2) atomicAdd(&hot_cnt[lane], lane == 0 ? hot : hot_lds);
        }
        __syncthreads();
        int32_t *x = from; from = to; to = x;
    }
    const int32_t n_short = n_le >= kPackMinRows && nnz > 0 && !row_split ? n_le : 0;
    if (tid == 0) {
        int32_t cls[3][5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            cls[1][k] = cnt[4 + k];
            cls[2][k] = cnt[9 + k];
            cls[0][k] = cls[1][k] + cls[2][k];
        }
        if (!row_split)   // a class that cannot fill its last work-group hands its rows up (plan_rows in api.hip)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t left = cls[0][k] % (kWavesPerBlock >> k), above = kWavesPerBlock >> (k + 1);
                const bool room = (cls[0][k + 1] + left + above - 1) / above == (cls[0][k + 1] + above - 1) / above;
                const int32_t up = room ? left : 0;
                cls[0][k] -= up;
                cls[0][k + 1] += up;
            }
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int k = 0; k < 5; ++k) C.cls[v][k] = cls[v][k];
        C.longest_row = longest;
        C.hot_nnz = hot_cnt[0];
        C.hot_lds_nnz = hot_cnt[1];
        C.n_dense = dense_cnt[0];
        C.dense_nnz = dense_cnt[1];
        C.long_nnz = static_cast<int32_t>(long_nnz);
        C.n_huge_rows = n_huge;
        C.n_huge_blocks = parts;
        C.n_long_rows = n - n_le;
        C.n_short = n_short;
        C.n_blocks = parts + blocks_of(cls[0]);
        C.n_long_blocks = n_short > 0 ? parts + blocks_of(cls[1]) : 0;
        C.n_rest_blocks = n_short > 0 && n_short < n ? blocks_of(cls[2]) : 0;
    }

    // the staged plan: of the long rows alone where the rows differ widely, of all rows otherwise
    const int32_t cblocks = (S.other + kStageRows - 1) / kStageRows;
    const int32_t n_dense = __builtin_amdgcn_readfirstlane(dense_cnt[0]), dense_nnz = __builtin_amdgcn_readfirstlane(dense_cnt[1]),
                  below = __builtin_amdgcn_readfirstlane(dense_cnt[2]);
    int32_t min_len = 0, want = 0;
    int32_t ranges = 0, quad_len = 0, n_cov = 0, longest_share = 0;
    if (n_short > 0 && n_short < n && A.mode == kPlanBalanced && static_cast<int64_t>(longest) * n > 4ll * nnz) {
        min_len = kPackMaxLen + 1;
        want = staged_ranges_wanted(n - n_le - n_dense, long_nnz - dense_nnz, S.other, A.max_batch, A.mode, S.range_bound);
    }
    const bool partial = want > 0;
    if (want == 0) {
        min_len = 0;
        want = staged_ranges_wanted(n - n_dense, nnz - dense_nnz, S.other, A.max_batch, A.mode, S.range_bound);
    }
    if (want > 0) {
        auto cost = [&](int32_t len) { return static_cast<int64_t>(len) + 2 * min(len, cblocks) + 1; };
        int64_t sum = 0;
        int32_t covered = 0;
        for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
            const int32_t i = i0 + lane;
            const int32_t len = i < k_hi ? lens[i] : -1;
            const bool in = len >= min_len && len < below;
            if (in) sum += cost(len);
            covered += __popcll(__ballot(in));
        }
        sum = wave_sum(sum);
        if (lane == 0) { wtot[wv][2] = sum; wtot[wv][3] = covered; }
        __syncthreads();
        int64_t total = 0, done = 0;
        int32_t k_at = 0;
        for (int w = 0; w < kWaves; ++w) {
            total += wtot[w][2];
            n_cov += static_cast<int32_t>(wtot[w][3]);
            done += w < wv ? wtot[w][2] : 0;
            k_at += w < wv ? static_cast<int32_t>(wtot[w][3]) : 0;
        }
        quad_len = static_cast<int32_t>(max(static_cast<int64_t>(256), total / want / 32));
        // slots before the wave's chunk
        int32_t slots = 0, longest_single = 0, longest_in = 0;
        for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
            const int32_t i = i0 + lane;
            const int32_t len = i < k_hi ? lens[i] : -1;
            const bool in = len >= min_len && len < below;
            slots += in ? (len >= quad_len ? 4 : 1) : 0;
            if (in && len < quad_len) longest_single = max(longest_single, len);
            if (in) longest_in = max(longest_in, len);
        }
        slots = wave_sum(slots);
        longest_single = wave_max(longest_single);
        longest_in = wave_max(longest_in);
        if (lane == 0) { wtot[wv][4] = slots; wtot[wv][5] = longest_single; wtot[wv][7] = longest_in; }
        __syncthreads();
        slots = 0;
        for (int w = 0; w < kWaves; ++w) {
            slots += w < wv ? static_cast<int32_t>(wtot[w][4]) : 0;
            longest_single = max(longest_single, static_cast<int32_t>(wtot[w][5]));
            longest_in = max(longest_in, static_cast<int32_t>(wtot[w][7]));
        }
        // covered rows in row order, with the part of the total cost and the slots before them
        for (int32_t i0 = k_lo; i0 < k_hi; i0 += kWave) {
            const int32_t i = i0 + lane;
            const int32_t len = i < k_hi ? lens[i] : -1;
            const bool in = len >= min_len && len < below;
            const uint64_t mask = __ballot(in);
            const int64_t c = in ? cost(len) : 0, c_incl = wave_inclusive(c);
            const int32_t s = in ? (len >= quad_len ? 4 : 1) : 0, s_incl = wave_inclusive(s);
            if (in) {
                const int32_t k = k_at + lanes_below(mask);
                S.work.covered[k] = i;
                cut[k] = staged_cut(done + c_incl - c, want, total);
                sl[k] = slots + s_incl - s;
            }
            k_at += __popcll(mask);
            done += __shfl(c_incl, kWave - 1, kWave);
            slots += last_lane(s_incl);
        }
        __syncthreads();
        // a range begins where the cut does, and after every kStageRangeFill slots of it: a thread per cut finds its
        // first row and how many ranges it makes
        auto first_of_cut = [&](int32_t c) { return lower_bound(cut, 0, n_cov, c); };
        for (int32_t c0 = 0; c0 < want; c0 += kBig) {   // (one round up to 1024 ranges)
            const int32_t c = c0 + tid;
            int32_t k0 = 0, pieces = 0, s0 = 0;
            if (c < want) {
                k0 = first_of_cut(c);
                const int32_t k1 = first_of_cut(c + 1);
                if (k0 < k1) {
                    s0 = sl[k0];
                    pieces = (sl[k1 - 1] - s0) / kStageRangeFill + 1;
                }
            }
            const int32_t incl = wave_inclusive(pieces);
            __syncthreads();
            if (lane == kWave - 1) wtot[wv][6] = incl;
            __syncthreads();
            int32_t at = ranges + incl - pieces;
            for (int w = 0; w < kWaves; ++w) {
                at += w < wv ? static_cast<int32_t>(wtot[w][6]) : 0;
                ranges += static_cast<int32_t>(wtot[w][6]);
            }
            // (every piece has a row of its own: slots grow by 4 at most from row to row)
            for (int32_t piece = 0; piece < pieces; ++piece)
                S.work.range_first[at + piece] = piece == 0 ? k0 : lower_bound(sl, k0, n_cov, s0 + piece * kStageRangeFill);
        }
        if (tid == 0) S.work.range_first[ranges] = n_cov;
        longest_share = max(longest_in >= quad_len ? (longest_in + 3) / 4 : 0, longest_single);
    }
    if (tid == 0) {
        C.staged_ranges = ranges;
        C.staged_partial = partial;
        C.staged_quad_len = quad_len;
        C.staged_rows = n_cov;
        C.staged_nnz = static_cast<int32_t>(want == 0 ? 0 : (min_len > 0 ? long_nnz : nnz) - dense_nnz);
        C.staged_longest_share = longest_share;
        if (S.strip_blocks > 0) S.work.strip_count[0] = S.work.strip_count[1] = 0;
    }
    __syncthreads();
    // (a word a thread: pinned memory is a long way off)
    static_assert(sizeof(PlanCounts) / 4 <= kWave, "");
    if (tid < sizeof(PlanCounts) / 4) {
        const int32_t word = reinterpret_cast<const int32_t *>(&C)[tid];
        reinterpret_cast<int32_t *>(S.work.counts)[tid] = word;
        reinterpret_cast<int32_t *>(&A.result->plan[blockIdx.x])[tid] = word;
    }
}

// Wave w of work-group b of a partition: huge rows' work-groups first, then the classes, heaviest first, whose rows
// are `order` from position `first` on.
__device__ __forceinline__ int4 wave_record(const PlanSide &S, const PlanCounts &C, const int32_t (&cls)[5], int32_t first, int32_t huge_blocks,
                                            int32_t cap, int32_t b, int w)
{
    int32_t row = -1, lg = 4, p0 = 0, p1 = 0, index = 0;
    bool lead = false;
    const bool huge = b < huge_blocks;
    if (huge) {
        int32_t lo = 0, hi = C.n_huge_rows - 1;   // the last huge row whose first work-group is not beyond b
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) / 2;
            if (S.tables.huge_rows[mid].y <= b) lo = mid; else hi = mid - 1;
        }
        const int4 h = S.tables.huge_rows[lo];
        row = h.x;
        index = lo;
        const int32_t q = b - h.y, len = S.indptr[row + 1] - S.indptr[row], share = (len + h.z - 1) / h.z;
        p0 = S.indptr[row] + min(q * share, len);
        p1 = S.indptr[row] + min(q * share + share, len);
        lead = w == 0 && q == 0;
    } else {
        int32_t rest = b - huge_blocks, f = first;
        for (lg = 4; lg >= 0; --lg) {
            const int32_t per = kWavesPerBlock >> lg, nb = (cls[lg] + per - 1) / per;
            if (rest < nb) {
                const int32_t k = rest * per + (w >> lg);
                if (k < cls[lg]) row = S.work.order[f + k];
                break;
            }
            rest -= nb;
            f += cls[lg];
        }
        lg = max(lg, 0);
        if (row >= 0) {
            p0 = S.indptr[row];
            p1 = S.indptr[row + 1];
            lead = (w & ((1 << lg) - 1)) == 0;
        }
    }
    const int part = w & ((1 << lg) - 1);
    int32_t per = ((p1 - p0) + (1 << lg) - 1) >> lg;
    per = (per + 3) / 4 * 4;
    const int32_t s0 = min(static_cast<int64_t>(p0) + static_cast<int64_t>(part) * per, static_cast<int64_t>(p1));
    const int32_t s1 = min(static_cast<int64_t>(s0) + per, static_cast<int64_t>(p1));
    return make_int4(row, s0, s1, part | (lg << 4) | (lead ? 256 : 0) | (huge ? 512 : 0) | (index << 10));
}

// A record of a partition as the launch of the rows that are not dense sees it.
__device__ __forceinline__ int4 without_dense(const PlanSide &S, int4 d)
{
    if (d.x >= 0 && S.tables.dense_flag[d.x]) d.x = -1;
    return d;
}

// The tables of both orientations (blockIdx.y).  Staged ranges: a work-group per range ranks its rows by counting
// the longer ones; records and short rows: an element per thread.
__global__ __launch_bounds__(kStageRangeRows) void plan_fill_kernel(const PlanArgs A)
{
    __shared__ int32_t len_s[kStageRangeRows], out[kStageRangeRows];
    __shared__ int32_t n_quads;
    if (A.status[0] != 0) return;
    const PlanSide S = blockIdx.y ? A.side[1] : A.side[0];
    const PlanCounts C = *S.work.counts;
    const int tid = threadIdx.x;
    for (int32_t q = blockIdx.x; q < C.staged_ranges; q += gridDim.x) {
        const int32_t k0 = S.work.range_first[q], m = S.work.range_first[q + 1] - k0;
        const int32_t row = tid < m ? S.work.covered[k0 + tid] : 0;
        const int32_t len = tid < m ? S.indptr[row + 1] - S.indptr[row] : -1;
        len_s[tid] = len;
        out[tid] = -1;
        if (tid == 0) n_quads = 0;
        __syncthreads();
        const bool quad = tid < m && len >= C.staged_quad_len;
        const uint64_t mask = __ballot(quad);
        if (lane_id() == 0 && mask) atomicAdd(&n_quads, __popcll(mask));
        int32_t rank = 0;
        for (int u = 0; u < m; ++u) rank += len_s[u] > len || (len_s[u] == len && u < tid);
        __syncthreads();
        const int32_t nq = n_quads;
        if (tid < m) {
            if (quad)
                for (int c = 0; c < 4; ++c) out[rank * 4 + c] = row | kStageQuad;
            else
                out[nq * 4 + (rank - nq)] = row;
        }
        __syncthreads();
        S.tables.staged_rows[static_cast<int64_t>(q) * kStageRangeRows + tid] = out[tid];
        if (tid == 0) S.tables.staged_groups[q] = (m + 3 * nq + 63) / 64;
        __syncthreads();
    }
    const int32_t cap = min(max(A.nnz / 16384, 8), 64) * kWavesPerBlock;
    const int64_t n_w = static_cast<int64_t>(C.n_blocks) * kWavesPerBlock, n_l = n_w + static_cast<int64_t>(C.n_long_blocks) * kWavesPerBlock;
    const int64_t n_r = n_l + static_cast<int64_t>(C.n_rest_blocks) * kWavesPerBlock, n_all = n_r + rows_table_size(S.rows);
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kStageRangeRows + tid; k < n_all; k += static_cast<int64_t>(gridDim.x) * kStageRangeRows) {
        if (k < n_w) {
            const int4 d = wave_record(S, C, C.cls[0], C.n_huge_rows, C.n_huge_blocks, cap, k / kWavesPerBlock, k % kWavesPerBlock);
            S.tables.waves[k] = d;
            if (C.n_dense > 0) S.tables.other_waves[k] = without_dense(S, d);
        } else if (k < n_l) {
            const int64_t e = k - n_w;
            const int4 d = wave_record(S, C, C.cls[1], C.n_huge_rows, C.n_huge_blocks, cap, e / kWavesPerBlock, e % kWavesPerBlock);
            S.tables.long_waves[e] = d;
            if (C.n_dense > 0) S.tables.other_long_waves[e] = without_dense(S, d);
        } else if (k < n_r) {
            const int64_t e = k - n_l;
            S.tables.rest_waves[e] = wave_record(S, C, C.cls[2], C.n_long_rows, 0, cap, e / kWavesPerBlock, e % kWavesPerBlock);
        } else {
            const int64_t e = k - n_r;
            int4 d = make_int4(-1, 0, 0, 0);
            if (e < S.rows) {
                const int32_t r = S.work.order[e];
                d = make_int4(r, S.indptr[r], S.indptr[r + 1] - S.indptr[r], 0);
            }
            S.tables.rows_by_length[e] = d;
        }
    }
}

// Segment bounds of the staged product: per slot of every range and per column block b, the position
// of the slot's first stored entry with column >= b * kStageRows (b = n_cb: one past the row's last
// entry; unused slots: 0 throughout).
__device__ __forceinline__ void staged_ends(const PlanSide &S, int64_t thread, int64_t threads)
{
    const int32_t n_cb = (S.other + kStageRows - 1) / kStageRows;
    const int64_t total = static_cast<int64_t>(S.work.counts->staged_ranges) * (n_cb + 1) * kStageRangeRows;
    for (int64_t idx = thread; idx < total; idx += threads) {
        const int32_t slot = static_cast<int32_t>(idx % kStageRangeRows);
        const int32_t b = static_cast<int32_t>((idx / kStageRangeRows) % (n_cb + 1));
        const int64_t q = idx / (static_cast<int64_t>(kStageRangeRows) * (n_cb + 1));
        const int32_t r = S.tables.staged_rows[q * kStageRangeRows + slot];
        S.tables.staged_ends[idx] = r < 0 ? 0 : lower_bound(S.indices, S.indptr[r & ~kStageQuad], S.indptr[(r & ~kStageQuad) + 1], b * kStageRows);
    }
}

// Plan of the product in strips (Strips), a work-group per kStripGroup rows of rows_by_length: where the blocks cut each row; which rows go together; the longest segment of every
// set and block, and its place in the stream.  Sixteen rows run side by side for as long as the longest of them has entries in a block, so rows of about one length are put together by
// their entries in the first block, and 64 at a time of these by theirs in the second: of the steps 0.82 are entries of 8192^2 at 0.74 % (0.71 by length alone), 0.97 of
// 8192 x 3072 at 1.4 % (0.79), 0.77 of 16384^2 at 1 % (0.73).  Product and stream 68 -> 58, 49 -> 41, 257 -> 245 us at batch 1024.
constexpr int kStripGroup = 256, kStripSubgroup = 64, kStripParts = kBig / kStripGroup, kStripSets = kStripGroup / kStripSet;
static_assert(kStripSets * kStripMaxBlocks <= kBig, "a thread per segment");
__device__ __forceinline__ void strip_plan(const PlanArgs &A, const int32_t block, int32_t *cuts)
{
    __shared__ __attribute__((aligned(16))) int32_t key[kStripGroup], place[kStripGroup], listed[kStripGroup];
    __shared__ int32_t wtot[kWaves][2], base;
    const PlanSide &S = A.side[0];
    const int32_t nb = S.strip_blocks, block_rows = strip_block_rows_of(S.other), n_sets = (S.rows + kStripSet - 1) / kStripSet;
    const int32_t tid = threadIdx.x, r = tid % kStripGroup, part = tid / kStripGroup, k = block * kStripGroup + r;
    const int lane = lane_id(), wv = wave_id();
    const int4 d = k < S.rows ? S.tables.rows_by_length[k] : make_int4(-1, 0, 0, 0);
    for (int32_t b = part; b <= nb; b += kStripParts) cuts[b * kStripGroup + r] = b == 0 ? d.y : b == nb ? d.y + d.z : lower_bound(S.indices, d.y, d.y + d.z, b * block_rows);
    if (part == 0) place[r] = 0;
    __syncthreads();
    auto entries = [&](int32_t row, int32_t b) { return cuts[(b + 1) * kStripGroup + row] - cuts[b * kStripGroup + row]; };
    // places in the order of the keys, within groups of `size` that the parts search a share each of (equal ones as they are)
    auto rank_in = [&](int32_t first, int32_t size) {
        int32_t rank = 0;
        const int32_t mine = key[r], u0 = first + part * (size / kStripParts);
#pragma unroll 4
        for (int32_t u = u0; u < u0 + size / kStripParts; u += 4) {
            const int4 o = *reinterpret_cast<const int4 *>(key + u);
            rank += (o.x > mine || (o.x == mine && u < r)) + (o.y > mine || (o.y == mine && u + 1 < r)) + (o.z > mine || (o.z == mine && u + 2 < r)) + (o.w > mine || (o.w == mine && u + 3 < r));
        }
        atomicAdd(&place[r], rank);
    };
    // (rows past the last one come behind all others)
    if (part == 0) key[r] = d.x < 0 ? -1 : entries(r, 0);
    __syncthreads();
    rank_in(0, kStripGroup);
    __syncthreads();
    if (part == 0) listed[place[r]] = r;
    __syncthreads();
    if (nb > 1) {
        const int32_t here = listed[r], first = r / kStripSubgroup * kStripSubgroup;
        if (part == 0) {
            key[r] = block * kStripGroup + here < S.rows ? entries(here, 1) : -1;
            place[r] = first;
        }
        __syncthreads();
        rank_in(first, kStripSubgroup);
        __syncthreads();
        if (part == 0) listed[place[r]] = here;
        __syncthreads();
    }
    const int32_t set0 = block * kStripSets, sets = min(kStripSets, n_sets - set0), row = listed[r];
    if (r < sets * kStripSet) {
        if (part == 0) S.tables.strip_rows[set0 * kStripSet + r] = block * kStripGroup + row < S.rows ? S.tables.rows_by_length[block * kStripGroup + row].x : -1;
        for (int32_t b = part; b <= nb; b += kStripParts) S.tables.strip_cuts[(static_cast<int64_t>(set0 + r / kStripSet) * (nb + 1) + b) * kStripSet + r % kStripSet] = cuts[b * kStripGroup + row];
    }
    int32_t n = 0;
    if (tid < sets * nb)
#pragma unroll
        for (int q = 0; q < kStripSet; ++q) n = max(n, entries(listed[tid / nb * kStripSet + q], tid % nb));
    const int32_t chunks = (n + kStripChunk - 1) / kStripChunk, incl = wave_inclusive(chunks), steps = wave_sum(n);
    if (lane == kWave - 1) wtot[wv][0] = incl;
    if (lane == 0) wtot[wv][1] = steps;
    __syncthreads();
    int32_t before = 0, total = 0;
    unsigned long long all_steps = 0;
    for (int w = 0; w < kWaves; ++w) {
        before += w < wv ? wtot[w][0] : 0;
        total += wtot[w][0];
        all_steps += static_cast<unsigned long long>(wtot[w][1]);
    }
    if (tid == 0) {
        // (the order in which the work-groups take their places has no bearing on any result)
        const int32_t first = static_cast<int32_t>(atomicAdd(&S.work.strip_count[0], static_cast<unsigned long long>(total) | all_steps << 32));
        base = first;
        unsigned long long one = 1;
        asm volatile("" : "+v"(one) : "v"(first));   // (counted as done once it has its place)
        if (atomicAdd(&S.work.strip_count[1], one) == static_cast<unsigned long long>((S.rows + kStripGroup - 1) / kStripGroup - 1)) A.result->strip = atomicAdd(&S.work.strip_count[0], 0ull);
    }
    __syncthreads();
    if (tid < sets * nb) S.tables.strip_segs[static_cast<int64_t>(set0) * nb + tid] = make_int2(base + before + incl - chunks, n);
}

// Both, after the tables that they read: the first strip_groups work-groups plan strips, kEndsBlocks for each orientation cut the staged plan's rows.
constexpr int kEndsBlocks = 256;
__global__ __launch_bounds__(kBig) void plan_cuts_kernel(const PlanArgs A, const int strip_groups)
{
    extern __shared__ int32_t strip_lds[];
    if (A.status[0] != 0) return;
    const int32_t block = blockIdx.x;
    if (block < strip_groups) {
        if (A.prefer_strips || strip_even(A.side[0].work.counts->longest_row, A.side[0].rows, A.nnz)) strip_plan(A, block, strip_lds);
        return;
    }
    const int32_t e = block - strip_groups;
    const PlanSide &S = e < kEndsBlocks ? A.side[0] : A.side[1];
    staged_ends(S, static_cast<int64_t>(e % kEndsBlocks) * kBig + threadIdx.x, static_cast<int64_t>(kEndsBlocks) * kBig);
}

// Entries of the mirror rows in the order of HotRows: every row's place among the longest, or -1; then a wave per mirror row.
__global__ __launch_bounds__(kSetupBlock) void hot_place_kernel(const int4 *rows_by_length, const int32_t n, int32_t *place)
{
    const int32_t e = blockIdx.x * kSetupBlock + threadIdx.x;
    if (e < n) place[rows_by_length[e].x] = e < kHotRowsLds ? e : -1;
}
__global__ __launch_bounds__(kSetupBlock) void hot_order_kernel(const int32_t *indptr_t, const int32_t *indices_t, const int32_t rows, const int32_t *perm,
                                                                const int32_t *place, int32_t *entry, int32_t *at, int32_t *hot_perm, int32_t *count)
{
    const int32_t row = blockIdx.x * (kSetupBlock / kWave) + wave_id();
    if (row >= rows) return;
    const int32_t p0 = indptr_t[row], p1 = indptr_t[row + 1], lane = lane_id();
    int32_t hot = 0;
    for (int32_t p = p0; p < p1; p += kWave) hot += __popcll(__ballot(p + lane < p1 && place[indices_t[min(p + lane, p1 - 1)]] >= 0));
    if (lane == 0) count[row] = hot;
    int32_t next_hot = p0, next_cold = p0 + hot;
    for (int32_t p = p0; p < p1; p += kWave) {
        const bool in = p + lane < p1;
        const int32_t i = indices_t[min(p + lane, p1 - 1)], slot = place[i];
        const uint64_t hots = __ballot(in && slot >= 0), colds = __ballot(in && slot < 0);
        if (in) {
            const int32_t to = slot >= 0 ? next_hot + lanes_below(hots) : next_cold + lanes_below(colds);
            entry[to] = slot >= 0 ? slot * 256 : i;
            at[to] = p + lane;
            hot_perm[to] = perm[p + lane];
        }
        next_hot += __popcll(hots);
        next_cold += __popcll(colds);
    }
}

// Rows of about one length, kHotGroup at a time, by their hot entries: what runs side by side then has as many of either kind (16384^2 power-law at 1 %: 16 -> 6 % of the steps without an entry).
constexpr int kHotGroup = 256;
__global__ __launch_bounds__(kHotGroup) void hot_sets_kernel(const int4 *mirror_rows, const int32_t rows, const int32_t *count, int4 *sets)
{
    __shared__ int32_t key[kHotGroup];
    const int32_t r = threadIdx.x, k = blockIdx.x * kHotGroup + r;
    int4 d = make_int4(-1, 0, 0, 0);
    if (k < rows) {
        d = mirror_rows[k];
        d.w = count[d.x];
    }
    key[r] = k < rows ? d.w : -1;
    __syncthreads();
    int32_t rank = 0;
    const int32_t mine = key[r];
    for (int u = 0; u < kHotGroup; ++u) rank += key[u] > mine || (key[u] == mine && u < r);
    sets[blockIdx.x * kHotGroup + rank] = d;
}

}  // namespace

hipError_t launch_hot_order(const int4 *rows_by_length, int32_t x_rows, const int32_t *indptr_t, const int32_t *indices_t, int32_t rows, const int32_t *perm,
                            int32_t *place, int32_t *entry, int32_t *at, int32_t *hot_perm, const int4 *mirror_rows, int4 *sets, hipStream_t s)
{
    hipLaunchKernelGGL(hot_place_kernel, dim3((x_rows + kSetupBlock - 1) / kSetupBlock), dim3(kSetupBlock), 0, s, rows_by_length, x_rows, place);
    int32_t *count = place + x_rows;
    hipLaunchKernelGGL(hot_order_kernel, dim3((rows + kSetupBlock / kWave - 1) / (kSetupBlock / kWave)), dim3(kSetupBlock), 0, s, indptr_t, indices_t, rows, perm, place, entry, at, hot_perm, count);
    hipLaunchKernelGGL(hot_sets_kernel, dim3((rows + kHotGroup - 1) / kHotGroup), dim3(kHotGroup), 0, s, mirror_rows, rows, count, sets);
    return hipGetLastError();
}

MirrorGeometry mirror_geometry(int32_t rows, int32_t cols, int32_t nnz)
{
    MirrorGeometry g;
    // About 256 bins, of at most 64 columns, narrower where that keeps a bin's bitmap in one piece (else it covers the
    // rows in several); at most 8192 bins a launch, of at most 4096 columns: matrices of more than 2^25 columns are
    // built block of columns by block of columns.
    const int32_t row_words = static_cast<int32_t>((static_cast<int64_t>(rows) + 31) / 32);
    g.block_cols = cols < (1 << 25) ? cols : (1 << 25);
    g.bin_shift = 0;
    while (g.bin_shift < 6 && (2 << g.bin_shift) <= g.block_cols / 256) ++g.bin_shift;
    while (g.bin_shift > 0 && (static_cast<int64_t>(row_words) << g.bin_shift) > kBinWords) --g.bin_shift;
    while (((g.block_cols + (1 << g.bin_shift) - 1) >> g.bin_shift) > 8192) ++g.bin_shift;
    g.bins = (g.block_cols + (1 << g.bin_shift) - 1) >> g.bin_shift;
    const int32_t width = 1 << g.bin_shift;
    g.seg_words = row_words < kBinWords / width ? row_words : kBinWords / width;
    // tiles of about 2048 entries, 1024 of them at most unless a tile would have more than 2^17 (its row starts are
    // marked in LDS)
    int64_t T = nnz / 2048;
    T = T < 1 ? 1 : (T > 1024 ? 1024 : T);
    if (T < nnz / (1 << 17) + 1) T = nnz / (1 << 17) + 1;
    g.tiles = static_cast<int32_t>(T);
    g.tile_entries = static_cast<int32_t>((nnz + T - 1) / T);
    if (g.tile_entries < 1) g.tile_entries = 1;
    return g;
}

hipError_t launch_bind(const MirrorArgs &whole, const PlanArgs &p, hipStream_t s)
{
    hipLaunchKernelGGL(status_init_kernel, dim3(1), dim3(kWave), 0, s, whole.status, whole.block_base);
    const MirrorGeometry &g = whole;
    const int width = 1 << g.bin_shift;
    MirrorArgs m = whole;
    for (int64_t col_lo = 0; col_lo < m.cols; col_lo += g.block_cols, ++m.block_base) {   // (one block up to 2^25 columns)
        m.col_lo = static_cast<int32_t>(col_lo);
        m.cols_here = static_cast<int32_t>(m.cols - col_lo < g.block_cols ? m.cols - col_lo : g.block_cols);
        m.bins = static_cast<int32_t>((static_cast<int64_t>(m.cols_here) + width - 1) >> g.bin_shift);
        const size_t check_lds = (static_cast<size_t>(m.bins) + (m.tile_entries + 31) / 32) * 4;
        hipLaunchKernelGGL(bind_check_kernel, dim3(m.tiles), dim3(kBig), check_lds, s, m);
        hipLaunchKernelGGL(bin_scan_kernel, dim3((m.bins + kSetupBlock / kWave - 1) / (kSetupBlock / kWave)), dim3(kSetupBlock), 0, s, m);
        if (m.nnz > 0) hipLaunchKernelGGL(bin_scatter_kernel, dim3(m.tiles), dim3(kBig), static_cast<size_t>(m.bins) * 4, s, m);
        hipLaunchKernelGGL(bin_place_kernel, dim3(m.bins), dim3(kPlaceBlock), (3ll * width + 2ll * width * m.seg_words) * 4, s, m);
    }
    return launch_plan(p, 2, s);
}

hipError_t launch_plan(const PlanArgs &p, int sides, hipStream_t s)
{
    const int64_t plan_rows = p.side[0].rows > p.side[1].rows ? p.side[0].rows : p.side[1].rows;
    const int64_t plan_arrays = kPlanLds / 4 / plan_rows < 3 ? kPlanLds / 4 / plan_rows : 3;   // of the larger side; the smaller one may keep more
    const int64_t small = p.side[0].rows + p.side[1].rows - plan_rows, small_arrays = kPlanLds / 4 / small < 3 ? kPlanLds / 4 / small : 3;
    const int64_t plan_lds = 4 * (plan_arrays * plan_rows > small_arrays * small ? plan_arrays * plan_rows : small_arrays * small);
    hipLaunchKernelGGL(plan_kernel, dim3(sides), dim3(kBig), static_cast<size_t>(plan_lds), s, p);
    hipLaunchKernelGGL(plan_fill_kernel, dim3(256, sides), dim3(kStageRangeRows), 0, s, p);
    const int strip_groups = p.side[0].strip_blocks > 0 ? (p.side[0].rows + kStripGroup - 1) / kStripGroup : 0;
    const int ends_sides = sides > 1 && p.side[1].range_bound > 0 ? 2 : p.side[0].range_bound > 0 ? 1 : 0;
    if (strip_groups + ends_sides > 0)
        hipLaunchKernelGGL(plan_cuts_kernel, dim3(strip_groups + ends_sides * kEndsBlocks), dim3(kBig),
                           strip_groups > 0 ? static_cast<size_t>(p.side[0].strip_blocks + 1) * kStripGroup * 4 : 0, s, p, strip_groups);
    return hipGetLastError();
}

}  // namespace nerva
