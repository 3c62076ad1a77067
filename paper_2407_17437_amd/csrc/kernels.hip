// gfx950 kernels of the truly sparse MLP training step.
//
// Mapping shared by the sparse kernels: lanes of a 64-wide wavefront run along the batch
// dimension, so every gather of a dense row is one contiguous, coalesced read (one example
// per column, batch contiguous).  Where a gather fills the whole wave (wide batches) row
// pointers, column indices and weights are wave-uniform and travel through the scalar path;
// for narrow batches and column tiles several stored entries share one gather instruction, their
// indices loaded one per lane and handed round with ds_bpermute.  Rows are handed to work-groups
// by a static partition (RowBlocks) that gives long rows several waves, each with a contiguous
// share of the row's stored entries; partial sums of one row meet in LDS and are added in a
// fixed order.  No float is added atomically: every output element is produced by one lane in one
// order, so results are bit-reproducible from run to run.  (The exceptions to "along the batch":
// spmv_kernel, spmv_rows_kernel and head_kernel, whose lanes run across a row's entries, and the MFMA
// products of dense.hip: dense layers, dense rows, sampled gradients.)
#include "device.h"
#include "kernels.h"

#include <numeric>
#include <utility>

namespace nerva {
namespace {

constexpr int kBlock = kWave * kWavesPerBlock;
constexpr int kEwBlock = 256;  // work-group of the element-wise kernels

// Which row, and which contiguous run [s0, s1) of its stored entries, the calling wave serves.
struct WaveTask {
    int row;     // -1: nothing to do
    int part;    // index of this wave among the waves that share the row inside this work-group
    int lg;      // log2(waves that share the row in this work-group); uniform over the work-group
    int s0, s1;  // the wave's stored entries
    bool huge;   // the work-group holds one share of a huge row: its result is a partial sum
    bool lead;   // first wave of the row's first share (owner of per-row by-products)
    int index;   // of a huge row in RowBlocks::huge_rows
};
// One 16-byte scalar load per wave: the partition table is spelled out per wave when the
// pattern is bound, so nothing about the row has to be looked up before its entries are fetched.
// W: waves of the work-group, fewer than the partition's where they share nothing.
template <int W = kWavesPerBlock>
__device__ __forceinline__ WaveTask wave_task(const RowBlocks &b, int block)
{
    const int4 d = b.waves[block * W + wave_in_block()];
    WaveTask t;
    t.row = d.x;
    t.s0 = d.y;
    t.s1 = d.z;
    t.part = d.w & 15;
    t.lg = (d.w >> 4) & 15;
    t.lead = (d.w >> 8) & 1;
    t.huge = (d.w >> 9) & 1;
    t.index = d.w >> 10;
    return t;
}

__device__ __forceinline__ void fma_into(float (&acc)[4], float w, float4 x)
{
    acc[0] = fmaf(w, x.x, acc[0]);
    acc[1] = fmaf(w, x.y, acc[1]);
    acc[2] = fmaf(w, x.z, acc[2]);
    acc[3] = fmaf(w, x.w, acc[3]);
}

// f(i) for 0 <= i < n, a work-group's threads side by side, in eight runs: n_blocks work-groups (a multiple of 8, the launch's first) go to the XCDs in turn, and each
// XCD walks a run of its own in order.  For passes that step through one orientation's entries and reach the other's through the position map: entries of
// neighbouring rows there lie side by side here, so the 128-byte lines that one XCD's run touches are a band that its L2 holds, and every line is
// brought to (or written back from) one or two L2s instead of all eight.
// The mirror's values of 16384^2 at 1 / 10 %, power-law: 20.9 -> 17.6 and 307 -> 192 us (what is left is a line from L2 per value); second pass of both gradients, at 1 % 52 -> 39 us, of a
// step's 8192^2 layer at 0.6 % 24.5 -> 21.0.  Steps of 3072-8192-8192-10 at 5 %, batch 512 726 -> 694, of 1000-3000-3000-3000-30 262 -> 251.
struct XcdRun {
    int64_t first, end, step;   // the work-group's first item, its XCD's last, the way from one turn to the next
};
template <int EACH = 1>
__device__ __forceinline__ XcdRun xcd_run(int64_t n, int n_blocks, uint32_t block = blockIdx.x)
{
    constexpr int kItems = kEwBlock * EACH;
    const int64_t per = ((n + kItems - 1) / kItems + 7) / 8 * kItems, first = (block & 7) * per;
    return XcdRun{first + static_cast<int64_t>(block >> 3) * kItems, min(n, first + per), static_cast<int64_t>(n_blocks >> 3) * kItems};
}
template <typename F>
__device__ __forceinline__ void for_runs_of_xcds(int64_t n, int n_blocks, F &&f, uint32_t block = blockIdx.x)
{
    const XcdRun run = xcd_run(n, n_blocks, block);
    for (int64_t i = run.first + threadIdx.x; i < run.end; i += run.step) f(i);
}
// dst[i] = src[perm[i]]: many in kGatherEach a thread, whose reads travel together, few in one
constexpr int kGatherEach = 4;
constexpr int64_t kGatherMany = 1 << 20;
__device__ __forceinline__ void gather_runs(float *__restrict__ dst, const float *__restrict__ src, const int32_t *__restrict__ perm, int64_t n, int n_blocks)
{
    if (n < kGatherMany) return for_runs_of_xcds(n, n_blocks, [&](int64_t i) { dst[i] = src[perm[i]]; });
    const XcdRun run = xcd_run<kGatherEach>(n, n_blocks);
    for (int64_t base = run.first + threadIdx.x; base < run.end; base += run.step) {
        float x[kGatherEach];
#pragma unroll
        for (int u = 0; u < kGatherEach; ++u) x[u] = src[perm[min(base + u * kEwBlock, run.end - 1)]];
#pragma unroll
        for (int u = 0; u < kGatherEach; ++u)
            if (base + u * kEwBlock < run.end) dst[base + u * kEwBlock] = x[u];
    }
}

// U consecutive stored entries starting at p: all index/weight fetches, then all gathers, then
// the FMAs, so that U reads are in flight per wave.
template <bool XMASK, int U>
__device__ __forceinline__ void spmm_step(const SpmmArgs &a, int p, uint32_t ldxb, uint32_t ldmb, uint32_t off, float (&acc)[4])
{
    int j[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        j[u] = a.indices[p + u];
        w[u] = a.values[p + u];
    }
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        x[u] = gload4(row_base(a.X, j[u], ldxb), off);
        if constexpr (XMASK) x[u] = keep_where_positive(x[u], gload4(row_base(a.XM, j[u], ldmb), off));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) fma_into(acc, w[u], x[u]);
}

// Bias, ReLU and the optional output mask on the four columns from `col` on of one row, and their store: of those from `own`
// on, where the lane's columns were shifted to end with the batch (the others may be another work-group's, summed in another order).
__device__ __forceinline__ void spmm_store(const SpmmArgs &a, int row, int col, int own, const float (&acc)[4])
{
    const float b = a.bias ? a.bias[row] : 0.f;
    float y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        y[k] = acc[k] + b;
        if (a.relu) y[k] = y[k] > 0.f ? y[k] : 0.f;
    }
    float4 o = make_float4(y[0], y[1], y[2], y[3]);
    if (a.YM) o = keep_where_positive(o, ld4(a.YM + static_cast<int64_t>(row) * a.ldym + col));
    float *out = a.Y + static_cast<int64_t>(row) * a.ldy + col;
    if (own == col) {
        st4(out, o);
    } else {
        if (own <= col + 1) out[1] = o.y;
        if (own <= col + 2) out[2] = o.z;
        out[3] = o.w;
    }
}

// The share of a huge row that a work-group has summed, for the columns from col0 on (its first wave holds it in acc, lane l the columns
// from col on): left in the work-group's scratch row; the work-group that comes last adds up the shares, a wave every 16th, and
// stores the row.  Called by all waves of the work-group, none with something pending in red.  The shares of a row come from any XCD: they go
// out and come back as relaxed atomics of agent scope, which pass the L2s by, and the wait before the ticket is taken makes
// them arrive first (a release fence would write back a whole L2).  The ticket counts modulo the number of shares: it is 0 after
// every product, whatever ran beside it (products of one layer that overlap spoil each other's partial rows, but none after them).
// Instead of a second launch: forward product of the power-law 16384^2 matrix at 0.1 %, batch 128: 21.4 -> 18.3 us.
// ALONE: the first wave does it all and the others end at once.  In column tiles the work-groups outnumber what the chip holds,
// and 16 waves that wait for one wave's round trips keep others out: the same matrix at batch 512 / 1024, with a second launch instead
// 55.7 / 104 us, all waves waiting 58.8 / 114.4, one alone 56.2 / 107.2.
template <bool ALONE, int N, int LANES>
__device__ __forceinline__ void huge_row_share(const SpmmArgs &a, const WaveTask &task, int block, int col0, int col, int own, bool on,
                                               float (&acc)[N], float (&red)[kWavesPerBlock][N][LANES])
{
    __shared__ int turn_s;
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block();
    if (ALONE && wv != 0) return;
    const int4 h = a.blocks.huge_rows[task.index];
    int turn = 0;
    if (wv == 0) {
        float *mine = a.scratch + static_cast<int64_t>(block) * a.scratch_ld + col;
        if (on) {
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (col + k >= own) __hip_atomic_store(mine + k, acc[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) {
            int *ticket = a.tickets + 2 * task.index * huge_row_tickets(a.scratch_ld) + col0 / 32;
            turn = static_cast<int>(atomicInc(reinterpret_cast<unsigned *>(ticket), static_cast<unsigned>(h.z - 1)));
        }
        turn = __builtin_amdgcn_readfirstlane(turn);
    }
    constexpr int step = ALONE ? 1 : kWavesPerBlock;   // shares from one of the wave's to its next
    if constexpr (!ALONE) {
        if (threadIdx.x == 0) turn_s = turn;
        __syncthreads();
        turn = turn_s;
    }
    if (turn != h.z - 1) return;  // uniform
    if (on) {
        const float *first = a.scratch + static_cast<int64_t>(h.y) * a.scratch_ld + col;
#pragma unroll
        for (int k = 0; k < N; ++k) acc[k] = 0.f;
        constexpr int U = 4;   // (8 of them cost the packed kernel its second work-group per compute unit)
        for (int q = wv; q < h.z; q += U * step) {
            float v[U][N];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < N; ++k)
                    v[u][k] = __hip_atomic_load(first + static_cast<int64_t>(min(q + u * step, h.z - 1)) * a.scratch_ld + k, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            if constexpr (ALONE) {   // (in pairs: one chain over all shares would round more often than the 16 waves' sums do)
#pragma unroll
                for (int k = 0; k < N; ++k) {
#pragma unroll
                    for (int u = 1; u < U; ++u) v[u][k] = q + u < h.z ? v[u][k] : 0.f;
                    acc[k] += (v[0][k] + v[1][k]) + (v[2][k] + v[3][k]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int k = 0; k < N; ++k) acc[k] = q + u * step < h.z ? acc[k] + v[u][k] : acc[k];
            }
        }
        if constexpr (!ALONE)
#pragma unroll
            for (int k = 0; k < N; ++k) red[wv][k][lane] = acc[k];
    }
    if constexpr (!ALONE) __syncthreads();
    if (wv != 0 || !on) return;
    if constexpr (!ALONE)
        for (int w = 1; w < min(h.z, kWavesPerBlock); ++w)
#pragma unroll
            for (int k = 0; k < N; ++k) acc[k] += red[w][k][lane];
    if constexpr (N == 4) {
        spmm_store(a, task.row, col, own, acc);
    } else {
        float y = acc[0] + (a.bias ? a.bias[task.row] : 0.f);
        if (a.relu) y = y > 0.f ? y : 0.f;
        if (a.YM) y = keep_where_positive(y, a.YM[static_cast<int64_t>(task.row) * a.ldym + col]);
        a.Y[static_cast<int64_t>(task.row) * a.ldy + col] = y;
    }
}

// ---------------------------------------------------------------------------------------
// SpMM on 256 columns: a wave covers them with one 16-byte access per lane and entry.
// ---------------------------------------------------------------------------------------
template <bool XMASK>
__device__ __forceinline__ void spmm_body(const SpmmArgs &a, const int block, const int col0)
{
    constexpr int U = 8;
    __shared__ float red[kWavesPerBlock][4][kWave];

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const WaveTask task = wave_task(a.blocks, block);
    // Lanes whose columns lie beyond the batch re-read the tile's first columns and are never stored.
    const bool on = col0 + lane * 4 < a.batch;
    const int col = four_columns(on ? col0 + lane * 4 : col0, a.batch);
    const uint32_t off = static_cast<uint32_t>(col) * 4u;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};

    if (task.row >= 0) {
        const uint32_t ldxb = static_cast<uint32_t>(a.ldx) * 4u;
        const uint32_t ldmb = XMASK ? static_cast<uint32_t>(a.ldxm) * 4u : 0u;
        int p = task.s0;
        const int pe = task.s1;
        // only entries of this wave's share are gathered: the gather stream is what the kernel pays for
        for (; p + U <= pe; p += U) spmm_step<XMASK, U>(a, p, ldxb, ldmb, off, acc);
        if (p + 4 <= pe) { spmm_step<XMASK, 4>(a, p, ldxb, ldmb, off, acc); p += 4; }
        if (p + 2 <= pe) { spmm_step<XMASK, 2>(a, p, ldxb, ldmb, off, acc); p += 2; }
        if (p < pe) spmm_step<XMASK, 1>(a, p, ldxb, ldmb, off, acc);
    }

    if (task.lg > 0) {  // uniform over the work-group
        if (task.part != 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) red[wv][k][lane] = acc[k];
        }
        __syncthreads();
        if (task.part == 0) {
            for (int s = 1; s < (1 << task.lg); ++s)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] += red[wv + s][k][lane];
        }
    }
    if (task.row >= 0 && task.huge) {  // uniform over the work-group
        huge_row_share<false>(a, task, block, col0, col, col0 + lane * 4, on, acc, red);
        return;
    }
    if (task.row < 0 || task.part != 0 || !on) return;
    spmm_store(a, task.row, col, col0 + lane * 4, acc);
}

// One pass of U gather instructions of the grouped SpMM: every index move, then every gather,
// then the FMAs.  Straight-line on purpose: with no branch between the gathers the compiler
// counts outstanding loads exactly (vmcnt U-1 ... 0) and all U stay in flight; a branch inside
// makes it wait for every earlier load before each later one.
// src: byte address (lane * 4) of the lane that holds this group's entry of the pass's first
// step; consecutive steps lie STEP_BYTES further on.
template <int U, int STEP_BYTES, bool XMASK>
__device__ __forceinline__ void grouped_pass(gmem_ptr Xg, gmem_ptr Mg, int src, int my_ro, int my_mo, float my_w,
                                             uint32_t off, float (&acc)[4])
{
    uint32_t ro[U], mo[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        ro[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src + u * STEP_BYTES, my_ro));
        w[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src + u * STEP_BYTES, __builtin_bit_cast(int, my_w)));
        if constexpr (XMASK) mo[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src + u * STEP_BYTES, my_mo));
    }
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = gload4(Xg, ro[u] + off);
    if constexpr (XMASK) {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = keep_where_positive(x[u], gload4(Mg, mo[u] + off));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        acc[0] = fmaf(w[u], x[u].x, acc[0]);
        acc[1] = fmaf(w[u], x[u].y, acc[1]);
        acc[2] = fmaf(w[u], x[u].z, acc[2]);
        acc[3] = fmaf(w[u], x[u].w, acc[3]);
    }
}

// SpMM for batches of at most GS*4 columns, GS in {8, 16, 32}: a gather instruction costs the
// memory pipeline the same whether 25 or 64 lanes take part, so each group of GS lanes works on
// its own stored entry and one instruction fetches 64/GS rows of the dense operand.  Entries of
// the wave's share are dealt to the groups round-robin; the groups' partial sums meet in LDS
// together with those of the other waves of the row and are added in (wave, group) order (GS < 16: the groups first, by shuffles).
// Narrow groups for narrow batches: 4096^2 at 10 % and batch 32 took 19.1 us in groups of 16, 15.5 in groups of 8 (and 14.5 at batch
// 16 in groups of 4, but 5.3 instead of 5.1 on 1000 x 3000: not kept).
// Row offsets are 32-bit byte offsets from the operand's base: the operand (and its mask) must
// span less than 4 GiB, which the launcher checks.
template <int GS, bool XMASK, bool TILED = false>
__device__ __forceinline__ void spmm_body_grouped(const SpmmArgs &a, const int block, const int col0 = 0)
{
    constexpr int NE = kWave / GS;   // entries per gather instruction
    constexpr int SB = NE * 4;       // lane-address distance between consecutive steps
    __shared__ float red[kWavesPerBlock][4][kWave];

    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int grp = lane / GS;
    const int lig = lane % GS;
    const WaveTask task = wave_task(a.blocks, block);
    const bool on = col0 + lig * 4 < a.batch;
    const int col = four_columns(on ? col0 + lig * 4 : col0, a.batch);
    const uint32_t off = static_cast<uint32_t>(col) * 4u;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};

    if (task.row >= 0) {
        const uint32_t ldxb = static_cast<uint32_t>(a.ldx) * 4u;
        const uint32_t ldmb = XMASK ? static_cast<uint32_t>(a.ldxm) * 4u : 0u;
        const gmem_ptr Xg = as_gmem(a.X);
        const gmem_ptr Mg = as_gmem(a.XM);
        for (int pc = task.s0; pc < task.s1; pc += kWave) {
            const int n = min(kWave, task.s1 - pc);
            // Entry pc+l of the chunk sits in lane l; step u hands entry u*NE+grp to group grp.
            // Lanes past the chunk's end repeat its first entry with weight 0: a gather of theirs
            // reads a row this output row reads anyway, and adds nothing.
            const int q = lane < n ? lane : 0;
            const int my_j = a.indices[pc + q];
            float my_w = a.values[pc + q];
            my_w = lane < n ? my_w : 0.f;
            const int my_ro = static_cast<int>(static_cast<uint32_t>(my_j) * ldxb);
            const int my_mo = XMASK ? static_cast<int>(static_cast<uint32_t>(my_j) * ldmb) : 0;
            const int steps = (n + NE - 1) / NE;
            int src = grp * 4;
            int u0 = 0;
            for (; u0 + 8 <= steps; u0 += 8, src += 8 * SB)
                grouped_pass<8, SB, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
            if (u0 + 4 <= steps) {
                grouped_pass<4, SB, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
                u0 += 4; src += 4 * SB;
            }
            if (u0 + 2 <= steps) {
                grouped_pass<2, SB, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
                u0 += 2; src += 2 * SB;
            }
            if (u0 < steps) grouped_pass<1, SB, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
        }
    }

    // every wave leaves its 64 lanes' partial sums in LDS; the row's first wave adds them up
    if constexpr (GS < 16) {
#pragma unroll
        for (int d = GS; d < kWave; d <<= 1)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], d, kWave);
    }
    constexpr int kParts = GS < 16 ? 1 : NE;   // of a wave
    if (kParts > 1 || grp == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) red[wv][k][lane] = acc[k];
    }
    __syncthreads();
    if (task.row < 0 || (!task.huge && (task.part != 0 || grp != 0))) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) acc[k] = 0.f;
    if (task.part == 0 && grp == 0) {
        for (int s = 0; s < (1 << task.lg); ++s)
#pragma unroll
            for (int g = 0; g < kParts; ++g)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] += red[wv + s][k][g * GS + lig];
    }
    if (task.huge) {  // uniform over the work-group
        huge_row_share<TILED>(a, task, block, col0, col, col0 + lig * 4, on && grp == 0, acc, red);
        return;
    }
    if (on) spmm_store(a, task.row, col, col0 + lig * 4, acc);
}

// Packed SpMM for short rows: each group of GS lanes owns one row, so a gather instruction
// fetches one entry of each of 64/GS rows and no sum across groups or waves is needed.  The rows
// come from RowBlocks::short_rows, longest first, so the rows of a set have nearly the same
// length; a group whose row is exhausted repeats that row's first entry with weight 0.  A wave
// can serve kPackSets sets one after the other, fetching the next set's rows and indices one
// step ahead; measured, one set per wave is best (more, shorter work-groups balance better than
// the saved start-up is worth).
template <int GS, bool XMASK, int W>
__device__ __forceinline__ void spmm_body_packed(const SpmmArgs &a, const int block, const int col0, const int n_pack_blocks)
{
    constexpr int NE = kWave / GS;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int grp = lane / GS;
    const int lig = lane % GS;
    const bool on = col0 + lig * 4 < a.batch;
    const int col = four_columns(on ? col0 + lig * 4 : col0, a.batch);
    const uint32_t off = static_cast<uint32_t>(col) * 4u;
    const uint32_t ldxb = static_cast<uint32_t>(a.ldx) * 4u;
    const uint32_t ldmb = XMASK ? static_cast<uint32_t>(a.ldxm) * 4u : 0u;
    const gmem_ptr Xg = as_gmem(a.X);
    const gmem_ptr Mg = as_gmem(a.XM);
    const int n_sets = (a.blocks.n_short + NE - 1) / NE;
    const int src0 = grp * GS * 4;  // byte address of the group's first lane
    // The sets are sorted by length, so they are dealt to the waves round-robin: wave k of the
    // launch's n_waves takes sets k, k + n_waves, k + 2 n_waves, ... and every wave gets its share
    // of long and of short rows (consecutive sets per wave left the first work-groups 1.4x the work
    // of the average on rows of 40..85 entries, and a launch is one round of work-groups).
    const int n_waves = n_pack_blocks * W;
    const int first_set = block * W + wv;
    if (first_set >= n_sets) return;  // wave-uniform
    const int last_set = first_set + ((n_sets - 1 - first_set) / n_waves) * n_waves;  // <= first_set + (kPackSets - 1) * n_waves

    // Entry base+lig of the group's row: column index and weight (0 past the row's end, where the
    // row's first entry is repeated; an empty row reads entry 0 of the matrix and is zeroed below).
    auto fetch = [&](int s0, int len, int base, int &j, float &w) {
        const int e = base + lig;
        const bool ok = e < len;
        const int p = len > 0 ? s0 + (ok ? e : 0) : 0;
        j = a.indices[p];
        w = a.values[p];
        w = ok ? w : 0.f;
    };

    // One step ahead: while a chunk of GS entries per row is gathered, the indices and weights of
    // the next chunk (or of the next set's first chunk) and the next set's rows are on their way.
    int4 d = a.blocks.short_rows[first_set * NE + grp];  // the table is padded to whole sets
    int cur_j;
    float cur_w;
    fetch(d.y, d.z, 0, cur_j, cur_w);
    for (int set = first_set; set <= last_set; set += n_waves) {
        const int row = d.x, s0 = d.y, len = d.z;
        const int maxlen = __builtin_amdgcn_readfirstlane(len);  // group 0 holds the set's longest row
        const int4 dn = a.blocks.short_rows[min(set + n_waves, last_set) * NE + grp];
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        int base = 0;
        do {
            const bool more = base + GS < maxlen;  // wave-uniform
            int next_j;
            float next_w;
            fetch(more ? s0 : dn.y, more ? len : dn.z, more ? base + GS : 0, next_j, next_w);
            const int my_ro = static_cast<int>(static_cast<uint32_t>(cur_j) * ldxb);
            const int my_mo = XMASK ? static_cast<int>(static_cast<uint32_t>(cur_j) * ldmb) : 0;
            const float my_w = cur_w;
            const int steps = min(GS, maxlen - base);  // 0 for a set of empty rows
            int src = src0;
            int u0 = 0;
            for (; u0 + 8 <= steps; u0 += 8, src += 32) grouped_pass<8, 4, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
            if (u0 + 4 <= steps) {
                grouped_pass<4, 4, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
                u0 += 4; src += 16;
            }
            if (u0 + 2 <= steps) {
                grouped_pass<2, 4, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
                u0 += 2; src += 8;
            }
            if (u0 < steps) grouped_pass<1, 4, XMASK>(Xg, Mg, src, my_ro, my_mo, my_w, off, acc);
            cur_j = next_j;
            cur_w = next_w;
            base += GS;
        } while (base < maxlen);
        d = dn;
        if (row < 0 || !on) continue;
        if (len == 0) acc[0] = acc[1] = acc[2] = acc[3] = 0.f;  // an empty row gathered (with weight 0) from entry 0 of the matrix
        spmm_store(a, row, col, col, acc);
    }
}

// Which column tile, and which of the launch's n_blocks work-groups of rows, a work-group serves (they go to the XCDs in turn).  One by one: tile by tile, all XCDs on one tile.
// Whole: every eighth tile to an XCD, so that eight of them side by side are read at a time.  Otherwise the list of all work-groups is cut into eight equal runs, one per XCD, so that
// an L2 sees an eighth of the tiles and one more; the stride, which has no factor in common with n_blocks, is the order within a tile.  (tile_order chooses.)
enum : int { kTilesOneByOne = 0, kTilesWhole = -1 };
struct TileOrder {
    int per, stride;   // an eighth of the grid (an argument: the grid's size costs a load), or one of the above
};
__device__ __forceinline__ bool tile_of_block(int n_tiles, int n_blocks, TileOrder order, int &tile, int &block, uint32_t id = blockIdx.x)
{
    const int stride = order.stride;
    int at = id;
    if (order.per > 0) at = (id & 7) * order.per + (id >> 3);
    if (order.per < 0) at = id >> 3;
    tile = at / n_blocks;
    block = at - tile * n_blocks;
    if (order.per < 0) tile = tile * 8 + (id & 7);
    if (stride > 1) block = static_cast<int>(static_cast<uint32_t>(block) * static_cast<uint32_t>(stride) % static_cast<uint32_t>(n_blocks));
    return tile < n_tiles;
}

// Short rows through the packed body, the remaining rows through the grouped body, in one grid, for every column tile.
template <int GS, bool XMASK>
__global__ __launch_bounds__(kBlock) void spmm_packed_kernel(const SpmmArgs a, const int n_tiles, const TileOrder order,
                                                             const int n_pack_blocks)
{
    const int nrb = n_pack_blocks + a.blocks.n_long_blocks;
    int tile, rb;
    if (!tile_of_block(n_tiles, nrb, order, tile, rb)) return;
    if (rb < n_pack_blocks) {
        spmm_body_packed<GS, XMASK, kWavesPerBlock>(a, rb, tile * GS * 4, n_pack_blocks);
    } else {
        SpmmArgs al = a;
        al.blocks.waves = a.blocks.long_waves;
        spmm_body_grouped<GS, XMASK, true>(al, rb - n_pack_blocks, tile * GS * 4);
    }
}

// The same without long rows, in work-groups of kPackWaves: nothing is shared among the waves, and where the launch is a round of work-groups and a little, the
// little starts on every compute unit as waves end (infer 3072-8192-8192-10 at 1 %, batch 300: 74.8 us in work-groups of 16 waves, 70.8 of 8, 70.0 of 4, 69.8 of 1; 8192^2 at 1 %,
// batch 300 48.9 -> 42.9; 3000 x 7000 at 1 %, batch 600 32.4 -> 28.8; wide MLP at batch 1024 as before).
constexpr int kPackWaves = 4;
template <int GS, bool XMASK>
__global__ __launch_bounds__(kPackWaves * kWave) __attribute__((amdgpu_waves_per_eu(XMASK ? 1 : 8))) void spmm_packed_only_kernel(const SpmmArgs a, const int n_tiles,
                                                                                                                            const TileOrder order, const int n_pack_blocks)
{
    int tile, rb;
    if (!tile_of_block(n_tiles, n_pack_blocks, order, tile, rb)) return;
    spmm_body_packed<GS, XMASK, kPackWaves>(a, rb, tile * GS * 4, n_pack_blocks);
}

template <int GS, bool XMASK>
__global__ __launch_bounds__(kBlock) void spmm_grouped_kernel(const SpmmArgs a)
{
    spmm_body_grouped<GS, XMASK>(a, blockIdx.x);
}

// Column-tiled launch for dense operands that do not fit an L2: the batch is cut into tiles of
// GS*4 columns, narrow enough that one tile of the whole operand (x_rows x GS*4 floats) stays
// resident in a 4 MiB L2 while every stored entry gathers from it.  TileOrder says which XCD works on which tiles.
template <int GS, bool XMASK>
__global__ __launch_bounds__(kBlock) void spmm_tiled_kernel(const SpmmArgs a, const int n_tiles, const TileOrder order)
{
    const int nrb = a.blocks.n_blocks;
    int tile, rb;
    if (!tile_of_block(n_tiles, nrb, order, tile, rb)) return;
    spmm_body_grouped<GS, XMASK, true>(a, rb, tile * GS * 4);
}

// Wide batches: the columns in tiles of 256, a work-group of the row partition each -- more, shorter work-groups than one
// wave carrying up to 1024 columns of its entries (power-law 2957 x 948 at batch 585: 22.4 us, 12.4 in tiles; 1024 x 600 at
// batch 1024: 19.3, 10.0; even rows the same) -- and what is left of the batch in the kernels for as few columns.
template <bool XMASK>
__device__ __forceinline__ void spmm_wide_body(const SpmmArgs &a, const int block, const int col0)
{
    const int left = a.batch - col0;
    if (left > 128 || a.wide_offsets)
        spmm_body<XMASK>(a, block, col0);
    else if (left > 64)
        spmm_body_grouped<32, XMASK>(a, block, col0);
    else if (left > 32)
        spmm_body_grouped<16, XMASK>(a, block, col0);
    else
        spmm_body_grouped<8, XMASK>(a, block, col0);
}
template <bool XMASK>
__global__ __launch_bounds__(kBlock) void spmm_kernel(const SpmmArgs a)
{
    spmm_wide_body<XMASK>(a, blockIdx.x, blockIdx.y * 256);
}

// SpMM for batches of at most 4 columns (inference on one or a few examples): there is no batch
// dimension to spread lanes over, so lanes run across the stored entries of the wave's share
// instead -- coalesced index/weight reads, a 4-byte gather per entry and column, a DPP sum over
// the wave, and the usual ordered LDS combine of the row's shares.  Any leading dimension.
template <int NB>
__global__ __launch_bounds__(kBlock) void spmv_kernel(const SpmmArgs a)
{
    __shared__ float red[kWavesPerBlock][NB], shares[kWavesPerBlock][1][NB];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const WaveTask task = wave_task(a.blocks, blockIdx.x);
    float acc[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = 0.f;
    if (task.row >= 0) {
        for (int p = task.s0 + lane; p < task.s1; p += kWave) {
            const int64_t j = a.indices[p];
            const float w = a.values[p];
            const float *xr = a.X + j * a.ldx;
            const float *mr = a.XM ? a.XM + j * a.ldxm : nullptr;
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c < a.batch) {
                    float x = xr[c];
                    if (mr) x = keep_where_positive(x, mr[c]);
                    acc[c] = fmaf(w, x, acc[c]);
                }
        }
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = group_sum<kWave>(acc[c]);  // all lanes of every wave take part
    if (task.lg > 0) {
        if (lane == 0)
#pragma unroll
            for (int c = 0; c < NB; ++c) red[wv][c] = acc[c];
        __syncthreads();
        if (task.part == 0)
            for (int s = 1; s < (1 << task.lg); ++s)
#pragma unroll
                for (int c = 0; c < NB; ++c) acc[c] += red[wv + s][c];
    }
    if (task.row < 0 || (!task.huge && (task.part != 0 || lane >= a.batch || lane >= NB))) return;
    float y = acc[0];
#pragma unroll
    for (int c = 1; c < NB; ++c) y = lane == c ? acc[c] : y;
    if (task.huge) {  // uniform over the work-group
        float one[1] = {y};
        huge_row_share<false>(a, task, blockIdx.x, 0, lane, lane, lane < a.batch && lane < NB, one, shares);
        return;
    }
    y += a.bias ? a.bias[task.row] : 0.f;
    if (a.relu) y = y > 0.f ? y : 0.f;
    if (a.YM) y = keep_where_positive(y, a.YM[static_cast<int64_t>(task.row) * a.ldym + lane]);
    a.Y[static_cast<int64_t>(task.row) * a.ldy + lane] = y;
}

// The same for matrices of more entries than the chip's waves hold at 64 each: there a wave took one load of its share and
// waited out three round trips for it, wave after wave (3030 x 2039 at 33 %, 2 M entries, 1 / 4 examples: 16.6 / 36 us, now 11.6 / 11.8).
// Here the waves are as many as the chip holds, 2^lg to a row, rows longest first, with four or eight loads of a lane in flight.
template <int NB>
__global__ __launch_bounds__(kBlock) void spmv_rows_kernel(const SpmmArgs a, const int lg)
{
    constexpr int U = NB == 1 ? 8 : 4;
    __shared__ float red[kWavesPerBlock][NB];
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block(), part = wv & ((1 << lg) - 1);
    const int at = (blockIdx.x * kWavesPerBlock + wv) >> lg;
    const int4 d = at < a.rows ? a.blocks.rows_by_length[at] : make_int4(-1, 0, 0, 0);
    const int share = (((d.z + (1 << lg) - 1) >> lg) + kWave - 1) / kWave * kWave, end = d.y + d.z;
    const int s0 = min(d.y + part * share, end), s1 = min(s0 + share, end);
    const gmem_ptr X = as_gmem(a.X), M = as_gmem(a.XM);
    const uint32_t ldxb = static_cast<uint32_t>(a.ldx) * 4u, ldmb = static_cast<uint32_t>(a.ldxm) * 4u;
    float acc[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = 0.f;
    for (int p = s0 + lane; p - lane < s1; p += kWave * U) {   // wave-uniform
        int j[U];
        float w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at_u = min(p + u * kWave, s1 - 1);
            j[u] = a.indices[at_u];
            w[u] = a.values[at_u];
        }
        float x[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (NB == 4 && a.batch == 4) {   // uniform
                float4 v = gload4(X, static_cast<uint32_t>(j[u]) * ldxb);
                if (a.XM) v = keep_where_positive(v, gload4(M, static_cast<uint32_t>(j[u]) * ldmb));
                x[u][0] = v.x; x[u][1 % NB] = v.y; x[u][2 % NB] = v.z; x[u][3 % NB] = v.w;
                continue;
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                const uint32_t column = static_cast<uint32_t>(min(c, a.batch - 1)) * 4u;
                x[u][c] = gload1(X, static_cast<uint32_t>(j[u]) * ldxb + column);
                if (a.XM) x[u][c] = keep_where_positive(x[u][c], gload1(M, static_cast<uint32_t>(j[u]) * ldmb + column));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool mine = p + u * kWave < s1;   // (past the end: the last entry again, not added)
#pragma unroll
            for (int c = 0; c < NB; ++c) acc[c] = mine ? fmaf(w[u], x[u][c], acc[c]) : acc[c];
        }
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = group_sum<kWave>(acc[c]);
    if (lane == 0)
#pragma unroll
        for (int c = 0; c < NB; ++c) red[wv][c] = acc[c];
    __syncthreads();
    if (d.x < 0 || part != 0 || lane >= a.batch || lane >= NB) return;
    float y = 0.f;
    for (int s = 0; s < (1 << lg); ++s) y += red[wv + s][lane];
    y += a.bias ? a.bias[d.x] : 0.f;
    if (a.relu) y = y > 0.f ? y : 0.f;
    if (a.YM) y = keep_where_positive(y, a.YM[static_cast<int64_t>(d.x) * a.ldym + lane]);
    a.Y[static_cast<int64_t>(d.x) * a.ldy + lane] = y;
}

// Product with a FULL matrix of few rows (every entry stored, rows <= kFullMaxRows): values[] is
// the row-major dense matrix, so instead of gathering the operand once per row the kernel streams
// it once for all rows.  A work-group of 4 waves owns kFullSlice consecutive operand rows and 256
// batch columns (4 per lane); wave w walks the slice's operand rows w*32 .. w*32+31, eight 16-byte
// loads in flight, weights through uniform loads, one accumulator per matrix row; the waves'
// accumulators meet in LDS and are added in wave order.  The slice's partial result goes to
// full_scratch; full_rows_finish_kernel adds the slices in order and applies the epilogue.
constexpr int kFullWaves = 4;  // 4 waves x 16 rows x 1 KiB of LDS at most: 64 KiB
__global__ __launch_bounds__(kFullWaves * kWave) void full_rows_kernel(const SpmmArgs a)
{
    extern __shared__ float4 full_red[];  // [kFullWaves][rows][kWave]
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int K = a.x_rows;
    const int slice = blockIdx.x;
    const bool on = static_cast<int>((blockIdx.y * kWave + lane) * 4) < a.batch;
    const int col = on ? four_columns((blockIdx.y * kWave + lane) * 4, a.batch) : 0;
    const int64_t xoff = col;
    constexpr int KW = kFullSlice / kFullWaves;  // operand rows per wave: all requested before the first use
    static_assert(KW <= 64 && (KW & (KW - 1)) == 0, "one weight per lane");
    const int k_begin = slice * kFullSlice + wv * KW;
    float4 acc[kFullMaxRows];
    float4 x[KW];
#pragma unroll
    for (int u = 0; u < KW; ++u) {
        const int64_t k = k_begin + u < K ? k_begin + u : K - 1;  // rows past the end are re-read and get weight 0
        x[u] = ld4(a.X + k * a.ldx + xoff);
    }
    // lane u (and u + 32) holds row r's weight of operand row k_begin + u
    float wrow[kFullMaxRows];
    const int kl = k_begin + (lane & (KW - 1));
#pragma unroll
    for (int r = 0; r < kFullMaxRows; ++r)
        wrow[r] = (r < a.rows && kl < K) ? a.values[static_cast<int64_t>(r) * K + kl] : 0.f;
#pragma unroll
    for (int r = 0; r < kFullMaxRows; ++r) {
        acc[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < a.rows) {  // uniform
#pragma unroll
            for (int u = 0; u < KW; ++u) {
                const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wrow[r]), u));
                acc[r].x = fmaf(w, x[u].x, acc[r].x);
                acc[r].y = fmaf(w, x[u].y, acc[r].y);
                acc[r].z = fmaf(w, x[u].z, acc[r].z);
                acc[r].w = fmaf(w, x[u].w, acc[r].w);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < kFullMaxRows; ++r)
        if (r < a.rows) full_red[(wv * a.rows + r) * kWave + lane] = acc[r];
    __syncthreads();
    if (!on) return;
    for (int r = wv; r < a.rows; r += kFullWaves) {
        float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int w = 0; w < kFullWaves; ++w) {
            const float4 p = full_red[(w * a.rows + r) * kWave + lane];
            y.x += p.x; y.y += p.y; y.z += p.z; y.w += p.w;
        }
        st4(a.full_scratch + (static_cast<int64_t>(slice) * a.rows + r) * a.full_scratch_ld + col, y);
    }
}

__global__ __launch_bounds__(kEwBlock) void full_rows_finish_kernel(const SpmmArgs a, const int n_slices)
{
    const int r = blockIdx.x;
    const int c = blockIdx.y * kEwBlock + threadIdx.x;
    if (c >= a.batch) return;
    const float *p = a.full_scratch + static_cast<int64_t>(r) * a.full_scratch_ld + c;
    const int64_t step = static_cast<int64_t>(a.rows) * a.full_scratch_ld;
    float y = 0.f;
    int q = 0;
    for (; q + 8 <= n_slices; q += 8) {  // eight loads in flight, added in slice order
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * step];
#pragma unroll
        for (int u = 0; u < 8; ++u) y += v[u];
    }
    for (; q < n_slices; ++q) y += p[q * step];
    y += a.bias ? a.bias[r] : 0.f;
    if (a.relu) y = y > 0.f ? y : 0.f;
    if (a.YM) y = keep_where_positive(y, a.YM[static_cast<int64_t>(r) * a.ldym + c]);
    a.Y[static_cast<int64_t>(r) * a.ldy + c] = y;
}

// The same finish pass for an output layer, with the softmax cross-entropy on top: wave r of a work-group adds the
// slices of row r for 64 columns, the rows meet in LDS, and every wave then forms its own row of the loss gradient
// (each lane repeats the column's maximum and sum over the <= 16 rows, in the order of softmax_ce_kernel, so the
// gradient has the same bits); wave 0 also stores the column's loss.
__global__ __launch_bounds__(kBlock) void full_rows_finish_softmax_kernel(const SpmmArgs a, const int n_slices)
{
    __shared__ float zs[kWavesPerBlock][kWave];
    static_assert(kFullMaxRows <= kWavesPerBlock, "one wave per row");
    const int lane = threadIdx.x & (kWave - 1);
    const int r = wave_in_block();
    const int c = blockIdx.x * kWave + lane;
    const bool on = r < a.rows && c < a.batch;
    float y = 0.f;
    if (on) {
        const float *p = a.full_scratch + static_cast<int64_t>(r) * a.full_scratch_ld + c;
        const int64_t step = static_cast<int64_t>(a.rows) * a.full_scratch_ld;
        int q = 0;
        for (; q + 8 <= n_slices; q += 8) {  // eight loads in flight, added in slice order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(q + u) * step];
#pragma unroll
            for (int u = 0; u < 8; ++u) y += v[u];
        }
        for (; q < n_slices; ++q) y += p[q * step];
        y += a.bias ? a.bias[r] : 0.f;
        a.Y[static_cast<int64_t>(r) * a.ldy + c] = y;
    }
    zs[r][lane] = y;
    __syncthreads();
    if (!on) return;
    const int t = a.ce_labels[c];
    float z[kFullMaxRows];
#pragma unroll
    for (int i = 0; i < kFullMaxRows; ++i) z[i] = i < a.rows ? zs[i][lane] : -INFINITY;
    float m = z[0];
#pragma unroll
    for (int i = 1; i < kFullMaxRows; ++i) m = fmaxf(m, z[i]);
    float sum = 0.f, zt = 0.f;
#pragma unroll
    for (int i = 0; i < kFullMaxRows; ++i) {
        if (i < a.rows) sum += expf(z[i] - m);
        zt = i == t ? z[i] : zt;
    }
    const float lse = m + logf(sum);
    a.ce_dZ[static_cast<int64_t>(r) * a.ce_lddz + c] = (expf(y - lse) - (r == t ? 1.f : 0.f)) * (1.0f / static_cast<float>(a.batch));
    if (r == 0) a.ce_loss_cols[c] = lse - zt;
}

// ---- staged product ----------------------------------------------------------------------
// For wide batches and matrices with many entries per operand row the gathers are served from LDS instead of the L2, and the results stay in
// registers until they are complete.  A work-group of 16 waves owns a range of at most kStageRangeRows rows and kStageCols columns of the batch; a
// row of 16 lanes owns up to kStageJ of those rows, a float4 of the batch per lane and row.  The work-group walks the column blocks of the matrix in
// order: it copies the block's kStageRows operand rows (128 KiB) into LDS, then every lane row serves, out of that copy, the segment (row, block) of
// each of its rows.  A segment's (column, weight) pairs are loaded one per lane, two segments ahead, and reach the other lanes of the row through DPP
// row broadcasts, so the only LDS traffic is the gather itself.  The next block's operand rows travel to registers while a block is served.  Bias,
// ReLU and the output mask are applied when the rows are stored, once, after the last block.  What bounds it: the latency of short runs of LDS
// gathers at four waves a SIMD (vector ALUs 65 % busy, LDS 45 %; a loop of nothing but whole chunks runs 1.5 times as fast), not either pipe.
// Segments, masks and offsets worked out once per block and not per use, the rows brought ahead, no wait for memory among the gathers, the weight's
// move in the multiply-add: 16384^2 power-law rows at 10 %, batch 1024, under the profiler 1087 -> 745 us (10.3 -> 6.5 vector instructions a gather;
// among other passes it takes 640 to 680); forward products of uniform 8192^2 at 5 %, batch 1024, 374 -> 278, 16384^2 at 2 %, batch 512, 448 -> 334,
// 5000 x 7000 at 8 %, batch 511, 146 -> 115.  The waves of a SIMD take turns by age, so that the oldest were through a block while the youngest,
// alone, could not fill the LDS pipe: their priorities fall as they go through their slots, and who is behind goes first.  Power-law 16384^2 at 10 %,
// batch 1024, dense rows included, 1311 -> 1243, uniform at 10 % 1780 -> 1650; 8192^2 at 5 % 291 -> 270; weight gradients of 16384^2 at 10 / 2 % 2571
// -> 2483, 827 -> 798, 5000 x 7000 at 8 %, batch 511, 153 -> 142.  (48 KB of code, the gradient's 56, the instruction cache 64.  Two registers are
// stored before the block loop and reloaded after it; with a mask four, two of them reloaded once a block.) Slots dealt to the waves there and back
// change nothing, two runs of 8 gathers made one of 16 neither.  A row marked kStageQuad is shared by the four lane rows of a wave, a quarter of each
// segment each, and their four results are added in a fixed order before the store.  Every output element is summed in one order.  With a partial
// plan (RowBlocks::staged_partial) the kernel serves the long rows only and a second launch, the packed kernel, the others.
constexpr int kStageWaves = kWavesPerBlock;
// LDS byte offset of a zero-filled row behind the staged block: where a lane with no entry of its own
// gathers from, so that it multiplies its weight 0 with 0 and not with an operand row that the
// output row does not reference (which may hold Inf or NaN).
constexpr int kStageZeroRow = kStageRows * kStageCols * 4;
static_assert(kStageRangeRows == kStageWaves * 4 * kStageJ && kStageJ <= 16, "a lane row owns kStageJ rows of the range");

template <int... I, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// lane i of every row of 16 lanes receives the value of the row's lane I
template <int I>
__device__ __forceinline__ int row_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + I, 0xF, 0xF, true); }
// acc += w of the row's lane I times x, the move of w in the multiply-add itself (the compiler makes it an instruction of its own, one in six of
// a step).  Such an operand is only there two cycles after it is written, the compiler sees to that in its own instructions alone, and nothing keeps it from writing w
// (a copy, a reload) right before any step: each waits for itself.  Against one wait per run of steps: forward products of 16384^2 power-law at 10 %, batch 1024 1223 -> 1229 us, uniform at 10 %,
// batch 512 891 -> 914, 8192^2 at 1.95 / 5 %, batch 1024 171 -> 173, 278 -> 285; two steps of one wait 1290, 936, 193, 304, as each then waits for two gathers.
template <int I>
__device__ __forceinline__ void fma_row_lane(float4 &acc, float w, const float4 &x)
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %4, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %6 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %4, %7 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc.x), "+&v"(acc.y), "+&v"(acc.z), "+&v"(acc.w)
        : "v"(w), "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w), "n"(I));
}
// Entries B .. B + N - 1 of every lane row, in that order, out of the 16 that its lanes hold as (LDS byte offset, weight): four gathers
// ahead of the one whose products are added.
template <int B, int N>
__device__ __forceinline__ void staged_steps(const char *lds, int off, float w, float4 &acc)
{
    constexpr int kAhead = N < 4 ? N : 4;
    float4 x[N];
    auto gather = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        x[i] = *reinterpret_cast<const float4 *>(lds + row_lane<B + i>(off));
    };
    static_for(std::make_integer_sequence<int, kAhead>{}, gather);
    __builtin_amdgcn_sched_barrier(0);
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i + kAhead < N) gather(std::integral_constant<int, i + kAhead>{});
        fma_row_lane<B + i>(acc, w, x[i]);  // (in this order: each adds to acc)
        if constexpr (i + kAhead < N) __builtin_amdgcn_sched_barrier(0);
    });
}
// the first n entries (n > 0) of lanes B .. B + 7, and one more at most.  (One if after the other: with else the sums of one way are kept
// while the other is gone, and are copied back and forth.)
template <int B>
__device__ __forceinline__ void staged_half(const char *lds, int n, int off, float w, float4 &acc)
{
    int ways = n > 6 ? 1 : n > 4 ? 6 : n > 2 ? 2 : 8;
    asm("" : "+s"(ways));
    if (ways & 1) staged_steps<B, 8>(lds, off, w, acc);
    if (ways & 2) staged_steps<B, 4>(lds, off, w, acc);
    if (ways & 4) staged_steps<B + 4, 2>(lds, off, w, acc);
    if (ways & 8) staged_steps<B, 2>(lds, off, w, acc);
}

// Work-group barrier that orders LDS accesses only: global loads issued before it stay in flight
// across it (the staged kernel has no global data that one wave writes and another reads).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Work-groups of one column tile stage the same operand rows: where there are eight tiles or
// more, each of eight tiles gets an XCD (consecutive work-groups go to consecutive XCDs) and its
// L2 to itself; left-over tiles are dealt out plainly.
__device__ __forceinline__ void staged_ids(int n_ranges, int n_tiles, int &range, int &tile)
{
    const int aligned = (n_tiles >> 3) * 8 * n_ranges;
    if (static_cast<int>(blockIdx.x) < aligned) {
        const int slot = blockIdx.x >> 3;
        range = slot % n_ranges;
        tile = (slot / n_ranges) * 8 + (blockIdx.x & 7);
    } else {
        const int rest = blockIdx.x - aligned, left = n_tiles & 7;
        tile = (n_tiles >> 3) * 8 + rest % left;
        range = rest / left;
    }
}

// A slot's entries [e_lo, e_hi) of a block, or this lane row's quarter of them where the four lane rows share a long row; the
// longest of the four segments that a wave serves side by side sets the number of steps, shorter ones ride along with weight 0.
struct StagedSegments {
    uint32_t at;     // bytes to its first entry, or entries (UNIT 4, 1)
    int left, most;  // 4 times its length; the longest of the four
};
template <int UNIT = 4>
__device__ __forceinline__ StagedSegments staged_segments(int e_lo, int e_hi, bool quad, int lrow)
{
    int p0 = e_lo, len = e_hi - e_lo;
    if (quad) {
        const int from = (len * lrow) >> 2;
        p0 += from;
        len = ((len * (lrow + 1)) >> 2) - from;
    }
    int most = max(len, __shfl_xor(len, 16));
    most = max(most, __shfl_xor(most, 32));
    return StagedSegments{static_cast<uint32_t>(p0) * UNIT, len * 4, most};
}

// MANY: 2^30 entries or more, which 32-bit byte offsets do not reach; they are counted instead.  (65536 x 131072 at 12.5 %, batch 128, forward /
// transposed, with the mirror's values: 8.5 / 29 ms, gathered from memory 70 / 72.)
template <bool XMASK, bool MANY>
__global__ __launch_bounds__(kStageWaves * kWave) void spmm_staged_kernel(const SpmmArgs a, const int n_tiles)
{
    __shared__ float4 stage[kStageRows * kStageCols / 4 + kStageCols / 4];  // the block, then one row of zeros
    const int n_ranges = a.blocks.staged_ranges;
    int range, tile;
    staged_ids(n_ranges, n_tiles, range, tile);
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int lrow = lane >> 4, lig = lane & 15;
    const bool col_on = tile * kStageCols + lig * 4 < a.batch;
    const int col = four_columns(tile * kStageCols + lig * 4, a.batch);
    const char *lds = reinterpret_cast<const char *>(stage) + lig * 16;
    if (threadIdx.x < kStageCols / 4) stage[kStageRows * kStageCols / 4 + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);  // (visible after the first barrier)
    const int n_cb = a.blocks.staged_cblocks;
    // The lane row's J-th row sits in slot (J * 16 + wave) * 4 + lrow of the range; lane J of the
    // lane row keeps that slot's row id and, block after block, its segment.
    const int my_slot = ((lig & (kStageJ - 1)) * kStageWaves + wv) * 4 + lrow;
    const int my_row = a.blocks.staged_rows[range * kStageRangeRows + my_slot];
    const bool my_quad = my_row >= 0 && (my_row & kStageQuad);
    const int n_j = a.blocks.staged_groups[range];  // rows of the range / 64, rounded up
    const int32_t *ends = a.blocks.staged_ends + static_cast<int64_t>(range) * (n_cb + 1) * kStageRangeRows + my_slot;
    constexpr auto all_j = std::make_integer_sequence<int, kStageJ>{};
    float4 acc[kStageJ];
    static_for(all_j, [&](auto jc) { acc[decltype(jc)::value] = make_float4(0.f, 0.f, 0.f, 0.f); });
    // 16 entries of a segment, one per lane, as they are stored.  at: byte offset (MANY: number) of the lane's one in the first chunk; left: 4 times the entries
    // from there to the segment's end; lanes past it read near entry 0
    struct Chunk {
        int index;
        float w;
    };
    constexpr int kUnit = MANY ? 1 : 4;
    const int lig4 = lig * 4;
    auto load_chunk = [&](uint32_t at, int left, int first) {
        const uint32_t o = left > first * 4 ? at : 0u;
        if constexpr (MANY) return Chunk{a.indices[static_cast<int64_t>(o) + first], a.values[static_cast<int64_t>(o) + first]};
        return Chunk{__builtin_bit_cast(int, gload1(as_gmem(a.indices), o + static_cast<uint32_t>(first * 4))), gload1(as_gmem(a.values), o + static_cast<uint32_t>(first * 4))};
    };
    // the same as LDS byte offset and weight
    auto placed = [&](const Chunk &c, bool on, int base, int &off, float &w) {
        off = on ? (c.index << 8) - base : kStageZeroRow;
        w = on ? c.w : 0.f;
    };
    static_assert(kStageCols * 4 == 1 << 8, "");
    // The first two chunks of every slot are asked for kAheadJ slots before they are used, across the end of a block too.
    constexpr int kAheadJ = 2, kHeld = 4;
    static_assert(kStageJ % kHeld == 0 && kAheadJ < kHeld, "");
    Chunk held[kHeld][2];
    auto ask = [&](auto jc, const StagedSegments &s) {
        constexpr int j = decltype(jc)::value;
        const uint32_t at = static_cast<uint32_t>(row_lane<j>(static_cast<int>(s.at)) + lig * kUnit);
        const int left = row_lane<j>(s.left) - lig4;
        held[j % kHeld][0] = load_chunk(at, left, 0);
        held[j % kHeld][1] = load_chunk(at, left, 16);
    };
    // A block's operand rows on their way to LDS: thread t holds four columns of rows t / 16, t / 16 + 64, ... of it.  The last block starts
    // early enough to be whole, and of fewer rows than a block's some are brought twice.
    constexpr int kShare = kStageRows / 64;
    static_assert(kShare % 2 == 0 && kShare / 2 <= kStageJ, "two of them are asked for beside each slot");
    float4 v[kShare];
    const float *const my_x = a.X + static_cast<int64_t>(threadIdx.x >> 4) * a.ldx + col;
    const int last_block = max(a.x_rows - kStageRows, 0), last_rows = a.x_rows - 64;
    auto block_row = [&](int b) { return min(b * kStageRows, last_block); };
    // (Behind the last block there is nothing to ask for: the requests go to the first 64 rows, all of a slot to the same, and find them in the L1.  Asking for the last block again was a
    // third pass over an operand of two blocks: forward products of 16384 x 300 / 1000 / 2000 at 8 %, batch 1024 47.4 -> 45.9, 112.6 -> 113.0, 199.8 -> 194.8 us, 8192^2 at 1.95 % 177.9 -> 172.6; a
    // branch around them 2 % slower on short segments.  The gradient as before: 79 / 143 / 265 -> 79 / 145 / 265.)
    auto ask_rows = [&](int i, int cb0, int last) { v[i] = ld4(my_x + static_cast<int64_t>(min(cb0 + i * 64, last)) * a.ldx); };
    auto put_rows = [&](int cb0) {
#pragma unroll
        for (int i = 0; i < kShare; ++i) {
            const int k = min(cb0 + i * 64, last_rows);
            if constexpr (XMASK) v[i] = keep_where_positive(v[i], ld4(a.XM + static_cast<int64_t>(k + static_cast<int>(threadIdx.x >> 4)) * a.ldxm + col));
            stage[(k - cb0) * 16 + static_cast<int>(threadIdx.x)] = v[i];
        }
    };
    int e1 = ends[kStageRangeRows];
    StagedSegments now = staged_segments<kUnit>(ends[0], e1, my_quad, lrow);
    int e2 = n_cb >= 2 ? ends[2 * kStageRangeRows] : e1;
    static_for(std::make_integer_sequence<int, kAheadJ>{}, [&](auto jc) { ask(jc, now); });
#pragma unroll
    for (int i = 0; i < kShare; ++i) ask_rows(i, 0, last_rows);
    for (int b = 0; b < n_cb; ++b) {
        const int cb0 = block_row(b), cb_next = block_row(b + 1), last_next = b + 1 < n_cb ? last_rows : 0;
        const int e3 = ends[min(b + 3, n_cb) * kStageRangeRows];
        const StagedSegments next = staged_segments<kUnit>(e1, e2, my_quad, lrow);  // (empty behind the last block)
        lds_barrier();  // the previous block's gathers are done
        put_rows(cb0);
        lds_barrier();
        const int base = cb0 << 8;
        static_for(all_j, [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j < kShare / 2) {   // (early: their way is long, and a range of few rows has no last slots)
                ask_rows(2 * j, cb_next, last_next);
                ask_rows(2 * j + 1, cb_next, last_next);
            }
            if constexpr (j + kAheadJ < kStageJ) ask(std::integral_constant<int, j + kAheadJ>{}, now);
            else ask(std::integral_constant<int, j + kAheadJ - kStageJ>{}, next);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j % 2 == 0) __builtin_amdgcn_s_setprio(3 - j / 2);
            const int most = __builtin_amdgcn_readlane(now.most, j);
            if (most > 0) {
                uint32_t at = static_cast<uint32_t>(row_lane<j>(static_cast<int>(now.at)) + lig * kUnit);
                int left = row_lane<j>(now.left) - lig4;
                int off, off1;
                float w, w1;
                placed(held[j % kHeld][0], left > 0, base, off, w);
                placed(held[j % kHeld][1], left > 64, base, off1, w1);
                int n = most;
                // (a loop of its own, so that whatever it asks for has come at its end, and the loop after it waits for no memory)
                for (; n > 32; n -= 16, at += 16 * kUnit, left -= 64) {
                    const Chunk c2 = load_chunk(at, left, 32);
                    staged_steps<0, 16>(lds, off, w, acc[j]);
                    off = off1;
                    w = w1;
                    placed(c2, left > 128, base, off1, w1);
                }
                for (;;) {
                    staged_half<0>(lds, n, off, w, acc[j]);
                    if (n > 8) staged_half<8>(lds, n - 8, off, w, acc[j]);
                    n -= 16;
                    if (n <= 0) break;
                    off = off1;
                    w = w1;
                }
            }
        });
        now = next;
        e1 = e2;
        e2 = e3;
    }
    static_for(all_j, [&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int slot_row = row_lane<j>(my_row);
        const bool quad = slot_row >= 0 && (slot_row & kStageQuad);
        const int row = slot_row < 0 ? -1 : (slot_row & ~kStageQuad);
        if (j < n_j && __builtin_amdgcn_readfirstlane(quad)) {
            // the four lane rows hold a quarter of the row's sum each: (0 + 1) + (2 + 3), in every lane row
            acc[j].x += __shfl_xor(acc[j].x, 16); acc[j].y += __shfl_xor(acc[j].y, 16);
            acc[j].z += __shfl_xor(acc[j].z, 16); acc[j].w += __shfl_xor(acc[j].w, 16);
            acc[j].x += __shfl_xor(acc[j].x, 32); acc[j].y += __shfl_xor(acc[j].y, 32);
            acc[j].z += __shfl_xor(acc[j].z, 32); acc[j].w += __shfl_xor(acc[j].w, 32);
        }
        if (j < n_j && row >= 0 && col_on && (!quad || lrow == 0)) {
            const float bb = a.bias ? a.bias[row] : 0.f;
            float4 r = make_float4(acc[j].x + bb, acc[j].y + bb, acc[j].z + bb, acc[j].w + bb);
            if (a.relu) r = make_float4(r.x > 0.f ? r.x : 0.f, r.y > 0.f ? r.y : 0.f, r.z > 0.f ? r.z : 0.f, r.w > 0.f ? r.w : 0.f);
            if (a.YM) r = keep_where_positive(r, ld4(a.YM + static_cast<int64_t>(row) * a.ldym + col));
            st4(a.Y + static_cast<int64_t>(row) * a.ldy + col, r);
        }
    });
}

// ---- product out of LDS in strips of 16 columns ------------------------------------------------------
// The staged product in narrower tiles, for even rows of some 20 to some hundred entries a block at wide batches: a strip of kStripCols columns
// leaves room for kStripRows operand rows at a time (128 KiB), four times as many as there, so that segments are four times as long and the operand
// is copied by a quarter of the work-groups.  A quad of lanes serves a row (four columns a lane), a wave a set of sixteen rows, and an entry reaches
// the lanes of its quad by DPP quad_perm.  What all strips of a product have in common is done once, by strip_stream_kernel: it writes every entry as
// the LDS offset of its operand row and its weight, in the order in which the waves take them, segments as long as the longest of the set, so that
// the product has nothing to look up and nothing to mask (with its entries as they are stored, masked by every strip, 80 vector instructions a chunk:
// 371 us for the first matrix below, 92 for the second).  What bounds it: LDS and vector ALUs together, 4.2 ns a gather (62 TB/s; rows of 64 bytes
// meet in a bank group one time in four), of which 0.7 to 0.97 carry an entry (strip_plan in structure.hip); around them a launch, 4.4 us until the
// first block is there, and 1 to 3 us a block for the last wave of it: the waves' priorities fall as they go through their sets, so that who is
// behind goes first (270 -> 257, 62 -> 58).  Results are stored as the last block completes them, under the gathers of the sets that follow (49 ->
// 47).  Forward products at batch 1024, stream included, gathered from the L2s (staged: *) -> in strips: 16384^2 at 1 % 456* -> 245, at 0.3 % 198 ->
// 133; 8192^2 at 0.74 % 93 -> 58; 8192 x 3072 at 1.4 % 59 -> 41; 5818 x 7889 at 1.6 %, batch 806 131* -> 63.
constexpr int kStripJ = 8, kStripWaves = kWavesPerBlock;
constexpr int kStripZeroRow = kStripRows * kStripCols * 4;   // as kStageZeroRow
static_assert(kStripCols * 4 == 1 << 6 && kStripSet * 4 == kWave && kStripChunk == 8, "");

// Chunk c of a segment: lane 4 q + l of the wave holds entries 8 c + 2 l and the next of row q, {offset, weight} each.  A wave per segment, a matrix per blockIdx.y.
constexpr int kStripStreamWaves = 4;
__global__ __launch_bounds__(kStripStreamWaves * kWave) void strip_stream_kernel(const StripStreams list)
{
    const StripStream &m = list.of[blockIdx.y];
    const int at = blockIdx.x * kStripStreamWaves + wave_in_block();
    if (at >= m.sets * m.blocks) return;
    const int set = at / m.blocks, b = at - set * m.blocks;
    const int lane = threadIdx.x & (kWave - 1);
    const int2 seg = m.segs[at];
    const int32_t *cuts = m.cuts + (static_cast<int64_t>(set) * (m.blocks + 1) + b) * kStripSet + (lane >> 2);
    const int lo = cuts[0], hi = cuts[kStripSet], base = strip_block_base(b, m.block_rows, m.x_rows);
    float4 *out = m.out + static_cast<int64_t>(seg.x) * kWave + lane;
#pragma unroll 4
    for (int e = 0; e < seg.y; e += kStripChunk, out += kWave) {
        const int p = lo + e + (lane & 3) * 2, p0 = min(p, m.nnz - 1), p1 = min(p + 1, m.nnz - 1);
        const int j0 = m.indices[p0], j1 = m.indices[p1];
        const float w0 = m.values[p0], w1 = m.values[p1];
        *out = make_float4(__builtin_bit_cast(float, p < hi ? (j0 - base) * (kStripCols * 4) : kStripZeroRow), p < hi ? w0 : 0.f,
                           __builtin_bit_cast(float, p + 1 < hi ? (j1 - base) * (kStripCols * 4) : kStripZeroRow), p + 1 < hi ? w1 : 0.f);
    }
}

// every lane of a quad receives the value of the quad's lane I
template <int I>
__device__ __forceinline__ int quad_lane(int v) { return __builtin_amdgcn_update_dpp(0, v, I * 0x55, 0xF, 0xF, true); }
// acc += w of the quad's lane I times x (see fma_row_lane)
template <int I>
__device__ __forceinline__ void fma_quad_lane(float4 &acc, float w, const float4 &x)
{
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %4, %5 quad_perm:[%9,%9,%9,%9] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %4, %6 quad_perm:[%9,%9,%9,%9] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %4, %7 quad_perm:[%9,%9,%9,%9] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %4, %8 quad_perm:[%9,%9,%9,%9] row_mask:0xf bank_mask:0xf"
        : "+&v"(acc.x), "+&v"(acc.y), "+&v"(acc.z), "+&v"(acc.w)
        : "v"(w), "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w), "n"(I));
}
// Entries B .. B + N - 1 of a chunk of every quad, in that order, four gathers ahead of the one whose products are added.
template <int B, int N>
__device__ __forceinline__ void strip_steps(const char *lds, const float4 &c, float4 &acc)
{
    constexpr int kAhead = N < 4 ? N : 4;
    float4 x[N];
    auto gather = [&](auto ic) {
        constexpr int i = decltype(ic)::value, e = B + i;
        x[i] = *reinterpret_cast<const float4 *>(lds + quad_lane<e / 2>(__builtin_bit_cast(int, e & 1 ? c.z : c.x)));
    };
    static_for(std::make_integer_sequence<int, kAhead>{}, gather);
    __builtin_amdgcn_sched_barrier(0);
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value, e = B + i;
        if constexpr (i + kAhead < N) gather(std::integral_constant<int, i + kAhead>{});
        fma_quad_lane<e / 2>(acc, e & 1 ? c.w : c.y, x[i]);
        if constexpr (i + kAhead < N) __builtin_amdgcn_sched_barrier(0);
    });
}

struct StripGrid {
    int n_tiles, n_ranges, per;     // strips, ranges of sets, an eighth of the grid
};
__global__ __launch_bounds__(kStripWaves * kWave) void spmm_strip_kernel(const SpmmArgs a, const StripGrid g, const Strips f, const float4 *const strip_stream)
{
    __shared__ float4 strip[kStripRows * kStripCols / 4 + kStripCols / 4];  // the block, then one row of zeros
    // (neighbouring tiles share lines of the operand, all ranges of a tile its rows: a run of the list of both to an XCD)
    const int at_block = static_cast<int>(blockIdx.x & 7) * g.per + static_cast<int>(blockIdx.x >> 3);
    const int tile = at_block / g.n_ranges, range = at_block - tile * g.n_ranges;
    if (tile >= g.n_tiles) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int lig = lane & 3, lig4 = lig * 4;
    const bool col_on = tile * kStripCols + lig4 < a.batch;
    const int col = four_columns(tile * kStripCols + lig4, a.batch);
    const char *lds = reinterpret_cast<const char *>(strip) + lig * 16;
    if (threadIdx.x < kStripCols / 4) strip[kStripRows * kStripCols / 4 + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);  // (visible after the first barrier)
    constexpr auto all_j = std::make_integer_sequence<int, kStripJ>{};
    // Set J of the wave (longest first, dealt there and back); lane J keeps its segment, block after block.
    const int n_sets = (a.rows + kStripSet - 1) / kStripSet, round = kStripWaves * g.n_ranges, mine = wv * g.n_ranges + range, n_blocks = f.blocks;
    auto set_of = [&](int j) { return j * round + (j & 1 ? round - 1 - mine : mine); };
    const int my_set = set_of(lane & (kStripJ - 1));
    const int2 *my_segs = f.segs + static_cast<int64_t>(my_set) * n_blocks;
    auto segment = [&](int b) { return b < n_blocks && my_set < n_sets ? my_segs[b] : make_int2(0, 0); };
    float4 acc[kStripJ];
    static_for(all_j, [&](auto jc) { acc[decltype(jc)::value] = make_float4(0.f, 0.f, 0.f, 0.f); });
    // the first two chunks of a segment are asked for a set ahead (of an empty one or a short one, others', which nothing is done with)
    const float4 *stream = strip_stream + lane;
    float4 held[2][2];
    auto ask = [&](auto jc, const int2 &s) {
        constexpr int j = decltype(jc)::value;
        const float4 *p = stream + static_cast<int64_t>(__builtin_amdgcn_readlane(s.x, j)) * kWave;
        held[j % 2][0] = p[0];
        held[j % 2][1] = p[kWave];
    };
    // operand rows on their way to LDS: thread t holds four columns of rows t / 4, t / 4 + 256, ... of a block (see spmm_staged_kernel)
    constexpr int kShare = kStripRows / 256;
    float4 v[kShare];
    const float *const my_x = a.X + static_cast<int64_t>(threadIdx.x >> 2) * a.ldx + col;
    const int last_rows = a.x_rows - 256, last_i = (f.block_rows >> 8) - 1;
    auto ask_rows = [&](int i, int cb0, int last) { v[i] = ld4(my_x + static_cast<int64_t>(min(cb0 + min(i, last_i) * 256, last)) * a.ldx); };
    auto put_rows = [&](int cb0) {
#pragma unroll
        for (int i = 0; i < kShare; ++i) strip[(min(cb0 + min(i, last_i) * 256, last_rows) - cb0) * 4 + static_cast<int>(threadIdx.x)] = v[i];
    };
    int2 now = segment(0), next = segment(1);
#pragma unroll
    for (int i = 0; i < kShare; ++i) ask_rows(i, 0, last_rows);
    ask(std::integral_constant<int, 0>{}, now);
    // the wave's segments of a block, the next block's rows asked for beside them; of the last block with what is done to a row once it is complete
    auto serve = [&](int b, auto last_one) {
        constexpr bool last = decltype(last_one)::value;
        const int cb0 = strip_block_base(b, f.block_rows, a.x_rows), cb_next = strip_block_base(b + 1, f.block_rows, a.x_rows);
        const int2 after = segment(b + 2);
        int row[kStripJ / 4];     // lane k of a quad: of sets k, k + 4
        float bias[kStripJ / 4];
        lds_barrier();  // the previous block's gathers are done
        put_rows(cb0);
        if constexpr (last)
#pragma unroll
            for (int k = 0; k < kStripJ / 4; ++k) {
                const int set = set_of(k * 4 + lig);
                row[k] = set < n_sets ? f.rows[set * kStripSet + (lane >> 2)] : -1;
                bias[k] = a.bias ? a.bias[max(row[k], 0)] : 0.f;
            }
        lds_barrier();
        static_for(all_j, [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (!last && j < kShare / 2) {
                ask_rows(2 * j, cb_next, last_rows);
                ask_rows(2 * j + 1, cb_next, last_rows);
            }
            if constexpr (j + 1 < kStripJ) ask(std::integral_constant<int, j + 1>{}, now);
            else if constexpr (!last) ask(std::integral_constant<int, 0>{}, next);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j % 2 == 0) __builtin_amdgcn_s_setprio(3 - j / 2);   // (whoever is behind goes first)
            int n = __builtin_amdgcn_readlane(now.y, j);
            if (n > 0) {
                float4 c = held[j % 2][0], d = held[j % 2][1];
                const float4 *p = stream + static_cast<int64_t>(__builtin_amdgcn_readlane(now.x, j)) * kWave + 2 * kWave;
                for (; n > 16; n -= 8, p += kWave) {
                    const float4 e = *p;
                    strip_steps<0, 8>(lds, c, acc[j]);
                    c = d;
                    d = e;
                }
                if (n > 8) {
                    strip_steps<0, 8>(lds, c, acc[j]);
                    c = d;
                    n -= 8;
                }
                // (one if after the other: see staged_half)
                int ways = n > 6 ? 1 : n > 4 ? 6 : n > 2 ? 2 : 8;
                asm("" : "+s"(ways));
                if (ways & 1) strip_steps<0, 8>(lds, c, acc[j]);
                if (ways & 2) strip_steps<0, 4>(lds, c, acc[j]);
                if (ways & 4) strip_steps<4, 2>(lds, c, acc[j]);
                if (ways & 8) strip_steps<0, 2>(lds, c, acc[j]);
            }
            if constexpr (last) {
                const int r = quad_lane<j % 4>(row[j / 4]);
                const float bb = __builtin_bit_cast(float, quad_lane<j % 4>(__builtin_bit_cast(int, bias[j / 4])));   // (all lanes: moves read from active ones only)
                if (r >= 0 && col_on) {
                    float4 y = make_float4(acc[j].x + bb, acc[j].y + bb, acc[j].z + bb, acc[j].w + bb);
                    if (a.relu) y = make_float4(y.x > 0.f ? y.x : 0.f, y.y > 0.f ? y.y : 0.f, y.z > 0.f ? y.z : 0.f, y.w > 0.f ? y.w : 0.f);
                    if (a.YM) y = keep_where_positive(y, ld4(a.YM + static_cast<int64_t>(r) * a.ldym + col));
                    st4(a.Y + static_cast<int64_t>(r) * a.ldy + col, y);
                }
            }
        });
        now = next;
        next = after;
    };
    for (int b = 0; b + 1 < n_blocks; ++b) serve(b, std::false_type{});
    serve(n_blocks - 1, std::true_type{});
}

// ---------------------------------------------------------------------------------------
// SDDMM.  The row of dZ stays in registers; the wave is cut into 64/G groups of G lanes, each
// group computing the dot product of one stored entry at a time (lanes along the batch, 4
// columns per lane and tile, NV tiles: G*4*NV >= batch; 4096^2 at 10 % and batch 16 / 32: 21.0 us in groups of 16, 12.9 / 14.7 in
// groups of 4 / 8), reduced inside the group with DPP
// moves.  Results of up to 64 consecutive entries are collected one per lane, so the store of
// g -- or the fused momentum step on values/velocity -- is a coalesced access.
// Lanes whose columns lie beyond the batch hold dZ = 0 and re-read the row's first columns.  SPARE: there are such lanes, or lanes
// that share columns; a result that is NaN, which an Inf there would make it, is formed again from every lane's own columns
// (asked once per 64 entries; dropping the gathered side of every entry instead takes four selects beside its four multiply-adds).
// ---------------------------------------------------------------------------------------
// By-product carried by an SDDMM launch: the mean of the per-column losses the head kernel left.
__device__ __forceinline__ void mean_loss_task(const SddmmArgs &a, int block)
{
    if (a.loss_cols && block == 0 && wave_in_block() == 0) mean_of(a.loss_cols, a.loss_n, a.loss_out);  // wave-uniform
}

// One pass of the SDDMM over U stored entries per group: every index move, then every gather,
// then the dot products and their reductions.  Straight-line, so that all U*NV gathers stay in
// flight (see grouped_pass).  Group `grp` works on slot it*NG+grp of the chunk in iteration it;
// that slot's row offset sits in lane grp*G+it, and its result is kept by the lane with lig == it.
template <int G, int NV, int U>
__device__ __forceinline__ void sddmm_pass(gmem_ptr Xg, int it0, int my_ro, const uint32_t (&off)[NV],
                                           const float4 (&dz)[NV], float &res)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int lig = lane % G;
    uint32_t ro[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (G == kWave)
            ro[u] = static_cast<uint32_t>(__builtin_amdgcn_readlane(my_ro, it0 + u));
        else
            ro[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(((lane / G) * G + it0 + u) * 4, my_ro));
    }
    float4 x[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < NV; ++t) x[u][t] = gload4(Xg, ro[u] + off[t]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            part = fmaf(dz[t].x, x[u][t].x, part);
            part = fmaf(dz[t].y, x[u][t].y, part);
            part = fmaf(dz[t].z, x[u][t].z, part);
            part = fmaf(dz[t].w, x[u][t].w, part);
        }
        part = group_sum<G>(part);
        if (lig == it0 + u) res = part;
    }
}

// The results of `iters` such iterations from every lane's own columns alone (col0: first column of the pass).
template <int G, int NV>
__device__ __forceinline__ float sddmm_own_columns(gmem_ptr Xg, int iters, int my_ro, const uint32_t (&off)[NV], const float4 (&dz)[NV], int col0,
                                                   int batch)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int lig = lane % G;
    float res = 0.f;
#pragma unroll 1
    for (int it = 0; it < iters; ++it) {
        const uint32_t ro = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(((lane / G) * G + it) * 4, my_ro));
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            part = add_own_products(part, dz[t], gload4(Xg, ro + off[t]), col0 + (t * G + lig) * 4, static_cast<int>(off[t] >> 2), batch);
        }
        part = group_sum<G>(part);
        if (lig == it) res = part;
    }
    return res;
}

// col0: first column of the pass, which covers G*4*NV columns of the batch.  HELD: the wave's task and its row of dZ (without
// the columns that are not the lanes' own) are there already.
template <int G, int NV, bool SPARE, bool HELD = false, int W = kWavesPerBlock>
__device__ __forceinline__ void sddmm_body(const SddmmArgs &a, const int block, const int col0 = 0, const WaveTask *held_task = nullptr,
                                           const float4 *held_dz = nullptr)
{
    constexpr int NG = kWave / G;
    constexpr int UI = NV >= 3 ? 2 : (NV == 2 ? 4 : 8);   // 32 registers of gathered data: two 16-wave work-groups fit a compute unit
    const int lane = threadIdx.x & (kWave - 1);
    if constexpr (!HELD) mean_loss_task(a, block);
    WaveTask task;
    if constexpr (HELD) task = *held_task;
    else task = wave_task<W>(a.blocks, block);
    if (task.row < 0) return;
    const int row = task.row;
    const int grp = lane / G;
    const int lig = lane % G;

    // the row of dZ: all its loads together, whole waves (lanes beyond the batch re-read columns of the pass and are zeroed)
    float4 dz[NV];
    uint32_t off[NV];
    if constexpr (HELD) {
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const int own = col0 + (t * G + lig) * 4;
            off[t] = static_cast<uint32_t>(four_columns(own < a.batch ? own : col0, a.batch)) * 4u;
            dz[t] = held_dz[t];
        }
    } else {
        const gmem_ptr zr = as_gmem(a.dZ + static_cast<int64_t>(row) * a.lddz);
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const int own = col0 + (t * G + lig) * 4;
            off[t] = static_cast<uint32_t>(four_columns(own < a.batch ? own : col0, a.batch)) * 4u;
            dz[t] = gload4(zr, off[t]);
        }
        if (a.ZM) {
            const gmem_ptr zm = as_gmem(a.ZM + static_cast<int64_t>(row) * a.ldzm);
            float4 m[NV];
#pragma unroll
            for (int t = 0; t < NV; ++t) m[t] = gload4(zm, off[t]);
#pragma unroll
            for (int t = 0; t < NV; ++t) dz[t] = keep_where_positive(dz[t], m[t]);
        }
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const int own = col0 + (t * G + lig) * 4;
            dz[t] = own < a.batch ? drop_shared(dz[t], own, static_cast<int>(off[t] >> 2)) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }

    if (task.lead && (a.db || (a.fused && a.bias))) {
        float s = 0.f;
#pragma unroll
        for (int t = 0; t < NV; ++t) s += (dz[t].x + dz[t].y) + (dz[t].z + dz[t].w);
        s = group_sum<G>(s);
        if (lane == 0) {
            if (a.db) a.db[row] = s;
            if (a.fused && a.bias) {
                float w = a.bias[row], v = a.bias_velocity[row];
                momentum_step(w, v, s, a.lr, a.momentum, a.nesterov);
                a.bias[row] = w;
                a.bias_velocity[row] = v;
            }
        }
    }
    if (a.skip_products) return;

    const int s0 = task.s0;
    const int s1 = task.s1;
    const uint32_t ldxb = static_cast<uint32_t>(a.ldx) * 4u;
    const gmem_ptr Xg = as_gmem(a.X);
    const int q_mine = lig * NG + grp;  // slot of this lane inside a chunk of 64 entries
    const bool spare = SPARE && col0 + G * 4 * NV > a.batch;  // uniform

    for (int pc = s0; pc < s1; pc += kWave) {
        const int n = min(kWave, s1 - pc);
        const bool mine = q_mine < n;
        // lanes whose slot lies past the chunk's end work on its first entry and store nothing
        const int p = pc + (mine ? q_mine : 0);
        const int my_j = a.indices[p];
        // operands of the fused update travel together with the column index
        float w_old = 0.f, v_old = 0.f;
        int mirror_pos = 0;
        if (a.fused) {
            w_old = a.values[p];
            v_old = a.velocity[p];
            if (a.values_t) mirror_pos = a.pos_t[p];
        }
        const int my_ro = static_cast<int>(static_cast<uint32_t>(my_j) * ldxb);
        const int iters = (n + NG - 1) / NG;
        float res = 0.f;
        int it = 0;
        for (; it + UI <= iters; it += UI) sddmm_pass<G, NV, UI>(Xg, it, my_ro, off, dz, res);
        if constexpr (UI >= 8)
            if (it + 4 <= iters) { sddmm_pass<G, NV, 4>(Xg, it, my_ro, off, dz, res); it += 4; }
        if constexpr (UI >= 4)
            if (it + 2 <= iters) { sddmm_pass<G, NV, 2>(Xg, it, my_ro, off, dz, res); it += 2; }
        if (it < iters) sddmm_pass<G, NV, 1>(Xg, it, my_ro, off, dz, res);
        if (spare && __any(res != res)) res = sddmm_own_columns<G, NV>(Xg, iters, my_ro, off, dz, col0, a.batch);
        if (mine) {
            if (a.g) a.g[p] = res;
            if (a.fused) {
                momentum_step(w_old, v_old, res, a.lr, a.momentum, a.nesterov);
                a.values[p] = w_old;
                a.velocity[p] = v_old;
                if (a.values_t) a.values_t[mirror_pos] = w_old;
                if (a.dense) a.dense[static_cast<int64_t>(row) * a.dense_ld + my_j] = w_old;
            }
        }
    }
}

template <int G, int NV, bool SPARE>
__global__ __launch_bounds__(kBlock) void sddmm_kernel(const SddmmArgs a)
{
    sddmm_body<G, NV, SPARE>(a, blockIdx.x);
}

// Column-tiled SDDMM for operands X that no L2 holds: tile t covers columns [t*W, t*W + W), W = G*4*NV; a work-group computes the partial products of
// its rows over one tile and stores them (and the partial row sums of dZ) in the tile's slice of the partial buffer.  Tiles go to the XCDs as in
// spmm_tiled_kernel, so that an operand tile stays in one L2 while every entry gathers from it.  In work-groups of four waves, a quarter of one of
// the partition's (nothing is shared among them; see spmm_packed_only_kernel): of 16 / of 4 waves, weight gradients of 12000 x 5000 power-law at 0.5
// %, batch 300 / 450 / 700 30.0 / 30.4, 52.5 / 47.3, 74.8 / 66.2 us; 5000^2 at 1.2 % 28.0 / 28.0, 40.1 / 37.0, 56.0 / 51.1; 8192 x 3072 at 1.3 %,
// batch 700 / 1024 56.7 / 53.8, 68.3 / 67.1.
constexpr int kSddmmWaves = 4, kSddmmParts = kWavesPerBlock / kSddmmWaves;
template <int G, int NV, bool SPARE>
__device__ __forceinline__ void sddmm_tile(const SddmmArgs &a, int n_tiles, TileOrder order, uint32_t id)
{
    const int nrb = a.blocks.n_blocks * kSddmmParts;
    int tile, rb;
    if (!tile_of_block(n_tiles, nrb, order, tile, rb, id)) return;
    SddmmArgs t = a;
    t.fused = 0;
    t.g = a.partial + static_cast<int64_t>(tile) * a.partial_stride;
    t.db = t.g + a.partial_db_at;
    if (tile != 0) t.loss_cols = nullptr;
    sddmm_body<G, NV, SPARE, false, kSddmmWaves>(t, rb, tile * (G * 4 * NV));
}
template <int G, int NV, bool SPARE>
__global__ __launch_bounds__(kSddmmWaves * kWave) __attribute__((amdgpu_waves_per_eu(8))) void sddmm_tiled_kernel(const SddmmArgs a, const int n_tiles, const TileOrder order)
{
    sddmm_tile<G, NV, SPARE>(a, n_tiles, order, blockIdx.x);
}

// ---- staged SDDMM --------------------------------------------------------------------------
// The SDDMM on the staged product's plan: same ranges, tiles, column blocks and LDS copy of the
// operand; a lane row keeps the tile's 64 columns of dZ of its 8 rows in registers instead of
// results.  An entry's product is a dot product over the lane row: each lane multiplies its four
// columns, and up to 16 entries at a time are summed across the 16 lanes by a transposing butterfly
// (33 instructions per 16 entries instead of 6 per entry), after which lane i holds entry i's sum
// and the lane row stores 16 consecutive partial products.  Partial products and partial row
// sums of dZ go to the tile's slice of the partial buffer; sddmm_finish_kernel adds the tiles.
// What bounds it: the vector ALUs (8 instructions a gather of 4 x 64 columns: its address, four multiply-adds, the butterfly's share) beside the LDS.
// As in the product, segments worked out once per block, indices and the next block's rows brought ahead, 32-bit offsets; the butterfly under bank
// masks, and as short as the segment's end.  Weight gradient with its second pass, batch 1024: uniform 8192^2 at 5 % 580 -> 414 us, 16384^2 at 2 / 10 %
// 1261 -> 840 and 3425 -> 2483, power-law 16384^2 at 10 % (dense rows apart) 2292 -> 1776; 5000 x 7000 at 8 %, batch 511: 213 -> 175.  Same bits.
// d[i] is this lane's share of value i < N; returns, in lane i of every row of 16 lanes, the sum of
// the 16 lanes' d[i] (in lanes N and up nothing of use).  Fixed pairing: lane l with l^8, l^7, l^2, l^1 in turn.  The first two levels add under a bank
// mask, the lanes of one value and then those of the other, which needs no selects; in one piece, as an operand moved between lanes is there two
// instructions after it is written.
template <int N>
__device__ __forceinline__ float row16_transpose_sum(float (&d)[16], int lig)
{
    static_assert(N == 4 || N == 8 || N == 12 || N == 16, "");
#define NERVA_ADD8(a, b, banks) "v_add_f32_dpp %" #a ", %" #b ", %" #b " row_ror:8 row_mask:0xf bank_mask:" banks "\n\t"
#define NERVA_ADD4(a, b, banks) "v_add_f32_dpp %" #a ", %" #b ", %" #b " row_half_mirror row_mask:0xf bank_mask:" banks "\n\t"
    if constexpr (N == 16)
        asm("s_nop 1\n\t"
            NERVA_ADD8(0, 0, "0x3") NERVA_ADD8(0, 8, "0xc") NERVA_ADD8(1, 1, "0x3") NERVA_ADD8(1, 9, "0xc")
            NERVA_ADD8(2, 2, "0x3") NERVA_ADD8(2, 10, "0xc") NERVA_ADD8(3, 3, "0x3") NERVA_ADD8(3, 11, "0xc")
            NERVA_ADD8(4, 4, "0x3") NERVA_ADD8(4, 12, "0xc") NERVA_ADD8(5, 5, "0x3") NERVA_ADD8(5, 13, "0xc")
            NERVA_ADD8(6, 6, "0x3") NERVA_ADD8(6, 14, "0xc") NERVA_ADD8(7, 7, "0x3") NERVA_ADD8(7, 15, "0xc")
            NERVA_ADD4(0, 0, "0x5") NERVA_ADD4(0, 4, "0xa") NERVA_ADD4(1, 1, "0x5") NERVA_ADD4(1, 5, "0xa")
            NERVA_ADD4(2, 2, "0x5") NERVA_ADD4(2, 6, "0xa") NERVA_ADD4(3, 3, "0x5") NERVA_ADD4(3, 7, "0xa")
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4]), "+&v"(d[5]), "+&v"(d[6]), "+&v"(d[7])
            : "v"(d[8]), "v"(d[9]), "v"(d[10]), "v"(d[11]), "v"(d[12]), "v"(d[13]), "v"(d[14]), "v"(d[15]));
    else if constexpr (N == 12)
        asm("s_nop 1\n\t"
            NERVA_ADD8(0, 0, "0x3") NERVA_ADD8(0, 8, "0xc") NERVA_ADD8(1, 1, "0x3") NERVA_ADD8(1, 9, "0xc")
            NERVA_ADD8(2, 2, "0x3") NERVA_ADD8(2, 10, "0xc") NERVA_ADD8(3, 3, "0x3") NERVA_ADD8(3, 11, "0xc")
            NERVA_ADD8(4, 4, "0x3") NERVA_ADD8(5, 5, "0x3") NERVA_ADD8(6, 6, "0x3") NERVA_ADD8(7, 7, "0x3")
            NERVA_ADD4(0, 0, "0x5") NERVA_ADD4(0, 4, "0xa") NERVA_ADD4(1, 1, "0x5") NERVA_ADD4(1, 5, "0xa")
            NERVA_ADD4(2, 2, "0x5") NERVA_ADD4(2, 6, "0xa") NERVA_ADD4(3, 3, "0x5") NERVA_ADD4(3, 7, "0xa")
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4]), "+&v"(d[5]), "+&v"(d[6]), "+&v"(d[7])
            : "v"(d[8]), "v"(d[9]), "v"(d[10]), "v"(d[11]));
    else if constexpr (N == 8)
        asm("s_nop 1\n\t"
            NERVA_ADD8(0, 0, "0x3") NERVA_ADD8(1, 1, "0x3") NERVA_ADD8(2, 2, "0x3") NERVA_ADD8(3, 3, "0x3")
            NERVA_ADD8(4, 4, "0x3") NERVA_ADD8(5, 5, "0x3") NERVA_ADD8(6, 6, "0x3") NERVA_ADD8(7, 7, "0x3")
            NERVA_ADD4(0, 0, "0x5") NERVA_ADD4(0, 4, "0xa") NERVA_ADD4(1, 1, "0x5") NERVA_ADD4(1, 5, "0xa")
            NERVA_ADD4(2, 2, "0x5") NERVA_ADD4(2, 6, "0xa") NERVA_ADD4(3, 3, "0x5") NERVA_ADD4(3, 7, "0xa")
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]), "+&v"(d[4]), "+&v"(d[5]), "+&v"(d[6]), "+&v"(d[7]));
    else
        asm("s_nop 1\n\t"
            NERVA_ADD8(0, 0, "0x3") NERVA_ADD8(1, 1, "0x3") NERVA_ADD8(2, 2, "0x3") NERVA_ADD8(3, 3, "0x3")
            NERVA_ADD4(0, 0, "0x5") NERVA_ADD4(1, 1, "0x5") NERVA_ADD4(2, 2, "0x5") NERVA_ADD4(3, 3, "0x5")
            : "+&v"(d[0]), "+&v"(d[1]), "+&v"(d[2]), "+&v"(d[3]));
#undef NERVA_ADD8
#undef NERVA_ADD4
    const bool b1 = lig & 2, b0 = lig & 1;
    float g[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) g[k] = (b1 ? d[k + 2] : d[k]) + dpp<0x4E>(b1 ? d[k] : d[k + 2]);  // quad_perm [2,3,0,1]
    return (b0 ? g[1] : g[0]) + dpp<0xB1>(b0 ? g[0] : g[1]);                                      // quad_perm [1,0,3,2]
}

// The first N entries of every lane row, whose LDS byte offsets its lanes hold: their sums, in lane i entry i's.
template <int N>
__device__ __forceinline__ float staged_dots(const char *lds, int off, const float4 &z, int lig)
{
    constexpr int kAhead = 4;
    float4 x[N];
    float d[16];
    auto gather = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        x[i] = *reinterpret_cast<const float4 *>(lds + row_lane<i>(off));
    };
    static_for(std::make_integer_sequence<int, kAhead>{}, gather);
    __builtin_amdgcn_sched_barrier(0);
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i + kAhead < N) gather(std::integral_constant<int, i + kAhead>{});
        d[i] = fmaf(x[i].w, z.w, fmaf(x[i].z, z.z, fmaf(x[i].y, z.y, x[i].x * z.x)));
        if constexpr (i + kAhead < N) __builtin_amdgcn_sched_barrier(0);
    });
    return row16_transpose_sum<N>(d, lig);
}

__global__ __launch_bounds__(kStageWaves * kWave) void sddmm_staged_kernel(const SddmmArgs a, const int n_tiles)
{
    __shared__ float4 stage[kStageRows * kStageCols / 4];
    const int n_ranges = a.blocks.staged_ranges;
    int range, tile;
    staged_ids(n_ranges, n_tiles, range, tile);
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int lrow = lane >> 4, lig = lane & 15;
    const int own_col = tile * kStageCols + lig * 4;
    const bool col_on = own_col < a.batch;
    const int col = four_columns(own_col, a.batch);
    const char *lds = reinterpret_cast<const char *>(stage) + lig * 16;
    const int n_cb = a.blocks.staged_cblocks;
    const int my_slot = ((lig & (kStageJ - 1)) * kStageWaves + wv) * 4 + lrow;
    const int my_row = a.blocks.staged_rows[range * kStageRangeRows + my_slot];
    const bool my_quad = my_row >= 0 && (my_row & kStageQuad);
    const int n_j = a.blocks.staged_groups[range];
    const int32_t *ends = a.blocks.staged_ends + static_cast<int64_t>(range) * (n_cb + 1) * kStageRangeRows + my_slot;
    float *gp = a.partial + static_cast<int64_t>(tile) * a.partial_stride;
    constexpr auto all_j = std::make_integer_sequence<int, kStageJ>{};
    // the tile's columns of dZ for the lane row's rows, and their sums (the tile's share of db)
    float4 z[kStageJ];
    static_for(all_j, [&](auto jc) {
        constexpr int j = decltype(jc)::value;
        z[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j < n_j) {
            const int slot_row = row_lane<j>(my_row);
            const int row = slot_row < 0 ? -1 : (slot_row & ~kStageQuad);
            if (row >= 0 && col_on) {
                z[j] = ld4(a.dZ + static_cast<int64_t>(row) * a.lddz + col);
                if (a.ZM) z[j] = keep_where_positive(z[j], ld4(a.ZM + static_cast<int64_t>(row) * a.ldzm + col));
                z[j] = drop_shared(z[j], own_col, col);
            }
            const float sum = row16_sum((z[j].x + z[j].y) + (z[j].z + z[j].w));
            // (the four lane rows of a split row hold the same dZ: the first one reports it)
            if (row >= 0 && lig == 0 && (!(slot_row & kStageQuad) || lrow == 0)) gp[a.partial_db_at + row] = sum;
        }
    });
    // segments and chunks as in spmm_staged_kernel, without weights; a lane without an entry gathers from the block's first row, for a sum that is not stored
    const int lig4 = lig * 4;
    auto load_chunk = [&](uint32_t at, int left, int first) {
        return __builtin_bit_cast(int, gload1(as_gmem(a.indices), (left > first * 4 ? at : 0u) + static_cast<uint32_t>(first * 4)));
    };
    auto placed = [&](int index, bool on, int base) { return on ? (index << 8) - base : 0; };
    constexpr int kAheadJ = 2, kHeld = 4;
    static_assert(kStageJ % kHeld == 0 && kAheadJ < kHeld, "");
    int held[kHeld][2];
    auto ask = [&](auto jc, const StagedSegments &s) {
        constexpr int j = decltype(jc)::value;
        const uint32_t at = static_cast<uint32_t>(row_lane<j>(static_cast<int>(s.at)) + lig4);
        const int left = row_lane<j>(s.left) - lig4;
        held[j % kHeld][0] = load_chunk(at, left, 0);
        held[j % kHeld][1] = load_chunk(at, left, 16);
    };
    constexpr int kShare = kStageRows / 64;
    static_assert(kShare % 2 == 0 && kShare / 2 <= kStageJ, "two of them are asked for beside each slot");
    float4 v[kShare];
    const float *const my_x = a.X + static_cast<int64_t>(threadIdx.x >> 4) * a.ldx + col;
    const int last_block = max(a.x_rows - kStageRows, 0), last_rows = a.x_rows - 64;
    auto block_row = [&](int b) { return min(b * kStageRows, last_block); };
    auto ask_rows = [&](int i, int cb0, int last) { v[i] = ld4(my_x + static_cast<int64_t>(min(cb0 + i * 64, last)) * a.ldx); };
    auto put_rows = [&](int cb0) {
#pragma unroll
        for (int i = 0; i < kShare; ++i) {
            const int k = min(cb0 + i * 64, last_rows);
            stage[(k - cb0) * 16 + static_cast<int>(threadIdx.x)] = col_on ? drop_shared(v[i], own_col, col) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    int e1 = ends[kStageRangeRows];
    StagedSegments now = staged_segments(ends[0], e1, my_quad, lrow);
    int e2 = n_cb >= 2 ? ends[2 * kStageRangeRows] : e1;
    static_for(std::make_integer_sequence<int, kAheadJ>{}, [&](auto jc) { ask(jc, now); });
#pragma unroll
    for (int i = 0; i < kShare; ++i) ask_rows(i, 0, last_rows);
    for (int b = 0; b < n_cb; ++b) {
        const int cb0 = block_row(b), cb_next = block_row(b + 1), last_next = b + 1 < n_cb ? last_rows : 0;
        const int e3 = ends[min(b + 3, n_cb) * kStageRangeRows];
        const StagedSegments next = staged_segments(e1, e2, my_quad, lrow);  // (empty behind the last block)
        lds_barrier();  // the previous block's gathers are done
        put_rows(cb0);
        lds_barrier();
        const int base = cb0 << 8;
        static_for(all_j, [&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr (j < kShare / 2) {
                ask_rows(2 * j, cb_next, last_next);
                ask_rows(2 * j + 1, cb_next, last_next);
            }
            if constexpr (j + kAheadJ < kStageJ) ask(std::integral_constant<int, j + kAheadJ>{}, now);
            else ask(std::integral_constant<int, j + kAheadJ - kStageJ>{}, next);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (j % 2 == 0) __builtin_amdgcn_s_setprio(3 - j / 2);
            int n = __builtin_amdgcn_readlane(now.most, j);
            if (n > 0) {
                uint32_t at = static_cast<uint32_t>(row_lane<j>(static_cast<int>(now.at)) + lig4);
                int left = row_lane<j>(now.left) - lig4;
                int off = placed(held[j % kHeld][0], left > 0, base), off1 = placed(held[j % kHeld][1], left > 64, base);
                for (; n > 32; n -= 16, at += 64, left -= 64) {
                    const int c2 = load_chunk(at, left, 32);
                    const float sum = staged_dots<16>(lds, off, z[j], lig);
                    if (left > 0) gstore1(gp, at, sum);
                    off = off1;
                    off1 = placed(c2, left > 128, base);
                }
                for (;;) {
                    float sum;
                    if (n > 12) sum = staged_dots<16>(lds, off, z[j], lig);
                    else if (n > 8) sum = staged_dots<12>(lds, off, z[j], lig);
                    else if (n > 4) sum = staged_dots<8>(lds, off, z[j], lig);
                    else sum = staged_dots<4>(lds, off, z[j], lig);
                    if (left > 0) gstore1(gp, at, sum);
                    n -= 16;
                    if (n <= 0) break;
                    at += 64;
                    left -= 64;
                    off = off1;
                }
            }
        });
        now = next;
        e1 = e2;
        e2 = e3;
    }
}

// SDDMM of a full matrix of few rows (every entry stored, rows <= kFullMaxRows): dZ, a few rows,
// is copied into LDS once per work-group and X is streamed once, a wave per row of X: the lane
// multiplies its columns of the X row with the same columns of every dZ row, the row's `rows`
// products are summed over the wave by the transposing butterfly, and lane i stores (or applies the
// momentum step to) entry (i, row of X).  The first work-group also sums the rows of dZ for db.
// WITH_T: the layer's transposed product in the same pass -- row j of W^T is column j of the full matrix,
// the very entries this wave updates, and its result is masked by the row of X the wave holds:
//     dX[j, :] = (sum_i W(i, j) dZ[i, :]) * [X[j, :] > 0],  i ascending, the weights of the step's start
// (read before the update; no other wave touches column j).  X is read once for both.
template <bool WITH_T>
__global__ __launch_bounds__(kBlock) void full_sddmm_kernel(const SddmmArgs a, const int n_chunks, float *__restrict__ dX, const int lddx)
{
    extern __shared__ float4 dz_s[];  // [rows][n_chunks][kWave]
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int R = a.rows, K = a.x_rows;
    for (int idx = threadIdx.x; idx < R * n_chunks * kWave; idx += kBlock) {
        const int i = idx / (n_chunks * kWave), c4 = idx % (n_chunks * kWave);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c4 * 4 < a.batch) {
            const int c = four_columns(c4 * 4, a.batch);
            v = ld4(a.dZ + static_cast<int64_t>(i) * a.lddz + c);
            if (a.ZM) v = keep_where_positive(v, ld4(a.ZM + static_cast<int64_t>(i) * a.ldzm + c));
            v = drop_shared(v, c4 * 4, c);
        }
        dz_s[idx] = v;
    }
    __syncthreads();
    mean_loss_task(a, blockIdx.x);
    if (blockIdx.x == 0 && wv < R && (a.db || (a.fused && a.bias))) {
        float sum = 0.f;
        for (int ch = 0; ch < n_chunks; ++ch) {
            const float4 z = dz_s[(wv * n_chunks + ch) * kWave + lane];
            sum += (z.x + z.y) + (z.z + z.w);
        }
        sum = group_sum<kWave>(sum);
        if (lane == 0) {
            if (a.db) a.db[wv] = sum;
            if (a.fused && a.bias) {
                float w = a.bias[wv], v = a.bias_velocity[wv];
                momentum_step(w, v, sum, a.lr, a.momentum, a.nesterov);
                a.bias[wv] = w;
                a.bias_velocity[wv] = v;
            }
        }
    }
    for (int j = blockIdx.x * kWavesPerBlock + wv; j < K; j += gridDim.x * kWavesPerBlock) {
        float d[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) d[i] = 0.f;
        const float *xr = a.X + static_cast<int64_t>(j) * a.ldx;
        float w_own = 0.f;  // lane i: W(i, j)
        float below = 0.f;  // the lane's share of the row sum of dX[j, :]
        if constexpr (WITH_T)
            if (lane < R) w_own = a.values[static_cast<int64_t>(lane) * K + j];
        for (int ch = 0; ch < n_chunks; ++ch) {
            const int own = (ch * kWave + lane) * 4;
            const int col = four_columns(own, a.batch);
            const float4 x = own < a.batch ? drop_shared(ld4(xr + col), own, col) : make_float4(0.f, 0.f, 0.f, 0.f);
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < kFullMaxRows; ++i) {
                if (i < R) {  // uniform
                    const float4 z = dz_s[(i * n_chunks + ch) * kWave + lane];
                    d[i] = fmaf(x.w, z.w, fmaf(x.z, z.z, fmaf(x.y, z.y, fmaf(x.x, z.x, d[i]))));
                    if constexpr (WITH_T) {
                        const float wi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w_own), i));
                        t.x = fmaf(wi, z.x, t.x);
                        t.y = fmaf(wi, z.y, t.y);
                        t.z = fmaf(wi, z.z, t.z);
                        t.w = fmaf(wi, z.w, t.w);
                    }
                }
            }
            if constexpr (WITH_T) {
                const float4 o = keep_where_positive(t, x);  // (columns beyond the batch: x = 0, so o = 0)
                if (own < a.batch) st4(dX + static_cast<int64_t>(j) * lddx + col, o);  // (batch % 4 == 0: no columns are shared)
                below += (o.x + o.y) + (o.z + o.w);
            }
        }
        if constexpr (WITH_T) {
            if (a.below_bias) {  // uniform
                below = group_sum<kWave>(below);
                if (lane == 0) {
                    float w = a.below_bias[j], v = a.below_bias_velocity[j];
                    momentum_step(w, v, below, a.lr, a.momentum, a.nesterov);
                    a.below_bias[j] = w;
                    a.below_bias_velocity[j] = v;
                }
            }
        }
        // lane i of each row of 16 lanes gets that row's sum of product i; then the four rows: (0 + 1) + (2 + 3)
        float g = row16_transpose_sum<16>(d, lane & 15);
        g += __shfl_xor(g, 16);
        g += __shfl_xor(g, 32);
        if (lane < R) {
            const int64_t p = static_cast<int64_t>(lane) * K + j;
            if (a.g) a.g[p] = g;
            if (a.fused) {
                float w = WITH_T ? w_own : a.values[p], v = a.velocity[p];
                momentum_step(w, v, g, a.lr, a.momentum, a.nesterov);
                a.values[p] = w;
                a.velocity[p] = v;
                if (a.values_t) a.values_t[a.pos_t[p]] = w;
            }
        }
    }
}

// Second pass of the tiled SDDMM: adds the tiles' partial products in tile order, then stores the
// gradient or applies the fused momentum step (and the mirror scatter); the same for the biases.
// Rows that another launch serves (DenseRows) are runs of entries and left alone: `ahead` is the first listed row that does
// not end before the work-group's entries.
__global__ __launch_bounds__(kEwBlock) void sddmm_finish_kernel(const SddmmArgs a, const int n_tiles, const DenseRows dense,
                                                               const uint8_t *__restrict__ dense_flag)
{
    const int64_t stride = static_cast<int64_t>(blockDim.x) * gridDim.x;
    const bool skip = dense.n > 0;
    // (only where new weights go to the mirror: 26.8 M gradients alone 213 us in turn, 233 in runs)
    const XcdRun run = a.fused && a.values_t ? xcd_run(a.nnz, gridDim.x) : XcdRun{static_cast<int64_t>(blockIdx.x) * kEwBlock, a.nnz, stride};
    for (int64_t base = run.first; base < run.end; base += run.step) {
        const int64_t p = base + threadIdx.x;
        bool mine = p < run.end;
        if (skip) {
            int ahead = 0, hi = dense.n;
            while (ahead < hi) {
                const int mid = (ahead + hi) / 2;
                if (a.indptr[dense.list[mid] + 1] <= base)
                    ahead = mid + 1;
                else
                    hi = mid;
            }
            for (; ahead < dense.n; ++ahead) {   // uniform: one or two rows
                const int row = dense.list[ahead];
                const int from = a.indptr[row], to = a.indptr[row + 1];
                if (from >= base + static_cast<int>(blockDim.x)) break;
                mine = mine && !(p >= from && p < to);
            }
        }
        if (!mine) continue;
        float g = 0.f;
        int t = 0;
        for (; t + 8 <= n_tiles; t += 8) {  // eight loads in flight, added in tile order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = a.partial[static_cast<int64_t>(t + u) * a.partial_stride + p];
#pragma unroll
            for (int u = 0; u < 8; ++u) g += v[u];
        }
        for (; t < n_tiles; ++t) g += a.partial[static_cast<int64_t>(t) * a.partial_stride + p];
        if (a.g) a.g[p] = g;
        if (a.fused) {
            float w = a.values[p], v = a.velocity[p];
            momentum_step(w, v, g, a.lr, a.momentum, a.nesterov);
            a.values[p] = w;
            a.velocity[p] = v;
            if (a.values_t) a.values_t[a.pos_t[p]] = w;
        }
    }
    if (!(a.db || (a.fused && a.bias))) return;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.rows; i += stride) {
        if (skip && dense_flag[i]) continue;
        float s = 0.f;
        for (int t = 0; t < n_tiles; ++t) s += a.partial[static_cast<int64_t>(t) * a.partial_stride + a.partial_db_at + i];
        if (a.db) a.db[i] = s;
        if (a.fused && a.bias) {
            float w = a.bias[i], v = a.bias_velocity[i];
            momentum_step(w, v, s, a.lr, a.momentum, a.nesterov);
            a.bias[i] = w;
            a.bias_velocity[i] = v;
        }
    }
}

// ---- both gradients of a layer in one gather stream ---------------------------------------------
// The transposed product dX = W^T dZ and the SDDMM g = (dZ X^T) on W's pattern gather the same
// rows: taken in the mirror's order (row j of W^T, its entries i ascending), stored entry (i, j)
// needs dZ[i, :] for both.  One kernel walks the mirror like spmm_body_packed (one mirror row per
// group of GS lanes, inside column tiles), gathers dZ[i, tile] once and uses it twice:
//     acc[j, tile]        += values_t[q] * dZ[i, tile]
//     partial[tile][q]     = <dZ[i, tile], X[j, tile]>        (X[j, tile] is held by the lane group)
// and stores dX[j, tile] = acc * [X[j, tile] > 0] (the ReLU derivative of the layer below, whose
// output X is; a call on its own stores acc).  The per-tile partial products, in mirror order, are added in tile order by
// backward_finish_kernel, which stores the gradient or applies the momentum step through perm (mirror -> CSR position) and
// forms the bias gradient (row sums of dZ).  A single tile needs no second pass.  Where the mirror rows do not make enough
// waves several groups share a row.  What bounds it is the gathers, half of what the two products apart take: backward call
// on 16384^2 power-law rows at 1 %, batch 1024: 1088 -> 570 us (452 with the longest rows of dZ in LDS, backward_hot_kernel); uniform 8192^2 at 0.5 % / 5 %: 146 -> 91, 982 -> 648; at batch
// 32: 18.1 -> 10.8, 100 -> 68; 1000 x 1000 at 0.5 %, one launch instead of three: 13.5 -> 5.8.
constexpr int kBwdWaves = 4;  // waves per work-group: no sums across waves, and smaller groups schedule finer (measured on the wide MLP:
                              // 134 / 138 / 142 us with 4 / 8 / 16 waves; gather depth 4 instead of 8 and a register cap of 64 change nothing)

// Lanes may re-read columns that are not their own.  What they have gathered there is dropped by a bitwise and with a mask
// of all ones or zeros; of the result they store their own columns.  One tile without / with: the 1585-521 layer in a step of
// 355-1585-521-1999-10 at 32 %, batch 66, 19.0 / 18.9 us; 713 x 2042 at 6.6 %, batch 36, 6.2 / 5.7; 15969 x 11666 at 0.6 %, batch 51, 29.5 / 32.3;
// 64-column tiles, 14024 x 5061 at 0.3 %, batch 845, 79.5 / 79.4.  (Forming a NaN result again, as sddmm_body does, takes registers
// of the pass itself: the first of these 23.1.)  In tiles, where batches are multiples of 4 and lanes have all four columns or
// none, masking the product alone leaves the registers as they are: 7413 x 4010 at 0.5 %, batch 212, 17.4 without, 18.3 with four masks, 17.7 with one.
enum BackwardSpare { kSpareNone, kSpareLanes, kSpareColumns };
__device__ __forceinline__ float keep_bits(float x, uint32_t mask) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & mask); }
// APART: every gather before the first product, which the compiler else mixes to save registers, with two or three in flight.  One tile on 4096 x 3072 at
// 5 %, batch 128: 25.3 -> 23.4 us; column tiles lose with fewer waves (wide MLP 97.3 -> 99.2), and masked gathers take too many registers.  One tile loses as well
// where its waves are more than fit at once with that many registers (backward_gathers_apart).
template <int U, int GS, bool XMASK, BackwardSpare SPARE, bool APART>
__device__ __forceinline__ void bwd_pass(gmem_ptr Zg, gmem_ptr Mg, int src, int my_ro, int my_mo, float my_w, uint32_t off, const float4 &ax,
                                         const uint32_t (&own)[4], int it0, int lig, float (&acc)[4], float &res)
{
    uint32_t ro[U], mo[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        ro[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src + u * 4, my_ro));
        if constexpr (XMASK) mo[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src + u * 4, my_mo));
        w[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src + u * 4, __builtin_bit_cast(int, my_w)));
    }
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = gload4(Zg, ro[u] + off);
    if constexpr (XMASK) {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = keep_where_positive(x[u], gload4(Mg, mo[u] + off));
    }
    if constexpr (APART) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if constexpr (SPARE == kSpareColumns) x[u] = make_float4(keep_bits(x[u].x, own[0]), keep_bits(x[u].y, own[1]), keep_bits(x[u].z, own[2]), keep_bits(x[u].w, own[3]));
        acc[0] = fmaf(w[u], x[u].x, acc[0]);
        acc[1] = fmaf(w[u], x[u].y, acc[1]);
        acc[2] = fmaf(w[u], x[u].z, acc[2]);
        acc[3] = fmaf(w[u], x[u].w, acc[3]);
        float part = fmaf(ax.w, x[u].w, fmaf(ax.z, x[u].z, fmaf(ax.y, x[u].y, ax.x * x[u].x)));
        if constexpr (SPARE == kSpareLanes) part = keep_bits(part, own[3]);
        part = group_sum<GS>(part);
        res = lig == it0 + u ? part : res;
    }
}

// The same for one tile in groups of 16 or 32 lanes: a chunk is sixteen entries, one in each lane of every sixteen, n of them (or one more) used.  The weight is moved between lanes in
// the multiply-add, and the products are added up across the lanes sixteen at a time: 11 vector instructions a gather where bwd_pass has 17 and three moves through the LDS crossbar.
// Figures are at bwd_sixteens.
template <int GS>
__device__ __forceinline__ float bwd_chunk(gmem_ptr Zg, int n, int ro, float w, uint32_t off, const float4 &ax, float4 &acc, int lig)
{
    float d[16];
    auto pass = [&](auto first, auto count) {
        constexpr int B = decltype(first)::value, N = decltype(count)::value;
        float4 x[N];
        static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
            constexpr int i = decltype(ic)::value;
            x[i] = gload4(Zg, static_cast<uint32_t>(row_lane<B + i>(ro)) + off);
        });
        static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (i + 1 < N || n > B + i) fma_row_lane<B + i>(acc, w, x[i]);   // (uniform; the one more may hold an infinity)
            float part = fmaf(x[i].w, ax.w, fmaf(x[i].z, ax.z, fmaf(x[i].y, ax.y, x[i].x * ax.x)));
            d[B + i] = part;
        });
    };
    using std::integral_constant;
    auto half = [&](auto first, int m) {
        constexpr int B = decltype(first)::value;
        int ways = m > 6 ? 1 : m > 4 ? 6 : m > 2 ? 2 : 8;   // (one if after the other: see staged_half)
        asm("" : "+s"(ways));
        if (ways & 1) pass(first, integral_constant<int, 8>{});
        if (ways & 2) pass(first, integral_constant<int, 4>{});
        if (ways & 4) pass(integral_constant<int, B + 4>{}, integral_constant<int, 2>{});
        if (ways & 8) pass(first, integral_constant<int, 2>{});
    };
    half(integral_constant<int, 0>{}, n);
    float res;
    if (n > 8) {
        half(integral_constant<int, 8>{}, n - 8);
        res = row16_transpose_sum<16>(d, lig);
    } else {
        res = row16_transpose_sum<8>(d, lig);
    }
    if constexpr (GS == 32) res += __shfl_xor(res, 16, kWave);
    return res;
}

// Sums of the rows of dZ, a wave per row: the bias gradient, stored or applied.
__device__ __forceinline__ void backward_row_sums(const BackwardArgs &a, int64_t wave, int64_t n_waves)
{
    const int lane = threadIdx.x & (kWave - 1);
    for (int64_t i = wave; i < a.x_rows; i += n_waves) {
        const float *zr = a.dZ + i * a.lddz;
        float s = 0.f;
        for (int c = lane * 4; c < a.batch; c += kWave * 4) {
            const int first = four_columns(c, a.batch);
            float4 z = ld4(zr + first);
            if (a.ZM) z = keep_where_positive(z, ld4(a.ZM + i * a.ldzm + first));
            z = drop_shared(z, c, first);
            s += (z.x + z.y) + (z.z + z.w);
        }
        s = group_sum<kWave>(s);
        if (lane == 0) {
            if (a.db) a.db[i] = s;
            if (a.fused && a.bias) {
                float w = a.bias[i], v = a.bias_velocity[i];
                momentum_step(w, v, s, a.lr, a.momentum, a.nesterov);
                a.bias[i] = w;
                a.bias_velocity[i] = v;
            }
        }
    }
}

// Otherwise than in kBackwardTiles there is no second pass -- the products are whole and are stored as the gradient by the work-groups that form them, and
// the work-groups after those of the rows sum the rows of dZ.  For a single column tile, or where the rows are no longer than
// the lane groups and the matrix is small: then a wave takes its entries through all tiles.  XMASK: dZ is dY times
// [Y > 0], gathered from both.
enum BackwardPass { kBackwardTiles, kBackwardOneTile, kBackwardLooped };
// SIXTEENS: bwd_chunk instead of bwd_pass, where the gathers would be APART.
template <int GS, bool SIXTEENS, BackwardPass PASS, bool XMASK, BackwardSpare SPARE, bool APART>
__global__ __launch_bounds__(kBwdWaves * kWave) void backward_fused_kernel(const BackwardArgs a, const int n_tiles, const TileOrder order,
                                                                          const int n_pack_blocks, const int lg_split)
{
    constexpr bool ONE = PASS != kBackwardTiles, LOOPED = PASS == kBackwardLooped;
    if (ONE && static_cast<int>(blockIdx.x) >= n_pack_blocks) {
        backward_row_sums(a, static_cast<int64_t>(blockIdx.x - n_pack_blocks) * kBwdWaves + wave_in_block(),
                          static_cast<int64_t>(gridDim.x - n_pack_blocks) * kBwdWaves);
        return;
    }
    int tile, rb;
    if constexpr (ONE) {
        tile = 0;
        rb = blockIdx.x;
        if (n_tiles <= 0) return;   // (never; the loop over all tiles takes 10 to 20 registers more where it might not run: 5000^2 at 0.1 %, batch 260 9.4 -> 11.6 us)
    } else {
        if (!tile_of_block(n_tiles, n_pack_blocks, order, tile, rb)) return;
    }
    constexpr int NE = kWave / GS;
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    const int grp = lane / GS;
    const int lig = lane % GS;
    constexpr int CH = SIXTEENS ? 16 : GS;   // entries of a row in a chunk; lane lig % CH has its one
    const int mine = lig % CH;
    const uint32_t ldzb = static_cast<uint32_t>(a.lddz) * 4u, ldmb = XMASK ? static_cast<uint32_t>(a.ldzm) * 4u : 0u;
    const gmem_ptr Zg = as_gmem(a.dZ), Mg = as_gmem(a.ZM);
    const int per_set = NE >> lg_split, part = grp & ((1 << lg_split) - 1);   // rows per wave; the group's share of its row
    const int n_sets = (a.rows + per_set - 1) / per_set;
    const int src0 = grp * GS * 4;
    const int n_waves = n_pack_blocks * kBwdWaves;
    const int first_set = rb * kBwdWaves + wv;
    if (first_set >= n_sets) return;  // wave-uniform
    float *gp = ONE ? nullptr : a.partial + static_cast<int64_t>(tile) * a.partial_stride;

    auto fetch = [&](int s0, int len, int base, int &j, float &w, int &at, float &v) {  // as in spmm_body_packed
        const int e = base + part * CH + mine;
        const bool ok = e < len;
        const int p = len > 0 ? s0 + (ok ? e : 0) : 0;
        j = a.indices[p];
        if (ONE || a.refresh) at = a.perm[p];
        if (a.refresh) {   // uniform
            w = a.refresh[at];
            if (ok && (ONE || tile == 0) && lig < CH) a.w_t[p] = w;
        } else {
            w = a.values[p];
        }
        if (ONE && a.fused) v = a.velocity[at];
        w = ok ? w : 0.f;
    };

    for (int set = first_set; set < n_sets; set += n_waves) {
        const int4 d = a.blocks.rows_by_length[set * per_set + (grp >> lg_split)];  // the table is padded to whole sets
        const int row = d.x, s0 = d.y, len = d.z;
        const int maxlen = __builtin_amdgcn_readfirstlane(len);  // group 0 holds the set's longest row
        float whole = 0.f;   // the lane's product over all tiles
        for (int tile_now = tile; tile_now < (LOOPED ? n_tiles : tile + 1); ++tile_now) {
                const int col0 = tile_now * GS * 4, own_col = col0 + lig * 4;
                const bool on = own_col < a.batch;
                const int col = four_columns(on ? own_col : col0, a.batch);
                const uint32_t off = static_cast<uint32_t>(col) * 4u;
                // the group's row of X: the second operand of its entries' products, and the mask of its result;
                // lanes beyond the batch hold zeros, so that the columns they re-read add nothing to a product
                float4 ax = make_float4(0.f, 0.f, 0.f, 0.f), mask = ax;
                if (row >= 0 && on) {
                    mask = ld4(a.X + static_cast<int64_t>(row) * a.ldx + col);
                    ax = drop_shared(mask, own_col, col);
                }
                uint32_t own[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) own[k] = on && col + k >= own_col ? ~0u : 0u;
                float acc[4] = {0.f, 0.f, 0.f, 0.f};
                float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
                int cur_j, cur_at = 0;
                float cur_w, cur_v = 0.f;
                fetch(s0, len, 0, cur_j, cur_w, cur_at, cur_v);
                for (int base = 0; base < maxlen; base += CH << lg_split) {
                    int next_j = 0, next_at = 0;
                    float next_w = 0.f, next_v = 0.f;
                    if (base + (CH << lg_split) < maxlen)  // wave-uniform: one chunk ahead
                        fetch(s0, len, base + (CH << lg_split), next_j, next_w, next_at, next_v);
                    const int my_ro = static_cast<int>(static_cast<uint32_t>(cur_j) * ldzb);
                    const int my_mo = XMASK ? static_cast<int>(static_cast<uint32_t>(cur_j) * ldmb) : 0;
                    float res = 0.f;
                    if constexpr (SIXTEENS) {
                        res = bwd_chunk<GS>(Zg, min(CH, maxlen - base), my_ro, cur_w, off, ax, sum, lig & 15);
                    } else {
                        const int steps = min(GS, maxlen - base);
                        int src = src0;
                        int u0 = 0;
                        for (; u0 + 8 <= steps; u0 += 8, src += 32) bwd_pass<8, GS, XMASK, SPARE, APART>(Zg, Mg, src, my_ro, my_mo, cur_w, off, ax, own, u0, lig, acc, res);
                        if (u0 + 4 <= steps) {
                            bwd_pass<4, GS, XMASK, SPARE, APART>(Zg, Mg, src, my_ro, my_mo, cur_w, off, ax, own, u0, lig, acc, res);
                            u0 += 4; src += 16;
                        }
                        if (u0 + 2 <= steps) {
                            bwd_pass<2, GS, XMASK, SPARE, APART>(Zg, Mg, src, my_ro, my_mo, cur_w, off, ax, own, u0, lig, acc, res);
                            u0 += 2; src += 8;
                        }
                        if (u0 < steps) bwd_pass<1, GS, XMASK, SPARE, APART>(Zg, Mg, src, my_ro, my_mo, cur_w, off, ax, own, u0, lig, acc, res);
                    }
                    const int e = base + part * CH + mine;
                    if (row >= 0 && e < len && lig < CH) {
                        if constexpr (ONE) {
                            if constexpr (LOOPED) {   // (the row has one chunk)
                                whole += res;
                                if (tile_now + 1 < n_tiles) continue;
                                res = whole;
                            }
                            if (a.g) a.g[cur_at] = res;
                            if (a.fused) {
                                momentum_step(cur_w, cur_v, res, a.lr, a.momentum, a.nesterov);
                                a.w[cur_at] = cur_w;
                                a.velocity[cur_at] = cur_v;
                                a.w_t[s0 + e] = cur_w;
                            }
                        } else {
                            gp[s0 + e] = res;  // GS consecutive entries of the row: one coalesced store
                        }
                    }
                    cur_j = next_j;
                    cur_w = next_w;
                    cur_at = next_at;
                    cur_v = next_v;
                }
                if constexpr (SIXTEENS) { acc[0] = sum.x; acc[1] = sum.y; acc[2] = sum.z; acc[3] = sum.w; }
                for (int d = GS; d < GS << lg_split; d <<= 1)   // the shares of a row, in one fixed order
#pragma unroll
                    for (int k = 0; k < 4; ++k) acc[k] += __shfl_xor(acc[k], d, kWave);
                if (row < 0 || !on || part != 0) continue;
                float4 y = len > 0 ? make_float4(acc[0], acc[1], acc[2], acc[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
                if (a.mask) y = keep_where_positive(y, mask);
                float *out = a.dX + static_cast<int64_t>(row) * a.lddx + col;
                if (SPARE != kSpareColumns || col == own_col) {
                    st4(out, y);
                } else {   // (the lane's own columns of the batch's last four)
                    if (own_col <= col + 1) out[1] = y.y;
                    if (own_col <= col + 2) out[2] = y.z;
                    out[3] = y.w;
                }
        }
    }
}

// Second pass: work-groups [0, n_entry_blocks) add the tiles' partial products of mirror entry q in tile
// order and apply the momentum step to the entry's CSR position perm[q] (or store the gradient there);
// the remaining work-groups, a wave per row of W, sum the rows of dZ for the bias gradient.
__device__ __forceinline__ void backward_finish(const BackwardArgs &a, const int32_t *hot_at, int n_tiles, int n_entry_blocks, int n_blocks, int block)
{
    if (block < n_entry_blocks) {
        for_runs_of_xcds(a.nnz, n_entry_blocks, [&](int64_t q) {
            const int p = a.perm[q];
            float g = 0.f;
            // (eight loads in flight, added in pairs: sixteen slices are then no further off than eight one after the other, 8.7e-8 and 9.2e-8; one after the other 1.0e-7)
            for (int t = 0; t < n_tiles; t += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = t + u < n_tiles ? a.partial[static_cast<int64_t>(t + u) * a.partial_stride + q] : 0.f;   // (uniform)
                g += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            }
            if (a.g) a.g[p] = g;
            if (a.fused) {
                float w = a.w[p], v = a.velocity[p];
                momentum_step(w, v, g, a.lr, a.momentum, a.nesterov);
                a.w[p] = w;
                a.velocity[p] = v;
                a.w_t[hot_at ? hot_at[q] : q] = w;
            }
        }, block);
        return;
    }
    if (!(a.db || (a.fused && a.bias))) return;
    backward_row_sums(a, static_cast<int64_t>(block - n_entry_blocks) * (kEwBlock / kWave) + wave_in_block(),
                      static_cast<int64_t>(n_blocks - n_entry_blocks) * (kEwBlock / kWave));
}
__global__ __launch_bounds__(kEwBlock) void backward_finish_kernel(const BackwardArgs a, const int32_t *const hot_at, const int n_tiles, const int n_entry_blocks)
{
    backward_finish(a, hot_at, n_tiles, n_entry_blocks, gridDim.x, blockIdx.x);
}

// The same among the work-groups of the column-tiled SDDMM of the layer below, which only needs the dZ that this layer's pass has formed: a launch and one drained chip less.  Every `every`-th eight
// work-groups (one to an XCD) are the finish pass's.  Wide MLP 322 -> 318 us a step (21 + 64 in turn, 83 together: the second pass's scattered lines take the same L2 requests as the gathers;
// at twice to eight times the rate, or first of all, 305-310 where this order gives 303).
template <int NV, bool SPARE>
__global__ __launch_bounds__(kSddmmWaves * kWave) __attribute__((amdgpu_waves_per_eu(8)))
void sddmm_tiled_finish_kernel(const SddmmArgs a, const int n_tiles, const TileOrder order, const BackwardArgs f, const int32_t *const hot_at, const int f_tiles,
                               const int n_entry_blocks, const int n_finish, const int every)
{
    static_assert(kSddmmWaves * kWave == kEwBlock, "");
    const int eight = blockIdx.x >> 3, turn = eight / every, groups = (n_finish + 7) / 8;
    if (turn < groups && eight - turn * every == every - 1) {
        const int block = turn * 8 + (blockIdx.x & 7);
        if (block < n_finish) backward_finish(f, hot_at, f_tiles, n_entry_blocks, n_finish, block);
        return;
    }
    sddmm_tile<16, NV, SPARE>(a, n_tiles, order, (eight - min(turn, groups)) * 8 + (blockIdx.x & 7));
}

// ---- both gradients where a few rows of dZ take most gathers ------------------------------------------
// The backward pass on one gather stream (backward_fused_kernel) for matrices a few of whose rows hold most of the entries: the kHotRowsLds longest rows of W -- two thirds of the entries of 16384^2
// power-law rows at 1 % -- are gathered from LDS, in which a work-group keeps its 64 columns of their dZ, the others from memory.  The entries of a mirror row are taken hot ones first
// (HotRows, launch_hot_order).  Sixteen lanes serve a mirror row, four of which run side by side in a wave; a gathered row goes into the row's result with the weight moved
// between lanes in the multiply-add (fma_row_lane), and into the entry's product with the mirror row's X, sixteen products at a time added up across the lanes (row16_transpose_sum).
// What bounds it: the vector ALUs (11.3 instructions a gather of four rows by 64 columns, 74 % busy at the 1.8 GHz that the card then holds; texture-address units 67 %, where the pass without LDS has
// them 79 % busy).  16384^2 at 1 %, batch 1024: 490 -> 370 us; of it, weights and sums in the order of the walk (stored through the mirror's positions: 50 more), rows side by side of like
// counts and half a chunk of cold rows on its way while hot ones are served 10, sets taken by whichever wave is free 10.  (Twice the slices of partial products: the second pass 38 -> 45.)
constexpr int kHotWaves = kWavesPerBlock, kHotZeroRow = kHotRowsLds * 256;
template <int N>
__device__ __forceinline__ float hot_steps(const char *lds, int off, float w, const float4 &ax, float4 &acc, int lig)
{
    constexpr int kAhead = 4;
    float4 x[N];
    float d[16];
    auto gather = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        x[i] = *reinterpret_cast<const float4 *>(lds + row_lane<i>(off));
    };
    static_for(std::make_integer_sequence<int, kAhead>{}, gather);
    __builtin_amdgcn_sched_barrier(0);
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (i + kAhead < N) gather(std::integral_constant<int, i + kAhead>{});
        fma_row_lane<i>(acc, w, x[i]);
        d[i] = fmaf(x[i].w, ax.w, fmaf(x[i].z, ax.z, fmaf(x[i].y, ax.y, x[i].x * ax.x)));
        if constexpr (i + kAhead < N) __builtin_amdgcn_sched_barrier(0);
    });
    return row16_transpose_sum<N>(d, lig);
}
// Entries B .. B + N - 1 of a cold chunk: asked for, and, when they have come, used.  (Lane i < N holds entry B + i's sum.)
template <int B, int N>
__device__ __forceinline__ void cold_ask(gmem_ptr Zg, int ro, uint32_t col_bytes, float4 (&x)[N])
{
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        x[i] = gload4(Zg, static_cast<uint32_t>(row_lane<B + i>(ro)) + col_bytes);
    });
    __builtin_amdgcn_sched_barrier(0);
}
template <int B, int N, bool SPARE>
__device__ __forceinline__ float cold_use(float4 (&x)[N], float w, const float4 &ax, const uint32_t (&own)[4], float4 &acc, int lig)
{
    float d[16];
    static_for(std::make_integer_sequence<int, N>{}, [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (SPARE) x[i] = make_float4(keep_bits(x[i].x, own[0]), keep_bits(x[i].y, own[1]), keep_bits(x[i].z, own[2]), keep_bits(x[i].w, own[3]));
        fma_row_lane<B + i>(acc, w, x[i]);
        d[i] = fmaf(x[i].w, ax.w, fmaf(x[i].z, ax.z, fmaf(x[i].y, ax.y, x[i].x * ax.x)));
    });
    const float sum = row16_transpose_sum<N>(d, lig);
    __builtin_amdgcn_sched_barrier(0);
    return sum;
}

// The mirror's values in the hot rows' order, out of the mirror, or, with perm (the CSR position of each), out of values[], from which the mirror's
// are brought up to date as well (gather_kernel's work).
__global__ __launch_bounds__(kEwBlock) void hot_values_kernel(float *out, const float *values, float *values_t, const int32_t *at, const int32_t *perm, const int64_t n)
{
    for_runs_of_xcds(n, gridDim.x, [&](int64_t k) {
        const int q = at[k];
        const float v = perm ? values[perm[k]] : values[q];
        out[k] = v;
        if (perm) values_t[q] = v;
    });
}
template <bool SPARE>
__global__ __launch_bounds__(kHotWaves * kWave) void backward_hot_kernel(const BackwardArgs a, const StripGrid g, const HotRows f, const float *const hot_values)
{
    __shared__ float4 hot[kHotRowsLds * 16 + 16];   // the rows, then one of zeros
    __shared__ int taken;
    const int at_block = static_cast<int>(blockIdx.x & 7) * g.per + static_cast<int>(blockIdx.x >> 3);
    const int tile = at_block / g.n_ranges, range = at_block - tile * g.n_ranges;
    if (tile >= g.n_tiles) return;
    const int lane = threadIdx.x & (kWave - 1), lrow = lane >> 4, lig = lane & 15;
    const int own_col = tile * 64 + lig * 4;
    const bool on = own_col < a.batch;
    const int col = four_columns(own_col, a.batch);
    uint32_t own[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) own[k] = on && col + k >= own_col ? ~0u : 0u;
    auto owned = [&](const float4 &x) { return SPARE ? make_float4(keep_bits(x.x, own[0]), keep_bits(x.y, own[1]), keep_bits(x.z, own[2]), keep_bits(x.w, own[3])) : x; };
    if (threadIdx.x == 0) taken = 0;
    if (threadIdx.x < 16) hot[kHotRowsLds * 16 + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);
    {
        float4 v[kHotRowsLds / 64];
#pragma unroll
        for (int i = 0; i < kHotRowsLds / 64; ++i)
            v[i] = ld4(a.dZ + static_cast<int64_t>(f.rows[i * 64 + static_cast<int>(threadIdx.x >> 4)].x) * a.lddz + col);
#pragma unroll
        for (int i = 0; i < kHotRowsLds / 64; ++i) hot[i * 1024 + static_cast<int>(threadIdx.x)] = owned(v[i]);
    }
    __syncthreads();
    const char *lds = reinterpret_cast<const char *>(hot) + lig * 16;
    const uint32_t col_bytes = static_cast<uint32_t>(col) * 4u, ldzb = static_cast<uint32_t>(a.lddz) * 4u;
    const gmem_ptr Zg = as_gmem(a.dZ);
    float *gp = a.partial + static_cast<int64_t>(tile) * a.partial_stride;
    const int n_sets = (a.rows + 3) >> 2;
    auto take = [&] {   // the next of the range's sets
        int k = 0;
        if (lane == 0) k = atomicAdd(&taken, 1);
        return __builtin_amdgcn_readfirstlane(k) * g.n_ranges + range;
    };
    // a mirror row of each lane row, and what the four take side by side: chunks of sixteen hot entries, then of cold ones
    struct Set {
        int row, s0, len, n_hot, most_hot, most_cold;
    };
    auto set_of = [&](const int4 &d) {
        auto most_of = [&](int n) {
            n = max(n, __shfl_xor(n, 16, kWave));
            return __builtin_amdgcn_readfirstlane(max(n, __shfl_xor(n, 32, kWave)));
        };
        return Set{d.x, d.y, d.z, d.w, most_of(d.w), most_of(d.z - d.w)};
    };
    // sixteen entries from `first` on of the hot or the cold ones, a lane's one: {offset or row, weight}; on: there is one
    struct Chunk {
        int entry;
        float w;
    };
    auto ask = [&](const Set &s, bool is_hot, int first) {
        const int e = first + lig, n = is_hot ? s.n_hot : s.len - s.n_hot;
        const uint32_t o = e < n ? static_cast<uint32_t>(s.s0 + (is_hot ? 0 : s.n_hot) + e) * 4u : 0u;
        return Chunk{__builtin_bit_cast(int, gload1(as_gmem(f.entry), o)), gload1(as_gmem(hot_values), o)};
    };
    auto record = [&](int set) { return set < n_sets ? f.sets[set * 4 + lrow] : make_int4(-1, 0, 0, 0); };
    auto input = [&](const Set &s) { return ld4(a.X + static_cast<int64_t>(max(s.row, 0)) * a.ldx + col); };
    int set = take(), set_next = take();
    Set now = set_of(record(set));
    float4 mask = input(now);
    Chunk hot_now = ask(now, true, 0), cold_now = ask(now, false, 0);
    int4 d_next = record(set_next);
    while (set < n_sets) {   // (every wave's tickets grow)
        const int set_after = take();
        const int4 d_after = record(set_after);
        const Set next = set_of(d_next);
        const float4 mask_next = input(next), ax = now.row >= 0 ? owned(mask) : make_float4(0.f, 0.f, 0.f, 0.f);
        const Chunk hot_first = ask(next, true, 0), cold_first = ask(next, false, 0);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), acc_cold = acc;   // (apart, so that neither sum is long)
        const int n_cold = now.len - now.n_hot;
        int fill = 0;
        if (now.most_cold > 0) {
            // what a lane without a cold entry gathers, with weight 0: a row of dZ that the mirror row references anyway, its first cold one, or, without any, a hot one
            // (an empty row: row 0, for a result that is not taken)
            fill = row_lane<0>(cold_now.entry);
            if (__any(n_cold == 0)) fill = n_cold > 0 ? fill : now.len > 0 ? f.rows[f.entry[now.s0] >> 8].x : 0;
        }
        auto hot_sums = [&](const Chunk &c, int e) {   // (a row of zeros for a lane without an entry)
            const bool ok = e + lig < now.n_hot;
            const int off = ok ? c.entry : kHotZeroRow, n = now.most_hot - e;
            const float w = ok ? c.w : 0.f;
            if (n > 12) return hot_steps<16>(lds, off, w, ax, acc, lig);
            if (n > 8) return hot_steps<12>(lds, off, w, ax, acc, lig);
            if (n > 4) return hot_steps<8>(lds, off, w, ax, acc, lig);
            return hot_steps<4>(lds, off, w, ax, acc, lig);
        };
        const uint32_t gp_hot = static_cast<uint32_t>(now.s0 + lig) * 4u, gp_cold = static_cast<uint32_t>(now.s0 + now.n_hot + lig) * 4u;
        int h = 0, c = 0;   // entries done
        // two chunks of hot entries beside one of cold ones: half of the latter are on their way while a hot chunk is served from LDS
        while (h + 16 < now.most_hot && c + 8 < now.most_cold) {
            const bool ok = c + lig < n_cold;
            const int ro = static_cast<int>(static_cast<uint32_t>(ok ? cold_now.entry : fill) * ldzb);
            const float w = ok ? cold_now.w : 0.f;
            const Chunk hot_next = ask(now, true, h + 16);
            float4 x[8];
            cold_ask<0, 8>(Zg, ro, col_bytes, x);
            const bool ok_hot = h + lig < now.n_hot;
            const float sum_hot = hot_steps<16>(lds, ok_hot ? hot_now.entry : kHotZeroRow, ok_hot ? hot_now.w : 0.f, ax, acc, lig);
            __builtin_amdgcn_sched_barrier(0);
            const float sum_0 = cold_use<0, 8, SPARE>(x, w, ax, own, acc_cold, lig);
            hot_now = ask(now, true, h + 32);
            cold_now = ask(now, false, c + 16);
            cold_ask<8, 8>(Zg, ro, col_bytes, x);
            if (ok_hot) gstore1(gp, gp_hot + static_cast<uint32_t>(h) * 4u, sum_hot);
            if (lig < 8 && ok) gstore1(gp, gp_cold + static_cast<uint32_t>(c) * 4u, sum_0);
            const float sum_hot2 = hot_sums(hot_next, h + 16);
            __builtin_amdgcn_sched_barrier(0);
            const float sum_1 = cold_use<8, 8, SPARE>(x, w, ax, own, acc_cold, lig);
            if (h + 16 + lig < now.n_hot) gstore1(gp, gp_hot + static_cast<uint32_t>(h) * 4u + 64u, sum_hot2);
            if (lig < 8 && c + 8 + lig < n_cold) gstore1(gp, gp_cold + static_cast<uint32_t>(c) * 4u + 32u, sum_1);
            h += 32;
            c += 16;
        }
        for (; h < now.most_hot; h += 16) {
            const Chunk hot_next = ask(now, true, h + 16);
            const float sum = hot_sums(hot_now, h);
            if (h + lig < now.n_hot) gstore1(gp, gp_hot + static_cast<uint32_t>(h) * 4u, sum);
            hot_now = hot_next;
        }
        for (; c < now.most_cold; c += 16) {
            const bool ok = c + lig < n_cold;
            const int ro = static_cast<int>(static_cast<uint32_t>(ok ? cold_now.entry : fill) * ldzb);
            const float w = ok ? cold_now.w : 0.f;
            cold_now = ask(now, false, c + 16);
            float4 x[8];
            cold_ask<0, 8>(Zg, ro, col_bytes, x);
            const float sum_0 = cold_use<0, 8, SPARE>(x, w, ax, own, acc_cold, lig);
            if (lig < 8 && ok) gstore1(gp, gp_cold + static_cast<uint32_t>(c) * 4u, sum_0);
            if (c + 8 < now.most_cold) {
                cold_ask<8, 8>(Zg, ro, col_bytes, x);
                const float sum_1 = cold_use<8, 8, SPARE>(x, w, ax, own, acc_cold, lig);
                if (lig < 8 && c + 8 + lig < n_cold) gstore1(gp, gp_cold + static_cast<uint32_t>(c) * 4u + 32u, sum_1);
            }
        }
        const int row = now.row, len = now.len;
        const float4 mask_now = mask;
        set = set_next;
        set_next = set_after;
        now = next;
        mask = mask_next;
        hot_now = hot_first;
        cold_now = cold_first;
        d_next = d_after;
        if (row < 0 || !on) continue;
        // (an empty row gathered, with weight 0, from row 0 of dZ)
        float4 y = len > 0 ? make_float4(acc.x + acc_cold.x, acc.y + acc_cold.y, acc.z + acc_cold.z, acc.w + acc_cold.w) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.mask) y = keep_where_positive(y, mask_now);
        float *out = a.dX + static_cast<int64_t>(row) * a.lddx + col;
        if (!SPARE || col == own_col) {
            st4(out, y);
        } else {   // (the lane's own columns of the batch's last four)
            if (own_col <= col + 1) out[1] = y.y;
            if (own_col <= col + 2) out[2] = y.z;
            out[3] = y.w;
        }
    }
}

// ---- the end of a training step in one launch ----------------------------------------------------
// Row j of dZ_0 = (W_1^T dZ_1) * [A_0 > 0] takes the mirror row j of W_1 only, and row j of W_0's gradient takes that row of dZ_0
// only: the waves that serve row j of W_0 (its partition) form dZ_0[j, :] from their shares of the mirror row, each gathered row of
// dZ_1 giving the products of W_1's gradient as well (as in backward_fused_kernel; a mirror entry is read and updated by one wave), add them up in LDS, and
// go on to the entries of W_0.  After them in the grid: the waves that sum the rows of dZ_1 for W_1's biases, and, where a layer above still waits for its
// update, that (sddmm_body).
// What bounds it: the chain of memory round trips of its two halves; what it saves is a launch and the way of dZ_0 through
// memory.  Steps of 3072-1024-512-10 at batch 100, 99 / 90 %: 23.2 -> 21.7 and 38.4 -> 34.6 us, 3001-1501-777-10 at
// 5 %, batch 77: 39.0 -> 36.5; the launch 8.9 / 17.1 us, the two before 4.6 + 5.9 and 5.9 + 15.5.  (The column indices of the second half asked for
// ahead, and the mask kept: 21.6, 34.9 and 37.7.)
template <int G, int NV, int U, bool WHOLE>
__device__ __forceinline__ void chain_pass(gmem_ptr Zg, int it0, int my_ro, float my_w, const uint32_t (&off)[NV], const float4 (&ax)[NV], float4 (&acc)[NV],
                                           float &res)
{
    const int lane = threadIdx.x & (kWave - 1), lig = lane % G;
    uint32_t ro[U];
    float w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int src = ((lane / G) * G + it0 + u) * 4;
        ro[u] = static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(src, my_ro));
        w[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, __builtin_bit_cast(int, my_w)));
    }
    float4 z[U][NV];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < NV; ++t) z[u][t] = gload4(Zg, ro[u] + off[t]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            if constexpr (WHOLE) {
                part = fmaf(ax[t].x, z[u][t].x, part);
                part = fmaf(ax[t].y, z[u][t].y, part);
                part = fmaf(ax[t].z, z[u][t].z, part);
                part = fmaf(ax[t].w, z[u][t].w, part);
            }
            acc[t].x = fmaf(w[u], z[u][t].x, acc[t].x);
            acc[t].y = fmaf(w[u], z[u][t].y, acc[t].y);
            acc[t].z = fmaf(w[u], z[u][t].z, acc[t].z);
            acc[t].w = fmaf(w[u], z[u][t].w, acc[t].w);
        }
        if constexpr (WHOLE) {
            part = group_sum<G>(part);
            if (lig == it0 + u) res = part;
        }
    }
}

template <int G, int NV, bool SPARE, bool WHOLE>
__device__ __forceinline__ void chain_body(const ChainArgs &c, const SddmmArgs &a, const int block)
{
    constexpr int NG = kWave / G;
    constexpr int UI = NV >= 3 ? 1 : (NV == 2 ? 2 : 4);
    __shared__ float4 red[kWavesPerBlock][NV][G];
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block(), grp = lane / G, lig = lane % G;
    const WaveTask task = wave_task(a.blocks, block);
    const int row = task.row;
    uint32_t off[NV];
    float4 acc[NV];
    const gmem_ptr ar = as_gmem(c.A + static_cast<int64_t>(max(row, 0)) * c.lda);
#pragma unroll
    for (int t = 0; t < NV; ++t) {
        const int own = (t * G + lig) * 4;
        off[t] = static_cast<uint32_t>(four_columns(own < a.batch ? own : 0, a.batch)) * 4u;
        acc[t] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (row >= 0) {
        float4 ax[NV];
#pragma unroll
        for (int t = 0; t < NV; ++t) ax[t] = gload4(ar, off[t]);
        int q0 = c.indptr_t[row], q1 = c.indptr_t[row + 1];
        const int share = (q1 - q0 + (1 << task.lg) - 1) >> task.lg;
        q0 = min(q0 + task.part * share, q1);
        q1 = min(q0 + share, q1);
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            const int own = (t * G + lig) * 4;
            ax[t] = own < a.batch ? drop_shared(ax[t], own, static_cast<int>(off[t] >> 2)) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const uint32_t ldzb = static_cast<uint32_t>(c.lddz) * 4u;
        const gmem_ptr Zg = as_gmem(c.dZ);
        const int q_mine = lig * NG + grp;  // slot of this lane inside a chunk of 64 entries, as in sddmm_body
        const bool spare = SPARE && G * 4 * NV > a.batch;  // uniform
        for (int pc = q0; pc < q1; pc += kWave) {
            const int n = min(kWave, q1 - pc);
            const bool mine = q_mine < n;
            const int p = pc + (mine ? q_mine : 0);
            const int my_i = c.indices_t[p];
            float w = c.values_t[p], v = 0.f;
            int at = 0;
            if constexpr (WHOLE) {
                at = c.perm[p];
                v = c.velocity[at];
            }
            const int my_ro = static_cast<int>(static_cast<uint32_t>(my_i) * ldzb);
            const float my_w = mine ? w : 0.f;
            const int iters = (n + NG - 1) / NG;
            float res = 0.f;
            int it = 0;
            for (; it + UI <= iters; it += UI) chain_pass<G, NV, UI, WHOLE>(Zg, it, my_ro, my_w, off, ax, acc, res);
            if constexpr (UI >= 4)
                if (it + 2 <= iters) { chain_pass<G, NV, 2, WHOLE>(Zg, it, my_ro, my_w, off, ax, acc, res); it += 2; }
            if constexpr (UI >= 2)
                if (it < iters) chain_pass<G, NV, 1, WHOLE>(Zg, it, my_ro, my_w, off, ax, acc, res);
            if constexpr (!WHOLE) continue;
            if (spare && __any(res != res)) res = sddmm_own_columns<G, NV>(Zg, iters, my_ro, off, ax, 0, a.batch);
            if (mine) {
                momentum_step(w, v, res, a.lr, a.momentum, a.nesterov);
                c.w[at] = w;
                c.velocity[at] = v;
                c.values_t[p] = w;
            }
        }
    }
    // the groups' sums, then the waves', each in one fixed order
#pragma unroll
    for (int d = G; d < kWave; d <<= 1)
#pragma unroll
        for (int t = 0; t < NV; ++t) {
            acc[t].x += __shfl_xor(acc[t].x, d, kWave);
            acc[t].y += __shfl_xor(acc[t].y, d, kWave);
            acc[t].z += __shfl_xor(acc[t].z, d, kWave);
            acc[t].w += __shfl_xor(acc[t].w, d, kWave);
        }
    if (task.lg > 0) {   // uniform over the work-group
        if (grp == 0)
#pragma unroll
            for (int t = 0; t < NV; ++t) red[wv][t][lig] = acc[t];
        __syncthreads();
        const int first = wv - task.part;
#pragma unroll
        for (int t = 0; t < NV; ++t) acc[t] = red[first][t][lig];
        for (int s = 1; s < (1 << task.lg); ++s)
#pragma unroll
            for (int t = 0; t < NV; ++t) {
                const float4 r = red[first + s][t][lig];
                acc[t].x += r.x; acc[t].y += r.y; acc[t].z += r.z; acc[t].w += r.w;
            }
    }
    if (row < 0) return;
    float4 dz[NV];
#pragma unroll
    for (int t = 0; t < NV; ++t) {
        const int own = (t * G + lig) * 4;
        const float4 y = keep_where_positive(acc[t], gload4(ar, off[t]));   // (read again: registers)
        if (task.part == 0 && grp == 0 && own < a.batch) st4(c.dZ_below + static_cast<int64_t>(row) * c.lddz_below + (off[t] >> 2), y);
        dz[t] = own < a.batch ? drop_shared(y, own, static_cast<int>(off[t] >> 2)) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if constexpr (WHOLE) sddmm_body<G, NV, SPARE, true>(a, block, 0, &task, dz);
}

// Biases of W_1: a group of lanes per row of dZ_1, added up as sddmm_body does.
template <int G, int NV>
__device__ __forceinline__ void chain_row_sums(const ChainArgs &c, const SddmmArgs &a, const int block)
{
    const int lane = threadIdx.x & (kWave - 1), lig = lane % G, i = (block * kWavesPerBlock + wave_in_block()) * (kWave / G) + lane / G;
    const float *zr = c.dZ + static_cast<int64_t>(min(i, c.rows - 1)) * c.lddz;
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < NV; ++t) {
        const int own = (t * G + lig) * 4, first = four_columns(own < a.batch ? own : 0, a.batch);
        float4 z = ld4(zr + first);
        z = own < a.batch ? drop_shared(z, own, first) : make_float4(0.f, 0.f, 0.f, 0.f);
        s += (z.x + z.y) + (z.z + z.w);
    }
    s = group_sum<G>(s);
    if (lig != 0 || i >= c.rows) return;
    float w = c.bias[i], v = c.bias_velocity[i];
    momentum_step(w, v, s, a.lr, a.momentum, a.nesterov);
    c.bias[i] = w;
    c.bias_velocity[i] = v;
}

// GB, NVB: lanes of the layer that waits, those of a launch of its own.
template <int G, int NV, int GB, int NVB, bool SPARE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(8))) void chain_kernel(const ChainArgs c, const SddmmArgs a, const SddmmArgs b, const int n_sum_blocks)
{
    int block = blockIdx.x;
    if (block < a.blocks.n_blocks) return chain_body<G, NV, SPARE, true>(c, a, block);
    block -= a.blocks.n_blocks;
    if (block < n_sum_blocks) return chain_row_sums<G, NV>(c, a, block);
    sddmm_body<GB, NVB, SPARE || GB != G>(b, block - n_sum_blocks);
}

// Its first half alone, dZ_0: for a step whose launches are kept apart, so that both form the same sums.
template <int G, int NV>
__global__ __launch_bounds__(kBlock) void chain_transposed_kernel(const ChainArgs c, const SddmmArgs a)
{
    chain_body<G, NV, false, false>(c, a, blockIdx.x);
}

// Two independent launches of a training step in one grid: work-groups [0, na) run the first,
// the rest the second.  Saves a launch (and its drain) on the step's critical path.
template <int GS_S, int G, int NV_D, bool SPARE>
__global__ __launch_bounds__(kBlock) void spmm_sddmm_pair_kernel(const SpmmArgs a, const SddmmArgs b, const int na)
{
    if (static_cast<int>(blockIdx.x) < na) {
        if constexpr (GS_S < kWave)
            spmm_body_grouped<GS_S, false>(a, blockIdx.x);
        else
            spmm_wide_body<false>(a, blockIdx.x % a.blocks.n_blocks, blockIdx.x / a.blocks.n_blocks * 256);
    } else {
        sddmm_body<G, NV_D, SPARE>(b, blockIdx.x - na);
    }
}
template <int G, int NV_D, bool SPARE>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(SPARE ? 8 : 1))) void sddmm_pair_kernel(const SddmmArgs a, const SddmmArgs b, const int na)
{
    if (static_cast<int>(blockIdx.x) < na)
        sddmm_body<G, NV_D, SPARE>(a, blockIdx.x);
    else
        sddmm_body<G, NV_D, SPARE>(b, blockIdx.x - na);
}

// Any batch size, operands of any span: one column per lane and pass, both operands re-read per stored
// entry.  For batches below 4, untiled ones beyond 1024 and operands of 4 GiB or more.
__global__ __launch_bounds__(kBlock) void sddmm_generic(const SddmmArgs a)
{
    const int lane = threadIdx.x & (kWave - 1);
    mean_loss_task(a, blockIdx.x);
    const WaveTask task = wave_task(a.blocks, blockIdx.x);
    if (task.row < 0) return;
    const int row = task.row;
    const float *zr = a.dZ + static_cast<int64_t>(row) * a.lddz;
    const float *zm = a.ZM ? a.ZM + static_cast<int64_t>(row) * a.ldzm : nullptr;

    if (task.lead && (a.db || (a.fused && a.bias))) {
        float s = 0.f;
        for (int c = lane; c < a.batch; c += kWave) {
            float z = zr[c];
            if (zm) z = keep_where_positive(z, zm[c]);
            s += z;
        }
        s = group_sum<kWave>(s);
        if (lane == 0) {
            if (a.db) a.db[row] = s;
            if (a.fused && a.bias) {
                float w = a.bias[row], v = a.bias_velocity[row];
                momentum_step(w, v, s, a.lr, a.momentum, a.nesterov);
                a.bias[row] = w;
                a.bias_velocity[row] = v;
            }
        }
    }
    if (a.skip_products) return;

    const int s0 = task.s0;
    const int s1 = task.s1;
    for (int p = s0; p < s1; ++p) {
        const float *xr = a.X + static_cast<int64_t>(a.indices[p]) * a.ldx;
        float part = 0.f;
        for (int c = lane; c < a.batch; c += kWave) {
            float z = zr[c];
            if (zm) z = keep_where_positive(z, zm[c]);
            part = fmaf(z, xr[c], part);
        }
        part = group_sum<kWave>(part);
        if (lane == 0) {
            if (a.g) a.g[p] = part;
            if (a.fused) {
                float w = a.values[p], v = a.velocity[p];
                momentum_step(w, v, part, a.lr, a.momentum, a.nesterov);
                a.values[p] = w;
                a.velocity[p] = v;
                if (a.values_t) a.values_t[a.pos_t[p]] = w;
                if (a.dense) a.dense[static_cast<int64_t>(row) * a.dense_ld + a.indices[p]] = w;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Element-wise kernels
// ---------------------------------------------------------------------------------------

__global__ __launch_bounds__(kEwBlock) void momentum_kernel(float *__restrict__ w, float *__restrict__ v,
                                                            const float *__restrict__ g, int64_t n,
                                                            float lr, float mu, int nesterov, int vec4)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (vec4) {
        const int64_t n4 = n >> 2;
        for (int64_t k = i; k < n4; k += stride) {
            float4 ww = ld4(w + 4 * k), vv = ld4(v + 4 * k);
            const float4 gg = ld4(g + 4 * k);
            momentum_step(ww.x, vv.x, gg.x, lr, mu, nesterov);
            momentum_step(ww.y, vv.y, gg.y, lr, mu, nesterov);
            momentum_step(ww.z, vv.z, gg.z, lr, mu, nesterov);
            momentum_step(ww.w, vv.w, gg.w, lr, mu, nesterov);
            st4(v + 4 * k, vv);
            st4(w + 4 * k, ww);
        }
        i += n4 << 2;  // tail: elements 4*n4 .. n-1, one per thread of the first work-group
        if (i < n) {
            float ww = w[i], vv = v[i];
            momentum_step(ww, vv, g[i], lr, mu, nesterov);
            v[i] = vv;
            w[i] = ww;
        }
    } else {
        for (; i < n; i += stride) {
            float ww = w[i], vv = v[i];
            momentum_step(ww, vv, g[i], lr, mu, nesterov);
            v[i] = vv;
            w[i] = ww;
        }
    }
}

__global__ __launch_bounds__(kEwBlock) void gather_kernel(float *__restrict__ dst, const float *__restrict__ src,
                                                          const int32_t *__restrict__ perm, int64_t n)
{
    gather_runs(dst, src, perm, n, gridDim.x);
}

// What a stand-alone backward pass needs before its products, in one grid: the mirror's values (work-groups [0, n_gather)),
// and dZ = dY * [Y > 0] of a ReLU layer, four columns per thread.  The transposed product gathers a row of dZ per stored
// entry; with the mask as a second operand it gathered two (4096 x 3072 at 5 %, batch 128: 37.9 us, 16.4 from dZ,
// which takes 0.8 us more than the values alone).
__global__ __launch_bounds__(kEwBlock) void backward_prep_kernel(float *__restrict__ values_t, const float *__restrict__ values,
                                                                 const int32_t *__restrict__ perm, int64_t nnz, int n_gather,
                                                                 const float *__restrict__ dY, int64_t lddy, const float *__restrict__ Y,
                                                                 int64_t ldy, float *__restrict__ dZ, int64_t lddz, int rows, int batch)
{
    if (static_cast<int>(blockIdx.x) < n_gather) {
        gather_runs(values_t, values, perm, nnz, n_gather);
        return;
    }
    const int quads = (batch + 3) / 4;   // batch >= 4
    const int64_t n = static_cast<int64_t>(rows) * quads, stride = static_cast<int64_t>(gridDim.x - n_gather) * kEwBlock;
    for (int64_t k = static_cast<int64_t>(blockIdx.x - n_gather) * kEwBlock + threadIdx.x; k < n; k += stride) {
        const int64_t row = k / quads;
        const int c = four_columns(static_cast<int>(k - row * quads) * 4, batch);
        st4(dZ + row * lddz + c, keep_where_positive(ld4(dY + row * lddy + c), ld4(Y + row * ldy + c)));
    }
}

__global__ __launch_bounds__(kEwBlock) void copy_kernel(float *__restrict__ dst, const float *__restrict__ src,
                                                        int64_t n, int vec4)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (vec4) {
        const int64_t n4 = n >> 2;
        for (int64_t k = i; k < n4; k += stride) st4(dst + 4 * k, ld4(src + 4 * k));
        i += n4 << 2;
        if (i < n) dst[i] = src[i];
    } else {
        for (; i < n; i += stride) dst[i] = src[i];
    }
}

// Softmax cross-entropy for up to 16 classes, one column (example) per thread with its logits in registers, a single
// work-group so that the mean over the batch is summed in one fixed order (wave sums by DPP, then the wave leaders'
// values in wave order).
constexpr int kSoftmaxBlock = 1024;
constexpr int kSoftmaxWaves = kSoftmaxBlock / kWave;
constexpr int kSoftmaxFew = 16;

// *loss_out = mean over the batch of the threads' shares; every thread of the work-group arrives here
__device__ __forceinline__ void softmax_mean(float loss, float inv_b, float (&wave_loss)[kSoftmaxWaves], float *loss_out)
{
    loss = group_sum<kWave>(loss);
    if ((threadIdx.x & (kWave - 1)) == 0) wave_loss[threadIdx.x >> 6] = loss;
    __syncthreads();
    if (threadIdx.x == 0 && loss_out) {
        float total = 0.f;
        for (int w = 0; w < static_cast<int>(blockDim.x >> 6); ++w) total += wave_loss[w];
        *loss_out = total * inv_b;
    }
}

__global__ __launch_bounds__(kSoftmaxBlock) void softmax_ce_few_kernel(const float *Z, int64_t ldz, const int32_t *__restrict__ labels,
                                                                       int classes, int batch, float *dZ, int64_t lddz, float *loss_out)
{
    __shared__ float wave_loss[kSoftmaxWaves];
    const float inv_b = 1.0f / static_cast<float>(batch);
    float loss = 0.f;
    for (int c = threadIdx.x; c < batch; c += blockDim.x) {
        const int t = labels[c];
        float z[kSoftmaxFew];
#pragma unroll
        for (int i = 0; i < kSoftmaxFew; ++i) z[i] = i < classes ? Z[static_cast<int64_t>(i) * ldz + c] : -INFINITY;
        float m = z[0];
#pragma unroll
        for (int i = 1; i < kSoftmaxFew; ++i) m = fmaxf(m, z[i]);
        float s = 0.f, zt = 0.f;
#pragma unroll
        for (int i = 0; i < kSoftmaxFew; ++i) {
            if (i < classes) s += expf(z[i] - m);
            zt = i == t ? z[i] : zt;
        }
        const float lse = m + logf(s);
        loss += lse - zt;
#pragma unroll
        for (int i = 0; i < kSoftmaxFew; ++i)
            if (i < classes) dZ[static_cast<int64_t>(i) * lddz + c] = (expf(z[i] - lse) - (i == t ? 1.f : 0.f)) * inv_b;
    }
    softmax_mean(loss, inv_b, wave_loss, loss_out);
}

// The same for more classes.  Work-group b < n_tiles forms the gradient of 64 columns, a column per lane, wave w taking the
// classes w, w + 16, ...: eight of a lane's logits are read at a time (and kept, up to 128 classes), and the waves meet in LDS for
// the maximum and for the sum.  The loss needs every column, so the last work-group forms it on its own from all the
// logits, with as many waves to a column as there are to spare: it waits for nobody, and one launch does.
// (One thread per column that walked the classes three times: 49 us for 85 classes at batch 256.)
// dZ may be Z: then the loss takes its own launch, before the gradients overwrite the logits.
constexpr int kSoftmaxKept = 8;
__device__ __forceinline__ float finite_or_zero(float m) { return m == -INFINITY ? 0.f : m; }   // (-Inf logits: exp(z - m) is 0, not NaN)

__device__ __forceinline__ void softmax_loss(const float *Z, int64_t ldz, const int32_t *__restrict__ labels, int classes, int batch,
                                             float *loss_out, float (&red)[2][kSoftmaxWaves][kWave], float (&wave_loss)[kSoftmaxWaves])
{
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block();
    int lg = 0;   // waves per column
    while (lg < 4 && ((batch - 1) >> (10 - lg - 1)) == 0) ++lg;
    const int share = wv & ((1 << lg) - 1), step = 1 << lg, wide = (kSoftmaxWaves >> lg) * kWave;
    float loss = 0.f;
    for (int base = 0; base < batch; base += wide) {
        const int own = base + (wv >> lg) * kWave + lane, c = min(own, batch - 1);
        float m = -INFINITY, s = 0.f;
        for (int i0 = share; i0 < classes; i0 += step * kSoftmaxKept) {
            float z[kSoftmaxKept], top = m;
#pragma unroll
            for (int u = 0; u < kSoftmaxKept; ++u) z[u] = Z[static_cast<int64_t>(min(i0 + u * step, classes - 1)) * ldz + c];
#pragma unroll
            for (int u = 0; u < kSoftmaxKept; ++u) top = i0 + u * step < classes ? fmaxf(top, z[u]) : top;
            const float shift = finite_or_zero(top);
            s *= expf(m - shift);
#pragma unroll
            for (int u = 0; u < kSoftmaxKept; ++u) s += i0 + u * step < classes ? expf(z[u] - shift) : 0.f;
            m = top;
        }
        red[0][wv][lane] = m;
        red[1][wv][lane] = s;
        __syncthreads();
        if (share == 0 && own < batch) {
            float top = m;
            for (int w = 1; w < step; ++w) top = fmaxf(top, red[0][wv + w][lane]);
            const float shift = finite_or_zero(top);
            float sum = 0.f;
            for (int w = 0; w < step; ++w) sum += red[1][wv + w][lane] * expf(red[0][wv + w][lane] - shift);
            loss += (top + logf(sum)) - Z[static_cast<int64_t>(labels[c]) * ldz + c];
        }
        __syncthreads();
    }
    softmax_mean(loss, 1.0f / static_cast<float>(batch), wave_loss, loss_out);
}

__global__ __launch_bounds__(kSoftmaxBlock) void softmax_ce_kernel(const float *Z, int64_t ldz, const int32_t *__restrict__ labels, int classes,
                                                                   int batch, float *dZ, int64_t lddz, float *loss_out, const int n_tiles)
{
    __shared__ float red[2][kSoftmaxWaves][kWave];
    __shared__ float wave_loss[kSoftmaxWaves];
    if (static_cast<int>(blockIdx.x) == n_tiles) {
        softmax_loss(Z, ldz, labels, classes, batch, loss_out, red, wave_loss);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block();
    const int own = blockIdx.x * kWave + lane, c = min(own, batch - 1);
    const int t = labels[c];
    constexpr int kStep = kSoftmaxWaves * kSoftmaxKept;
    float z[kSoftmaxKept];
    auto fetch = [&](int i0) {
#pragma unroll
        for (int u = 0; u < kSoftmaxKept; ++u) z[u] = Z[static_cast<int64_t>(min(i0 + u * kSoftmaxWaves, classes - 1)) * ldz + c];
    };
    float m = -INFINITY;
    for (int i0 = wv; i0 < classes; i0 += kStep) {
        fetch(i0);
#pragma unroll
        for (int u = 0; u < kSoftmaxKept; ++u) m = fmaxf(m, z[u]);   // (past the end: the last class again)
    }
    red[0][wv][lane] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSoftmaxWaves; ++w) m = fmaxf(m, red[0][w][lane]);
    float s = 0.f;
    for (int i0 = wv; i0 < classes; i0 += kStep) {
        if (classes > kStep) fetch(i0);
#pragma unroll
        for (int u = 0; u < kSoftmaxKept; ++u) s += i0 + u * kSoftmaxWaves < classes ? expf(z[u] - m) : 0.f;
    }
    red[1][wv][lane] = s;
    __syncthreads();
    s = 0.f;
#pragma unroll
    for (int w = 0; w < kSoftmaxWaves; ++w) s += red[1][w][lane];
    const float lse = m + logf(s), inv_b = 1.0f / static_cast<float>(batch);
    if (own >= batch) return;
    for (int i0 = wv; i0 < classes; i0 += kStep) {
        if (classes > kStep) fetch(i0);
#pragma unroll
        for (int u = 0; u < kSoftmaxKept; ++u) {
            const int i = i0 + u * kSoftmaxWaves;
            if (i < classes) dZ[static_cast<int64_t>(i) * lddz + c] = (expf(z[u] - lse) - (i == t ? 1.f : 0.f)) * inv_b;
        }
    }
}

// Output-layer head (see HeadArgs).  A work-group first brings what its three phases gather from into LDS, in one
// round of loads: its four columns of the layer's input (IN_LDS), every entry of the mirror (MIRROR_LDS), and, in
// registers, the first chunks of every wave's row.  Forward: wave w takes rows w, w+16, ..., lanes run across the row's stored
// entries, DPP sum.  Softmax-CE: one wave per column, one class per lane.  Transposed product: one thread per row of
// W^T.  Each column's loss goes to loss_cols; their mean is taken by a later launch of the step (SddmmArgs::loss_cols).
// What bounds it is the chain of dependent memory round trips, a few microseconds for a few thousand entries: with
// gathers and mirror reads straight from memory, entry after entry, a full 10 x 777 layer took 15.1 us, now 8.2
// (a layer with an entry or less per column has nothing to share: read directly, 4.8 us at 10 x 512 and 1 %).
constexpr int kHeadCols = 4;
constexpr int kHeadChunks = 8;              // chunks of 64 entries of a row whose loads travel together
constexpr int kHeadMaxLds = 60 << 10;
__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, kWave));
    return x;
}
template <bool IN_LDS, bool MIRROR_LDS>
__global__ __launch_bounds__(kBlock) void head_kernel(const HeadArgs a)
{
    extern __shared__ float4 head_lds[];    // [cols] input columns (IN_LDS), then the mirror's values and rows
    __shared__ float4 z[kHeadMaxRows];
    float4 *xs = head_lds;
    float *wt = reinterpret_cast<float *>(head_lds + (IN_LDS ? a.cols : 0));
    unsigned char *it = reinterpret_cast<unsigned char *>(wt + a.nnz);
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = wave_in_block();
    // (the last work-group's columns move back to the batch's last four; those it shares with its neighbour get the same bits)
    const int nc = min(kHeadCols, a.batch);
    const int c0 = a.batch >= kHeadCols ? four_columns(blockIdx.x * kHeadCols, a.batch) : 0;
    auto four_of = [&](int j) {
        const float *xr = a.X + static_cast<int64_t>(j) * a.ldx + c0;
        if (nc == kHeadCols) return ld4(xr);
        return make_float4(xr[0], nc > 1 ? xr[1] : 0.f, nc > 2 ? xr[2] : 0.f, 0.f);
    };

    // One round of loads: first chunks of the wave's row, mirror row bounds, label, mirror, input columns.  No load
    // hides behind a lane's condition (lanes without an entry repeat the last one): a branch would make the compiler
    // wait for what is in flight.
    const int j0 = threadIdx.x;
    const int j_first = min(j0, a.cols - 1);
    int q0 = a.indptr_t[j_first], q1 = a.indptr_t[j_first + 1];
    float4 mask = four_of(j_first);
    const int label = wv < nc ? a.labels[c0 + wv] : 0;
    int row_b = 0, row_e = 0, idx[kHeadChunks];
    float w[kHeadChunks];
    auto load_chunks = [&](int p0) {        // p0 < row_e
        auto chunk = [&](int k) {
            const int p = min(p0 + k * kWave + lane, row_e - 1);
            idx[k] = a.indices[p];
            w[k] = a.values[p];
        };
        chunk(0);
        if (p0 + kWave < row_e)             // uniform
#pragma unroll
            for (int k = 1; k < kHeadChunks; ++k) chunk(k);
    };
    if (wv < a.rows && MIRROR_LDS) {
        row_b = a.indptr[wv];
        row_e = a.indptr[wv + 1];
        if (row_b < row_e) load_chunks(row_b);
    }
    constexpr int kM = 8;                   // nnz <= 8 * 1024 (head_ok)
    float mw[kM];
    int mi[kM];
    auto mirror_load = [&](int k) {
        const int q = min(k * kBlock + static_cast<int>(threadIdx.x), a.nnz - 1);
        mw[k] = a.values_t[q];
        mi[k] = a.indices_t[q];
    };
    auto mirror_keep = [&](int k) {
        const int q = k * kBlock + threadIdx.x;
        if (q < a.nnz) {
            wt[q] = mw[k];
            it[q] = static_cast<unsigned char>(mi[k]);
        }
    };
    if constexpr (MIRROR_LDS) {
        if (a.nnz > 0) mirror_load(0);
        if (a.nnz > kBlock)                 // uniform
#pragma unroll
            for (int k = 1; k < kM; ++k) mirror_load(k);
    }
    if constexpr (IN_LDS) {
        if (j0 < a.cols) xs[j0] = mask;
        for (int j = j0 + kBlock; j < a.cols; j += kBlock) xs[j] = four_of(j);
    }
    if constexpr (MIRROR_LDS) {
        if (a.nnz > 0) mirror_keep(0);
        if (a.nnz > kBlock)
#pragma unroll
            for (int k = 1; k < kM; ++k) mirror_keep(k);
    }
    if constexpr (IN_LDS || MIRROR_LDS) __syncthreads();

    for (int i = wv; i < a.rows; i += kWavesPerBlock) {
        if (i != wv || !MIRROR_LDS) {
            row_b = a.indptr[i];
            row_e = a.indptr[i + 1];
            if (row_b < row_e && MIRROR_LDS) load_chunks(row_b);
        }
        float acc[kHeadCols] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (!MIRROR_LDS)
            for (int p = row_b + lane; p < row_e; p += kWave) fma_into(acc, a.values[p], four_of(a.indices[p]));
        for (int p0 = MIRROR_LDS ? row_b : row_e; p0 < row_e; p0 += kHeadChunks * kWave) {
            float4 x[kHeadChunks];
#pragma unroll
            for (int k = 0; k < kHeadChunks; ++k)
                if (p0 + k * kWave < row_e) x[k] = IN_LDS ? xs[idx[k]] : four_of(idx[k]);  // uniform
            float wk[kHeadChunks];
#pragma unroll
            for (int k = 0; k < kHeadChunks; ++k) wk[k] = w[k];
            if (p0 + kHeadChunks * kWave < row_e) load_chunks(p0 + kHeadChunks * kWave);  // travel while these are added
#pragma unroll
            for (int k = 0; k < kHeadChunks; ++k)
                if (p0 + k * kWave + lane < row_e) fma_into(acc, wk[k], x[k]);
        }
#pragma unroll
        for (int c = 0; c < kHeadCols; ++c) acc[c] = group_sum<kWave>(acc[c]);
        if (lane == 0) {
            const float b = a.bias ? a.bias[i] : 0.f;
            z[i] = make_float4(acc[0] + b, acc[1] + b, acc[2] + b, acc[3] + b);
        }
    }
    __syncthreads();

    // softmax cross-entropy of column c0+wv by wave wv: one class per lane (rows <= 32)
    if (wv < nc) {
        float *zc = reinterpret_cast<float *>(z) + wv;
        const bool live = lane < a.rows;
        const float zi = live ? zc[lane * kHeadCols] : -INFINITY;
        const float m = wave_max(zi);
        const float lse = m + logf(group_sum<kWave>(live ? expf(zi - m) : 0.f));
        const float zt = group_sum<kWave>(lane == label ? zi : 0.f);  // one non-zero term: exact
        const float d = (expf(zi - lse) - (lane == label ? 1.f : 0.f)) / static_cast<float>(a.batch);
        if (live) {
            a.Z[static_cast<int64_t>(lane) * a.ldz + c0 + wv] = zi;
            a.dZ[static_cast<int64_t>(lane) * a.lddz + c0 + wv] = d;
            zc[lane * kHeadCols] = d;
        }
        if (lane == 0) a.loss_cols[c0 + wv] = lse - zt;
    }
    __syncthreads();

    for (int j = j0; j < a.cols; j += kBlock) {
        if (j != j0) {
            q0 = a.indptr_t[j];
            q1 = a.indptr_t[j + 1];
            mask = IN_LDS ? xs[j] : four_of(j);
        }
        float acc[kHeadCols] = {0.f, 0.f, 0.f, 0.f};
        for (int q = q0; q < q1; ++q) {
            if constexpr (MIRROR_LDS)
                fma_into(acc, wt[q], z[it[q]]);
            else
                fma_into(acc, a.values_t[q], z[a.indices_t[q]]);
        }
        const float4 o = keep_where_positive(make_float4(acc[0], acc[1], acc[2], acc[3]), mask);
        float *dr = a.dX + static_cast<int64_t>(j) * a.lddx + c0;
        if (nc == kHeadCols) {
            st4(dr, o);
        } else {
            dr[0] = o.x;
            if (nc > 1) dr[1] = o.y;
            if (nc > 2) dr[2] = o.z;
        }
    }
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline int elementwise_blocks(int64_t work_items)
{
    int64_t b = (work_items + kEwBlock - 1) / kEwBlock;
    if (b < 1) b = 1;
    if (b > 256 * 32) b = 256 * 32;  // 256 compute units; grid-stride beyond that
    return static_cast<int>(b);
}

// ... of for_runs_of_xcds, kEwBlock * each items to a work-group and turn: a turn for all, for the second would not follow the first's neighbours
inline int xcd_run_blocks(int64_t work_items, int each = 1)
{
    const int64_t b = (work_items + kEwBlock * each - 1) / (kEwBlock * each);
    return static_cast<int>(b < 1 ? 8 : b > (1 << 18) ? 1 << 18 : (b + 7) / 8 * 8);
}
inline int gather_blocks(int64_t n) { return xcd_run_blocks(n, n < kGatherMany ? 1 : kGatherEach); }

bool spmm_offsets_ok(const SpmmCall &a);

hipError_t spmm_go(SpmmCall a, hipStream_t s)
{
    a.wide_offsets = !spmm_offsets_ok(a);
    dim3 grid(a.blocks.n_blocks, (a.batch + 255) / 256);
    if (a.XM)
        hipLaunchKernelGGL(spmm_kernel<true>, grid, dim3(kBlock), 0, s, a);
    else
        hipLaunchKernelGGL(spmm_kernel<false>, grid, dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

template <int GS>
hipError_t spmm_grouped_go(const SpmmCall &a, hipStream_t s)
{
    dim3 grid(a.blocks.n_blocks);
    if (a.XM)
        hipLaunchKernelGGL((spmm_grouped_kernel<GS, true>), grid, dim3(kBlock), 0, s, a);
    else
        hipLaunchKernelGGL((spmm_grouped_kernel<GS, false>), grid, dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

// The gathered operand (and its mask) should stay in one 4 MiB L2 while it is being gathered
// from: if the whole operand is too large for that, the batch is walked in column tiles of
// 4 * (return value) columns.  0: no tiling.
int spmm_tile_group(const SpmmCall &a)
{
    if (static_cast<int64_t>(a.blocks.n_blocks) * ((a.batch + 31) / 32 + 8) >= (1ll << 31)) return 0;
    return tile_columns(a.x_rows, a.batch, a.nnz, a.rows, a.blocks.staged_longest_row, a.blocks.hot_share, a.XM != nullptr) / 4;
}

constexpr int64_t kMaxGridIds = (1ll << 31) - 1;

// Grid and order of launches in column tiles (tile_of_block).  Whole tiles leave some XCDs idle in the last round; equal runs do not, but an L2 then sees one tile more and
// shares two.  From eight tiles on runs pay where whole tiles waste an eighth or more: 8192^2 uniform at 0.6 %, batch 600 / 700 (10 / 11 tiles), forward 70.1 -> 48.7
// and 71.9 -> 57.8 us; 16384^2 at 1 %, batch 600: 633 -> 406, at batch 850 (14): 702 -> 625, at 900 (15) 707 -> 665; 1314 x 6656 at 0.6 %, batch 850: 33.7 -> 31.1, 2000 x 8192
// at 1.2 %: 52.5 -> 47.5; but 4000 x 9000 at 1.2 %, batch 850 / 900: 77.1 -> 84.0, 77.1 -> 87.6, and
// with rows of different lengths 3000 x 12000 at 0.4 %: 66.9 -> 73.7, 66.5 -> 77.2.
// Fewer tiles, which all XCDs walk together otherwise: only products whose tile is well within an L2 (8192^2 at 0.6 %, batch 300, 5 tiles: 35.9 -> 31.5), as gradients lose
// (5000^2 at 2 %, batch 200: 39.5 -> 42.9) and so do tiles that fill one (16384^2 at 1 %, batch 200: 161 -> 168), and where an operand row is gathered so
// rarely that bringing the tile counts: 4000 x 9000 at 1.2 % (48 entries a row), batch 300: 20 % faster, 8192^2 at 1.2 % (98), batch 200 / 300: 49.0 -> 53.0, 8 % faster, at 3 %
// (245) 101 -> 110, 127 -> 145; power-law 8192^2 at 1.2 %, batch 256, transposed: 47.0 -> 58.3; 5000^2 at 7 %, batch 350 / 700 (3 / 6): 86 -> 93, 168 -> 152.
// Rows of very different lengths are strewn over a run that does not hold whole tiles, for the long ones come first in each.
struct TiledLaunch {
    int x_rows, rows, longest_row;
    int64_t nnz;
    float hot_share;
};
inline TileOrder tile_order(int n_tiles, int64_t n_blocks, int gs, bool product, const TiledLaunch &t)
{
    const int64_t tile_bytes = static_cast<int64_t>(t.x_rows) * gs * 16;
    const bool small = product && tile_bytes <= (5 << 19);   // (2.5 MiB)
    const bool skewed = static_cast<int64_t>(t.longest_row) * t.rows > 4 * t.nnz, hot = t.hot_share >= 0.5f;
    if (n_tiles < 8) {
        const bool rarely = t.nnz <= (skewed || hot ? (n_tiles == 7 ? 128ll : 40ll) : n_tiles >= 5 ? 128ll : 90ll) * t.x_rows;
        const bool long_rows = skewed && !hot && n_tiles >= (gs == 32 && tile_bytes >= (15 << 17) ? 5 : 7);   // (among short ones)
        if (!small || !(rarely || long_rows)) return TileOrder{kTilesOneByOne, 1};
    } else {
        const double waste = (n_tiles + 7) / 8 * 8 / static_cast<double>(n_tiles);
        const bool runs = waste >= 1.15 || (!skewed && (waste >= 1.13 ? !small || 2 * t.rows >= t.x_rows || t.rows <= 2048 : waste >= 1.06 && tile_bytes >= (7 << 19) && t.nnz <= 512ll * t.x_rows));
        if (!runs) return TileOrder{kTilesWhole, 1};
    }
    TileOrder order{static_cast<int>((n_tiles * n_blocks + 7) / 8), 1};
    if (n_blocks < 8 || n_blocks >= (1 << 16) || !skewed) return order;   // (so many are strewn widely enough: gradients of 300000 x 8192 power-law at 0.2 %, batch 600 1374 us either way)
    order.stride = static_cast<int>(n_blocks * 0.618);
    while (std::gcd(order.stride, static_cast<int>(n_blocks)) != 1) ++order.stride;
    return order;
}
inline int64_t tile_grid(const TileOrder &order, int64_t n_tiles, int64_t n_blocks)
{
    return order.per > 0 ? 8ll * order.per : order.per == kTilesWhole ? (n_tiles + 7) / 8 * 8 * n_blocks : n_tiles * n_blocks;
}
template <typename Args>
inline TiledLaunch tiled_launch(const Args &a) { return TiledLaunch{a.x_rows, a.rows, a.blocks.staged_longest_row, a.nnz, a.blocks.hot_share}; }

template <int GS>
hipError_t spmm_tiled_go(const SpmmCall &a, hipStream_t s)
{
    const int n_tiles = (a.batch + GS * 4 - 1) / (GS * 4);
    const TileOrder order = tile_order(n_tiles, a.blocks.n_blocks, GS, true, tiled_launch(a));
    const int64_t ids = tile_grid(order, n_tiles, a.blocks.n_blocks);
    dim3 grid(static_cast<unsigned>(ids));
    if (a.XM)
        hipLaunchKernelGGL((spmm_tiled_kernel<GS, true>), grid, dim3(kBlock), 0, s, a, n_tiles, order);
    else
        hipLaunchKernelGGL((spmm_tiled_kernel<GS, false>), grid, dim3(kBlock), 0, s, a, n_tiles, order);
    return hipGetLastError();
}

// Work-groups of the packed launch for lane groups of gs lanes: those that serve the short rows, and
// the launch's grid size.  One place, so that the launch and the checks that the grid fits agree.
struct PackedGrid {
    int n_tiles, n_pack_blocks;
    TileOrder order;
    int64_t ids;
    bool long_rows;   // (else spmm_packed_only_kernel)
};
PackedGrid packed_grid(const SpmmCall &a, int gs, bool with_long_rows)
{
    PackedGrid g;
    const int ne = kWave / gs;
    g.n_tiles = (a.batch + gs * 4 - 1) / (gs * 4);
    const int64_t n_sets = (static_cast<int64_t>(a.blocks.n_short) + ne - 1) / ne;
    g.long_rows = with_long_rows && a.blocks.n_long_blocks > 0;
    const int sets = (g.long_rows ? kWavesPerBlock : kPackWaves) * kPackSets;   // of a work-group
    g.n_pack_blocks = static_cast<int>((n_sets + sets - 1) / sets);
    const int64_t nrb = static_cast<int64_t>(g.n_pack_blocks) + (g.long_rows ? a.blocks.n_long_blocks : 0);
    g.order = tile_order(g.n_tiles, nrb, gs, true, tiled_launch(a));
    g.ids = tile_grid(g.order, g.n_tiles, nrb);
    return g;
}
template <int GS>
hipError_t spmm_packed_go(const SpmmCall &a, hipStream_t s)
{
    const PackedGrid pg = packed_grid(a, GS, true);
    const int n_tiles = pg.n_tiles, n_pack_blocks = pg.n_pack_blocks;
    const TileOrder order = pg.order;
    if (pg.ids > kMaxGridIds) return hipErrorInvalidConfiguration;  // (callers check before choosing this path)
    dim3 grid(static_cast<unsigned>(pg.ids));
    if (!pg.long_rows) {
        const auto kernel = a.XM ? spmm_packed_only_kernel<GS, true> : spmm_packed_only_kernel<GS, false>;
        hipLaunchKernelGGL(kernel, grid, dim3(kPackWaves * kWave), 0, s, a, n_tiles, order, n_pack_blocks);
    } else if (a.XM)
        hipLaunchKernelGGL((spmm_packed_kernel<GS, true>), grid, dim3(kBlock), 0, s, a, n_tiles, order, n_pack_blocks);
    else
        hipLaunchKernelGGL((spmm_packed_kernel<GS, false>), grid, dim3(kBlock), 0, s, a, n_tiles, order, n_pack_blocks);
    return hipGetLastError();
}

// go(SPARE) for kernels whose work-groups cover `columns` of the batch at a time
template <typename F>
void with_spare(int batch, int columns, F &&go)
{
    if (batch % columns) go(std::true_type{});
    else go(std::false_type{});
}

template <int G, int NV>
hipError_t sddmm_go(const SddmmCall &a, hipStream_t s)
{
    dim3 grid(a.blocks.n_blocks);
    with_spare(a.batch, G * 4 * NV, [&](auto spare) { hipLaunchKernelGGL((sddmm_kernel<G, NV, decltype(spare)::value>), grid, dim3(kBlock), 0, s, a); });
    return hipGetLastError();
}

// The grouped kernels address the gathered operand with 32-bit byte offsets from its base.
inline bool spans_below_4gib(int64_t rows, int64_t ld) { return rows * ld * 4 < (1ll << 32); }

// The staged product pays where a work-group finds several stored entries per operand row it
// copies into LDS, fills its column tiles, and has enough siblings to occupy the chip; where the
// segments are long (the gathers then dominate everything else) or the operand is beyond any
// L2 and evenly used (the gathers of the other kernels then go to memory); and where no single lane row's share,
// served at about one entry per 60 ns, outlasts the rest of the matrix, which
// the chip's 256 LDS serve at about one entry and tile per 3.3 ns each.
bool spmm_dense_rows_ok(const SpmmCall &a)
{
    return dense_rows_product_ok(a.split, a.x_rows, a.batch) && !a.XM && spmm_offsets_ok(a);
}
bool sddmm_dense_rows_ok(const SddmmCall &a)
{
    return dense_rows_sddmm_ok(a.split, a.batch) && sampled_operands_ok(a);
}

bool staged_pays(const RowBlocks &blocks, int32_t x_rows, int32_t batch, int32_t long_segment)
{
    if (!blocks.staged_rows || batch < kStageMinBatch) return false;
    // (an operand of a few rows is in cache wherever it is gathered from: config 4's 8192 x 10 mirror, 21 against 28 us)
    if (x_rows < kStageRows / 2 && !blocks.staged_preferred) return false;
    const int64_t rows = blocks.staged_row_count, nnz = blocks.staged_nnz;  // what the plan covers
    const int64_t n_tiles = (batch + kStageCols - 1) / kStageCols;
    if (!blocks.staged_preferred && static_cast<int64_t>(batch) * 5 < n_tiles * kStageCols * 4) return false;  // a fifth or more of the tiles' columns idle
    const int64_t groups = n_tiles * blocks.staged_ranges;
    if (groups >= (1ll << 31)) return false;
    if (blocks.staged_preferred) return true;
    // (three quarters of the compute units busy at least; half where the plan covers a matrix's long rows only,
    // whose alternative is gathering from memory: 580 long rows of the 0.3 % power-law matrix make 144 work-groups)
    if (groups < (blocks.staged_partial ? kStageTargetGroups / 2 : kStageTargetGroups * 3 / 4)) return false;
    if (static_cast<double>(nnz) < static_cast<double>(kStageMinReuse) * blocks.staged_ranges * x_rows) return false;
    if (static_cast<int64_t>(blocks.staged_longest_share) * 4096 > nnz * n_tiles) return false;
    // An operand beyond the L2s, evenly used, on rows of similar length: shorter segments already pay, because the other kernels' gathers partly go
    // to memory there (a few hot operand rows that take most gathers would stay cached on the other paths; on a power-law matrix most (row, block)
    // pairs hold one entry or none and cost a visit all the same).  16384^2 uniform matrices at batch 1024, column-tiled -> staged, us: products at
    // 0.6 / 0.7 / 0.79 / 1 / 2 % (3.1, 3.6, 4.0, 5.1 and 10.2 entries per segment) 345 -> 424, 414 -> 429, 525 -> 437, 662 -> 458, 1331 -> 598, SDDMM
    // 512 -> 500, 594 -> 521, 666 -> 572, 834 -> 680, 1656 -> 805; 44 others of 12300 columns and more, batch 768 and more: 0.88 to 1.06 below 4
    // entries, 0.50 to 0.92 from there on.
    const bool big_operand = static_cast<int64_t>(x_rows) * batch * 4 >= kStageBigOperand && blocks.hot_share < 0.5f &&
                             static_cast<int64_t>(blocks.staged_longest_row) * rows <= 4 * nnz;
    const int64_t segment = big_operand ? std::min(long_segment, kStageSegmentBigOperand) : long_segment;
    return nnz >= segment * rows * blocks.staged_cblocks;
}

// Entries times columns for the rules of shorter segments: of the rows that the plan covers, which beside dense rows (DenseSplit) or in a plan of the
// long rows are a part of the matrix (weight gradient of 5000^2 power-law at 10 %, batch 256, 640 M in all, 186 M staged: 78 us in column tiles, 103
// staged), and none where copying the operand weighs too much beside them (column tiles / staged, entries per copied row: products of 7278 x 12626
// and 8772 x 13004, batch 256 97 / 102 us (2.2), 101 / 106 (2.3), 6024 x 14996, batch 384 171 / 125 (2.6); gradients of 5901 x 11786, batch 192 93 /
// 104 (2.3), 4665 x 10700, batch 320 100 / 97 (2.6)).
static int64_t staged_work(const RowBlocks &blocks, int32_t x_rows, int32_t batch)
{
    return blocks.staged_nnz * 2ll >= 5ll * blocks.staged_ranges * x_rows ? static_cast<int64_t>(blocks.staged_nnz) * batch : 0;
}

// Short even rows in 64-column tiles for the sake of the packed kernel and its small work-groups, where the rule of the tiles (tile_columns) leaves
// the operand whole: one beyond an L2 whose rows are gathered a dozen times or more (and not so often that it stays in cache), tiles hardly empty.
// Uniform rows, whole -> in tiles, us: 15997 x 15191 at 0.35 %, batch 372 126 -> 79; 3894 x 6816 at 0.6 %, batch 227 15.9 -> 11.8; 16384^2 at 0.3 %,
// batch 300 103 -> 61; 10442 x 13851 at 0.37 %, batch 164 38.8 -> 27.9.  But tiles a fifth empty or more: 10681 x 8704 at 0.8 %, batch 134 36.5 ->
// 42.3, 11466 x 5888 at 0.5 %, batch 263 30.2 -> 34.0; operands near an L2: 4545 x 5628 at 0.7 %, batch 189 13.1 -> 14.1; often gathered: 16000 x
// 5000 at 0.8 %, batch 200 29.0 -> 31.2, 3182 x 2692 at 1.9 %, batch 580 25.7 -> 28.3; rarely: 3428 x 12999 at 0.33 %, batch 290 25.3 -> 26.7.  (More
// work than kFusedMinWork whatever the shape: in a training step such a transposed product shares its gathers, or both pipelines follow the chain's
// order (chain_shape_ok), and it is never in another launch's grid, which would add in another order.)
constexpr int64_t kFusedMinWork = 16 << 20;        // (backward_fused_ok)
constexpr int64_t kPackTilesOperand = 21ll << 18;  // operand bytes
constexpr int64_t kPackTilesGathers = 13;          // entries per operand row
static_assert(kPackTilesOperand / 4 * kPackTilesGathers >= kFusedMinWork, "");
static bool packed_tiles_pay(const SpmmCall &a)
{
    if (a.batch <= 128 || a.XM || a.blocks.n_short != a.rows || a.blocks.hot_share >= 0.5f) return false;
    if (static_cast<int64_t>(a.blocks.staged_longest_row) * a.rows > 4ll * a.nnz || (a.batch + 63) / 64 * 320 > 6 * a.batch) return false;
    const int64_t row_bytes = static_cast<int64_t>(a.x_rows) * 4, operand = row_bytes * a.batch, most = operand >= (11ll << 20) ? 90 : 55;
    return operand >= kPackTilesOperand && row_bytes * 64 <= (4ll << 20) && a.nnz >= 28ll * a.rows && a.nnz >= kPackTilesGathers * a.x_rows && a.nnz <= most * a.x_rows &&
           packed_grid(a, 16, true).ids <= kMaxGridIds;
}

int spmm_tile_group(const SpmmCall &a);
constexpr int64_t kSplitMinOperand = 48ll << 20;  // operand bytes from which long rows go into column tiles of their own: beyond the eight L2s

// Lanes per row (4 columns each) of the column tiles in which the LONG rows of a matrix run while its short rows run
// untiled: for an operand that the L2s together cannot hold, gathered about evenly, on a matrix whose long rows
// (beyond kPackMaxLen entries; they have a partition of their own) hold most of the stored entries.  0: no split.
int spmm_split_group(const SpmmCall &a)
{
    if (a.blocks.n_long_blocks <= 0 || a.blocks.n_rest_blocks <= 0 || a.batch < 128) return 0;
    if (static_cast<int64_t>(a.x_rows) * a.batch * 4 < kSplitMinOperand || a.blocks.hot_share >= 0.5f) return 0;
    if (static_cast<int64_t>(a.blocks.long_nnz) * 2 < a.nnz) return 0;
    const int64_t budget = (a.XM ? 5 : 10) * (1 << 18), row_bytes = static_cast<int64_t>(a.x_rows) * 4;
    // 64-column tiles as long as a tile of the operand fits an L2 at all (measured on a 16384-row operand at 1024
    // columns: 137 us with 64-column tiles, 150 with 128, 174 with 32 -- a pass over the long rows per tile
    // costs more than the misses of a tile that fills the L2 -- and 173 us unsplit)
    int g = 0;
    if (row_bytes * 128 <= budget) g = 32;
    else if (row_bytes * 64 <= (a.XM ? (2ll << 20) : (4ll << 20))) g = 16;
    else if (row_bytes * 32 <= budget) g = 8;
    if (g == 0) return 0;
    const int64_t n_tiles = (a.batch + g * 4 - 1) / (g * 4);
    if ((n_tiles + 8) * a.blocks.n_long_blocks > kMaxGridIds) return 0;
    return g;
}

bool spmm_staged_ok(const SpmmCall &a);
// The product in strips, us, with the ranges that make it shortest: rounds of 256 work-groups (one fits a compute unit), each the steps that its LDS
// serves, the sets that a wave takes one after the other, and the copy of the operand's strip; before them the stream.  Fitted, as the estimates of
// the other kernels below, to 28600 uniform matrices of 300 to 16384 rows, 1024 to 16384 columns, 0.1 to 10 %, batch 193 to 1024, and to the next
// best number of ranges: root mean square 6.6 %, 1 % off at any number of blocks.
struct StripPlan {
    StripGrid grid;
    double us;
};
static StripPlan strip_plan(int32_t rows, int32_t x_rows, int32_t batch, int32_t blocks, double steps, double chunks)
{
    StripPlan p{};
    p.grid.n_tiles = (batch + kStripCols - 1) / kStripCols;
    const int64_t sets = (static_cast<int64_t>(rows) + kStripSet - 1) / kStripSet, least = (sets + kStripWaves * kStripJ - 1) / (kStripWaves * kStripJ);
    const double per_set = steps / static_cast<double>(sets);
    for (int64_t more = 0, first = (p.grid.n_tiles * least + 255) / 256; more < 4; ++more) {   // (of the ranges that a number of rounds holds the most)
        const int64_t r = std::max(least, 256 * (first + more) / p.grid.n_tiles);
        const double rounds = static_cast<double>((p.grid.n_tiles * r + 255) / 256), most = static_cast<double>((sets + kStripWaves * r - 1) / (kStripWaves * r));
        const double us = rounds * (6.8 + 2.06e-3 * steps / static_cast<double>(r) + 20.7e-3 * most * per_set + 0.46e-3 * x_rows + 2.07 * blocks);
        if (p.grid.n_ranges == 0 || us < p.us) { p.us = us; p.grid.n_ranges = static_cast<int>(r); }
    }
    p.us += 6.6 + 0.62e-3 * chunks;
    p.grid.per = static_cast<int>((static_cast<int64_t>(p.grid.n_tiles) * p.grid.n_ranges + 7) / 8);
    return p;
}
static StripPlan strip_plan(const SpmmCall &a) { return strip_plan(a.rows, a.x_rows, a.batch, a.strips->blocks, a.strips->steps, a.strips->chunks); }
// The kernel that would run otherwise, us: staged, in column tiles (of 128, or of 64 and fewer) or over the whole batch; 3.5, 8.8, 17 (3 to 16 too
// short in the mean) and 10 % root mean square.  0: not known well enough for a comparison.
static double other_product_us(const SpmmCall &a)
{
    const double nnz = a.nnz * 1e-6, x_rows = a.x_rows * 1e-6, rows = a.rows * 1e-6, operand = 4. * x_rows * a.batch;   // (millions)
    if (spmm_staged_ok(a)) {
        const int tiles = (a.batch + kStageCols - 1) / kStageCols, ranges = a.blocks.staged_ranges;
        const double rounds = static_cast<double>((static_cast<int64_t>(tiles) * ranges + kStageTargetGroups - 1) / kStageTargetGroups);
        return 2.1 + tiles * (0.36 * nnz + 9.5 * rows * a.blocks.staged_cblocks) + rounds * (7.2 + 652. * nnz / ranges + 4600. * x_rows);
    }
    if (a.rows < kPackMinRows) return 0.;   // (few sets, which the strips' estimate is too kind to: 1223 x 4592 at 10 %, batch 466 46.8 -> 56.3)
    int tg = spmm_tile_group(a);
    if (tg == 0 && packed_tiles_pay(a)) tg = 16;
    if (tg == 0) return 6. + 4. * nnz * a.batch * (0.0228 + 0.0262 * std::max(operand - 4., 0.) / 8.) + 10.9 * nnz * ((a.batch + 255) / 256) + 0.3 * operand + 0.033 * rows * a.batch;
    const double gathers = nnz * ((a.batch + tg * 4 - 1) / (tg * 4)) * tg * 16., tile = x_rows * tg * 16. / 4.194304;
    if (tg == 32) return 7.4 + gathers * (0.0294 + 0.0118 * tile) + 0.36 * rows * a.batch;
    return 6.2 + gathers * (0.036 + 0.015 * std::min(tile, 2.)) + 0.2 * operand - 0.4 * rows * a.batch;
}
// Where strips pay: of the matrices above that take them 0.75 % are slower by 3 % or more, the worst by 14 %; all in all they are 1.32 times as fast.
// (A line that asks less of the strips, 0.98: 1.27 times, but 3 % of the matrices slower.)
static bool strip_pays(double strips, double other) { return strips < 0.94 * other; }
bool spmm_strip_ok(const SpmmCall &a)
{
    if (!a.strips || !a.strip_stream || a.XM || a.batch <= kStripFromBatch) return false;
    const int64_t groups = (static_cast<int64_t>(a.rows) + kStripSet * kStripWaves * kStripJ - 1) / (kStripSet * kStripWaves * kStripJ) * ((a.batch + kStripCols - 1) / kStripCols);
    return groups < (1 << 28) && (a.strips->preferred || strip_pays(strip_plan(a).us, other_product_us(a)));
}

bool spmm_staged_ok(const SpmmCall &a)
{
    if (a.x_rows < 64 || a.nnz < 64) return false;  // (it brings 64 operand rows at a time, and reads entries up to 32 past the first)
    if (!staged_pays(a.blocks, a.x_rows, a.batch, staged_work(a.blocks, a.x_rows, a.batch) >= kStageSomeWork ? kStageSegmentSomeWork : kStageLongSegment)) return false;
    return !a.blocks.staged_partial || a.blocks.n_rest_blocks > 0;  // (the rows the plan leaves out need a partition of their own)
}

// whether the rows a partial plan leaves out take the packed kernel, which runs inside column tiles only
bool staged_rest_packed(const SpmmCall &a, int tg)
{
    return a.blocks.n_short > 0 && tg != 0 && spmm_offsets_ok(a) && packed_grid(a, tg, false).ids <= kMaxGridIds;
}

bool sddmm_offsets_ok(const SddmmCall &a);

// a full matrix of few rows whose dZ fits in 64 KiB of LDS
bool sddmm_full_ok(const SddmmCall &a)
{
    if (a.rows > kFullMaxRows || a.x_rows < 256 || static_cast<int64_t>(a.nnz) != static_cast<int64_t>(a.rows) * a.x_rows) return false;
    if (a.batch < 64 || a.skip_products || a.dense || a.loss_cols || !sddmm_offsets_ok(a)) return false;
    return static_cast<int64_t>(a.rows) * ((a.batch + 255) / 256) <= 64;
}

// the staged SDDMM needs room for one slice of partial products per 64-column tile
bool sddmm_staged_ok(const SddmmCall &a)
{
    if (!a.partial || a.skip_products || a.dense || a.loss_cols || !sddmm_offsets_ok(a)) return false;
    if ((a.batch + kStageCols - 1) / kStageCols > a.partial_tiles) return false;
    if (a.x_rows < 64 || a.nnz < 64 || a.nnz >= (1 << 30)) return false;  // (as spmm_staged_ok; its byte offsets have 32 bits, and for so many entries there is no room for partial products)
    const int64_t work = staged_work(a.blocks, a.x_rows, a.batch);
    const int32_t segment = a.split_done && a.batch >= 512 ? kStageSegmentBesideDense : work >= kStageMuchWork ? kStageSegmentMuchWork : kStageLongSegmentSddmm;
    const int64_t rest_ids = static_cast<int64_t>(a.blocks.n_rest_blocks) * kSddmmParts * ((a.batch + kStageCols - 1) / kStageCols + 8);
    if (a.blocks.staged_partial && (a.blocks.n_rest_blocks <= 0 || rest_ids >= (1ll << 31))) return false;
    return staged_pays(a.blocks, a.x_rows, a.batch, segment);
}

bool spmm_offsets_ok(const SpmmCall &a)
{
    return spans_below_4gib(a.x_rows, a.ldx) && (!a.XM || spans_below_4gib(a.x_rows, a.ldxm));
}

void sddmm_finish_go(const SddmmCall &a, int n_tiles, hipStream_t s)
{
    const int64_t work = a.nnz > a.rows ? a.nnz : a.rows;
    hipLaunchKernelGGL(sddmm_finish_kernel, dim3(a.fused && a.values_t ? xcd_run_blocks(work) : elementwise_blocks(work)), dim3(kEwBlock), 0, s, a, n_tiles,
                       a.split_done ? a.split_done->rows : DenseRows{}, a.split_done ? a.split_done->flag : nullptr);
}

template <int G, int NV>
hipError_t sddmm_tiled_go(const SddmmCall &a, hipStream_t s, BackwardFinish *first = nullptr)
{
    const int W = G * 4 * NV;
    const int n_tiles = (a.batch + W - 1) / W;
    const int n_blocks = a.blocks.n_blocks * kSddmmParts;
    const TileOrder order = tile_order(n_tiles, n_blocks, W / 4, false, tiled_launch(a));
    const int64_t ids = tile_grid(order, n_tiles, n_blocks);
    dim3 grid(static_cast<unsigned>(ids));
    if (first && ids >= (1 << 23)) {   // (threads are counted in 32 bits)
        const hipError_t e = launch_backward_finish(*first, s);
        if (e != hipSuccess) return e;
    }
    with_spare(a.batch, W, [&](auto spare) {
        if constexpr (G == 16) {
            if (first && first->waiting) {
                const int n_finish = first->n_entry_blocks + first->n_row_blocks, groups = (n_finish + 7) / 8;
                const int64_t eights = (ids + 7) / 8 + groups;
                first->waiting = false;
                hipLaunchKernelGGL((sddmm_tiled_finish_kernel<NV, decltype(spare)::value>), dim3(static_cast<unsigned>(eights * 8)), dim3(kSddmmWaves * kWave), 0, s, a,
                                   n_tiles, order, first->a, first->hot_at, first->n_tiles, first->n_entry_blocks, n_finish, static_cast<int>(eights / groups));
                return;
            }
        }
        hipLaunchKernelGGL((sddmm_tiled_kernel<G, NV, decltype(spare)::value>), grid, dim3(kSddmmWaves * kWave), 0, s, a, n_tiles, order);
    });
    sddmm_finish_go(a, n_tiles, s);
    return hipGetLastError();
}

// what the SDDMM kernels but the generic one ask for: four columns, 32-bit offsets into X
bool sddmm_offsets_ok(const SddmmCall &a)
{
    return a.batch >= 4 && (a.skip_products || spans_below_4gib(a.x_rows, a.ldx));
}

template <int GS_S, int G, int NV_D>
hipError_t pair_go(const SpmmCall &a, const SddmmCall &b, hipStream_t s)
{
    const int na = a.blocks.n_blocks * (GS_S == kWave ? (a.batch + 255) / 256 : 1);
    dim3 grid(na + b.blocks.n_blocks);
    with_spare(b.batch, G * 4 * NV_D, [&](auto spare) {
        hipLaunchKernelGGL((spmm_sddmm_pair_kernel<GS_S, G, NV_D, decltype(spare)::value>), grid, dim3(kBlock), 0, s, a, b, na);
    });
    return hipGetLastError();
}

template <int G, int NV_D>
hipError_t sddmm_pair_go(const SddmmCall &a, const SddmmCall &b, hipStream_t s)
{
    const int na = a.blocks.n_blocks;
    dim3 grid(na + b.blocks.n_blocks);
    with_spare(b.batch, G * 4 * NV_D, [&](auto spare) {
        hipLaunchKernelGGL((sddmm_pair_kernel<G, NV_D, decltype(spare)::value>), grid, dim3(kBlock), 0, s, a, b, na);
    });
    return hipGetLastError();
}

// Lanes per entry and columns of 4 per lane of the SDDMM that covers a batch with the fewest columns to spare: go(G, NV).
// (1000 x 3000 at 10 %, groups of 16 lanes with 4 against 3 of them: batch 160 16.0 and 12.7 us, batch 300 in groups of 64 and 32: 24.4 and 19.9.)
template <typename F>
hipError_t with_sddmm_lanes(int batch, F &&go)
{
    using std::integral_constant;
    if (batch <= 16) return go(integral_constant<int, 4>{}, integral_constant<int, 1>{});
    if (batch <= 32) return go(integral_constant<int, 8>{}, integral_constant<int, 1>{});
    if (batch <= 48) return go(integral_constant<int, 4>{}, integral_constant<int, 3>{});
    if (batch <= 64) return go(integral_constant<int, 16>{}, integral_constant<int, 1>{});
    if (batch <= 96) return go(integral_constant<int, 8>{}, integral_constant<int, 3>{});
    if (batch <= 128) return go(integral_constant<int, 16>{}, integral_constant<int, 2>{});
    if (batch <= 192) return go(integral_constant<int, 16>{}, integral_constant<int, 3>{});
    if (batch <= 256) return go(integral_constant<int, 16>{}, integral_constant<int, 4>{});
    if (batch <= 384) return go(integral_constant<int, 32>{}, integral_constant<int, 3>{});
    if (batch <= 512) return go(integral_constant<int, 64>{}, integral_constant<int, 2>{});
    if (batch <= 768) return go(integral_constant<int, 64>{}, integral_constant<int, 3>{});
    return go(integral_constant<int, 64>{}, integral_constant<int, 4>{});
}

}  // namespace

int sddmm_tile_columns(const SddmmCall &a);

static int tile_columns_wanted(int32_t x_rows, int32_t batch, int64_t nnz, int32_t rows, bool skewed, float hot_share, bool masked, bool for_sddmm)
{
    const int64_t budget = (masked ? 5 : 10) * (1 << 18);  // 2.5 MiB (half of it with a mask operand)
    const int64_t row_bytes = static_cast<int64_t>(x_rows) * 4;
    if (x_rows <= 0 || row_bytes * batch <= budget) return 0;
    // A matrix of few rows is in flight as a whole: its rows gather the same operand rows at about
    // the same time, which serves them from cache without tiling (measured on a dense 10 x 8192 layer).
    if (rows <= 256) return 0;
    // (the SDDMM, whose second operand is a row per matrix row and not a gather, still gains from 128-column
    // tiles when they fill a whole L2: config 4's 8192-row operand, 120 -> 113 us, where the product loses 7 %)
    // (and so do rows of very different lengths, most of them too short for the pass over them that every tile costs:
    // 9106 x 9383 power-law at 0.1 %, batch 1000: forward 63 us in 64-column tiles, 49 in 128; SDDMM 79 and 54)
    if (row_bytes * 128 <= (for_sddmm || skewed ? (5ll << 20) : budget) && batch > 128) return 128;
    if (row_bytes * 64 <= budget && batch > 64) return 64;
    if (batch <= 32) return 0;
    // Short rows on an operand whose 64-column tile (4 MiB for 16384 rows) no longer fits beside the rest in an L2: wide tiles
    // still pay at wide batches, because they cut the set of operand rows in flight by 8 to 16 and what misses the L2
    // then hits the infinity cache.  Measured on 16384^2 matrices at batch 1024 (512): uniform rows at 0.1 / 0.3 %,
    // products 165 -> 83 and 458 -> 197 us with 64 columns (109 / 282 with 128), SDDMM 156 -> 111 and 442 -> 271 with
    // 128; power-law rows at 0.1 %, forward 142 -> 110 (85 -> 60), SDDMM 165 -> 134 (80 -> 69; 147 with 64 columns).
    // Where a few operand rows take most gathers (the transposed product of the power-law matrix) 64 columns lose
    // (57 -> 63, 554 -> 597 us at 0.1 / 1 %) and 128 do not (58, 475).
    // (Beside the staged long rows of the power-law matrix at 1 % the short rows then run in 64- instead of 32-column
    // tiles: forward 495 -> 450 us.)
    // (The same holds with tiles twice that size: 32768^2 at batch 1024, uniform rows at 0.1 / 0.5 %, products 629 -> 478
    // and 2577 -> 1814 us; 12288^2: 94 -> 49 and 395 -> 163.)
    if (batch >= 512 && row_bytes * 64 <= (8ll << 20)) return for_sddmm || hot_share >= 0.5f ? 128 : 64;
    // Narrower batches (128 .. 511) on such an operand: 64-column tiles from about 128 entries per row on, unless a few
    // operand rows take most gathers.  16384^2 at 1 %, batch 128 / 256: uniform rows, products 105 -> 90 and 252 -> 173 us
    // (32-column tiles: 136, 250), SDDMM 108 -> 97 and 225 -> 181; power-law rows, forward 96 -> 81 and 210 -> 154,
    // SDDMM 93 -> 89 and 204 -> 164, transposed (hot rows) 83 -> 100 and 131 -> 171: left untiled.  At 16 entries per
    // row tiles lose at these batches (power-law 0.1 %, batch 128: forward 24 -> 36 us).
    if (batch >= 128 && row_bytes * 64 <= (4ll << 20) && row_bytes * batch >= (8ll << 20) && hot_share < 0.5f &&
        nnz >= static_cast<int64_t>(rows) * 128)
        return 64;
    // Narrower tiles, for operands larger still: they multiply the per-wave set-up (one pass
    // over the row partition per tile) by 32 or more.  Measured on 16384^2 matrices at batch 1024 against untiled
    // launches: they pay from about 128 entries per row on (1 % density: 1.48 -> 1.18 ms, 10 %: 1.4x) unless a few
    // operand rows take most of the gathers (the transposed product of a power-law matrix: 0.58 -> 1.08 ms); at 16
    // entries per row they lose, and so they do on an 8 MiB operand (batch 128), half of which an L2 holds anyway.
    if (nnz >= static_cast<int64_t>(rows) * 1024) return 32;
    if (nnz >= static_cast<int64_t>(rows) * 128 && hot_share < 0.5f && row_bytes * batch >= (16ll << 20)) return 32;
    return 0;
}

int tile_columns(int32_t x_rows, int32_t batch, int64_t nnz, int32_t rows, int32_t longest_row, float hot_share, bool masked, bool for_sddmm)
{
    const bool skewed = static_cast<int64_t>(longest_row) * rows > 16 * nnz;
    const int w = tile_columns_wanted(x_rows, batch, nnz, rows, skewed, hot_share, masked, for_sddmm);
    const int n_tiles = w > 0 ? (batch + w - 1) / w : 0;
    if (w == 0 || n_tiles >= 8) return w;
    // Fewer tiles than XCDs: either every L2 sees every tile, and an eighth of the gathers from it, or it sees few and its share of the work is short
    // (tile_order).  The tiles then pay where an L2 gathers a row of one several times and the untiled operand is well beyond the L2; a product's
    // also on an operand beyond three L2s whose rows are gathered rarely.  Rows of very different lengths: where enough is gathered from an operand
    // of two L2s; in products rows and columns of 48 entries, and tiles that fill much of an L2 (narrower ones lose), but no more than one where the
    // last of seven is partly empty.  Untiled / in tiles.  Even rows, 9106 x 9383 at 0.3 % (27 entries per operand row), batch 100 / 182 / 400:
    // forward 11.2 / 17.7 / 40.5 and 16.1 / 18.4 / 39.7 us, at 0.1 %: SDDMM 7.8 / 11.2 / 22.4 and 10.4 / 16.1 / 28.1, forward at batch 400 18.9 and
    // 14.5; 5000^2 at 0.3 %, batch 300 / 700 / 850: 11.5 / 21.2 / 25.9 and 10.6 / 17.4 / 18.8, but transposed 6656 x 1314 at 0.3 %, batch 400 (10
    // MiB): 10.1 and 15.6.  Power-law rows, forward: 9106 x 9383 at 0.6 %, batch 256 / 700: 48.3 / 112 and 38.4 / 94; 3000 x 12000 at 3.5 %, batch
    // 256: 115 and 67, at 1.2 % 46.2 and 45.0; but 12000 x 3000 at 0.6 %, batch 700: 41.4 and 53.3, 5000^2 at 1.2 %: 52.6 and 61.3; 9106 x 9383 at
    // 1.2 %, batch 850: 209 and 225.  SDDMM: 5000^2 at 2 %, batch 300 / 700: 47.6 / 139 and 44.4 / 79; 8192^2 at 0.6 %, batch 256 / 850: 39.2 / 161
    // and 32.4 / 95, at 0.3 %, batch 400: 39.0 and 41.1; 12000 x 3000 at 0.3 %, batch 850: 40.7 and 58.0.
    const int64_t operand = static_cast<int64_t>(x_rows) * batch * 4, tile = static_cast<int64_t>(x_rows) * 4 * w;
    bool pays;
    if (!skewed)
        pays = operand >= (6ll << 20) && (nnz >= 24ll * x_rows || (operand >= (11ll << 20) && !for_sddmm && hot_share < 0.5f));
    else if (for_sddmm)
        pays = operand >= (8ll << 20) && nnz >= 24ll * rows && nnz * batch >= (90ll << 20);
    else
        pays = operand >= (8ll << 20) && nnz >= 48ll * x_rows && nnz >= 48ll * rows && tile > (5ll << 19) && (tile <= (4ll << 20) || n_tiles < 7);
    if (skewed) pays = pays || operand >= (32ll << 20) || (operand >= (8ll << 20) && nnz >= 128ll * x_rows);
    return pays ? w : 0;
}

// Few tiles of an operand whose rows are gathered rarely are for the product alone, with a gradient they lose: 9000 x 4000 at 0.3 %, batch 400, both
// gradients 30.2 -> 33.6 us in them; 9106 x 9383 at 0.1 % 28.9 -> 29.8.
static bool few_rare_tiles(const SpmmCall &a)
{
    const int columns = 4 * spmm_tile_group(a);
    return columns > 0 && (a.batch + columns - 1) / columns < 8 && a.nnz < 24ll * a.x_rows && static_cast<int64_t>(a.blocks.staged_longest_row) * a.rows <= 16 * a.nnz;
}

bool can_pair(const SpmmCall &a, const SddmmCall &b)
{
    return !sddmm_sampled_ok(b) && !sddmm_dense_rows_ok(b) && a.batch == b.batch && a.batch > 4 && a.batch <= 1024 && !a.XM && a.rows > 0 && b.rows > 0 &&
           a.blocks.n_blocks > 0 && b.blocks.n_blocks > 0 && spmm_offsets_ok(a) &&
           sddmm_offsets_ok(b) && (spmm_tile_group(a) == 0 || few_rare_tiles(a)) && !spmm_staged_ok(a) && sddmm_tile_columns(b) == 0 &&
           !sddmm_staged_ok(b) && !sddmm_full_ok(b);
}

bool can_pair(const SddmmCall &a, const SddmmCall &b)
{
    return !sddmm_sampled_ok(a) && !sddmm_sampled_ok(b) && !sddmm_dense_rows_ok(a) && !sddmm_dense_rows_ok(b) && a.batch == b.batch && a.batch > 0 && a.batch <= 1024 && a.rows > 0 && b.rows > 0 &&
           a.blocks.n_blocks > 0 && b.blocks.n_blocks > 0 && sddmm_offsets_ok(a) && sddmm_offsets_ok(b) &&
           sddmm_tile_columns(a) == 0 && sddmm_tile_columns(b) == 0 && !sddmm_staged_ok(a) && !sddmm_staged_ok(b) &&
           !sddmm_full_ok(a) && !sddmm_full_ok(b);
}

hipError_t launch_pair(const SpmmCall &a, const SddmmCall &b, hipStream_t s)
{
    return with_sddmm_lanes(a.batch, [&](auto g, auto nv) {
        // (the product's own lane groups for that many columns, as launch_spmm has them)
        constexpr int G = decltype(g)::value, NV = decltype(nv)::value, kColumns = G * NV * 4;
        return pair_go<(kColumns <= 32 ? 8 : kColumns <= 64 ? 16 : kColumns <= 128 ? 32 : 64), G, NV>(a, b, s);
    });
}

hipError_t launch_pair(const SddmmCall &a, const SddmmCall &b, hipStream_t s)
{
    return with_sddmm_lanes(a.batch, [&](auto g, auto nv) { return sddmm_pair_go<decltype(g)::value, decltype(nv)::value>(a, b, s); });
}

// Whether T_1 (t), S_1 (g1) and S_0 (g0) of a step can be one launch (chain_kernel): all three untiled, T_1's operand and mask those of S_1, its result
// that of S_0, no row of W_0 cut into several work-groups.  The waves of a row are those that W_0's partition gives it: the mirror must not be much the larger of the
// two or have long rows.  Steps at batch 100 apart / in one, us: 500-1000-1000-10 at 10 % (twice W_0's entries) 34.3 / 29.8, 300-1000-1000-10 (three times)
// 33.6 / 29.2.  Up to 192 columns: 2000-1500-400-10 at 5 %, batch 180 / 256: 37.2 / 34.4, 41.3 / 43.6.  Networks of a small hidden layer keep their two
// launches, which a profile of the step shows one by one (256-128-64-10 at 20 %: 20.9 / 18.6).
bool chain_pays(const SpmmCall &t, const SddmmCall &g0);
bool chain_shape_ok(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0)
{
    if (t.batch != g1.batch || t.batch > kChainMaxBatch || t.X != g1.dZ || t.ldx != g1.lddz || !t.YM || t.YM != g1.X || t.ldym != g1.ldx || t.Y != g0.dZ || t.ldy != g0.lddz) return false;
    if (!can_pair(t, g0) || !can_pair(t, g1) || t.nnz <= 0 || t.nnz != g1.nnz || t.rows != g0.rows) return false;
    if (g1.dense || g0.dense || g1.loss_cols || g0.loss_cols || g0.values_t || g0.ZM || g1.ZM) return false;
    return g0.blocks.n_huge_rows == 0 && t.rows >= kChainMinRows && t.blocks.staged_longest_row <= 2 * kPackMaxLen && t.nnz / 4 <= g0.nnz && chain_pays(t, g0);
}
bool chain_ok(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0)
{
    return g0.fused && g1.fused && g1.perm && g1.values_t && chain_shape_ok(t, g1, g0);
}

static ChainArgs chain_args(const SpmmCall &t, const SddmmCall &g1)
{
    ChainArgs c{};
    c.indptr_t = t.indptr; c.indices_t = t.indices; c.values_t = const_cast<float *>(t.values); c.perm = g1.perm; c.w = g1.values; c.velocity = g1.velocity;
    c.bias = g1.bias; c.bias_velocity = g1.bias_velocity; c.dZ = t.X; c.lddz = t.ldx; c.A = t.YM; c.lda = t.ldym; c.dZ_below = t.Y; c.lddz_below = t.ldy;
    c.rows = t.x_rows;
    return c;
}

// Lanes of chain_kernel: go(G, NV, GB, NVB).  Its first half waits for one gather after another, so three loads a lane, which spare the SDDMM columns (with_sddmm_lanes), are
// too many: steps of 3072-1024-512-10 at 2 %, batch 38 / 77 / 150, apart 24.1 / 24.3 / 27.1, with the SDDMM's lanes 24.9 / 24.6 / 26.6, with these 20.1 / 22.5 / 25.1;
// 1000-300-300-10 at 12 %: 23.6 / 22.8 / 24.9, 26.9 / 25.2 / 25.7, 20.6 / 22.3 / 23.7.
template <typename F>
hipError_t with_chain_lanes(int batch, F &&go)
{
    return with_sddmm_lanes(batch, [&](auto gb, auto nvb) {
        constexpr int kColumns = decltype(gb)::value * decltype(nvb)::value * 4, G = kColumns <= 16 ? 4 : kColumns <= 32 ? 8 : kColumns <= 128 ? 16 : 32,
                      NV = kColumns <= 64 ? 1 : 2;
        if constexpr (kColumns <= kChainMaxBatch) return go(std::integral_constant<int, G>{}, std::integral_constant<int, NV>{}, gb, nvb);
        else return hipErrorInvalidConfiguration;   // (chain_shape_ok)
    });
}

hipError_t launch_chain(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0, const SddmmCall *waiting, hipStream_t s)
{
    const ChainArgs c = chain_args(t, g1);
    SddmmCall b{};
    if (waiting) b = *waiting;
    return with_chain_lanes(t.batch, [&](auto g, auto nv, auto gb, auto nvb) {
        constexpr int G = decltype(g)::value, NV = decltype(nv)::value, kRows = kWavesPerBlock * (kWave / G);
        const int n_sum_blocks = c.bias ? (t.x_rows + kRows - 1) / kRows : 0;
        const dim3 grid(g0.blocks.n_blocks + n_sum_blocks + b.blocks.n_blocks);
        with_spare(t.batch, G * 4 * NV, [&](auto spare) {
            hipLaunchKernelGGL((chain_kernel<G, NV, decltype(gb)::value, decltype(nvb)::value, decltype(spare)::value>), grid, dim3(kBlock), 0, s, c, g0, b, n_sum_blocks);
        });
        return hipGetLastError();
    });
}

hipError_t launch_chain_transposed(const SpmmCall &t, const SddmmCall &g1, const SddmmCall &g0, hipStream_t s)
{
    return with_chain_lanes(t.batch, [&](auto g, auto nv, auto, auto) {
        hipLaunchKernelGGL((chain_transposed_kernel<decltype(g)::value, decltype(nv)::value>), dim3(g0.blocks.n_blocks), dim3(kBlock), 0, s, chain_args(t, g1), g0);
        return hipGetLastError();
    });
}

// The transposed product t and the SDDMM g of one layer can share their gathers when its result mask, if any, is the
// SDDMM's second operand (the output of the layer below), no mirror row outlasts the rest, and the layer's partial
// buffer has a slice per tile for the products in mirror order.
// Small work on short rows, two column tiles: a wave takes its entries through both, which leaves no second launch (546 x 2764 at
// 0.12 %, batch 300: 16.3 -> 6.4 us; through four tiles it is the longer way, 2592 x 702 at batch 933: 18).
constexpr int64_t kBackwardSmallWork = 8 << 20;   // entries times columns: a few us of gathers, a launch costs 3.5
static bool backward_looped(const SpmmCall &t)
{
    return t.batch > 128 && t.batch <= 512 && t.blocks.staged_longest_row <= kWave && static_cast<int64_t>(t.nnz) * t.batch <= kBackwardSmallWork;
}
// Lanes per mirror row of the fused backward pass: the transposed product's own tiles where it has any, else one tile up to 128
// columns, up to 256 where the operand is small or the rows are short (16384 x 2000 power-law at batch 256 in two tiles: 26 us, in one 29;
// 12000^2 at 0.1 %: 27 and 24), and tiles of 128 beyond; its own tiles are widened to 128 columns
// while a tile of dZ still fills no more than an L2 -- half as many tiles halve the partial products that go
// out and come back (wide MLP, 8192 x 8192 layer: 128.6 -> 122.6 us; the product alone loses 7 % with them).
static int backward_tile_group(const SpmmCall &t)
{
    if (backward_looped(t)) return 64;
    const int tg = few_rare_tiles(t) ? 0 : spmm_tile_group(t);
    if (tg == 16 && t.batch > 128 && static_cast<int64_t>(t.x_rows) * 4 * 128 <= (4ll << 20)) return 32;
    if (tg == 0) return t.batch <= 32 ? 8 : t.batch <= 64 ? 16 : t.batch <= 128 || t.batch > 256 || (t.x_rows > 4096 && t.nnz > 16 * static_cast<int64_t>(t.rows)) ? 32 : 64;
    if (tg == 8) return 16;
    return tg;
}
// log2 of the lane groups that share a mirror row: more of them where the rows alone do not make 4096 waves, as long as the
// shares are not shorter than a pass
static int backward_split(const SpmmCall &t, int tg, int n_tiles)
{
    int lg = 0;
    while ((tg << lg) < kWave && (static_cast<int64_t>(t.rows) * tg << lg) / kWave * n_tiles < 4096 && static_cast<int64_t>(t.rows) * (16 << lg) <= t.nnz) ++lg;
    return lg;
}
static int backward_tiles(const SpmmCall &t, int tg) { return (t.batch + tg * 4 - 1) / (tg * 4); }

// What the end of a step in one launch saves is 3 to 5 us whatever the work, and where there is much of it the launches apart are the faster ones,
// with more registers.  W_1: the entries of a mirror row lie a row of W_1 apart in its values and velocity.  Steps, us, apart -> in one (thousand
// entries of W_1 x thousand rows): 1000-2000-2000-10 at 5 / 10 % (200 x 2, 400 x 2), batch 64 39.8 -> 36.6, 51.9 -> 52.3, batch 16 33.9 -> 31.6, 39.8
// -> 45.0; 3000-3000-3000-10 at 1 / 2 / 5 % (90, 180, 450 x 3), batch 192 50.4 -> 48.6, 66.5 -> 67.5, 108 -> 112; 1500-3000-800-10 at 14 % (336 x
// 0.8), batch 64 54.5 -> 49.4, batch 16 39.6 -> 40.4; 1300-6600-700-10 (430 x 0.7), batch 80 78 -> 72; 3000-4000-4000-10 at 1 / 1.7 % (160, 272 x 4),
// batch 100 52.8 -> 48.9, 62.2 -> 64.1; 2498-7241-5799-13 at 0.5 / 1 / 1.7 % (29, 58 and 98 entries a mirror row), batch 64 47.4 -> 42.1, 62.8 ->
// 56.9, 80.9 -> 76.0, at 2.5 % 107 -> 112, batch 16 at 1 / 1.7 % 50.6 -> 51.6, 59.5 -> 68.6; where its backward pass alone takes two tiles, batch
// 150: 1.7 % 138 -> 122.  W_0's gradient beside a small W_1: 2500-700-64-10 at 30 % (525 and 13), batch 38 / 100: 34.0 -> 35.0, 42.9 -> 45.2, at 12 %
// 27.1 -> 25.0, 31.1 -> 30.2; 4000-6000-300-10 at 2.5 / 4 % (960 and 72), batch 80: 48.2 -> 45.5, 64.9 -> 68.7.
bool chain_pays(const SpmmCall &t, const SddmmCall &g0)
{
    const int64_t n = t.nnz, spread = n * t.x_rows, below = static_cast<int64_t>(g0.nnz) * t.batch;
    if ((n * 16 < g0.nnz && below > (24 << 20)) || (n * 8 < g0.nnz && below > (64 << 20))) return false;
    if (t.batch <= 32) return n <= (256 << 10) || (n <= (360 << 10) && spread <= 100'000'000);
    return n <= (172 << 10) || (n <= (360 << 10) && spread <= 500'000'000) || (n <= (440 << 10) && (spread <= 320'000'000 || n <= 58ll * t.rows)) ||
           (n <= (720 << 10) && backward_tiles(t, backward_tile_group(t)) > 1);
}

// (reading values[] through the position map costs a scattered read per entry and tile, a launch of its own 3.5 us)
bool backward_fused_refreshes(const SpmmCall &t, const SddmmCall &g)
{
    if (backward_hot_ok(t, g)) return true;
    const int tiles = backward_tiles(t, backward_tile_group(t));
    return tiles == 1 || backward_looped(t) || static_cast<int64_t>(tiles) * t.nnz <= (1 << 20);
}

// Within a training step small layers do better with T and S in the grids of their neighbours: entries times columns from which the pass pays there
// (steps of 3072-1024-512-10 at 10 %, batch 100, 5 M in the middle layer: 38.6 -> 42.5 us with it; 2000-4000-3000-10 at 3 %, batch 128, 46 M: 72.4 ->
// 70.2; three layers of 3000 at 5 %, batch 100: 128 -> 116): kFusedMinWork.  The transposed product staged through LDS and the gradient apart from it
// (staged too, or by matrix instructions sampled on the pattern) against one stream of L2 gathers for both: apart they read the operands twice, from
// LDS at up to three times the rate, and copy them there.  Which is faster goes by estimates of both, us.  A staged launch takes rounds of a
// work-group per compute unit, each a range's entries and the copy of its operand tile; the stream its gathers (more of them miss where dZ has many
// rows), and the strewing of results through the position map, whose share grows with the entries.  Root mean square from what was measured, apart /
// stream, batch 128 to 1024: 4 / 4 % on 330 uniform layers of 1500 to 16384 rows and columns, 3 to 15 %; 3 / 5 % on 94 power-law ones, where the
// staged gradient has the rows that are not dense, and the stream finds the operand rows of the dense ones in cache; 3 / 6 % on 75 of 15 to 40 % with
// a sampled gradient.  One stream -> apart: 12000 x 11500 at 7 %, batch 900 2103 -> 1677; 14000 x 6800 at 12 %, batch 640 1693 -> 1228; 9877 x 13217
// at 9 %, batch 192 636 -> 545; 16384^2 at 5 / 10 %, batch 1024 3246 -> 2596, 6435 -> 4595; power-law 14000 x 2800 at 12 %, batch 768 825 -> 593;
// 1896 x 8041 at 33 %, batch 300 360 -> 225; but 3336 x 14187 at 9 %, batch 640 483 -> 546, 6300 x 10100 at 9 %, batch 256 306 -> 334, power-law
// 11600 x 4700 at 5 %, batch 512 310 -> 346.  Far from the estimates: segments shorter than those fitted (16384^2 at 2 %, batch 300 478 -> 700),
// little work (1525 x 1453 at 15 %, batch 900 69 -> 89, 551 x 3748 at 31 %, batch 256 38 -> 46; steps of 604-1571-1495-10 at 8 %, batch 700 117 ->
// 129, 393-2977-692-10 at 17 %, batch 300 104 -> 110), and the stream of a mirror of few rows (11458 x 1073 at 8 %, batch 1024 198 -> 222).  In a
// training step the stream has the updates to strew over values and velocity as well, which the gradient's second pass finds in order: steps of
// 802-6257-6435-10 at 14 %, batch 320 732 -> 581, 751-8177-7029-10 at 8 %, batch 900 1264 -> 1174, 1055-7772-2917-10 at 24 %, batch 160 564 -> 423,
// but of 750-6610-5291-10 at 5 %, batch 640 382 -> 407; with dense rows much of the gradient goes by matrix instructions, and apart it stays.  A
// single call on a matrix with dense rows that would go apart stays together where its stream keeps its hot rows in LDS (backward_hot_ok) and takes
// less by 6 %: of 5000 power-law layers of 1500 to 16384 rows and columns, 1 to 14 %, batch 193 to 1024, 271 do, 1.10 times as fast, eight of them
// slower by 3 % or more, the worst by 5.  Apart -> with hot rows: 9349 x 10144 at 4.8 %, batch 1024 835 -> 733; 2128 x 4636 at 13 %, batch 901 228 ->
// 181; but 12085 x 6193 at 13 %, batch 656 951 -> 1329; 8119 x 5813 at 11 %, batch 450 445 -> 488.
static double hot_time(const SpmmCall &t, float share, bool update);
static double staged_launch_time(const RowBlocks &blocks, int64_t nnz, int32_t x_rows, int32_t batch)
{
    const int64_t groups = (static_cast<int64_t>(batch) + kStageCols - 1) / kStageCols * blocks.staged_ranges;
    const double rounds = static_cast<double>((groups + kStageTargetGroups - 1) / kStageTargetGroups);
    return rounds * (1.12e-3 * static_cast<double>(nnz) / blocks.staged_ranges + 5.9e-3 * x_rows);
}
static bool backward_apart_pays(const SpmmCall &t, const SddmmCall &g, bool alone)
{
    if (!spmm_staged_ok(t)) return false;
    const bool sampled = sddmm_sampled_ok(g), split = !sampled && sddmm_dense_rows_ok(g);
    SddmmCall others = g;
    if (split) {
        if (!alone) return true;
        others.blocks = g.split->others; others.split = nullptr; others.split_done = g.split;
    }
    if (!sampled && !sddmm_staged_ok(others)) return false;
    const int64_t work = static_cast<int64_t>(t.nnz) * t.batch, least = sampled ? (alone ? 300'000'000 : 120'000'000) : alone ? 600'000'000 : 400'000'000;
    if (work < least || t.nnz < 20ll * t.rows * t.blocks.staged_cblocks) return false;
    const int tg = backward_tile_group(t);
    const double million = t.nnz * 1e-6, gathers = million * backward_tiles(t, tg) * tg * 4., full = static_cast<double>(g.x_rows) * g.batch;   // (tiles: of 128 columns, or of fewer)
    double stream = 1.15 * million * std::min(million, 30.) + (alone ? 0. : 12. * million), apart = staged_launch_time(t.blocks, t.nnz, t.x_rows, t.batch);
    if (split) {
        const double other = static_cast<double>(t.nnz - g.split->dense_nnz);
        stream += 28. + gathers * (tg >= 32 ? 0.141 + 0.020 / 8192 * t.x_rows : 0.179);
        apart += 13. + staged_launch_time(others.blocks, others.blocks.staged_nnz, g.x_rows, g.batch) + 9.7e-9 * g.split->rows.n * full + 43e-6 * other +
                 196e-9 * (other - others.blocks.staged_nnz) * g.batch;
    } else {
        stream += 23. + gathers * (tg >= 32 ? 0.152 + 0.019 / 8192 * t.x_rows : 0.182 + 0.040 / 16384 * t.x_rows);
        if (sampled) apart = 22.5 + 0.69 * apart + 18.4e-9 * g.rows * full + 7.5 * million;
        else apart += 4. + staged_launch_time(others.blocks, t.nnz, g.x_rows, g.batch) + 5.5 * million;
    }
    if (split && backward_hot_ok(t, g) && apart > 1.06 * hot_time(t, t.hot->share, false)) return false;
    return apart < (!alone ? (sampled ? 1.03 : 0.96) : split ? 0.98 : t.rows < 2048 ? 0.93 : sampled ? 1.03 : 1.) * stream;
}
bool backward_fused_ok(const SpmmCall &t, const SddmmCall &g, bool alone)
{
    if (t.batch != g.batch || t.batch < 4 || t.X != g.dZ || t.ldx != g.lddz || t.XM != g.ZM || t.ldxm != g.ldzm) return false;
    if (t.YM && (t.YM != g.X || t.ldym != g.ldx)) return false;
    if (t.rows != g.x_rows || t.x_rows != g.rows || t.nnz != g.nnz || t.nnz <= 0) return false;
    if (g.skip_products || g.dense || g.loss_cols || !g.perm) return false;
    if (!spmm_offsets_ok(t) || !sddmm_offsets_ok(g) || backward_apart_pays(t, g, alone)) return false;
    const int tg = backward_tile_group(t);
    if (!alone && static_cast<int64_t>(t.nnz) * t.batch < kFusedMinWork) return false;
    const int n_tiles = backward_tiles(t, tg);
    // (a masked dZ only where gathering the mask as well costs less than the launch that would form dZ)
    if (t.XM && (!alone || static_cast<int64_t>(t.nnz) * t.batch > kBackwardSmallWork)) return false;
    const bool one = n_tiles == 1 || (alone && backward_looped(t));   // (then the products need no second pass)
    if (!one && (!g.partial || n_tiles > g.partial_tiles || g.partial_stride < t.nnz)) return false;
    // (no row so long that its lane groups outlast the rest of the launch; a pass over 128 entries is short enough on any matrix)
    const int64_t longest = t.blocks.staged_longest_row >> backward_split(t, tg, n_tiles);
    if (longest > kPackMaxLen && longest * 4096 > static_cast<int64_t>(t.nnz) * ((t.batch + 63) / 64)) return false;
    const int64_t per_set = (kWave / tg) >> backward_split(t, tg, n_tiles), sets = (static_cast<int64_t>(t.rows) + per_set - 1) / per_set;
    return ((n_tiles + 7) / 8) * 8 * ((sets + kBwdWaves - 1) / kBwdWaves) + 2048 <= kMaxGridIds;
}

bool strips_pay_somewhere(const RowBlocks &plan, int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch, double steps, double chunks)
{
    SpmmCall a{};
    a.blocks = plan; a.rows = rows; a.x_rows = cols; a.ldx = max_batch; a.nnz = nnz;
    // (asked at a quarter and at all of every 64 columns; beyond some thousand they all say the same)
    for (int32_t most = std::min(max_batch, 4096), hi = most; hi > kStripFromBatch; hi = (hi - 1) / 64 * 64)
        for (const int32_t batch : {hi, (hi - 1) / 64 * 64 + 16}) {
            if (batch > hi) continue;
            a.batch = batch;
            if (strip_pays(strip_plan(rows, cols, batch, strip_blocks_of(cols), steps, chunks).us, other_product_us(a))) return true;
        }
    return false;
}
bool strips_may_pay(int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch, int32_t staged_ranges)
{
    // at the best: every set's segments of one length, and whichever of the other kernels is the slowest
    const double steps = nnz / static_cast<double>(kStripSet), chunks = steps / kStripChunk;
    RowBlocks plan{};
    static constexpr int32_t some = 0;
    plan.n_short = nnz <= static_cast<int64_t>(kPackMaxLen) * rows ? rows : 0;
    plan.staged_longest_row = nnz / rows;
    for (const float hot : {0.f, 1.f}) {
        plan.hot_share = hot;
        plan.staged_rows = nullptr;
        if (strips_pay_somewhere(plan, rows, cols, nnz, max_batch, steps, chunks)) return true;
        if (staged_ranges == 0) continue;
        plan.staged_rows = &some;   // (asked whether it is there, never read)
        plan.staged_ranges = staged_ranges; plan.staged_cblocks = (cols + kStageRows - 1) / kStageRows;
        plan.staged_row_count = rows; plan.staged_nnz = nnz;
        if (strips_pay_somewhere(plan, rows, cols, nnz, max_batch, steps, chunks)) return true;
    }
    return false;
}

int32_t partial_tiles_wanted(const RowBlocks &plan, const RowBlocks &plan_t, int32_t rows, int32_t cols, int32_t nnz, int32_t max_batch)
{
    SpmmCall t{};
    t.blocks = plan_t; t.rows = cols; t.x_rows = rows; t.nnz = nnz;
    if (nnz <= 0) return 0;
    // The rules are asked at either end of every 64 columns, and tiles counted to the far end: none is narrower than 32 columns.
    constexpr int64_t kMostAsked = 1 << 18;
    if (max_batch > kMostAsked) return max_batch / 32 + 1;
    int64_t most = 0;
    for (int64_t lo = 0; lo < max_batch; lo += 64) {
        const int64_t hi = lo + 64 < max_batch ? lo + 64 : max_batch;
        for (const int64_t batch : {lo + 1, hi}) {
            t.batch = static_cast<int32_t>(batch);
            const int w = tile_columns(cols, t.batch, nnz, rows, plan.staged_longest_row, plan.hot_share, false, true);
            if (w > 0) most = most > (hi + w - 1) / w ? most : (hi + w - 1) / w;
            const int64_t columns = 4ll * backward_tile_group(t), n = (hi + columns - 1) / columns;
            if (n > 1 && !(backward_looped(t) && hi <= 512)) most = most > n ? most : n;
        }
    }
    return static_cast<int32_t>(most);
}

// The same sharing for a full matrix of few rows (a saturated output layer): its SDDMM streams the layer's
// input once, a wave per input row, and that row is also the mask of the transposed product's result row.
bool full_backward_ok(const SpmmCall &t, const SddmmCall &g)
{
    SddmmCall plain = g;
    plain.loss_cols = nullptr;  // (this launch can carry the mean of the losses, the plain one is not asked to)
    if (g.batch % 4 != 0 || !sddmm_full_ok(plain) || !g.fused || g.ZM || !g.values || !g.velocity) return false;
    if (t.batch != g.batch || t.XM || t.bias || t.relu || !t.YM || t.YM != g.X || t.ldym != g.ldx || t.X != g.dZ || t.ldx != g.lddz) return false;
    return t.rows == g.x_rows && t.x_rows == g.rows && t.nnz == g.nnz && t.Y;
}

hipError_t launch_full_backward(const SpmmCall &t, const SddmmCall &g, hipStream_t s)
{
    const int n_chunks = (g.batch + 255) / 256;
    const int groups = (g.x_rows + kWavesPerBlock - 1) / kWavesPerBlock;
    hipLaunchKernelGGL(full_sddmm_kernel<true>, dim3(groups < 1024 ? groups : 1024), dim3(kBlock),
                       static_cast<size_t>(g.rows) * n_chunks * kWave * sizeof(float4), s, g, n_chunks, t.Y, static_cast<int>(t.ldy));
    return hipGetLastError();
}

// Whether the waves of one tile have all gathers of a pass in flight (APART, 70 to 82 registers, 5 to 7 waves a SIMD) or two or three (62 to 78, 6 to
// 8): where few waves leave room anyway, and in groups of 16 where rows are short.  Uniform rows, us, mixed -> apart: batch 16, 8000 x 1000 at 12 % 3
// % faster, 700 x 6000 at 12 % 11.6 -> 12.6, 3000 x 16384 at 12 % 131 -> 150; batch 64, 2048 x 3000 at 10 / 40 % 21.2 -> 18.6, 60.5 -> 53.9, 2048 x
// 4096 at 10 / 40 % 24.4 -> 23.0, 73.9 -> 79.4, 2048 x 5500 at 10 / 40 % 30.2 -> 30.7, 107 -> 124, 3000 x 8192 at 5 / 40 % 34.8 -> 32.3, 226 -> 258;
// batch 128, 2048 x 3000 at 10 % 26.3 -> 25.1, 2048 x 3400 28.2 -> 28.6, 2048 x 6500 48.3 -> 50.6, 3000 x 13000 at 2 % 30.5 -> 33.2, 3000 x 16384 at
// 12 % 208 -> 200, 8192^2 at 0.3 / 0.6 / 2 / 7 % 14.3 -> 13.5, 20.9 -> 19.6, 51 -> 49.3, 151 -> 162, 9106 x 9383 at 0.3 / 0.6 / 2 % 16.7 -> 15.8,
// 24.4 -> 25.3, 65 -> 71.6; batch 256 not slower up to 25 %.  With the update, which loads more: steps of 3000-3000-3000-10, batch 64, at 15 / 25 %
// 121 -> 122, 185 -> 197, of 2000-2000-2000-10 at 25 % 97 -> 90.
static bool backward_gathers_apart(int gs, int64_t waves, const SpmmCall &t, bool update)
{
    if (update && gs < 64 && waves > 2048 && t.nnz > 400ll * t.rows) return false;
    if (gs == 8) return waves <= 2048;
    if (gs == 16) return waves <= 3072 || (t.nnz <= 256ll * t.rows && (waves <= 4096 || waves > 6144));
    return gs == 64 || waves <= 3072 || waves >= 16384 || t.nnz <= 40ll * t.rows || (waves <= 4608 && t.nnz <= 192ll * t.rows);
}

// Whether one tile in groups of 16 or 32 lanes, whose gathers would be apart, takes chunks of sixteen (80 registers, a third fewer instructions).
// Uniform rows, us, batch 64 / 128: 1200 x 1100 at 2 % 5.4 -> 5.1, 5.8 -> 5.2, at 6 % 6.4 -> 6.4, 8.9 -> 7.7; 2048 x 3000 at 6 % 12.3 -> 12.0, 17.3
// -> 16.1; 3000 x 4000 at 6 % 21.5 -> 20.8, 29.2 -> 27.5; 4000 x 3000 at 2 % 10.0 -> 9.6, 13.5 -> 12.6; 8192^2 at 0.6 / 2 % 15.6 -> 15.2, 37.4 ->
// 37.5, 19.9 -> 19.7, 50.3 -> 49.0.  Not with rows of one chunk (3000 x 4000 at 0.3 %, 9 entries a row, batch 128 5.0 -> 5.4), nor with long ones,
// which lose lines that the L1s would keep (2048 x 5500 at 25 % 67.7 -> 77.8, 98.5 -> 104; 9106 x 9383 at 6 %, batch 64 139 -> 158), nor with more
// waves than start at once (9106 x 9383 at 2 %, batch 128 65.0 -> 71.9, at 0.3 % 16.1 -> 16.8; but 2048 x 5500 at 2 % 14.0 -> 12.1).
static bool bwd_sixteens(int64_t waves, const SpmmCall &t) { return waves <= 4096 && t.nnz > 20ll * t.rows && t.nnz <= 400ll * t.rows; }

// Whether the pass with hot rows in LDS runs: where a tile's columns are on, there are mirror rows enough (a wave for
// each four of them and tile) and long ones (8068 x 4944 at 0.6 %, 46 entries a mirror row, batch 762 46.4 -> 50.9 us;
// with more rows of dZ beside the hot ones 14946 x 9731 at 0.5 %, 68, batch 252 51.5 -> 54.8), and where by the estimates
// of both it is the shorter way.  They are of 15400 matrices of 1024 to 16384 rows, power-law ones and even ones of up to
// 2400, batch 193 to 1024 (3.4 % root mean square each): those that take the pass are 1.13 times as fast, 0.7 % of them
// slower by 3 % or more.  From the L2s -> in LDS, us: power-law 16384^2 at 1 %, batch 1024 / 256 541 -> 446, 146 -> 133;
// 4000 x 8000 at 4 %, batch 256 77.7 -> 65.5; even 1100 x 2600 at 10 %, batch 1024 62.5 -> 53.1, 1200 x 16384 at 6 %,
// batch 320 91.8 -> 75.3.  But even 1500^2 at 5 %, batch 1024 32.4 -> 34.8 (a third of the gathers from LDS, few rounds of
// work-groups), and batches of up to 256 that otherwise need no second pass: power-law 3000 x 6000 at 3 % 33.7 -> 40.5,
// 2000 x 8000 31.5 -> 35.3, even 1500 x 8000 at 5 % 37.6 -> 44.5.  With the update, whose weights go back through the
// order of the walk, 1 us and 6 per million entries more (2450 training steps: of those that take the pass then one in
// 150 is slower by 2 % or more).
constexpr int64_t kHotTasks = 5000, kHotEntries = 45, kHotWork = 96ll << 20;
static double hot_time(const SpmmCall &t, float share, bool update)
{
    const double nnz = t.nnz * 1e-6, operand = 1e-6 * t.x_rows * t.batch, x = t.x_rows / 8192., tiles = (t.batch + 63) / 64;
    return (update ? 19 : 18) + nnz * ((update ? 17.8 : 11.8) + tiles * (5.8 + (1. - share) * (4.1 + 1.7 * x))) + 1.1 * operand + 0.05e-3 * tiles * t.rows;
}
static bool hot_pays(const SpmmCall &t, float share, bool update)
{
    const int64_t tiles = (static_cast<int64_t>(t.batch) + 63) / 64, sets = (static_cast<int64_t>(t.rows) + 3) / 4;
    if (t.batch < kHotFromBatch || t.batch * 20ll < tiles * 64 * 17 || sets * tiles < kHotTasks || t.nnz < (t.x_rows > 6144 ? 85ll : kHotEntries) * t.rows ||
        static_cast<int64_t>(t.nnz) * t.batch < kHotWork || t.x_rows < 1024 || t.blocks.hot_share < 0.5f || t.nnz >= (1 << 30)) return false;
    const int tg = backward_tile_group(t), n_tiles = backward_tiles(t, tg);
    const double nnz = t.nnz * 1e-6, operand = 1e-6 * t.x_rows * t.batch, x = t.x_rows / 8192.;
    const double stream = n_tiles == 1 ? 8 + nnz * (53 + 4.6 * x) + 0.2 * operand : 15.6 + nnz * (7.6 + n_tiles * tg / 16. * (10.45 + 0.1 * x)) + 0.65 * operand;
    return hot_time(t, share, update) < 0.98 * stream;
}
bool backward_hot_ok(const SpmmCall &t, const SddmmCall &g)
{
    if (!t.hot || !g.hot_values || t.XM || !g.partial || (t.batch + 63) / 64 > g.partial_tiles || g.partial_stride < t.nnz) return false;
    return hot_pays(t, t.hot->share, g.fused);
}
bool hot_rows_pay_somewhere(SpmmCall t, SddmmCall g, int32_t max_batch)
{
    static float some;
    t.X = g.dZ = g.partial = g.hot_values = &some;   // (asked whether they are there)
    // (asked of the fewest and the most columns that fill a number of tiles; beyond some thousand they all say the same)
    for (int32_t tiles = kHotFromBatch / 64, most = std::min((max_batch + 63) / 64, 256); tiles <= most; ++tiles)
        for (const int32_t batch : {(tiles * 64 * 17 + 19) / 20, std::min(tiles * 64, max_batch)})
            for (const bool alone : {true, false}) {
                if (batch > max_batch) continue;
                t.batch = g.batch = batch;
                t.ldx = g.lddz = g.ldx = batch;
                g.fused = !alone;
                if (backward_hot_ok(t, g) && backward_fused_ok(t, g, alone)) return true;
            }
    return false;
}

hipError_t launch_backward_finish(BackwardFinish &f, hipStream_t s)
{
    if (!f.waiting) return hipSuccess;
    f.waiting = false;
    hipLaunchKernelGGL(backward_finish_kernel, dim3(f.n_entry_blocks + f.n_row_blocks), dim3(kEwBlock), 0, s, f.a, f.hot_at, f.n_tiles, f.n_entry_blocks);
    return hipGetLastError();
}

hipError_t launch_backward_fused(const SpmmCall &t, const SddmmCall &g, bool alone, hipStream_t s, BackwardFinish *later)
{
    BackwardArgs a{};
    a.blocks = t.blocks; a.indices = t.indices; a.values = t.values;
    a.dZ = t.X; a.lddz = t.ldx; a.X = g.X; a.ldx = g.ldx; a.dX = t.Y; a.lddx = t.ldy; a.mask = t.YM != nullptr;
    a.ZM = t.XM; a.ldzm = t.ldxm;
    a.rows = t.rows; a.x_rows = t.x_rows; a.batch = t.batch; a.nnz = t.nnz;
    a.partial = g.partial; a.partial_stride = g.partial_stride; a.perm = g.perm;
    a.g = g.g; a.db = g.db; a.fused = g.fused; a.nesterov = g.nesterov; a.lr = g.lr; a.momentum = g.momentum;
    a.w = g.values; a.velocity = g.velocity; a.w_t = g.values_t; a.bias = g.bias; a.bias_velocity = g.bias_velocity;
    const int tg = backward_tile_group(t), n_tiles = backward_tiles(t, tg);
    if (alone && g.values && backward_fused_refreshes(t, g)) a.refresh = g.values;
    const int lg_split = backward_split(t, tg, n_tiles);
    const int64_t per_set = (kWave / tg) >> lg_split, sets = (static_cast<int64_t>(t.rows) + per_set - 1) / per_set;
    const int n_pack_blocks = static_cast<int>((sets + kBwdWaves - 1) / kBwdWaves);
    const bool one = n_tiles == 1 || (alone && backward_looped(t));
    const int64_t row_blocks = (static_cast<int64_t>(a.x_rows) + kBwdWaves - 1) / kBwdWaves;
    const int n_row_blocks = (a.db || (a.fused && a.bias)) ? static_cast<int>(row_blocks < 2048 ? row_blocks : 2048) : 0;
    auto finish = [&](int tiles, const int32_t *hot_at) {
        BackwardFinish f{a, hot_at, tiles, xcd_run_blocks(t.nnz), n_row_blocks, true};
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || !later) return e != hipSuccess ? e : launch_backward_finish(f, s);
        *later = f;
        return hipSuccess;
    };
    if (backward_hot_ok(t, g)) {
        StripGrid h;
        h.n_tiles = (t.batch + 63) / 64;
        // one round of work-groups, two tiles at a time on an XCD, where an L2 holds both (5001 x 9001 at 2 %, batch 999, in two: 133 -> 144 us),
        // else two (16384^2 at 1 %, batch 1024, in one: 438 -> 474)
        h.n_ranges = std::max(1, (t.x_rows * 512ll <= (3 << 20) ? 1 : 2) * 256 / h.n_tiles);
        h.per = (h.n_tiles * h.n_ranges + 7) / 8;
        const bool refresh = alone && g.values;   // (backward_fused_refreshes: the call leaves it to this launch)
        hipLaunchKernelGGL(hot_values_kernel, dim3(xcd_run_blocks(t.nnz)), dim3(kEwBlock), 0, s, g.hot_values, refresh ? g.values : t.values, g.values_t, t.hot->at,
                           refresh ? t.hot->perm : nullptr, t.nnz);
        hipLaunchKernelGGL(t.batch % 64 ? backward_hot_kernel<true> : backward_hot_kernel<false>, dim3(8u * h.per), dim3(kHotWaves * kWave), 0, s, a, h, *t.hot, g.hot_values);
        a.perm = t.hot->perm;
        return finish(h.n_tiles, t.hot->at);
    }
    const TileOrder order = tile_order(n_tiles, n_pack_blocks, tg, false, tiled_launch(t));
    const int64_t ids = one ? n_pack_blocks + n_row_blocks : tile_grid(order, n_tiles, n_pack_blocks);
    auto go = [&](auto group) {
        constexpr int GS = decltype(group)::value;
        const dim3 grid(static_cast<unsigned>(ids)), block(kBwdWaves * kWave);
        auto launch = [&](auto pass, auto mask) {
            constexpr bool kOne = decltype(pass)::value == kBackwardOneTile && !decltype(mask)::value;
            auto with = [&](auto spare) {
                constexpr BackwardSpare SPARE = decltype(spare)::value;
                constexpr BackwardPass P = decltype(pass)::value;
                constexpr bool MASK = decltype(mask)::value;
                const int64_t waves = static_cast<int64_t>(n_pack_blocks) * kBwdWaves;
                auto kernel = backward_fused_kernel<GS, false, P, MASK, SPARE, kOne>;
                if constexpr (kOne && (GS == 8 || SPARE == kSpareNone)) {   // (else both variants take the same registers)
                    if (!backward_gathers_apart(GS, waves, t, a.fused)) {
                        kernel = backward_fused_kernel<GS, false, P, MASK, SPARE, false>;
                    } else if constexpr (GS == 16 || GS == 32) {
                        if (bwd_sixteens(waves, t)) kernel = backward_fused_kernel<GS, true, P, MASK, SPARE, true>;
                    }
                }
                hipLaunchKernelGGL(kernel, grid, block, 0, s, a, n_tiles, order, n_pack_blocks, lg_split);
            };
            if (a.batch % (GS * 4) == 0) return with(std::integral_constant<BackwardSpare, kSpareNone>{});
            if constexpr (decltype(pass)::value == kBackwardTiles)
                if (a.batch % 4 == 0) return with(std::integral_constant<BackwardSpare, kSpareLanes>{});
            with(std::integral_constant<BackwardSpare, kSpareColumns>{});
        };
        using tiles = std::integral_constant<BackwardPass, kBackwardTiles>;
        using single = std::integral_constant<BackwardPass, kBackwardOneTile>;
        using looped = std::integral_constant<BackwardPass, kBackwardLooped>;
        if (!one && a.ZM) launch(tiles{}, std::true_type{});
        else if (!one) launch(tiles{}, std::false_type{});
        else if (n_tiles == 1 && a.ZM) launch(single{}, std::true_type{});
        else if (n_tiles == 1) launch(single{}, std::false_type{});
        else if constexpr (GS == kWave) {
            if (a.ZM) launch(looped{}, std::true_type{});
            else launch(looped{}, std::false_type{});
        }
    };
    switch (tg) {
        case 64: go(std::integral_constant<int, 64>{}); break;
        case 32: go(std::integral_constant<int, 32>{}); break;
        case 16: go(std::integral_constant<int, 16>{}); break;
        default: go(std::integral_constant<int, 8>{}); break;
    }
    if (one) return hipGetLastError();
    return finish(n_tiles, nullptr);
}

// whether launch_spmm serves `a` by streaming (full matrix of few rows), where the softmax epilogue can ride along
static bool spmm_full_rows_ok(const SpmmCall &a)
{
    return a.batch > 4 && a.full_scratch && !a.XM && a.batch >= 64 && a.rows <= kFullMaxRows;
}
bool spmm_softmax_epilogue_ok(const SpmmCall &a)
{
    return a.rows > 0 && a.blocks.n_blocks > 0 && spmm_full_rows_ok(a) && !a.relu && !a.YM && a.ce_labels && a.ce_dZ && a.ce_loss_cols;
}

// log2 of the waves per row of spmv_rows_kernel, -1: not for this matrix.  It needs more entries than 8192 waves hold at 64
// each, and no row that keeps its waves busy for more than 16 rounds.
static int spmv_rows_split(const SpmmCall &a)
{
    if (a.nnz < 8192 * kWave || !spmm_offsets_ok(a)) return -1;
    int lg = 0;
    while (lg < 4 && (static_cast<int64_t>(a.rows) << (lg + 1)) <= 8192) ++lg;
    return (a.blocks.staged_longest_row >> lg) <= 16 * 4 * kWave ? lg : -1;
}

bool spmm_takes_strip(const SpmmCall &a)
{
    return a.rows > 0 && a.batch > 4 && a.blocks.n_blocks > 0 && !spmm_full_rows_ok(a) && !spmm_dense_rows_ok(a) && spmm_strip_ok(a);
}

hipError_t launch_strip_streams(const SpmmCall *list, int n, hipStream_t s)
{
    StripStreams all{};
    unsigned most = 0;
    for (int k = 0; k < n; ++k) {
        const SpmmCall &a = list[k];
        all.of[k] = StripStream{a.strips->segs, a.strips->cuts, a.indices, a.values, a.strip_stream, (a.rows + kStripSet - 1) / kStripSet,
                                a.strips->blocks, a.strips->block_rows, a.x_rows, a.nnz};
        most = std::max(most, static_cast<unsigned>((all.of[k].sets * all.of[k].blocks + kStripStreamWaves - 1) / kStripStreamWaves));
    }
    hipLaunchKernelGGL(strip_stream_kernel, dim3(most, n), dim3(kStripStreamWaves * kWave), 0, s, all);
    return hipGetLastError();
}

hipError_t launch_spmm(const SpmmCall &a, hipStream_t s)
{
    if (a.rows <= 0 || a.batch <= 0 || a.blocks.n_blocks <= 0) return hipSuccess;
    if (a.batch <= 4) {
        if (const int lg = spmv_rows_split(a); lg >= 0) {
            const dim3 grid(static_cast<unsigned>(((static_cast<int64_t>(a.rows) << lg) + kWavesPerBlock - 1) / kWavesPerBlock));
            if (a.batch == 1)
                hipLaunchKernelGGL(spmv_rows_kernel<1>, grid, dim3(kBlock), 0, s, a, lg);
            else if (a.batch == 2)
                hipLaunchKernelGGL(spmv_rows_kernel<2>, grid, dim3(kBlock), 0, s, a, lg);
            else
                hipLaunchKernelGGL(spmv_rows_kernel<4>, grid, dim3(kBlock), 0, s, a, lg);
            return hipGetLastError();
        }
        if (a.batch == 1)
            hipLaunchKernelGGL(spmv_kernel<1>, dim3(a.blocks.n_blocks), dim3(kBlock), 0, s, a);
        else
            hipLaunchKernelGGL(spmv_kernel<4>, dim3(a.blocks.n_blocks), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    if (spmm_full_rows_ok(a)) {
        const int n_slices = (a.x_rows + kFullSlice - 1) / kFullSlice;
        hipLaunchKernelGGL(full_rows_kernel, dim3(n_slices, (a.batch + 255) / 256), dim3(kFullWaves * kWave),
                           static_cast<size_t>(kFullWaves) * a.rows * kWave * sizeof(float4), s, a);
        if (a.ce_labels)
            hipLaunchKernelGGL(full_rows_finish_softmax_kernel, dim3((a.batch + kWave - 1) / kWave), dim3(kBlock), 0, s, a, n_slices);
        else
            hipLaunchKernelGGL(full_rows_finish_kernel, dim3(a.rows, (a.batch + kEwBlock - 1) / kEwBlock), dim3(kEwBlock), 0, s, a, n_slices);
        return hipGetLastError();
    }
    if (spmm_dense_rows_ok(a)) {
        // the dense rows by matrix instructions, then the others as ever, told to leave these out
        const hipError_t e = launch_dense_rows(a, s);
        if (e != hipSuccess || a.split->rows.n == a.rows) return e;
        SpmmCall others = a;
        others.blocks = a.split->others;
        others.split = nullptr;
        others.strips = nullptr;   // (its rows are all, the dense ones too)
        return launch_spmm(others, s);
    }
    if (spmm_strip_ok(a)) {
        const StripGrid g = strip_plan(a).grid;
        if (!a.strip_ready) {
            const hipError_t e = launch_strip_streams(&a, 1, s);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(spmm_strip_kernel, dim3(8u * static_cast<unsigned>(g.per)), dim3(kStripWaves * kWave), 0, s, a, g, *a.strips, a.strip_stream);
        return hipGetLastError();
    }
    if (spmm_staged_ok(a)) {
        const int n_tiles = (a.batch + kStageCols - 1) / kStageCols;
        const dim3 grid(n_tiles * a.blocks.staged_ranges), block(kStageWaves * kWave);
        const bool many = a.nnz >= (1 << 30);
        const auto kernel = a.XM ? (many ? spmm_staged_kernel<true, true> : spmm_staged_kernel<true, false>) : many ? spmm_staged_kernel<false, true> : spmm_staged_kernel<false, false>;
        hipLaunchKernelGGL(kernel, grid, block, 0, s, a, n_tiles);
        if (a.blocks.staged_partial) {
            // the short rows: packed where that path runs (inside column tiles), and nothing else in that grid;
            // otherwise whatever kernel the batch asks for, on the short rows' own partition
            SpmmCall rest = a;
            rest.blocks.n_huge_rows = 0;
            const int tg = spmm_tile_group(a);
            if (staged_rest_packed(a, tg)) {
                rest.blocks.n_long_blocks = 0;
                switch (tg) {
                    case 32: return spmm_packed_go<32>(rest, s);
                    case 16: return spmm_packed_go<16>(rest, s);
                    default: return spmm_packed_go<8>(rest, s);
                }
            }
            rest.blocks.staged_rows = nullptr;
            rest.strips = nullptr;
            rest.blocks.n_short = 0;
            rest.blocks.waves = a.blocks.rest_waves;
            rest.blocks.n_blocks = a.blocks.n_rest_blocks;
            return launch_spmm(rest, s);
        }
        return hipGetLastError();
    }
    if (spmm_offsets_ok(a)) {
        int tg = spmm_tile_group(a);
        if (tg == 0 && packed_tiles_pay(a)) tg = 16;
        const int sg = tg == 0 ? spmm_split_group(a) : 0;
        if (sg != 0) {
            // Long rows inside column tiles (their gathers are most of the traffic and then hit in the L2s),
            // short rows outside (a pass over them per tile would cost more than their gathers): two launches.
            SpmmCall longs = a, rest = a;
            longs.blocks.waves = a.blocks.long_waves;
            longs.blocks.n_blocks = a.blocks.n_long_blocks;
            longs.blocks.n_short = 0;
            rest.blocks.waves = a.blocks.rest_waves;
            rest.blocks.n_blocks = a.blocks.n_rest_blocks;
            rest.blocks.n_huge_rows = 0;
            rest.blocks.n_short = 0;
            rest.blocks.n_long_blocks = 0;   // (nothing left to split off)
            rest.blocks.staged_rows = nullptr;
            rest.strips = nullptr;
            const hipError_t e = launch_spmm(rest, s);
            if (e != hipSuccess) return e;
            switch (sg) {
                case 32: return spmm_tiled_go<32>(longs, s);
                case 16: return spmm_tiled_go<16>(longs, s);
                default: return spmm_tiled_go<8>(longs, s);
            }
        }
        if (a.blocks.n_short > 0 && tg != 0 && packed_grid(a, tg, true).ids <= kMaxGridIds) {
            switch (tg) {
                case 32: return spmm_packed_go<32>(a, s);
                case 16: return spmm_packed_go<16>(a, s);
                default: return spmm_packed_go<8>(a, s);
            }
        }
        switch (tg) {
            case 32: return spmm_tiled_go<32>(a, s);
            case 16: return spmm_tiled_go<16>(a, s);
            case 8: return spmm_tiled_go<8>(a, s);
            default: break;
        }
        if (a.batch <= 32) return spmm_grouped_go<8>(a, s);
        if (a.batch <= 64) return spmm_grouped_go<16>(a, s);
        if (a.batch <= 128) return spmm_grouped_go<32>(a, s);
    }
    return spmm_go(a, s);
}

// Columns per tile of the column-tiled SDDMM, 0: one pass over the whole batch.
int sddmm_tile_columns(const SddmmCall &a)
{
    if (!a.partial || a.skip_products || a.dense || !sddmm_offsets_ok(a)) return 0;  // (the finish pass does not know an entry's row)
    // the operand rows an entry gathers are named by its column index: the matrix's own partition
    // carries the share of the most referenced ones
    const int w = tile_columns(a.x_rows, a.batch, a.nnz, a.rows, a.blocks.staged_longest_row, a.blocks.hot_share, false, true);
    if (w == 0) return 0;
    const int n_tiles = (a.batch + w - 1) / w;
    if (n_tiles > a.partial_tiles) return 0;
    if (static_cast<int64_t>(a.blocks.n_blocks) * kSddmmParts * (n_tiles + 8) >= (1ll << 31)) return 0;
    return w;
}

// Whether launch_sddmm takes a finish pass that waits into its grid.  It strews weights and velocity over the rows of the layer above, whose lines
// the gathers beside it push out of the L2s half written where they are many: not beyond 4096 rows (1 MiB in an L2) unless there are few entries, or
// half again as many as the gradient's at the most among eight tiles or more, whose last round has room.  Steps of 5400 networks of two hidden
// layers, apart -> in one launch: where it is taken 1.012 times as fast, else 0.999 in the mean: 1108-1879-8144-10 at 3 %, batch 1024 230 -> 241 us,
// 5871-5373-4349-10, batch 492 274 -> 288, 1134-7260-7945-10 at 1.2 %, batch 902 304 -> 320.
static bool sddmm_takes_finish(const SddmmCall &a, const BackwardArgs &f)
{
    if (a.rows <= 0 || a.batch <= 0 || a.blocks.n_blocks <= 0 || sddmm_sampled_ok(a) || sddmm_dense_rows_ok(a) || sddmm_full_ok(a) || sddmm_staged_ok(a)) return false;
    const int w = sddmm_tile_columns(a);
    return (w == 128 || w == 64) && (f.x_rows <= 4096 || f.nnz < 100'000 || (w == 128 && a.batch > 7 * 128 && f.nnz <= a.nnz + a.nnz / 2));
}

hipError_t launch_sddmm(const SddmmCall &a, hipStream_t s, BackwardFinish *first)
{
    if (first && first->waiting && !sddmm_takes_finish(a, first->a)) {
        const hipError_t e = launch_backward_finish(*first, s);
        if (e != hipSuccess) return e;
    }
    if (a.rows <= 0 || a.batch <= 0 || a.blocks.n_blocks <= 0) return hipSuccess;
    if (sddmm_sampled_ok(a)) {
        SampledArgs one{};
        add_sampled(one, a);
        return launch_sampled(one, s);
    }
    if (sddmm_dense_rows_ok(a)) {
        SampledArgs rows{};
        add_sampled_rows(rows, a);
        const hipError_t e = launch_sampled(rows, s);
        if (e != hipSuccess || a.split->rows.n == a.rows) return e;
        SddmmCall others = a;
        others.blocks = a.split->others;
        others.split = nullptr;
        others.split_done = a.split;
        return launch_sddmm(others, s);
    }
    if (sddmm_full_ok(a)) {
        const int n_chunks = (a.batch + 255) / 256;
        const int groups = (a.x_rows + kWavesPerBlock - 1) / kWavesPerBlock;  // one row of X per wave, up to two rounds of work-groups
        hipLaunchKernelGGL(full_sddmm_kernel<false>, dim3(groups < 1024 ? groups : 1024), dim3(kBlock),
                           static_cast<size_t>(a.rows) * n_chunks * kWave * sizeof(float4), s, a, n_chunks, static_cast<float *>(nullptr), 0);
        return hipGetLastError();
    }
    if (sddmm_staged_ok(a)) {
        const int n_tiles = (a.batch + kStageCols - 1) / kStageCols;
        hipLaunchKernelGGL(sddmm_staged_kernel, dim3(n_tiles * a.blocks.staged_ranges), dim3(kStageWaves * kWave), 0, s, a, n_tiles);
        if (a.blocks.staged_partial) {
            // the rows the plan leaves out: the column-tiled SDDMM on their own partition, same tiles, same partial buffer
            SddmmCall rest = a;
            rest.blocks.waves = a.blocks.rest_waves;
            rest.blocks.n_blocks = a.blocks.n_rest_blocks;
            TiledLaunch like = tiled_launch(a);
            like.longest_row = 0;   // (none of the rest is long)
            const int n_blocks = rest.blocks.n_blocks * kSddmmParts;
            const TileOrder order = tile_order(n_tiles, n_blocks, kStageCols / 4, false, like);
            const int64_t ids = tile_grid(order, n_tiles, n_blocks);
            with_spare(a.batch, kStageCols, [&](auto spare) {
                hipLaunchKernelGGL((sddmm_tiled_kernel<16, 1, decltype(spare)::value>), dim3(static_cast<unsigned>(ids)), dim3(kSddmmWaves * kWave), 0, s, rest, n_tiles,
                                   order);
            });
        }
        sddmm_finish_go(a, n_tiles, s);
        return hipGetLastError();
    }
    switch (sddmm_tile_columns(a)) {
        case 128: return sddmm_tiled_go<16, 2>(a, s, first);
        case 64: return sddmm_tiled_go<16, 1>(a, s, first);
        case 32: return sddmm_tiled_go<8, 1>(a, s);
        default: break;
    }
    if (a.chain_lanes)
        return with_chain_lanes(a.batch, [&](auto g, auto nv, auto, auto) { return sddmm_go<decltype(g)::value, decltype(nv)::value>(a, s); });
    if (sddmm_offsets_ok(a) && a.batch <= 1024)
        return with_sddmm_lanes(a.batch, [&](auto g, auto nv) { return sddmm_go<decltype(g)::value, decltype(nv)::value>(a, s); });
    hipLaunchKernelGGL(sddmm_generic, dim3(a.blocks.n_blocks), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_momentum(float *w, float *v, const float *g, int64_t n, float lr, float mu, int nesterov,
                           hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int vec4 = aligned16(w) && aligned16(v) && aligned16(g);
    hipLaunchKernelGGL(momentum_kernel, dim3(elementwise_blocks(vec4 ? (n + 3) / 4 : n)), dim3(kEwBlock), 0, s,
                       w, v, g, n, lr, mu, nesterov, vec4);
    return hipGetLastError();
}

hipError_t launch_gather(float *values_t, const float *values, const int32_t *perm, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_kernel, dim3(gather_blocks(n)), dim3(kEwBlock), 0, s, values_t, values, perm, n);
    return hipGetLastError();
}

hipError_t launch_backward_prep(float *values_t, const float *values, const int32_t *perm, int64_t nnz, const float *dY, int64_t lddy,
                                const float *Y, int64_t ldy, float *dZ, int64_t lddz, int32_t rows, int32_t batch, hipStream_t s)
{
    const int n_gather = nnz > 0 ? gather_blocks(nnz) : 0;
    const int n_mask = elementwise_blocks(static_cast<int64_t>(rows) * ((batch + 3) / 4));
    hipLaunchKernelGGL(backward_prep_kernel, dim3(n_gather + n_mask), dim3(kEwBlock), 0, s, values_t, values, perm, nnz, n_gather, dY, lddy, Y,
                       ldy, dZ, lddz, rows, batch);
    return hipGetLastError();
}

hipError_t launch_softmax_ce(const float *Z, int64_t ldz, const int32_t *labels, int32_t classes, int32_t batch,
                             float *dZ, int64_t lddz, float *loss, hipStream_t s)
{
    if (classes <= kSoftmaxFew) {
        int threads = (batch + kWave - 1) / kWave * kWave;
        if (threads > kSoftmaxBlock) threads = kSoftmaxBlock;
        hipLaunchKernelGGL(softmax_ce_few_kernel, dim3(1), dim3(threads), 0, s, Z, ldz, labels, classes, batch, dZ, lddz, loss);
        return hipGetLastError();
    }
    const int n_tiles = (batch + kWave - 1) / kWave;
    const bool in_place = dZ < Z + static_cast<int64_t>(classes) * ldz && Z < dZ + static_cast<int64_t>(classes) * lddz;
    if (in_place && loss) hipLaunchKernelGGL(softmax_ce_kernel, dim3(1), dim3(kSoftmaxBlock), 0, s, Z, ldz, labels, classes, batch, dZ, lddz, loss, 0);
    const bool with_loss = loss && !in_place;
    hipLaunchKernelGGL(softmax_ce_kernel, dim3(n_tiles + (with_loss ? 1 : 0)), dim3(kSoftmaxBlock), 0, s, Z, ldz, labels, classes, batch, dZ, lddz,
                       loss, n_tiles);
    return hipGetLastError();
}

// One work-group re-reads the whole layer for its 4 columns: only for layers of a few thousand entries.
// Its accesses to the layer's input and to dX are 16 bytes per row, so it loses to three launches on long layers and wide batches: steps of
// 300-cols-10 with it / without, at batch 16, 100, 1024: 1024 columns and 1 %: 13.0 / 18.8, 13.9 / 18.1, 26.1 / 26.1 us; 2048: 15.2 / 19.0,
// 17.5 / 19.1, 36.8 / 32.3 (10 %: 18.7 / 19.8, 21.3 / 21.0, 46.5 / 38.2); 8192: 33.7 / 24.3, 42.8 / 25.1, 101 / 51.
bool head_ok(int32_t rows, int32_t cols, int32_t nnz, int32_t batch)
{
    return rows > 0 && rows <= kHeadMaxRows && cols > 0 && nnz <= 8192 &&
           static_cast<double>(cols) * cols * (batch + 200.) <= 1.25e9;
}

hipError_t launch_head(const HeadArgs &a, hipStream_t s)
{
    const dim3 grid((a.batch + kHeadCols - 1) / kHeadCols);
    const size_t mirror = static_cast<size_t>(a.nnz) * 5, input = static_cast<size_t>(a.cols) * sizeof(float4);
    // Input columns and mirror come into LDS where the columns are gathered from more often than they are loaded (and
    // fit): with an entry or less per column there is nothing to share and the detour costs 0.3 us.
    if (a.nnz <= a.cols)
        hipLaunchKernelGGL((head_kernel<false, false>), grid, dim3(kBlock), 0, s, a);
    else if (mirror + input <= kHeadMaxLds)
        hipLaunchKernelGGL((head_kernel<true, true>), grid, dim3(kBlock), mirror + input, s, a);
    else
        hipLaunchKernelGGL((head_kernel<false, true>), grid, dim3(kBlock), mirror, s, a);
    return hipGetLastError();
}

hipError_t launch_copy(float *dst, const float *src, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int vec4 = aligned16(dst) && aligned16(src);
    hipLaunchKernelGGL(copy_kernel, dim3(elementwise_blocks(vec4 ? (n + 3) / 4 : n)), dim3(kEwBlock), 0, s, dst, src,
                       n, vec4);
    return hipGetLastError();
}

}  // namespace nerva
