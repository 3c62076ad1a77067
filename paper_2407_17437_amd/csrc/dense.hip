// Dense route of a layer whose density is high (the density-adaptive layer that the paper plans in
// "Discussion and Conclusion" and Appendix C.3: dense computation where it is the faster one).
// One zero-filled dense copy of the weights, D[i * ld + j] = W(i, j) (row-major, ld = cols rounded up to
// 64, zero off the pattern and in the padding), serves three fp32 MFMA products:
//     Y  = act(W X + b)          dense_nn_kernel      A operand = rows of D, 16 bytes per lane along k
//     dX = (W^T dZ) * [mask > 0]  dense_tn_kernel      A operand = D read down its columns: the same copy,
//                                                      16 bytes per lane along the output rows
//     G  = dZ X^T                sampled_update_kernel both operands 16 bytes per lane along the batch; the
//                                                      entries of G that lie on the pattern take the momentum step
//                                                      as they leave the accumulators (the state stays sparse)
//
// v_mfma_f32_16x16x4_f32: lane l supplies A(l % 16, l / 16) and B(l / 16, l % 16) of a 16 x 4 by 4 x 16
// step; register r of lane l holds C(4 * (l / 16) + r, l % 16).  A lane's four k slots need not be
// consecutive k as long as A and B agree, so one 16-byte load along k feeds four steps (slot q of
// step s: k = base + 4 q + s), and one 16-byte load along the output rows feeds four tiles (tile u
// holds the rows base + 4 r + u).  Small tiles on purpose: these products are a few hundred
// MFLOP, and only thousands of waves fill 1024 matrix units.  Every sum has one fixed order.
#include "device.h"
#include "kernels.h"

#include <algorithm>

namespace nerva {
namespace {

constexpr int kDenseWaves = 4;
constexpr int kDenseBlock = kWave * kDenseWaves;

__device__ __forceinline__ int wave_id() { return wave_in_block(); }
__device__ __forceinline__ v4f mfma(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

__device__ __forceinline__ void dense_epilogue(const DenseArgs &a, int row, int col, int m_rows, float y)
{
    if (row >= m_rows || col >= a.batch) return;
    if (a.bias) y += a.bias[row];
    if (a.relu) y = y > 0.f ? y : 0.f;
    if (a.YM) y = a.YM[static_cast<int64_t>(row) * a.ldym + col] > 0.f ? y : 0.f;
    a.Y[static_cast<int64_t>(row) * a.ldy + col] = y;
}

// Y (rows x batch) = act(D X + b).  Work-group: MB * 16 rows x NB * 16 columns; its kNnWaves waves split K = cols (or, where several work-groups
// share a tile, their part of it) into contiguous slices of whole chunks and meet in LDS, where wave w adds register w of all slices in
// slice order.  The loads of the next chunks of 16 k are on their way
// while a chunk's MFMA steps run; no branch stands between them, or every wait would be for all of them (and was: 1024 x 3072 at
// batch 512 60.9 us, 41.0 without; 2048 x 4096 at batch 256 78, 50, at 1024 279, 186; 1024 x 3072 at batch 100 16.8, 16.0).  Nor does the loop ask whether
// a chunk is whole: the last one of a K that is no multiple of 16 comes after it (1001 columns and 777 rows at batch 77 8.4, 7.2).
// (kSplitWaves: the same split in the transposed product.)
constexpr int kSplitWaves = 16;
constexpr int kSplitBlock = kSplitWaves * kWave;

// The NB columns of a lane are consecutive (tile t holds the columns n0 + NB * r + t), so that one load along the batch feeds the NB
// tiles; at the end of the batch the lane takes its last NB columns (which another lane has as well: both store the same).
template <int MB, int NB>
struct NnChunk {
    float4 w4[MB];
    float b[4][NB];
};

template <int NB>
__device__ __forceinline__ void nn_columns(const float *p, float (&b)[NB])
{
    typedef float columns __attribute__((ext_vector_type(NB == 1 ? 2 : NB), aligned(4)));   // (rows of any leading dimension)
    if constexpr (NB == 1) {
        b[0] = *p;
    } else {
        const columns v = *reinterpret_cast<const columns *>(p);
#pragma unroll
        for (int t = 0; t < NB; ++t) b[t] = v[t];
    }
}

// The slice's chunks one after another; past its last one the addresses stay there (what is read again is not used).
template <int MB, int NB>
struct NnReader {
    const float *w[MB], *x;
    int64_t ldx;
    int left;    // chunks from this one on

    __device__ __forceinline__ void load(NnChunk<MB, NB> &C)
    {
#pragma unroll
        for (int m = 0; m < MB; ++m) C.w4[m] = ld4(w[m]);
#pragma unroll
        for (int s = 0; s < 4; ++s) nn_columns<NB>(x + s * ldx, C.b[s]);
        const int step = left > 1 ? 16 : 0;   // uniform
        --left;
#pragma unroll
        for (int m = 0; m < MB; ++m) w[m] += step;
        x += step * ldx;
        __builtin_amdgcn_sched_barrier(0);   // chunk after chunk, or the first one's loads come last and its wait is for all
    }
};

template <int MB, int NB>
__device__ __forceinline__ void nn_mfma(const NnChunk<MB, NB> &C, v4f (&acc)[MB][NB])
{
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const float w = s == 0 ? C.w4[m].x : s == 1 ? C.w4[m].y : s == 2 ? C.w4[m].z : C.w4[m].w;
#pragma unroll
            for (int t = 0; t < NB; ++t) acc[m][t] = mfma(w, C.b[s][t], acc[m][t]);
        }
}

// 1024 x 3072 at batch 100, 4096 x 2048 at batch 256 with 4 / 8 / 16 waves: 16.0 / 16.5 / 17.7, 51.8 / 54.7 / 64.6 us; twice as many (W) where work-groups of one tile leave
// compute units idle: 512 x 1024 at batch 64 (with the copy's refresh) 9.6 -> 9.0, 1024 x 3072 at 20 24.0 -> 21.8, 300 x 5000 at 100 34.1 -> 31.2, but 512 x 1024 at 150 (320 work-groups)
// 11.2 -> 11.9.
constexpr int kNnWaves = 4;
constexpr int kNnAhead = 2;    // chunks of a wave; the same with 1 / 2 / 3 / 6: 23.8 / 16.1 / 16.4 / 17.1, 52.9 / 50.8 / 51.8 / 59.9
template <int MB, int NB, int W = kNnWaves>
__global__ __launch_bounds__(W * kWave) void dense_nn_kernel(const DenseArgs a, const int slices)
{
    __shared__ float part[W][MB][NB][4][kWave];
    __shared__ int turn_s;
    const int lane = threadIdx.x & (kWave - 1), wv = wave_id();
    const int r = lane & 15, q = lane >> 4;
    // Work-group ids go round the 8 XCDs: the column tiles of one row tile get ids 8 apart, so that they run on one
    // XCD and the rows of the copy they all read come out of its L2 after the first of them has fetched them.
    const int n_col_tiles = (a.batch + 16 * NB - 1) / (16 * NB);
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, in_row = n_col_tiles * slices;
    const int m_tile = (slot / in_row) * 8 + xcd, rest = slot % in_row, col_tile = rest % n_col_tiles, slice = rest / n_col_tiles;
    if (m_tile * 16 * MB >= a.rows) return;  // (the grid is padded to whole rounds of the XCDs)
    const int i0 = m_tile * 16 * MB, n0 = col_tile * (16 * NB);
    const int K = a.cols;
    const int col = min(n0 + NB * r, a.batch - NB);
    const int k16 = K / 16;                                          // whole chunks of 16 k; the rest is the last wave's
    const int per = (k16 + W * slices - 1) / (W * slices);
    const int c_begin = min((slice * W + wv) * per, k16), c_end = min(c_begin + per, k16);
    v4f acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int t = 0; t < NB; ++t) acc[m][t] = v4f{0.f, 0.f, 0.f, 0.f};
    const float *wrow[MB];   // (rows past the last one repeat the first, their results are never stored)
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int row = i0 + 16 * m + r;
        wrow[m] = a.W + static_cast<int64_t>(row < a.rows ? row : 0) * a.ldw + q * 4;
    }
    if (c_begin < c_end) {  // uniform
        NnChunk<MB, NB> ring[kNnAhead];
        NnReader<MB, NB> next;
#pragma unroll
        for (int m = 0; m < MB; ++m) next.w[m] = wrow[m] + c_begin * 16;
        next.x = a.X + static_cast<int64_t>(c_begin * 16 + q * 4) * a.ldx + col;
        next.ldx = a.ldx; next.left = c_end - c_begin;
#pragma unroll
        for (int d = 0; d < kNnAhead; ++d) next.load(ring[d]);
        int c = c_begin;
        for (; c + kNnAhead <= c_end; c += kNnAhead) {
#pragma unroll
            for (int d = 0; d < kNnAhead; ++d) {
                nn_mfma<MB, NB>(ring[d], acc);
                next.load(ring[d]);
            }
        }
#pragma unroll
        for (int d = 0; d < kNnAhead; ++d) {
            if (c + d >= c_end) break;  // wave-uniform
            nn_mfma<MB, NB>(ring[d], acc);
        }
    }
    if (k16 * 16 < K && wv == W - 1 && slice == slices - 1) {  // uniform
        NnChunk<MB, NB> C;   // the operand's rows past K count as 0 (the copy holds zeros there, which an infinity would not leave zero)
#pragma unroll
        for (int m = 0; m < MB; ++m) C.w4[m] = ld4(wrow[m] + k16 * 16);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = k16 * 16 + q * 4 + s;
            nn_columns<NB>(a.X + static_cast<int64_t>(min(k, K - 1)) * a.ldx + col, C.b[s]);
#pragma unroll
            for (int t = 0; t < NB; ++t) C.b[s][t] = k < K ? C.b[s][t] : 0.f;
        }
        nn_mfma<MB, NB>(C, acc);
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) part[wv][m][t][g][lane] = acc[m][t][g];
    __syncthreads();
    if (W > kNnWaves && wv >= kNnWaves) return;   // (four registers to add up)
    float y[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            y[m][t] = 0.f;
#pragma unroll
            for (int w = 0; w < W; ++w) y[m][t] += part[w][m][t][wv][lane];
        }
    if (W == kNnWaves && slices > 1) {  // uniform
        // as the shares of a huge row (huge_row_share): out and back past the L2s, the last work-group of the tile adds them in slice order
        constexpr int kShare = MB * NB * kNnWaves * kWave;
        const int tile = m_tile * n_col_tiles + col_tile;
        float *tile_shares = a.partial + static_cast<int64_t>(tile) * slices * kShare + wv * kWave + lane;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int t = 0; t < NB; ++t)
                __hip_atomic_store(tile_shares + slice * kShare + (m * NB + t) * (kNnWaves * kWave), y[m][t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) turn_s = static_cast<int>(atomicInc(reinterpret_cast<unsigned *>(a.tickets) + tile, static_cast<unsigned>(slices - 1)));
        __syncthreads();
        if (turn_s != slices - 1) return;  // uniform
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int t = 0; t < NB; ++t) y[m][t] = 0.f;
        for (int s = 0; s < slices; ++s)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int t = 0; t < NB; ++t)
                    y[m][t] += __hip_atomic_load(tile_shares + s * kShare + (m * NB + t) * (kNnWaves * kWave), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int t = 0; t < NB; ++t) dense_epilogue(a, i0 + 16 * m + 4 * q + wv, n0 + NB * r < a.batch ? col + t : a.batch, a.rows, y[m][t]);
}

// Y (cols x batch) = (D^T X) * [YM > 0].  Work-group: 64 output rows (four tiles fed by one 16-byte load along
// the row of D: tile u holds the output rows j0 + 4 r' + u) x NB * 16 columns; the waves split K = rows, kTnDepth
// steps of loads in flight.  Wave w adds tile (w / 4), register (w % 4) of all slices in slice order.  Two work-groups fit on a compute unit
// (64 registers with one column tile: (512 x 1024 at batch 100, 2048 x 4096 at batch 256) 6.1 and 58 us, with 78 7.2 and 66.5; eight steps
// requested and then multiplied 7.1 and 63.8).  The more columns of the batch a work-group has, the fewer loads there are to a product, each of
// which holds the compute unit's vector memory pipe; it has as many waves less, so that their slices fit in LDS.
constexpr int kTnDepth = 3;

template <int NB>
__global__ __launch_bounds__(kSplitBlock / NB, 8 / NB) void dense_tn_kernel(const DenseArgs a)
{
    constexpr int kWaves = kSplitWaves / NB;
    __shared__ float part[kWaves][4][NB][4][kWave];
    const int lane = threadIdx.x & (kWave - 1), wv = wave_id();
    const int r = lane & 15, q = lane >> 4;
    const int j0 = blockIdx.x * 64, n0 = blockIdx.y * (16 * NB);
    const int K = a.rows;
    const float *wcol = a.W + j0 + r * 4;     // (ld is a multiple of 64: the access stays inside the row)
    const int col = min(n0 + NB * r, a.batch - NB);
    const int k4 = (K + 3) / 4;                                     // steps of 4 k (one per slot)
    const int per = (k4 + kWaves - 1) / kWaves;
    const int c_begin = min(wv * per, k4), c_end = min(c_begin + per, k4);
    v4f acc[4][NB];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < NB; ++t) acc[u][t] = v4f{0.f, 0.f, 0.f, 0.f};
    float4 w4[kTnDepth];
    float b[kTnDepth][NB];
    int i = min(c_begin, k4 - 1) * 4 + q, left = c_end - c_begin - 1;   // (a slice may be empty)
    const float *wp = wcol + i * a.ldw, *xp = a.X + i * a.ldx + col;
    auto load = [&](int d) __attribute__((always_inline)) {   // as in NnReader: step after step, the last one again past the end
        const bool ok = i < K;
        w4[d] = ld4(ok ? wp : wcol);
        nn_columns<NB>(ok ? xp : a.X, b[d]);
        const int step = left > 0 ? 4 : 0;   // uniform
        --left;
        i += step; wp += step * a.ldw; xp += step * a.ldx;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int c, int d) __attribute__((always_inline)) {
        if (c * 4 + 4 > K) {  // uniform: the last step
            const bool i_ok = c * 4 + q < K;
            w4[d] = i_ok ? w4[d] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int t = 0; t < NB; ++t) b[d][t] = i_ok ? b[d][t] : 0.f;
        }
        const float wv4[4] = {w4[d].x, w4[d].y, w4[d].z, w4[d].w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < NB; ++t) acc[u][t] = mfma(wv4[u], b[d][t], acc[u][t]);
    };
#pragma unroll
    for (int d = 0; d < kTnDepth; ++d) load(d);
    int c = c_begin;
    for (; c + kTnDepth <= c_end; c += kTnDepth) {
#pragma unroll
        for (int d = 0; d < kTnDepth; ++d) {
            multiply(c + d, d);
            load(d);
        }
    }
#pragma unroll
    for (int d = 0; d < kTnDepth; ++d) {
        if (c + d >= c_end) break;  // wave-uniform
        multiply(c + d, d);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) part[wv][u][t][g][lane] = acc[u][t][g];
    __syncthreads();
    const int g = wv & 3;
#pragma unroll
    for (int u = wv >> 2; u < 4; u += kWaves / 4)
#pragma unroll
        for (int t = 0; t < NB; ++t) {
            float y = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) y += part[w][u][t][g][lane];
            dense_epilogue(a, j0 + 4 * (4 * q + g) + u, n0 + NB * r < a.batch ? col + t : a.batch, a.cols, y);
        }
}

// Sampled gradient: G = dZ X^T by MFMA tiles, of which only the entries on the pattern are used -- each tile takes the
// momentum step (or the store of the gradient) of its stored entries straight from its accumulators.  An entry is found
// through the layer's pattern table: 32 columns of a row are a word of bits and the CSR position of the first of them,
// so entry (i, j)'s position is that plus the bits below j.  K = batch is short, so there is no split: a work-group of 4
// waves owns 64 x 64 of G, a wave 32 x 32.  The waves of the first tile column add up the rows of dZ they hold for the bias
// gradient.  Up to kSampledLayers layers share the grid.
// What bounds it: the MFMA pipes (the 1024 x 3072 layer of the paper's MLP at batch 100: 4.5 us of steps) and the few
// round trips at either end.  Before, G went to memory and a second launch picked the pattern's entries: 18.8 + 11.8 us for
// that layer at 50 % sparsity, now 18.2 for both.
constexpr int kSampledWaves = 4;

constexpr int kSampledK = 64;                  // columns of the batch in LDS at a time
constexpr int kSampledLd = kSampledK + 4;      // floats per row there: the 16 rows of a fragment read start in different banks
constexpr int kSampledAhead = 4;               // entries per thread whose state is requested before the products are formed

__global__ __launch_bounds__(kSampledWaves * kWave) void sampled_update_kernel(const SampledArgs A)
{
    constexpr int kThreads = kSampledWaves * kWave;
    __shared__ float tile[2][64][kSampledLd];   // operands; afterwards the gradients of the tile's entries and their columns
    __shared__ uint2 tab[64][2];                // the tile's rows of the pattern table
    __shared__ int32_t first[65];               // entries of the tile before each row
    const int lane = threadIdx.x & (kWave - 1), wv = wave_id(), tid = threadIdx.x;
    if (A.loss_cols && blockIdx.x == 0 && wv == 0) mean_of(A.loss_cols, A.loss_n, A.loss_out);
    int k = 0;
#pragma unroll
    for (int i = 1; i < kSampledLayers; ++i)
        if (i < A.n && static_cast<int>(blockIdx.x) >= A.layer[i].first_block) k = i;
    const SampledLayer &L = A.layer[k];
    // Consecutive tiles -- down eight rows of tiles, then to the next column -- belong to one XCD (work-groups go to the
    // XCDs in turn): it then writes whole lines of values[], of which its neighbours' tiles hold the rest (tiles dealt
    // out plainly: 17.4 us for the 1024 x 3072 layer at 10 %, 14.0), and what its tiles read stays within its L2.
    const int block = blockIdx.x - L.first_block, per_xcd = (L.tiles_i * L.tiles_j + 7) >> 3;
    const int index = (block & 7) * per_xcd + (block >> 3), down = index / (8 * L.tiles_j) * 8, high = min(8, L.tiles_i - down);
    if (index >= L.tiles_i * L.tiles_j) return;
    const int in_band = index - down * L.tiles_j;
    const int ib = (down + in_band % high) * 64, jb = in_band / high * 64;
    const int wi = (wv >> 1) * 32, wj = (wv & 1) * 32;   // the wave's part of the tile
    const int r = lane & 15, q = lane >> 4;

    uint2 my_tab = make_uint2(0, 0);
    if (tid < 128) {
        const int i = ib + (tid >> 1), word = (jb >> 5) + (tid & 1);
        const uint2 e = L.table[static_cast<int64_t>(min(i, L.rows - 1)) * L.words + min(word, L.words - 1)];
        if (i < L.rows && word < L.words) my_tab = e;
    }
    // Operands go through LDS: read straight from memory, a fragment is 16 rows of 64 bytes each, a leading dimension apart,
    // which costs the memory pipeline several times what 256-byte row pieces do (the layer above: 31.7 us, 22.6 through LDS).
    // A thread brings four columns of rows sr, sr + 16, ... of both operands, a chunk ahead.
    const int sr = tid >> 4, sc = (tid & 15) * 4;
    float4 zn[4], xn[4];
    const gmem_ptr zb = as_gmem(L.dZ), xb = as_gmem(L.X);
    uint32_t z_row[4], x_row[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int zi = min(ib + sr + 16 * u, L.rows - 1);
        z_row[u] = static_cast<uint32_t>(L.list ? L.list[zi] : zi) * (static_cast<uint32_t>(L.lddz) * 4u);
        x_row[u] = static_cast<uint32_t>(min(jb + sr + 16 * u, L.cols - 1)) * (static_cast<uint32_t>(L.ldx) * 4u);
    }
    auto fetch = [&](int kb) {
        const int own = kb + sc, c = four_columns(own, A.batch);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            zn[u] = gload4(zb, z_row[u] + static_cast<uint32_t>(c) * 4u);
            xn[u] = gload4(xb, x_row[u] + static_cast<uint32_t>(c) * 4u);
        }
        if (kb + kSampledK > A.batch) {  // uniform: columns that another thread has, or none, count as 0
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                zn[u] = own < A.batch ? drop_shared(zn[u], own, c) : make_float4(0.f, 0.f, 0.f, 0.f);
                xn[u] = own < A.batch ? drop_shared(xn[u], own, c) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    };
    // The tiles start at different chunks: rows of wide batches lie a multiple of 4 KiB apart, and tiles that walked the
    // columns in step would meet in the same channels of the L2s (4096 x 4096 at batch 1024: 325 us in step, with row offsets kept in registers 290).
    const int n_chunks = (A.batch + kSampledK - 1) / kSampledK;
    int chunk = index % n_chunks;
    fetch(chunk * kSampledK);

    // where the tile's entries are: row by row they are runs of the CSR arrays
    if (tid < 128) {
        tab[tid >> 1][tid & 1] = my_tab;
        const int pair = __popc(my_tab.x) + __shfl_xor(__popc(my_tab.x), 1, kWave);
        if ((tid & 1) == 0) first[(tid >> 1) + 1] = pair;
        if (tid == 0) first[0] = 0;
    }
    __syncthreads();
    if (wv == 0) {
        int v = first[lane + 1];
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int y = __shfl_up(v, d, kWave);
            if (lane >= d) v += y;
        }
        first[lane + 1] = v;
    }
    __syncthreads();
    const int n_entries = first[64];
    // CSR position of the tile's e-th entry
    auto entry = [&](int e, int &row) {
        int lo = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1)
            if (first[lo + step] <= e) lo += step;
        row = lo;
        return static_cast<uint32_t>(tab[lo][0].y) + static_cast<uint32_t>(e - first[lo]);
    };
    // the state of the thread's first entries travels while the products are formed
    const gmem_ptr values = as_gmem(L.values), velocity = as_gmem(L.velocity), pos_t = as_gmem(L.pos_t);
    uint32_t at[kSampledAhead];
    int row_of[kSampledAhead];
    float w[kSampledAhead], v[kSampledAhead], to[kSampledAhead];
    if (L.fused && n_entries > 0) {  // uniform
#pragma unroll
        for (int u = 0; u < kSampledAhead; ++u) {
            if (u * kThreads < n_entries) {
                at[u] = entry(min(tid + u * kThreads, n_entries - 1), row_of[u]) * 4u;
                w[u] = gload1(values, at[u]);
                v[u] = gload1(velocity, at[u]);
                if (L.values_t) to[u] = gload1(pos_t, at[u]);
            }
        }
    }

    v4f acc[2][2];
    float row_sum[2] = {0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[m][t] = v4f{0.f, 0.f, 0.f, 0.f};
    const bool sum = jb + wj == 0 && (L.db || (L.fused && L.bias));
    for (int c = 0; c < n_chunks; ++c) {
        const int kb = chunk * kSampledK;
        if (c > 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            *reinterpret_cast<float4 *>(&tile[0][sr + 16 * u][sc]) = zn[u];
            *reinterpret_cast<float4 *>(&tile[1][sr + 16 * u][sc]) = xn[u];
        }
        __syncthreads();
        chunk = chunk + 1 == n_chunks ? 0 : chunk + 1;
        if (c + 1 < n_chunks) fetch(chunk * kSampledK);
        const int steps = min(kSampledK, A.batch - kb);
#pragma unroll
        for (int d = 0; d < kSampledK / 16; ++d) {
            if (16 * d >= steps) break;  // uniform
            float4 z[2], x[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                z[m] = *reinterpret_cast<const float4 *>(&tile[0][wi + 16 * m + r][16 * d + 4 * q]);
                x[m] = *reinterpret_cast<const float4 *>(&tile[1][wj + 16 * m + r][16 * d + 4 * q]);
            }
            if (sum)
#pragma unroll
                for (int m = 0; m < 2; ++m) row_sum[m] += (z[m].x + z[m].y) + (z[m].z + z[m].w);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[m][t] = mfma(s == 0 ? z[m].x : s == 1 ? z[m].y : s == 2 ? z[m].z : z[m].w,
                                         s == 0 ? x[t].x : s == 1 ? x[t].y : s == 2 ? x[t].z : x[t].w, acc[m][t]);
        }
    }

    if (sum) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            float s = row_sum[m];
            s += __shfl_xor(s, 16, kWave);
            s += __shfl_xor(s, 32, kWave);
            int i = ib + wi + 16 * m + r;
            if (q == 0 && i < L.rows) {
                if (L.list) i = L.list[i];
                if (L.db) L.db[i] = s;
                if (L.fused && L.bias) {
                    float bw = L.bias[i], bv = L.bias_velocity[i];
                    momentum_step(bw, bv, s, A.lr, A.momentum, A.nesterov);
                    L.bias[i] = bw;
                    L.bias_velocity[i] = bv;
                }
            }
        }
    }
    // The accumulators' elements that are stored entries, entry after entry in LDS: a thread per entry then finds runs of
    // consecutive positions in memory, and not one element in ten of a register.
    __syncthreads();
    float *grad = &tile[0][0][0];                                                    // [4096]
    unsigned char *column = reinterpret_cast<unsigned char *>(grad + 64 * 64);       // [4096]
    static_assert(sizeof(tile) >= 64 * 64 * 5, "the tile's entries fit where its operands were");
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int il = wi + 16 * m + 4 * q + g;
            const uint32_t bits = tab[il][wj >> 5].x;
            const int base = first[il] + (wj ? __popc(tab[il][0].x) : 0);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint32_t bit = 1u << (16 * t + r);
                const int e = base + __popc(bits & (bit - 1u));
                if (bits & bit) {
                    grad[e] = acc[m][t][g];
                    column[e] = static_cast<unsigned char>(wj + 16 * t + r);
                }
            }
        }
    __syncthreads();
    if (L.g)
        for (int e = tid; e < n_entries; e += kThreads) {
            int row;
            const uint32_t p = entry(e, row);
            gstore1(L.g, p * 4u, grad[e]);
        }
    if (!L.fused) return;
    auto update = [&](int e, uint32_t p4, int row, float pw, float pv, uint32_t pt) {
        momentum_step(pw, pv, grad[e], A.lr, A.momentum, A.nesterov);
        gstore1(L.values, p4, pw);
        gstore1(L.velocity, p4, pv);
        if (L.values_t) gstore1(L.values_t, pt * 4u, pw);
        if (L.dense) gstore1(L.dense, (static_cast<uint32_t>(ib + row) * static_cast<uint32_t>(L.dense_ld) + jb + column[e]) * 4u, pw);
    };
#pragma unroll
    for (int u = 0; u < kSampledAhead; ++u) {
        const int e = tid + u * kThreads;
        if (e < n_entries) update(e, at[u], row_of[u], w[u], v[u], __builtin_bit_cast(uint32_t, to[u]));
    }
    for (int e0 = kSampledAhead * kThreads; e0 < n_entries; e0 += kSampledAhead * kThreads) {
#pragma unroll
        for (int u = 0; u < kSampledAhead; ++u) {
            at[u] = entry(min(e0 + tid + u * kThreads, n_entries - 1), row_of[u]) * 4u;
            w[u] = gload1(values, at[u]);
            v[u] = gload1(velocity, at[u]);
            if (L.values_t) to[u] = gload1(pos_t, at[u]);
        }
#pragma unroll
        for (int u = 0; u < kSampledAhead; ++u) {
            const int e = e0 + tid + u * kThreads;
            if (e < n_entries) update(e, at[u], row_of[u], w[u], v[u], __builtin_bit_cast(uint32_t, to[u]));
        }
    }
}

// ---- dense rows ----------------------------------------------------------------------------------
// Y[i, :] = act(W[i, :] X + b[i]) for the rows of a sparse matrix that store an eighth of their columns or more (the heads
// of power-law matrices; evenly filled matrices of 30 to 40 %): an MFMA product whose left operand is made dense on the
// way into LDS.  A work-group of 4 waves owns 64 of the listed rows and 32 T columns of the batch; 64 columns of the matrix
// at a time, a wave places the entries of 16 rows, a lane per column: the pattern table says whether there is one and where
// (a row's entries are a run of values[]), the others are 0.  The operand's 64 rows come through LDS as well.  Both travel
// a step ahead, the table two.  K is cut into slices where the tiles do not fill the chip; dense_rows_finish_kernel adds them in
// slice order.  A step whose operand holds an Inf or NaN goes entry by entry, so that only rows that store the entry see it.
// What bounds it: the MFMA pipes, 4096 cycles of a step of T = 4.  Measured on 16384^2 power-law rows at 10 %, batch 1024:
// the 2611 dense rows (69 % of the entries) take 800 us (110 TFLOP/s), the others 1021 in the staged kernel, which took
// 3320 for all; at 3 %: 1787 -> 735.
constexpr int kDrRows = 64, kDrK = 64, kDrALd = kDrK + 4;

__device__ __forceinline__ void dense_rows_store(const SpmmArgs &a, int row, int col, float4 y)
{
    const float b = a.bias ? a.bias[row] : 0.f;
    y = make_float4(y.x + b, y.y + b, y.z + b, y.w + b);
    if (a.relu) y = make_float4(y.x > 0.f ? y.x : 0.f, y.y > 0.f ? y.y : 0.f, y.z > 0.f ? y.z : 0.f, y.w > 0.f ? y.w : 0.f);
    if (a.YM) y = keep_where_positive(y, ld4(a.YM + static_cast<int64_t>(row) * a.ldym + col));
    st4(a.Y + static_cast<int64_t>(row) * a.ldy + col, y);
}

template <int T>
__global__ __launch_bounds__(kDenseBlock) __attribute__((amdgpu_waves_per_eu(3))) void dense_rows_kernel(const SpmmArgs a, const DenseRows D,
                                                                                                             const int slices)
{
    constexpr int kCols = 32 * T, kQuads = kCols / 4, kRound = kDenseBlock / kQuads;   // operand rows the work-group brings at a time
    __shared__ float as[kDrRows][kDrALd];
    __shared__ float xs[kDrK][kCols + (T == 4 ? 4 : 8)];   // (rows that lanes read together start in different banks)
    __shared__ uint2 tab[2][kDrRows][2];
    __shared__ int4 odd_wave;   // per wave: it has brought an operand that is not finite
    const int lane = threadIdx.x & (kWave - 1), wv = wave_id(), tid = threadIdx.x;
    const int r = lane & 15, q = lane >> 4;
    const int row_tiles = (D.n + kDrRows - 1) / kDrRows;
    // consecutive work-groups share the slice of the operand: row tiles run fastest
    const int row_tile = blockIdx.x % row_tiles, rest = blockIdx.x / row_tiles, slice = rest % slices, n0 = rest / slices * kCols;
    const int ib = row_tile * kDrRows, wi = (wv >> 1) * 32, wj = (wv & 1) * 16 * T;
    const int chunks = (a.x_rows + kDrK - 1) / kDrK, per = (chunks + slices - 1) / slices;
    const int c_begin = min(slice * per, chunks), c_end = min(c_begin + per, chunks);
    const gmem_ptr X = as_gmem(a.X), values = as_gmem(a.values);
    const uint32_t last = static_cast<uint32_t>(a.nnz - 1) * 4u, ldxb = static_cast<uint32_t>(a.ldx) * 4u;

    uint2 tab_next;
    auto load_table = [&](int c) {  // threads 0 .. 127: row tid / 2, word tid & 1 of chunk c
        const int word = c * 2 + (tid & 1), i = min(ib + ((tid >> 1) & 63), D.n - 1);
        tab_next = D.table[static_cast<int64_t>(i) * D.words + min(word, D.words - 1)];
        if (word >= D.words || c >= c_end) tab_next.x = 0;
    };
    auto keep_table = [&](int buf) { if (tid < 2 * kDrRows) tab[buf][tid >> 1][tid & 1] = tab_next; };
    float av[16];
    uint32_t set = 0;
    float4 xv[kDrK / kRound];
    const int xr = tid / kQuads, xq = tid % kQuads;
    const int own = n0 + xq * 4, xcol = four_columns(own < a.batch ? own : n0, a.batch);
    auto fetch = [&](int c, int buf) {
        set = 0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const uint2 t = tab[buf][wv * 16 + u][lane >> 5];
            const uint32_t bit = 1u << (lane & 31);
            set |= t.x & bit ? 1u << u : 0u;
            av[u] = gload1(values, min((t.y + static_cast<uint32_t>(__popc(t.x & (bit - 1u)))) * 4u, last));
        }
#pragma unroll
        for (int u = 0; u < kDrK / kRound; ++u) {
            const int k = min(c * kDrK + xr + kRound * u, a.x_rows - 1);
            xv[u] = gload4(X, static_cast<uint32_t>(k) * ldxb + static_cast<uint32_t>(xcol) * 4u);
        }
    };
    v4f acc[2][T];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int t = 0; t < T; ++t) acc[m][t] = v4f{0.f, 0.f, 0.f, 0.f};
    load_table(c_begin);
    keep_table(0);
    __syncthreads();
    if (c_begin < c_end) fetch(c_begin, 0);
    load_table(c_begin + 1);
    for (int c = c_begin; c < c_end; ++c) {
        const int next = (c + 1 - c_begin) & 1;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) as[wv * 16 + u][lane] = set & (1u << u) ? av[u] : 0.f;
#pragma unroll
        for (int u = 0; u < kDrK / kRound; ++u) *reinterpret_cast<float4 *>(&xs[xr + kRound * u][xq * 4]) = xv[u];
        float zero = 0.f;
#pragma unroll
        for (int u = 0; u < kDrK / kRound; ++u) zero = fmaf(xv[u].x, 0.f, fmaf(xv[u].y, 0.f, fmaf(xv[u].z, 0.f, fmaf(xv[u].w, 0.f, zero))));
        const bool odd_here = __any(!(zero == 0.f));
        if (lane == 0) reinterpret_cast<int *>(&odd_wave)[wv] = odd_here;
        keep_table(next);
        __syncthreads();
        const int4 odd4 = odd_wave;
        const bool odd = __builtin_amdgcn_readfirstlane(odd4.x | odd4.y | odd4.z | odd4.w);
        if (c + 1 < c_end) {
            fetch(c + 1, next);
            load_table(c + 2);
        }
        if (odd) {  // an entry that is not stored must not meet an Inf or NaN with its 0: entry by entry
            for (int k = 0; k < kDrK; ++k) {
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int i = wi + 16 * m + 4 * q + g;
                        const bool stored = (tab[1 - next][i][k >> 5].x >> (k & 31)) & 1u;
                        const float w = as[i][k];
#pragma unroll
                        for (int t = 0; t < T; ++t) acc[m][t][g] = stored ? fmaf(w, xs[k][wj + T * r + t], acc[m][t][g]) : acc[m][t][g];
                    }
            }
            continue;
        }
#pragma unroll
        for (int d = 0; d < kDrK / 16; ++d) {
            float4 f[2];
            float x[4][T];
#pragma unroll
            for (int m = 0; m < 2; ++m) f[m] = *reinterpret_cast<const float4 *>(&as[wi + 16 * m + r][16 * d + 4 * q]);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float *p = &xs[16 * d + 4 * q + s][wj + T * r];   // (tile t holds the columns wj + T r + t)
                if constexpr (T == 4) {
                    const float4 v = *reinterpret_cast<const float4 *>(p);
                    x[s][0] = v.x; x[s][1] = v.y; x[s][2] = v.z; x[s][3] = v.w;
                } else {
                    const float2 v = *reinterpret_cast<const float2 *>(p);
                    x[s][0] = v.x; x[s][1] = v.y;
                }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const float fs = s == 0 ? f[m].x : s == 1 ? f[m].y : s == 2 ? f[m].z : f[m].w;
#pragma unroll
                    for (int t = 0; t < T; ++t) acc[m][t] = mfma(fs, x[s][t], acc[m][t]);
                }
        }
    }
    // A lane stores four columns at a time: with T = 2 it has two of them, and of a pair of lanes the even one takes all
    // four of its row of the first 16, the odd one of the other 16.
    auto store = [&](int k, int own_out, float4 y) {
        if (k >= D.n || own_out >= a.batch) return;
        const int col = four_columns(own_out, a.batch);
        if (slices > 1)
            st4(D.partial + (static_cast<int64_t>(slice) * D.n + k) * dense_rows_ld(a.batch) + col, y);
        else
            dense_rows_store(a, D.list[k], col, y);
    };
    if constexpr (T == 4) {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                store(ib + wi + 16 * m + 4 * q + g, n0 + wj + 4 * r, make_float4(acc[m][0][g], acc[m][1][g], acc[m][2][g], acc[m][3][g]));
    } else {
        const bool odd = r & 1;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float give0 = odd ? acc[0][0][g] : acc[1][0][g], give1 = odd ? acc[0][1][g] : acc[1][1][g];
            const float got0 = __shfl_xor(give0, 1, kWave), got1 = __shfl_xor(give1, 1, kWave);
            const float4 y = odd ? make_float4(got0, got1, acc[1][0][g], acc[1][1][g]) : make_float4(acc[0][0][g], acc[0][1][g], got0, got1);
            store(ib + wi + (odd ? 16 : 0) + 4 * q + g, n0 + wj + 4 * (r >> 1), y);
        }
    }
}

__global__ __launch_bounds__(kDenseBlock) void dense_rows_finish_kernel(const SpmmArgs a, const DenseRows D, const int slices)
{
    const int quads = (a.batch + 3) / 4;
    const int64_t n = static_cast<int64_t>(D.n) * quads, ld = dense_rows_ld(a.batch), step = D.n * ld;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kDenseBlock + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * kDenseBlock) {
        const int64_t k = i / quads;
        const int col = four_columns(static_cast<int>(i - k * quads) * 4, a.batch);
        const float *p = D.partial + k * ld + col;
        float4 y = ld4(p);
        for (int q = 1; q < slices; ++q) {
            const float4 v = ld4(p + q * step);
            y.x += v.x; y.y += v.y; y.z += v.z; y.w += v.w;
        }
        dense_rows_store(a, D.list ? D.list[k] : k, col, y);
    }
}

// The pattern table: a thread per 32 columns of a row finds the row's first entry among them and collects their bits.
__global__ __launch_bounds__(kDenseBlock) void pattern_table_kernel(const int32_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                                   const int32_t *__restrict__ list, int rows, int words, uint2 *__restrict__ table, const int32_t *status)
{
    if (status && status[0] != 0) return;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kDenseBlock, n = static_cast<int64_t>(rows) * words;
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kDenseBlock + threadIdx.x; k < n; k += stride) {
        const int at = static_cast<int>(k / words), row = list ? list[at] : at;
        const int64_t j0 = (k - static_cast<int64_t>(at) * words) * 32;
        int32_t lo = indptr[row], hi = indptr[row + 1];
        const int32_t end = hi;
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (indices[mid] >= j0)
                hi = mid;
            else
                lo = mid + 1;
        }
        uint32_t bits = 0;
        for (int32_t p = lo; p < end && indices[p] - j0 < 32; ++p) bits |= 1u << (indices[p] - j0);
        table[k] = make_uint2(bits, static_cast<uint32_t>(lo));
    }
}

// One wave per row of the CSR matrix: scatters the row's values into the dense copy.
__global__ __launch_bounds__(kDenseBlock) void dense_refresh_kernel(const int32_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                                   const float *__restrict__ values, int rows, float *D, int64_t ld)
{
    const int lane = threadIdx.x & (kWave - 1);
    for (int i = blockIdx.x * kDenseWaves + wave_id(); i < rows; i += gridDim.x * kDenseWaves)
        for (int p = indptr[i] + lane; p < indptr[i + 1]; p += kWave) D[static_cast<int64_t>(i) * ld + indices[p]] = values[p];
}

inline int blocks_for_rows(int64_t rows)
{
    int64_t b = (rows + kDenseWaves - 1) / kDenseWaves;
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return static_cast<int>(b);
}

}  // namespace

// Columns of the batch per work-group: as many as still leave the chip's 256 compute units a work-group each.
static int dense_nb(int64_t m_tiles, int batch)
{
    for (int nb = 4; nb > 1; nb >>= 1)
        if (m_tiles * ((batch + 16 * nb - 1) / (16 * nb)) >= 256) return nb;
    return 1;
}

// Tiles of 16 mb x 16 nb and slices of the sum of a forward product.  A compute unit takes a wave's loads in at 28 cycles each (its vector
// memory pipe was 90 % busy, the MFMA pipes 39, at 16 x 32), so tiles are as wide as 256 of them allow: 64 columns are loaded as fast as 32.  Where
// there are a few less and the sum is long, work-groups share a tile, which costs 3 to 4 us.  us, before -> with 16 x 64 in two slices:
// 1024 x 3072 at batch 100 15.1 -> 13.0, 1024 x 1536 10.0 -> 9.5, 2048 x 2048 at 64 11.2 -> 10.8, 2048 x 4096 at 64 19.0 -> 15.8 (512 x 1024 at 100
// 6.2 -> 7.7); in four: 1024 x 4096 at 64 16.3 -> 11.6, 512 x 3072 at 100 12.9 -> 10.2, 512 x 2048 9.4 -> 9.0, 1024 x 2000 at 64 9.6 -> 9.1 (1024 x 1536 at 64, with the copy's refresh,
// 13.1 -> 14.0).
// 32 x 64 is a tenth faster than two of 16 x 64 one after the other, so it pays where it leaves no compute unit with more of them (with the copy's refresh): 1024 x 3072 at batch 512 (256
// work-groups) 46.7 -> 40.8, 2048 x 2560 at 200 (256) 41.2 -> 36.9, 4096 x 2048 at 128 (256) 39.7 -> 36.0, at 1024 (2048) 203 -> 196; but 1024 x 3072 at 700 (352) 62.3 -> 76.5, 2048 x 3072 at
// 300 (320) 63.5 -> 77.9, 4096 x 4096 at 400 (896) 177 -> 194; 8192 x 2048 at 512 (2048) 204 -> 209.
struct NnCut {
    int mb, nb, slices;
};
static NnCut nn_cut(const DenseArgs &a)
{
    const int64_t wide = (a.batch + 63) / 64, tiles = (static_cast<int64_t>(a.rows) + 15) / 16 * wide;
    const int64_t pairs = (static_cast<int64_t>(a.rows) + 31) / 32 * wide;
    if (a.cols >= 2048 && (a.cols >= 2560 || pairs <= 512) && pairs >= 256 && (pairs + 255) / 256 * 2 <= (tiles + 255) / 256 && a.batch >= 4) return NnCut{2, 4, 1};
    if (a.cols >= (tiles < kNnShareTiles / 2 ? kNnShareFourCols : kNnShareCols) && a.batch > 32 && a.tickets && tiles >= kNnShareTiles / 4 && tiles < kNnShareTiles)
        return NnCut{1, 4, tiles < kNnShareTiles / 2 ? 4 : 2};
    int nb = dense_nb((static_cast<int64_t>(a.rows) + 15) / 16, a.batch);
    while (nb > a.batch) nb >>= 1;   // (a lane's columns lie within the batch)
    return NnCut{1, nb, 1};
}

hipError_t launch_dense_product(const DenseArgs &a, hipStream_t s)
{
    if (a.rows <= 0 || a.cols <= 0 || a.batch <= 0) return hipSuccess;
    if (!a.trans) {
        const NnCut cut = nn_cut(a);
        const int64_t mt = (a.rows + 16 * cut.mb - 1) / (16 * cut.mb);
        const dim3 grid(static_cast<unsigned>((mt + 7) / 8 * 8 * ((a.batch + 16 * cut.nb - 1) / (16 * cut.nb)) * cut.slices));
        DenseArgs own = a;
        if (cut.slices == 4) own.tickets += kNnShareTiles;
        auto go = [&](auto kernel, int waves = kNnWaves) { hipLaunchKernelGGL(kernel, grid, dim3(waves * kWave), 0, s, own, cut.slices); };
        if (cut.mb == 1 && cut.nb == 1 && mt * ((a.batch + 15) / 16) <= 256) go(dense_nn_kernel<1, 1, 2 * kNnWaves>, 2 * kNnWaves);
        else go(cut.mb == 2 ? dense_nn_kernel<2, 4> : cut.nb == 4 ? dense_nn_kernel<1, 4> : cut.nb == 2 ? dense_nn_kernel<1, 2> : dense_nn_kernel<1, 1>);
    } else {
        // One, two or four tiles of 16 columns, us: 2048 x 4096 at batch 256 54.9 / 47.7 / 50.3 (512 and 256 work-groups), at 1024 192 / 161 / 153;
        // 1024 x 4096 at 512 57.7 / 48.7 / 47.2, 4096 x 4096 at 100 53.8 / 49.6 with two, 1201 x 2201 at 301 (350) 33.8 / 29.0; a few more than one to a compute unit lose:
        // 2000 x 6000 at 77 (282) 57.9 / 62.6, 2048 x 4096 at 150 (320) 54.6 / 59.3, 1024 x 3072 at 200 (336, of 224 columns) 32.8 / 34.9, but 1000 x 4000 at 150 (315) 41.6 / 37.8.
        const int64_t across = (static_cast<int64_t>(a.cols) + 63) / 64, twos = across * ((a.batch + 31) / 32);
        const bool few_more = twos > 256 && twos <= 340 && (a.rows > 1024 || (a.batch + 31) / 32 * 200 > (a.batch + 15) / 16 * 106);
        const int nb = a.batch >= 4 && across * ((a.batch + 63) / 64) >= 512 ? 4 : a.batch >= 2 && twos >= 256 && !few_more ? 2 : 1;
        const dim3 grid(static_cast<unsigned>(across), (a.batch + 16 * nb - 1) / (16 * nb)), block(kSplitBlock / nb);
        if (nb == 4) hipLaunchKernelGGL(dense_tn_kernel<4>, grid, block, 0, s, a);
        else if (nb == 2) hipLaunchKernelGGL(dense_tn_kernel<2>, grid, block, 0, s, a);
        else hipLaunchKernelGGL(dense_tn_kernel<1>, grid, block, 0, s, a);
    }
    return hipGetLastError();
}

// what the sampled kernel asks of a layer's arrays: 32-bit byte offsets
bool sampled_operands_ok(const SddmmCall &a)
{
    return a.nnz > 0 && a.nnz < (1 << 30) && a.batch >= kSampledMinBatch && !a.ZM && !a.skip_products &&
           static_cast<int64_t>(a.rows) * a.lddz < (1 << 30) && static_cast<int64_t>(a.x_rows) * a.ldx < (1 << 30) &&
           (!a.dense || static_cast<int64_t>(a.rows) * a.dense_ld < (1 << 30));
}

bool sddmm_sampled_possible(const SddmmCall &a) { return a.table && sampled_operands_ok(a); }

bool sddmm_sampled_ok(const SddmmCall &a)
{
    if (!sddmm_sampled_possible(a) || a.rows < 64 || a.x_rows < 64) return false;
    // Measured against the gathering SDDMM, uniform patterns: 4096 x 3072 at batch 100 / 1024, 15 %: 42.6 / 242 us against 43.8 /
    // 238 there, 20 %: 43.5 / 238 against 59.5 / 299; 1024 x 3072, 20 %: 13.7 / 70 against 16.1 / 100.  Few tiles do not fill
    // the chip: 512 x 1024 (128 tiles) at 30 %: 8.9 / 32.4 against 7.3 / 38.9.
    const int64_t tiles = static_cast<int64_t>((a.rows + 63) / 64) * ((a.x_rows + 63) / 64);
    const double from = tiles >= 512 ? kTableFromDensity : 2.3 * kTableFromDensity;
    return a.dense || static_cast<double>(a.nnz) >= from * a.rows * a.x_rows;
}

// How a product of n dense rows is cut: columns of the batch per work-group, slices of K; on the bf16 units (split_dense_rows_kernel) or the
// fp32 ones.
struct DenseRowsCut {
    int cols, slices;
    int64_t tiles;
    bool split;
    double time;
};
// The cheapest by an estimate.  fp32: a compute unit holds 3 (4) work-groups of 128 (64) columns, which take 2.0 (1.1) us a step
// each when they keep its pipes busy together and 3.7 (2.6) alone; the slices' results go out and come back at 3.3 TB/s.
// (Within 3 to 7 % of the best of 20 cuts on matrices of 1024 to 16384 rows at batches of 128 to 1024.)
static DenseRowsCut dense_rows_fp32_cut(int32_t n, int32_t cols, int32_t batch)
{
    const int64_t chunks = (static_cast<int64_t>(cols) + kDrK - 1) / kDrK;
    DenseRowsCut best{};
    for (int wide = 1; wide >= 0; --wide) {
        const int tile_cols = wide ? 128 : 64, fit = wide ? 3 : 4;
        const double alone = wide ? 3.7 : 2.6, step = wide ? 2. : 1.1;
        const int64_t tiles = static_cast<int64_t>((n + kDrRows - 1) / kDrRows) * ((batch + tile_cols - 1) / tile_cols);
        for (int s = 1; s == 1 || (s <= 64 && s * 2 <= chunks); ++s) {
            const int64_t per_unit = (tiles * s + 255) / 256, full = per_unit / fit, left = per_unit % fit;
            const double rounds = full * std::max(alone, step * fit) + (left ? std::max(alone, step * left) : 0.);
            const double time = rounds * static_cast<double>((chunks + s - 1) / s) + (s > 1 ? 2. + 1.2e-6 * s * n * static_cast<double>(dense_rows_ld(batch)) : 0.);
            if (best.tiles == 0 || time < best.time) best = DenseRowsCut{tile_cols, s, tiles, false, time};
        }
    }
    return best;
}

// Split operands: one work-group per compute unit, 2.8 us per 32 columns of the matrix; before it the operand's parts are formed (10 bytes a number
// at 4.5 TB/s), after it the slices are added.  Within 12 % of 190 products measured.  fp32 -> split, us, matrices of 32 to 38 %: 2600 rows of 16384 at batch
// 1024 / 512 / 256: 833 -> 567, 459 -> 303, 237 -> 165; 873 of 11642: 254 -> 175, 124 -> 93, 74 -> 61; 8192 of 4096: 648 -> 420, 339 -> 235, 176 -> 124;
// 700 of 4096 at 1024: 75 -> 62; 2048 of 2048 at 1024 / 512: 95 -> 73, 53 -> 48.  The fp32 estimate is low on these by a quarter and a launch; 300 rows of 16384,
// 1024 of 3072 up to 640 columns and the like stay with it.
static DenseRowsCut dense_rows_split_cut(int32_t n, int32_t cols, int32_t batch)
{
    const int64_t chunks = (static_cast<int64_t>(cols) + 31) / 32, tiles = split_dense_rows_tiles(n, batch);
    const double parts = 3. + 10. * cols * static_cast<double>(operand_parts_ld(batch)) / 4.5e6;
    DenseRowsCut best{};
    for (int s = 1; s == 1 || (s <= 64 && s * 4 <= chunks); ++s) {
        if ((chunks + s - 1) / s > kSplitMaxChunks || chunks > 65535) continue;   // (65535: grid of the parts' launch)
        const double time = 2. + parts + 2.8 * static_cast<double>((tiles * s + 255) / 256 * ((chunks + s - 1) / s)) +
                            (s > 1 ? 3. + 8. * s * n * static_cast<double>(dense_rows_ld(batch)) / 4.5e6 : 0.);
        if (best.tiles == 0 || time < best.time) best = DenseRowsCut{0, s, tiles, true, time};
    }
    return best;
}

constexpr int64_t kPartsMaxInts = 1ll << 29;   // (32-bit byte offsets)
static DenseRowsCut dense_rows_cut(int32_t n, int32_t cols, int32_t batch, const DenseRowsCut &fp32)
{
    const DenseRowsCut split = dense_rows_split_cut(n, cols, batch);
    return split.tiles > 0 && split.time < 4. + 1.25 * fp32.time && operand_parts_ints(cols, batch) < kPartsMaxInts ? split : fp32;
}

// What gathering for a thin matrix (kThinDensity) takes, us.  Staged (as staged_pays has it): 0.84 ns an entry of a work-group's range and
// column tile, one work-group a compute unit, which copies its tile of the operand into LDS beside that at 57 GB/s; else about 25 TB/s of gathers.  Within 3 % (root mean square; 8 at most) of 139
// staged products of uniform matrices of 17 to 30 % with 600 to 16384 rows, each bound for the batch; within 10 % of most of 31 gathered ones (2600 x 16384 at 28 %, batch 256 takes 651 for 489).
static double thin_rows_gathered(const DenseSplit &d, int32_t cols, int32_t batch)
{
    const int64_t tiles = (static_cast<int64_t>(batch) + kStageCols - 1) / kStageCols, ranges = staged_ranges_aim(d.rows.n, d.max_batch), groups = tiles * ranges;
    if (static_cast<int64_t>(batch) * 5 < tiles * kStageCols * 4 || groups < kStageTargetGroups * 3 / 4) return static_cast<double>(d.thin_nnz) * batch * 4. / 25e6;
    return 7.5 + static_cast<double>((groups + kStageTargetGroups - 1) / kStageTargetGroups) * (0.84e-3 * static_cast<double>(d.thin_nnz) / static_cast<double>(ranges) + 4.5e-3 * cols);
}

// It goes to the bf16 units where they take less; their estimate is 4 to 8 % above what these matrices take.  Gathered / split, us: 8192 x 4096 at 20 %, batch 256 / 512 / 520 / 1024:
// 115 / 110, 205 / 201, 221 / 305, 408 / 380, at 24 %, batch 320 / 640 155 / 196, 295 / 310; 9019 x 2137 at 28 %, batch 256 / 1024 86 / 79, 317 / 296, at 24 %, batch 640 167 / 190;
// 2600 x 16384 at 20 %, batch 256 / 512 / 1024: 353 / 142, 306 / 267, 506 / 510; 3000 x 6000: 147 / 71, 123 / 123, 227 / 237; 2050 x 2100 at 28 %, batch 512 / 600 51 / 48, 58 / 59.
// (The fp32 units lose: 20 % of 4096^2 at batch 1024 235 / 326.)
static bool thin_rows_pay(const DenseSplit &d, int32_t cols, int32_t batch)
{
    if (batch < kThinBatch || d.thin_nnz * batch < kThinWork) return false;
    const DenseRowsCut cut = dense_rows_split_cut(d.rows.n, cols, batch);
    return cut.tiles > 0 && operand_parts_ints(cols, batch) <= d.rows.parts_ints &&
           (cut.slices == 1 || static_cast<int64_t>(cut.slices) * d.rows.n * dense_rows_ld(batch) <= d.rows.partial_floats) && cut.time * 0.92 < thin_rows_gathered(d, cols, batch);
}

bool thin_rows_pay_somewhere(const DenseSplit &d, int32_t cols)
{
    // (the estimates go in steps of 32 columns; beyond 2048, where tiles are many, every 64th is looked at)
    for (int32_t b = d.max_batch; b >= kThinBatch; b = (b - 1 - b / 64) / 32 * 32)
        if (thin_rows_pay(d, cols, b)) return true;
    return false;
}

bool dense_rows_product_ok(const DenseSplit *d, int32_t cols, int32_t batch)
{
    return d && d->rows.n > 0 && (d->thin_nnz > 0 ? thin_rows_pay(*d, cols, batch) : batch >= d->from_batch);
}

// (a thin matrix is one for sddmm_sampled_ok)
bool dense_rows_sddmm_ok(const DenseSplit *d, int32_t batch) { return d && d->rows.n > 0 && d->thin_nnz == 0 && batch >= d->from_batch; }

DenseRowsRoom dense_rows_room(int32_t n, int32_t cols, int32_t max_batch, bool thin)
{
    DenseRowsRoom room{0, 0};
    const int64_t step = thin ? 32 : 64;
    for (int64_t c = step; c - step < max_batch; c += step) {
        const int32_t batch = static_cast<int32_t>(c < max_batch ? c : max_batch);
        const DenseRowsCut fp32 = thin ? DenseRowsCut{} : dense_rows_fp32_cut(n, cols, batch), cut = thin ? dense_rows_split_cut(n, cols, batch) : dense_rows_cut(n, cols, batch, fp32);
        const int slices = std::max(cut.slices, fp32.slices);   // (the fp32 units take over where there is no room for the parts)
        if (slices > 1) room.partial_floats = std::max(room.partial_floats, static_cast<int64_t>(slices) * n * dense_rows_ld(batch));
        if (cut.split && operand_parts_ints(cols, batch) < kPartsMaxInts) room.parts_ints = std::max(room.parts_ints, operand_parts_ints(cols, batch));
    }
    room.partial_floats = std::min<int64_t>(room.partial_floats, 1ll << 28);   // (what does not fit is not sliced)
    return room;
}

hipError_t launch_dense_rows(const SpmmCall &a, hipStream_t s)
{
    const DenseRows &D = a.split->rows;
    const DenseRowsCut fp32 = dense_rows_fp32_cut(D.n, a.x_rows, a.batch);
    DenseRowsCut cut = a.split->thin_nnz > 0 ? dense_rows_split_cut(D.n, a.x_rows, a.batch) : dense_rows_cut(D.n, a.x_rows, a.batch, fp32);
    auto fits = [&] { return static_cast<int64_t>(cut.slices) * D.n * dense_rows_ld(a.batch) <= D.partial_floats; };
    // (a batch between those that the buffers were sized for may be cut finer than they are)
    if (cut.split && (operand_parts_ints(a.x_rows, a.batch) > D.parts_ints || (cut.slices > 1 && !fits()))) cut = fp32;
    if (cut.slices > 1 && !fits()) cut.slices = 1;
    const int slices = cut.slices;
    const dim3 grid(static_cast<unsigned>(cut.tiles * slices));
    if (cut.split)
        launch_split_dense_rows(a, D, slices, s);
    else if (cut.cols == 128)
        hipLaunchKernelGGL(dense_rows_kernel<4>, grid, dim3(kDenseBlock), 0, s, a, D, slices);
    else
        hipLaunchKernelGGL(dense_rows_kernel<2>, grid, dim3(kDenseBlock), 0, s, a, D, slices);
    if (slices > 1) {
        const int64_t work = static_cast<int64_t>(D.n) * ((a.batch + 3) / 4);
        const int64_t blocks = std::min<int64_t>((work + kDenseBlock - 1) / kDenseBlock, 4096);
        hipLaunchKernelGGL(dense_rows_finish_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kDenseBlock), 0, s, a, D, slices);
    }
    return hipGetLastError();
}

void add_sampled_rows(SampledArgs &list, const SddmmCall &a)
{
    add_sampled(list, a);
    SampledLayer &L = list.layer[list.n - 1];
    const DenseRows &D = a.split->rows;
    L.list = D.list; L.rows = D.n; L.table = D.table; L.words = D.words;
    if (D.n < a.rows) list.loss_cols = nullptr;   // (the other rows' launch takes the mean of the losses)
}

void add_sampled(SampledArgs &list, const SddmmCall &a)
{
    SampledLayer &L = list.layer[list.n++];
    L.table = a.table; L.words = a.table_words; L.rows = a.rows; L.cols = a.x_rows; L.nnz = a.nnz; L.fused = a.fused;
    L.dZ = a.dZ; L.lddz = a.lddz; L.X = a.X; L.ldx = a.ldx; L.g = a.g; L.db = a.db;
    L.values = a.values; L.velocity = a.velocity; L.values_t = a.values_t; L.pos_t = a.pos_t;
    L.dense = a.dense; L.dense_ld = a.dense_ld; L.bias = a.bias; L.bias_velocity = a.bias_velocity;
    list.batch = a.batch; list.nesterov = a.nesterov; list.lr = a.lr; list.momentum = a.momentum;
    if (a.loss_cols) { list.loss_cols = a.loss_cols; list.loss_out = a.loss_out; list.loss_n = a.loss_n; }
}

hipError_t launch_sampled(SampledArgs &a, hipStream_t s)
{
    int64_t blocks = 0;
    for (int k = 0; k < a.n; ++k) {
        SampledLayer &L = a.layer[k];
        L.tiles_i = (L.rows + 63) / 64;
        L.tiles_j = (L.cols + 63) / 64;
        L.first_block = static_cast<int32_t>(blocks);
        blocks += (static_cast<int64_t>(L.tiles_i) * L.tiles_j + 7) / 8 * 8;
    }
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(sampled_update_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kSampledWaves * kWave), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pattern_table(const int32_t *indptr, const int32_t *indices, const int32_t *list, int32_t rows, int32_t words, uint2 *table,
                                const int32_t *status, hipStream_t s)
{
    int64_t b = (static_cast<int64_t>(rows) * words + kDenseBlock - 1) / kDenseBlock;
    if (b > 8192) b = 8192;
    hipLaunchKernelGGL(pattern_table_kernel, dim3(static_cast<unsigned>(b)), dim3(kDenseBlock), 0, s, indptr, indices, list, rows, words, table, status);
    return hipGetLastError();
}

hipError_t launch_dense_refresh(const int32_t *indptr, const int32_t *indices, const float *values, int32_t rows, float *D, int64_t ld,
                                hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(dense_refresh_kernel, dim3(blocks_for_rows(rows)), dim3(kDenseBlock), 0, s, indptr, indices, values, rows, D, ld);
    return hipGetLastError();
}

}  // namespace nerva
