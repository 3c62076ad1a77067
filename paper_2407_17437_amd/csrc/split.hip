// Products on the bf16 matrix units at fp32 precision.
// An fp32 number is the sum of three bf16 numbers (8 + 8 + 8 bits of its 24: x = h + m + l exactly, unless x is so small, from 2^-110 down, that its
// last bits lie below the smallest bf16 number; blocks that hold such a number are left to fp32; the splitting is that of Henry, Tang and Heinecke, "Leveraging
// the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019), so a product of two is the
// sum of nine products, of which l l (below 2^-32 of it) is left out.  Without m l and l m as well, which can make 2^-24 of it, a result
// of a single product was off by up to 8.9e-8 where fp32 rounds once, by 6.0e-8 at most.  The bf16 units multiply exactly
// into fp32 and are 12 times as fast as the fp32 ones (1.73 against 0.14 PFLOP/s from registers on this card), so the eight
// products that are formed take two thirds of the time.  h h is added up in one accumulator and the seven small ones in another, which
// keeps the rounding of a small product from being that of the large sum.  Against 64 bits, error over the result's norm, fp32 units or gathered -> here:
// 1024 x 16384 at 35 % 6.8e-7 -> 1.9e-7, 8192 x 4096 at 25 % 5.7e-7 -> 1.6e-7, 2500 x 1057 at 36 % 3.5e-7 -> 0.8e-7; all numbers of one sign 2.7e-7 -> 0.9e-7,
// 4.4e-7 -> 1.3e-7, 2.9e-7 -> 0.6e-7 (no bias: the units round to nearest); one operand row in a column of the batch 2.9e-8 -> 2.9e-8.
//
// v_mfma_f32_32x32x16_bf16: lane l supplies A(l % 32, 8 (l / 32) + i) and B(8 (l / 32) + i, l % 32), i = 0 .. 7, of a
// 32 x 16 by 16 x 32 step; register r of lane l holds C(8 (r / 4) + 4 (l / 32) + r % 4, l % 32).
#include "device.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace nerva {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t bf16_pair(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf)); }
__device__ __forceinline__ float low_half(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float high_half(uint32_t p) { return __builtin_bit_cast(float, p & 0xFFFF0000u); }

// Numbers a and b become pair `i` of the parts.  `zero` stays 0 as long as every number is the sum of its three parts: not for an Inf, a NaN, one
// that rounds to an Inf in bf16 or one too small.  (The units take and give subnormal numbers as they are.)
__device__ __forceinline__ void split_pair(float a, float b, v4u (&part)[3], int i, float &zero)
{
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        const uint32_t h = bf16_pair(a, b);
        part[p][i] = h;
        a -= low_half(h);
        b -= high_half(h);
    }
    zero += fabsf(a) + fabsf(b);
}

// barrier for what is in LDS; global loads stay in flight across it
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// what lanes of a wave have put into LDS is there for the others of the wave (its LDS instructions run in order)
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

constexpr int kSpWaves = 8, kSpBlock = kSpWaves * kWave;
constexpr int kSpRows = 128, kSpK = 32;

// The operand's parts for the products below: planes[(8 rows) * 3 + part][column] of 16 bytes each, rows and columns beyond the
// operand's 0.  odd[(32 rows) * column tiles + column tile]: some of them are not the sum of their parts (split_pair), and all parts there are 0.
// A work-group: 32 rows, 256 columns, a thread 8 rows of a column at a time.
__global__ __launch_bounds__(kSplitCols) void split_operand_kernel(const float *__restrict__ X, int64_t ldx, int rows, int batch, v4u *__restrict__ planes,
                                                                int32_t *__restrict__ odd)
{
    const int col = blockIdx.x * kSplitCols + threadIdx.x, k0 = blockIdx.y * kSpK;
    const int64_t ld = static_cast<int64_t>(gridDim.x) * kSplitCols;
    float x[kSpK / 8][8];
#pragma unroll
    for (int g = 0; g < kSpK / 8; ++g)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = k0 + 8 * g + i;
            x[g][i] = X[static_cast<int64_t>(min(k, rows - 1)) * ldx + min(col, batch - 1)];
            if (k >= rows) x[g][i] = 0.f;   // uniform
        }
    float zero = 0.f;
    v4u part[kSpK / 8][3];
#pragma unroll
    for (int g = 0; g < kSpK / 8; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) split_pair(x[g][2 * i], x[g][2 * i + 1], part[g], i, zero);
    const int any = __syncthreads_or(!(zero == 0.f));
#pragma unroll
    for (int g = 0; g < kSpK / 8; ++g)
#pragma unroll
        for (int p = 0; p < 3; ++p) planes[((static_cast<int64_t>(blockIdx.y) * 4 + g) * 3 + p) * ld + col] = any ? v4u{} : part[g][p];
    if (threadIdx.x == 0) odd[blockIdx.y * gridDim.x + blockIdx.x] = any;
}

// ---- dense rows ----------------------------------------------------------------------------------
// Y[i, :] = act(W[i, :] X + b[i]) for the listed rows of a sparse matrix (DenseRows).  A work-group of 8 waves owns 128 of the rows
// and 256 columns of the batch, a wave all the rows and 32 columns; 32 columns of the matrix at a time (a chunk).  A wave brings 16 rows' entries, a
// lane per column of a row (the pattern table says whether there is one and where), turns them round in LDS and splits them for all waves, in
// steps between its products; its own columns of the operand come straight from the parts, a chunk ahead.  K is cut into slices
// where the tiles do not fill the chip.
// What bounds it: the card's power at these units (from registers they reach 1.73 PFLOP/s at 1.8 GHz), and the waits at either end of a chunk.
// Measured on the 2611 dense rows of 16384^2 power-law rows at 10 %, batch 1024: 490 to 510 us (1.4 PFLOP/s) after 32 for
// the parts and before 10 for the slices; dense_rows_kernel 813 + 9.
// Tried, with six of the products, which took 433: the operand split by the work-groups themselves (526), through LDS (480), one of a SIMD's two waves
// bringing entries while the other multiplies (450); without bringing entries and operand the same loop took 324.
__global__ __launch_bounds__(kSpBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) void split_dense_rows_kernel(const SpmmArgs a, const DenseRows D,
                                                                                                               const v4u *__restrict__ planes,
                                                                                                               const int32_t *__restrict__ x_odd, const int slices)
{
    __shared__ __align__(16) uint32_t as[2][kSpWaves * 768];   // [16 rows][8 k][part][row][4]
    __shared__ uint2 tab[4][kSpRows];
    __shared__ __align__(8) uint8_t odd[kSplitMaxChunks + 2][kSpWaves];         // per chunk and group of 16 rows: left out of the products
    const int lane = threadIdx.x & (kWave - 1), wv = wave_in_block(), tid = threadIdx.x;
    const int row_tiles = (D.n + kSpRows - 1) / kSpRows, col_tiles = (a.batch + kSplitCols - 1) / kSplitCols, total = row_tiles * col_tiles * slices;
    // an XCD gets consecutive tiles, row tiles running fastest: they share a slice of the operand
    const int index = (blockIdx.x & 7) * ((total + 7) >> 3) + (blockIdx.x >> 3);
    if (index >= total) return;
    const int rest = index / row_tiles, slice = rest % slices, col_tile = rest / slices, n0 = col_tile * kSplitCols, ib = index % row_tiles * kSpRows;
    const int chunks = D.words, per = (chunks + slices - 1) / slices;
    const int c_begin = min(slice * per, chunks), c_end = min(c_begin + per, chunks);
    const gmem_ptr values = as_gmem(a.values);
    const uint32_t last = static_cast<uint32_t>(a.nnz - 1) * 4u;
    const int r32 = lane & 31, half = lane >> 5;

    uint2 tab_next;
    const gmem_ptr table = row_base(D.table, ib, static_cast<uint32_t>(D.words) * 8u);
    const uint32_t tab_row = static_cast<uint32_t>(min(tid & (kSpRows - 1), D.n - 1 - ib)) * static_cast<uint32_t>(D.words) * 8u;
    auto load_table = [&](int c) {
        const v2u e = *reinterpret_cast<const __attribute__((address_space(1))) v2u *>(table + (tab_row + static_cast<uint32_t>(min(c, chunks - 1)) * 8u));
        tab_next = make_uint2(e.x, e.y);
    };
    auto keep_table = [&](int c) { tab[c & 3][tid & (kSpRows - 1)] = tab_next; };
    // A chunk's entries are brought in steps, so that they can run between products: where they are, their values,
    // the values in LDS (a lane has one column of eight rows), a row's eight columns per lane, their parts, the parts in LDS.
    float av[8], w[4];
    uint32_t set = 0;
    v4u parts[3];
    auto fetch = [&](int c, int u0, int u1) __attribute__((always_inline)) {
        if (u0 == 0) set = 0;
#pragma unroll
        for (int u = u0; u < u1; ++u) {
            const uint2 t = tab[c & 3][wv * 16 + 2 * u + half];
            const uint32_t bit = 1u << r32;
            set |= t.x & bit ? 1u << u : 0u;
            av[u] = gload1(values, min((t.y + static_cast<uint32_t>(__popc(t.x & (bit - 1u)))) * 4u, last));
        }
    };
    auto turn_in = [&](int buf) __attribute__((always_inline)) {
        uint32_t *mine = as[buf] + wv * 768;
#pragma unroll
        for (int u = 0; u < 8; ++u) mine[(2 * u + half) * 36 + r32] = set & (1u << u) ? __builtin_bit_cast(uint32_t, av[u]) : 0u;
        wave_lds_order();
    };
    auto turn_out = [&](int buf, int h) __attribute__((always_inline)) {
        const v4f q = *reinterpret_cast<const v4f *>(as[buf] + wv * 768 + (lane & 15) * 36 + 8 * (lane >> 4) + 4 * h);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = q[i];
        if (h == 1) wave_lds_order();
    };
    float zero = 0.f;
    auto split_half = [&](int h) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) split_pair(w[2 * i], w[2 * i + 1], parts, 2 * h + i, zero);
    };
    auto keep_parts = [&](int c, int buf) __attribute__((always_inline)) {
        uint32_t *mine = as[buf] + wv * 768 + (lane >> 4) * 192 + (lane & 15) * 4;
        const bool bad = __any(!(zero == 0.f));
        odd[c - c_begin][wv] = bad;
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<v4u *>(mine + p * 64) = bad ? v4u{} : parts[p];
        zero = 0.f;
    };
    const uint32_t plane_ld = static_cast<uint32_t>(col_tiles) * kSplitCols * 16u;
    const gmem_ptr X = as_gmem(planes);
    const uint32_t own = static_cast<uint32_t>(half * 3) * plane_ld + static_cast<uint32_t>(n0 + wv * 32 + r32) * 16u;
    v4u fb[2][3];   // the wave's fragments of the chunk's two steps of 16
    auto load_b = [&](int c, int s, v4u (&to)[3]) __attribute__((always_inline)) {
        const uint32_t group = static_cast<uint32_t>((min(c, chunks - 1) * 4 + 2 * s) * 3) * plane_ld;
#pragma unroll
        for (int p = 0; p < 3; ++p) to[p] = *reinterpret_cast<const __attribute__((address_space(1))) v4u *>(X + (own + (group + p * plane_ld)));
    };
    v16f acc[4], small[4];
    // Fragments of two row tiles at a time; those of the next two are read part by part into the registers that the products at
    // hand are done with (the compiler's own order waits for every read).
    auto multiply = [&](int buf, auto &&between) __attribute__((always_inline)) {
        const uint32_t *A = as[buf] + (r32 >> 4) * 768 + half * 192 + (r32 & 15) * 4;
        constexpr int kPairs = kSpK / 16 * 2;
        v8bf fa[2][3];
        auto read = [&](int pair, int p) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
                fa[h][p] = __builtin_bit_cast(v8bf, *reinterpret_cast<const v4u *>(A + (2 * (pair & 1) + h) * 1536 + (pair >> 1) * 384 + p * 64));
        };
#pragma unroll
        for (int p = 2; p >= 0; --p) read(0, p);
#pragma unroll
        for (int pair = 0; pair < kPairs; ++pair) {
            const int m = 2 * (pair & 1);
            auto product = [&](int pa, int pb) __attribute__((always_inline)) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v16f &sum = pa + pb == 0 ? acc[m + h] : small[m + h];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[h][pa], __builtin_bit_cast(v8bf, fb[pair >> 1][pb]), sum, 0, 0, 0);
                }
            };
#pragma unroll
            for (int p = 2; p >= 0; --p) {
#pragma unroll
                for (int pb = p == 2 ? 1 : 2; pb >= 0; --pb) product(p, pb);
                __builtin_amdgcn_sched_barrier(0);
                if (pair + 1 < kPairs) read(pair + 1, p);
                between(pair * 3 + 2 - p);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

#pragma unroll
    for (int i = 0; i < 3; ++i) {
        load_table(c_begin + i);
        keep_table(c_begin + i);
    }
    load_table(c_begin + 3);
    __syncthreads();
    auto bring = [&](int c, int buf) __attribute__((always_inline)) {   // chunk c's parts, then chunk c + 1's values on their way
        turn_in(buf);
        turn_out(buf, 0);
        split_half(0);
        turn_out(buf, 1);
        split_half(1);
        keep_parts(c, buf);
        fetch(c + 1, 0, 8);
    };
    fetch(c_begin, 0, 8);
    load_b(c_begin, 0, fb[0]);   // (in the order of the loop: what is asked for first is waited for first)
    bring(c_begin, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_b(c_begin, 1, fb[1]);
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = v16f{}, small[m] = v16f{};
    auto chunk = [&](int c, int buf) __attribute__((always_inline)) {
        lds_barrier();
        keep_table(c + 3);
        load_table(c + 4);
        multiply(buf, [&](int step) __attribute__((always_inline)) {
            if (step == 0) turn_in(1 - buf);
            if (step == 1) turn_out(1 - buf, 0);
            if (step == 2) split_half(0);
            if (step == 3) turn_out(1 - buf, 1);
            if (step == 4) split_half(1);
            if (step == 5) keep_parts(c + 1, 1 - buf);
            if (step == 6) load_b(c + 1, 0, fb[0]);
            if (step == 8) fetch(c + 2, 0, 4);
            if (step == 9) fetch(c + 2, 4, 8);
            if (step == 11) load_b(c + 1, 1, fb[1]);
        });
    };
    for (int c = c_begin; c < c_end; ++c) chunk(c, (c - c_begin) & 1);
    // What is left out: an entry that is not stored must not meet an Inf or NaN with its 0, and bits of a number that is too small are
    // missing in its parts, so entry by entry, in fp32.
    lds_barrier();
    auto left_out = [&](int c) {
        return x_odd[c * col_tiles + col_tile] ? 0x0101010101010101ull : *reinterpret_cast<const uint64_t *>(odd[c - c_begin]);
    };
    bool any = false;
    for (int c = c_begin + tid; c < c_end; c += kSpBlock) any |= left_out(c) != 0;
    any = __syncthreads_or(any);
    for (int c = any ? c_begin : c_end; c < c_end; ++c) {
        const uint64_t groups = left_out(c);
        if (groups == 0) continue;   // (the same for all threads)
        lds_barrier();
        load_table(c);
        keep_table(c);
        lds_barrier();
        fetch(c, 0, 8);
#pragma unroll
        for (int u = 0; u < 8; ++u) as[0][(wv * 16 + 2 * u + half) * kSpK + r32] = __builtin_bit_cast(uint32_t, av[u]);
        lds_barrier();
        for (int k = 0; k < kSpK; ++k) {
            const float x = gload1(row_base(a.X, min(c * kSpK + k, a.x_rows - 1), static_cast<uint32_t>(a.ldx) * 4u),
                                   static_cast<uint32_t>(min(n0 + wv * 32 + r32, a.batch - 1)) * 4u);
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int g = 0; g < 16; ++g) {
                    const int i = 32 * m + 8 * (g >> 2) + 4 * half + (g & 3);   // (of group 2 m + g / 8)
                    if ((groups >> (8 * (2 * m + (g >> 3))) & 1u) && (tab[c & 3][i].x >> k & 1u)) acc[m][g] = fmaf(__builtin_bit_cast(float, as[0][i * kSpK + k]), x, acc[m][g]);
                }
        }
    }
    const int col = n0 + wv * 32 + r32;
    if (col >= a.batch) return;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int k = ib + 32 * m + 8 * (g >> 2) + 4 * half + (g & 3);
            if (k >= D.n) continue;
            float y = acc[m][g] + small[m][g];
            if (slices > 1) {
                D.partial[(static_cast<int64_t>(slice) * D.n + k) * dense_rows_ld(a.batch) + col] = y;
                continue;
            }
            const int row = D.list ? D.list[k] : k;
            if (a.bias) y += a.bias[row];
            if (a.relu) y = y > 0.f ? y : 0.f;
            if (a.YM) y = a.YM[static_cast<int64_t>(row) * a.ldym + col] > 0.f ? y : 0.f;
            a.Y[static_cast<int64_t>(row) * a.ldy + col] = y;
        }
}

}  // namespace

int64_t split_dense_rows_tiles(int32_t n, int32_t batch) { return static_cast<int64_t>((n + kSpRows - 1) / kSpRows) * (operand_parts_ld(batch) / kSplitCols); }

void launch_split_dense_rows(const SpmmArgs &a, const DenseRows &D, int slices, hipStream_t s)
{
    v4u *parts = reinterpret_cast<v4u *>(D.parts);
    int32_t *odd = reinterpret_cast<int32_t *>(D.parts) + static_cast<int64_t>(D.words) * 48 * operand_parts_ld(a.batch);
    const unsigned col_tiles = static_cast<unsigned>(operand_parts_ld(a.batch) / kSplitCols);
    hipLaunchKernelGGL(split_operand_kernel, dim3(col_tiles, D.words), dim3(kSplitCols), 0, s, a.X, a.ldx, a.x_rows, a.batch, parts, odd);
    const int64_t tiles = split_dense_rows_tiles(D.n, a.batch) * slices;
    hipLaunchKernelGGL(split_dense_rows_kernel, dim3(static_cast<unsigned>((tiles + 7) / 8 * 8)), dim3(kSpBlock), 0, s, a, D, parts, odd, slices);
}

}  // namespace nerva
