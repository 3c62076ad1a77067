// Device helpers shared by the kernels of the products (kernels.hip, dense.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nerva {
namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int wave_in_block()
{
    return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
}

__device__ __forceinline__ float4 keep_where_positive(float4 x, float4 m)
{
    x.x = m.x > 0.f ? x.x : 0.f;
    x.y = m.y > 0.f ? x.y : 0.f;
    x.z = m.z > 0.f ? x.z : 0.f;
    x.w = m.w > 0.f ? x.w : 0.f;
    return x;
}
__device__ __forceinline__ float keep_where_positive(float x, float m) { return m > 0.f ? x : 0.f; }

// 16-byte accesses to global memory ask for 4-byte alignment only, which the hardware serves: matrices of any
// leading dimension run on the kernels below (a first layer of 1501 x 3001 at batch 77 stored without padding:
// forward 9.1 us and SDDMM 29.7 us on one-column-per-lane kernels, here 7.5 us, and 13.1 us for the SDDMMs of both
// layers, which now share a grid).
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 ld4(const float *p)
{
    const v4f_any r = *reinterpret_cast<const v4f_any *>(p);
    return make_float4(r.x, r.y, r.z, r.w);
}
__device__ __forceinline__ void st4(float *p, float4 v)
{
    v4f_any r = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<v4f_any *>(p) = r;
}
// First of the four columns that the lane at column `col` (a multiple of 4, below `batch`, batch >= 4) works on: where
// fewer than four are left the access moves back to the row's last four columns, so that nothing beyond the batch is
// read or written whatever the leading dimension.  The columns that it shares with its neighbour are computed by both,
// in the same order, to the same bits.
__device__ __forceinline__ int four_columns(int col, int batch) { return min(col, batch - 4); }
// ... and the lane's share of a sum over columns: those of its four that the neighbour does not have.  In a sum of products both
// factors are dropped: 0 times an Inf or NaN is no 0.
__device__ __forceinline__ float4 drop_shared(float4 x, int col, int first)
{
    if (first < col) x.x = 0.f;
    if (first + 1 < col) x.y = 0.f;
    if (first + 2 < col) x.z = 0.f;
    return x;
}
// sum + the products of z and x over the lane's own columns (as above; none where col lies beyond the batch), whatever the others hold
__device__ __forceinline__ float add_own_products(float sum, float4 z, float4 x, int col, int first, int batch)
{
    if (col >= batch) return sum;
    if (first >= col) sum = fmaf(z.x, x.x, sum);
    if (first + 1 >= col) sum = fmaf(z.y, x.y, sum);
    if (first + 2 >= col) sum = fmaf(z.z, x.z, sum);
    return fmaf(z.w, x.w, sum);
}

// Data-parallel-primitive move: lane l receives x from the lane that CTRL names; lanes in rows
// not selected by ROW_MASK receive 0.
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROW_MASK, 0xF, false));
}

// Sum over each row of 16 lanes, all 64 lanes active; every lane of a row gets the same bits.
__device__ __forceinline__ float row16_sum(float x)
{
    x += dpp<0xB1>(x);   // quad_perm [1,0,3,2]
    x += dpp<0x4E>(x);   // quad_perm [2,3,0,1]
    x += dpp<0x141>(x);  // row_half_mirror
    x += dpp<0x140>(x);  // row_mirror
    return x;
}

// Sum over groups of G lanes (4: per quad; 8: per half row; 16: per row; 64: whole wave, returned wave-uniform).
template <int G>
__device__ __forceinline__ float group_sum(float x)
{
    static_assert(G == 4 || G == 8 || G == 16 || G == 32 || G == 64, "group sizes with a reduction");
    if constexpr (G == 4) {
        x += dpp<0xB1>(x);   // quad_perm [1,0,3,2]
        x += dpp<0x4E>(x);   // quad_perm [2,3,0,1]
        return x;
    }
    if constexpr (G == 8) {
        x += dpp<0xB1>(x);   // quad_perm [1,0,3,2]
        x += dpp<0x4E>(x);   // quad_perm [2,3,0,1]
        x += dpp<0x141>(x);  // row_half_mirror
        return x;
    }
    x = row16_sum(x);
    if constexpr (G == 32) x += __shfl_xor(x, 16, kWave);  // the other row of the pair (through the LDS crossbar)
    if constexpr (G == 64) {
        x += dpp<0x142, 0xA>(x);  // row_bcast15 into rows 1 and 3
        x += dpp<0x143, 0xC>(x);  // row_bcast31 into rows 2 and 3
        x = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
    }
    return x;
}

// *out = mean of v[0 .. n), summed by one wave in one fixed order
__device__ __forceinline__ void mean_of(const float *v, int n, float *out)
{
    const int lane = threadIdx.x & (kWave - 1);
    float s = 0.f;
    for (int c = lane; c < n; c += kWave) s += v[c];
    s = group_sum<kWave>(s);
    if (lane == 0) *out = s / static_cast<float>(n);
}

// The momentum step of one element; the same expression in the fused and the stand-alone path.
// nesterov: the weight moves by the look-ahead mu*v_new - lr*g instead of v_new.
__device__ __forceinline__ void momentum_step(float &w, float &v, float g, float lr, float mu, int nesterov)
{
    const float step = lr * g;
    v = fmaf(mu, v, -step);
    w = nesterov ? w + fmaf(mu, v, -step) : w + v;
}

// Address of row j of a dense matrix whose rows are ld_bytes apart, kept in scalar registers:
// the readfirstlane fences stop the compiler from folding the per-lane column offset into a
// 64-bit vector multiply-add, so the gather uses the scalar-base + 32-bit lane offset form.
typedef const __attribute__((address_space(1))) char *gmem_ptr;  // global (device) memory
__device__ __forceinline__ gmem_ptr row_base(const void *base, int j, uint32_t ld_bytes)
{
    const uint64_t addr = reinterpret_cast<uint64_t>(base) + static_cast<uint64_t>(static_cast<uint32_t>(j)) * ld_bytes;
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(addr));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(addr >> 32));
    return reinterpret_cast<gmem_ptr>((static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ gmem_ptr as_gmem(const void *p) { return reinterpret_cast<gmem_ptr>(reinterpret_cast<uint64_t>(p)); }
__device__ __forceinline__ float4 gload4(gmem_ptr row, uint32_t byte_offset)
{
    const v4f_any r = *reinterpret_cast<const __attribute__((address_space(1))) v4f_any *>(row + byte_offset);
    return make_float4(r.x, r.y, r.z, r.w);
}

__device__ __forceinline__ float gload1(gmem_ptr base, uint32_t byte_offset)
{
    return *reinterpret_cast<const __attribute__((address_space(1))) float *>(base + byte_offset);
}
__device__ __forceinline__ void gstore1(float *base, uint32_t byte_offset, float x)
{
    *reinterpret_cast<__attribute__((address_space(1))) float *>(reinterpret_cast<__attribute__((address_space(1))) char *>(reinterpret_cast<uint64_t>(base)) + byte_offset) = x;
}

}  // namespace
}  // namespace nerva
