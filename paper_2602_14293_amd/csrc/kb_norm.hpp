// 1/|x| of a row by one wavefront: the one routine, and so the same bits, for keys and queries in every kernel (gfx950 only).
#pragma once
#include "kb_internal.hpp"

namespace kbi {

template <int DT> __device__ inline float piece_sum_squares(u32x4 v);
template <> __device__ inline float piece_sum_squares<KB_F32>(u32x4 v)
{
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = as_f32(v[e]);
        s += x * x;
    }
    return s;
}
template <> __device__ inline float piece_sum_squares<KB_F32_SPLIT>(u32x4 v) { return piece_sum_squares<KB_F32>(v); }
template <> __device__ inline float piece_sum_squares<KB_BF16>(u32x4 v)
{
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float lo = as_f32(v[e] << 16), hi = as_f32(v[e] & 0xffff0000u);
        s += lo * lo;
        s += hi * hi;
    }
    return s;
}
template <> __device__ inline float piece_sum_squares<KB_FP8_E4M3>(u32x4 v)
{
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8(v[e], false), b = __builtin_amdgcn_cvt_pk_f32_fp8(v[e], true);
        s += a.x * a.x;
        s += a.y * a.y;
        s += b.x * b.x;
        s += b.y * b.y;
    }
    return s;
}

__device__ inline float wave_sum(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One wavefront per row: lanes stride over the row's 16-byte pieces, fp32 sum of squares, butterfly
// reduction, inv = 1/sqrt(sum) or 0 for a zero row.
__device__ inline float inv_norm_of(float square_sum) { return square_sum > 0.f ? 1.0f / sqrtf(square_sum) : 0.f; }
template <int DT> __device__ inline float row_square_sum(const void *base, int64_t row, int row_bytes, int lane)
{
    const u32x4 *p = reinterpret_cast<const u32x4 *>(static_cast<const unsigned char *>(base) + (size_t)row * row_bytes);
    float s = 0.f;
    for (int i = lane; i < row_bytes / 16; i += 64) s += piece_sum_squares<DT>(__builtin_nontemporal_load(p + i));
    return wave_sum(s);
}
template <int DT> __device__ inline float row_inv_norm(const void *base, int64_t row, int row_bytes, int lane)
{
    return inv_norm_of(row_square_sum<DT>(base, row, row_bytes, lane));
}


// bytes of an element, and the type of the queries that go with keys of a type (kernel-side names)
constexpr int bytes_of(int t) { return t == KB_F32 || t == KB_F32_SPLIT ? 4 : t == KB_BF16 ? 2 : 1; }
constexpr int queries_of(int kt) { return kt == KB_F32 || kt == KB_F32_SPLIT ? kt : kt == KB_FP8_Q8 ? (int)KB_FP8_E4M3 : (int)KB_BF16; }

}  // namespace kbi
