// kb_quantize_rows: fp32 / bf16 rows to e4m3 codes with one fp32 scale per row, the storage form of
// compressed keys and of fp8 queries (gfx950).  Memory-bound: every element is read once from HBM (a
// second time from registers or the cache) and one byte is written.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kb.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int THREADS = 256;
constexpr int64_t STREAM_BYTES = 64 << 20;
constexpr int CACHED = 4;           // 16-byte pieces of the row a lane keeps in registers between the two passes
constexpr float E4M3_MAX = 448.0f;

// Four quotients to four e4m3 codes (nearest, ties to the even code, sign kept) with the conversion instruction
// of gfx950, which implements exactly that rounding for the OCP e4m3 format, subnormal range included.  No
// quotient exceeds 448 (1 + 2^-23), which rounds to 448, so the overflow behaviour of the instruction never
// comes into play.
__device__ inline uint32_t encode_e4m3_x4(float y0, float y1, float y2, float y3)
{
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(y0, y1, 0, false);
    w = __builtin_amdgcn_cvt_pk_fp8_f32(y2, y3, w, true);
    return (uint32_t)w;
}

template <int DT> struct Piece;     // 16 bytes of a row
template <> struct Piece<KB_F32> {
    static constexpr int ELEMS = 4;
    static __device__ float value(const u32x4 &v, int i) { return __uint_as_float(v[i]); }
};
template <> struct Piece<KB_BF16> {
    static constexpr int ELEMS = 8;
    static __device__ float value(const u32x4 &v, int i) { return __uint_as_float((i & 1) ? (v[i >> 1] & 0xFFFF0000u) : (v[i >> 1] << 16)); }
};

template <int DT> __device__ inline float piece_amax(const u32x4 &v)
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < Piece<DT>::ELEMS; ++i) m = fmaxf(m, fabsf(Piece<DT>::value(v, i)));
    return m;
}

// x / scale, correctly rounded, for many x and one scale: with recip = the correctly rounded 1 / scale, the first
// correction of x * recip leaves less than one unit in the last place, and the second one rounds correctly (Markstein,
// IBM J. Res. Dev. 34, 1990).  Six operations, where the general division takes a dozen; it wants remainders that do not
// underflow, which holds for scales in [2^-60, 2^60] and quotients that are not rounded to a zero code anyway.
template <bool EXACT> __device__ inline float quotient(float x, float scale, float recip)
{
    if constexpr (EXACT) return x / scale;
    float q = x * recip;
    q = __builtin_fmaf(__builtin_fmaf(-q, scale, x), recip, q);
    q = __builtin_fmaf(__builtin_fmaf(-q, scale, x), recip, q);
    return __builtin_copysignf(q, x);       // (the corrections turn a -0 into a +0)
}

template <int DT, bool EXACT, bool STREAM> __device__ inline void piece_store(const u32x4 &v, float scale, float recip, unsigned char *dst)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    uint32_t w[Piece<DT>::ELEMS / 4];
#pragma unroll
    for (int j = 0; j < Piece<DT>::ELEMS / 4; ++j) {
        w[j] = encode_e4m3_x4(quotient<EXACT>(Piece<DT>::value(v, 4 * j), scale, recip), quotient<EXACT>(Piece<DT>::value(v, 4 * j + 1), scale, recip),
                              quotient<EXACT>(Piece<DT>::value(v, 4 * j + 2), scale, recip), quotient<EXACT>(Piece<DT>::value(v, 4 * j + 3), scale, recip));
    }
    if constexpr (Piece<DT>::ELEMS == 8) {
        if constexpr (STREAM) __builtin_nontemporal_store(u32x2{w[0], w[1]}, reinterpret_cast<u32x2 *>(dst));
        else *reinterpret_cast<u32x2 *>(dst) = u32x2{w[0], w[1]};
    } else {
        if constexpr (STREAM) __builtin_nontemporal_store(w[0], reinterpret_cast<uint32_t *>(dst));
        else *reinterpret_cast<uint32_t *>(dst) = w[0];
    }
}

// LANES lanes (32 or 64) take a row: with rows of up to 128 pieces two rows share a wavefront, so that 96 pieces (768 bf16
// values) leave no lane idle and a wavefront has twice the bytes in flight.  500,000 x 768
// bf16 rows (1.15 GB): 0.198 ms = 5.8 TB/s, 0.264 ms with a wavefront per row, general divisions and cached loads and stores.
template <int DT, int LANES, bool STREAM> __global__ __launch_bounds__(THREADS) void quantize_rows_kernel(const unsigned char *rows, int64_t n, int d, unsigned char *codes, float *scale_out)
{
    constexpr int ELEMS = Piece<DT>::ELEMS, ROWS = THREADS / LANES;
    const int lane = threadIdx.x % LANES;
    const int pieces = d / ELEMS;
    for (int64_t row = (int64_t)blockIdx.x * ROWS + threadIdx.x / LANES; row < n; row += (int64_t)gridDim.x * ROWS) {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(rows + (size_t)row * d * (16 / ELEMS));
        u32x4 keep[CACHED];
        float m = 0.f;
#pragma unroll
        for (int c = 0; c < CACHED; ++c) {
            const int p = lane + LANES * c;
            keep[c] = p < pieces ? (STREAM ? __builtin_nontemporal_load(src + p) : src[p]) : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int c = 0; c < CACHED; ++c) m = fmaxf(m, piece_amax<DT>(keep[c]));
        for (int p = lane + LANES * CACHED; p < pieces; p += LANES) m = fmaxf(m, piece_amax<DT>(src[p]));
#pragma unroll
        for (int s = LANES / 2; s >= 1; s >>= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
        const float scale = m > 0.f ? m / E4M3_MAX : 1.0f, recip = 1.0f / scale;
        if (scale_out && lane == 0) scale_out[row] = scale;
        unsigned char *dst = codes + (size_t)row * d;
        if (scale >= 0x1p-60f && scale <= 0x1p60f) {
#pragma unroll
            for (int c = 0; c < CACHED; ++c) {
                const int p = lane + LANES * c;
                if (p < pieces) piece_store<DT, false, STREAM>(keep[c], scale, recip, dst + (size_t)p * ELEMS);
            }
            for (int p = lane + LANES * CACHED; p < pieces; p += LANES) piece_store<DT, false, STREAM>(src[p], scale, recip, dst + (size_t)p * ELEMS);
        } else {
            for (int p = lane; p < pieces; p += LANES) piece_store<DT, true, STREAM>(src[p], scale, recip, dst + (size_t)p * ELEMS);
        }
    }
}

template <int DT> void launch_quantize(const unsigned char *rows, int64_t n, int d, unsigned char *codes, float *scale, hipStream_t s)
{
    const int lanes = d / Piece<DT>::ELEMS <= 32 * CACHED ? 32 : 64, per_block = THREADS / lanes;
    const int64_t want = (n + per_block - 1) / per_block;
    const int grid = (int)(want < 256 * 32 ? want : 256 * 32);      // 32 workgroups per compute unit keep HBM busy; the rest loops
    // past the caches when the rows are more than they keep: a batch of queries is read and written where it is used
    const bool stream = n * (int64_t)d * (16 / Piece<DT>::ELEMS) > STREAM_BYTES;
    auto *fn = lanes == 32 ? (stream ? &quantize_rows_kernel<DT, 32, true> : &quantize_rows_kernel<DT, 32, false>)
                           : (stream ? &quantize_rows_kernel<DT, 64, true> : &quantize_rows_kernel<DT, 64, false>);
    hipLaunchKernelGGL(fn, dim3(grid), dim3(THREADS), 0, s, rows, n, d, codes, scale);
}

}  // namespace

extern "C" kb_status_t kb_quantize_rows(const void *rows_dev, kb_dtype_t dtype, int64_t n, int32_t d, void *codes_out_dev,
                                        float *scale_out_dev, void *hip_stream)
{
    if (!rows_dev || !codes_out_dev) return KB_ERR_NULL;
    if (dtype != KB_F32 && dtype != KB_BF16) return KB_ERR_DTYPE;
    if (n < 0 || n >= (int64_t(1) << 31) || d < 16 || d > 16384 || d % 16 != 0) return KB_ERR_INVALID_ARG;
    if (((reinterpret_cast<uintptr_t>(rows_dev) | reinterpret_cast<uintptr_t>(codes_out_dev)) & 15) != 0) return KB_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(scale_out_dev) & 3) != 0) return KB_ERR_INVALID_ARG;
    if (n == 0) return KB_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const unsigned char *rows = static_cast<const unsigned char *>(rows_dev);
    unsigned char *codes = static_cast<unsigned char *>(codes_out_dev);
    if (dtype == KB_F32) launch_quantize<KB_F32>(rows, n, d, codes, scale_out_dev, s);
    else launch_quantize<KB_BF16>(rows, n, d, codes, scale_out_dev, s);
    return hipGetLastError() == hipSuccess ? KB_OK : KB_ERR_DEVICE;
}
