// Scan kernel instantiations for f32 keys.
#include "kb_configs.hpp"
#include "kb_scan.hpp"

namespace kbi {

// The whole-store plan on some thousand f32 rows: one wavefront per workgroup scores 16 rows against CB blocks of 16
// queries.  Such a call is as long as one dot product's chain of matrix instructions: 32x32x2 takes 64 clocks per two
// elements, so 256 elements 3.4 us and 1024 elements 13.7 us; 16x16x4 takes 32 clocks per four, a quarter of that.  Both
// add the products to the accumulator one after the other, so with the elements of a 32-byte group dealt to the four
// lane groups in the order in which the wide instruction takes them (0 4 1 5, then 2 6 3 7) the sums are the same bits.
// 4096 x 256 rows, 8 queries: 6.2 us, 10.2 with 32x32 tiles.
template <int CB> struct SmallF32 {
    static constexpr int TK = 16, TQ = 16 * CB, NSTAGE = 9, RB = 128;
    static constexpr int A_BYTES = TK * RB, STAGE_BYTES = A_BYTES + TQ * RB, LOADS = STAGE_BYTES / 1024;
    static constexpr int SMEM_BYTES = NSTAGE * STAGE_BYTES;
    static_assert(LOADS * (NSTAGE - 2) < 64, "vmcnt is a 6-bit counter");
};

// DENSE: the scan of the dense plan; a workgroup per tile and block of queries, the rows of a tile are neighbours.
template <int CB, bool DENSE = false> __global__ __launch_bounds__(64) void kb_small_f32_kernel(ScanArgs p)
{
    typedef SmallF32<CB> C;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int lane = threadIdx.x, col = lane & 15, h = lane >> 4;
    const int tile = DENSE ? blockIdx.x / p.nqb : blockIdx.x, q0 = DENSE ? (int)(blockIdx.x % p.nqb) * C::TQ : 0;
    auto row_at = [&](int place) { return DENSE ? (int64_t)tile * C::TK + place : whole_row(tile, (int32_t)p.n_tiles, C::TK, place); };
    const int NC = p.d * 4 / C::RB;
    const uint32_t row_bytes = (uint32_t)p.d * 4;
    // load instruction j of a chunk fills rows 8 j .. 8 j + 7 (keys first, then queries) of 128 bytes, swizzled as in the
    // tiled kernel
    const unsigned char *src[C::LOADS];
#pragma unroll
    for (int j = 0; j < C::LOADS; ++j) {
        const int r = j * 8 + (lane >> 3), place = j < 2 ? r : r - 16;
        const uint32_t piece = (uint32_t)(((lane & 7) ^ swizzle<8>(place)) * 16);
        if (j < 2) {
            const int64_t row = row_at(place);
            src[j] = static_cast<const unsigned char *>(p.keys) + (size_t)(row < p.n_keys ? row : p.n_keys - 1) * row_bytes + piece;
        } else {
            src[j] = static_cast<const unsigned char *>(p.queries) + (size_t)(q0 + place < p.Q ? q0 + place : p.Q - 1) * row_bytes + piece;
        }
    }
    int issued = 0, slot = 0;
    auto issue = [&]() {
#pragma unroll
        for (int j = 0; j < C::LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const void *)(src[j] + (size_t)issued * C::RB), (lds_ptr)(smem + slot * C::STAGE_BYTES + j * 1024), 16, 0, 0);
        ++issued;
        slot = slot + 1 == C::NSTAGE ? 0 : slot + 1;
    };
    // side data of the lane's four rows and of its queries: asked for first, so that waiting for a chunk covers it
    float ik[4];
    uint64_t tg[4], qm[CB];
    bool live[4];
    const bool filter = p.qmask != nullptr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t row = row_at(4 * h + i);
        live[i] = row < p.n_keys;
        const int64_t r = live[i] ? row : p.n_keys - 1;
        ik[i] = p.inv_norm[r];
        tg[i] = filter ? p.tags[r] : 0ull;
    }
#pragma unroll
    for (int b = 0; b < CB; ++b) qm[b] = filter ? p.qmask[q0 + 16 * b + col < p.Q ? q0 + 16 * b + col : p.Q - 1] : 0ull;
    asm volatile("" ::: "memory");
    for (int s = 0; s < C::NSTAGE - 1 && s < NC; ++s) issue();

    f32x4 acc[CB] = {};
    int stage = 0;
    for (int c = 0; c < NC; ++c) {
        if (c + (C::NSTAGE - 2) < NC) __builtin_amdgcn_s_waitcnt(waitcnt_vm(C::LOADS * (C::NSTAGE - 2)));
        else __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        asm volatile("" ::: "memory");
        const unsigned char *sA = smem + stage * C::STAGE_BYTES, *sB = sA + C::A_BYTES;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int at = col * C::RB + (((2 * g + (h & 1)) ^ swizzle<8>(col)) << 4) + (h >> 1) * 4;
            const float a0 = *reinterpret_cast<const float *>(sA + at), a1 = *reinterpret_cast<const float *>(sA + at + 8);
#pragma unroll
            for (int b = 0; b < CB; ++b) {       // (16 rows further the swizzle is the same)
                const float b0 = *reinterpret_cast<const float *>(sB + b * 16 * C::RB + at), b1 = *reinterpret_cast<const float *>(sB + b * 16 * C::RB + at + 8);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[b], 0, 0, 0);
            }
        }
        stage = stage + 1 == C::NSTAGE ? 0 : stage + 1;
        // the slot of the chunk before this one is free: its fragments went into matrix instructions issued by now
        asm volatile("" ::: "memory");
        if (c + (C::NSTAGE - 1) < NC) issue();
    }

    // lane (col, h) holds rows 4 h .. 4 h + 3 of query 16 b + col
    if constexpr (DENSE) {
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = live[i] && !row_removed(ik[i]) && (!filter || (tg[i] & qm[b]) != 0) ? acc[b][i] * ik[i] : -__builtin_inff();
            const int q = q0 + 16 * b + col;
            if (q < p.Q) *reinterpret_cast<f32x4 *>(p.dense + (size_t)q * p.dense_stride + tile * C::TK + 4 * h) = v;
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < CB; ++b) {
        TopThree one[4], t = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), 0u};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool ok = live[i] && !row_removed(ik[i]) && (!filter || (tg[i] & qm[b]) != 0);
            one[i] = TopThree{ok ? acc[b][i] * ik[i] : -__builtin_inff(), -__builtin_inff(), -__builtin_inff(), (uint32_t)(4 * h + i)};
            t = join(t, one[i]);
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) t = join(t, other_half(t, o));
        if (__builtin_expect(unclear(t), 0)) {
            t = one[0];
#pragma unroll
            for (int i = 1; i < 4; ++i) t = join_in_order<C::TK>(t, one[i]);
#pragma unroll
            for (int o = 16; o < 64; o <<= 1) t = join_in_order<C::TK>(t, other_half(t, o));
        }
        const int q = 16 * b + col;
        if (h == 0 && q < p.Q) {
            const size_t at = (size_t)q * p.whole_groups + tile;
            p.whole_best[at] = t.first;
            p.whole_pair[at] = u32x4{as_u32(t.second), as_u32(t.third), t.rows, 0u};
        }
    }
}

template <int CB, bool DENSE = false> hipError_t launch_small_f32(int grid, const ScanArgs &a, hipStream_t s)
{
    static_assert(SmallF32<CB>::SMEM_BYTES <= 64 * 1024);
    hipExtLaunchKernelGGL((&kb_small_f32_kernel<CB, DENSE>), dim3(grid), dim3(64), SmallF32<CB>::SMEM_BYTES, s, scan_timing.start, scan_timing.stop, 0, a);
    return hipGetLastError();
}

hipError_t launch_scan_f32(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s)
{
    switch (config) {
#define X(ID, KT, TK, TQ, WM, WN, RBA, NSTAGE, WGPC) \
    case ID: return launch_scan_cfg<ScanCfg<KT, TK, TQ, WM, WN, RBA, NSTAGE, WGPC>>(sample, grid, a, s);
        KB_SCAN_CONFIGS_F32(X)
#undef X
    case SMALL_F32_CONFIG:
        if (a.dense) {      // one workgroup per tile of 16 rows and 32 queries (16 if there are no more)
            if (a.draw.enabled || grid != a.n_tiles * a.nqb) return hipErrorInvalidValue;
            return a.Q <= 16 ? launch_small_f32<1, true>(grid, a, s) : launch_small_f32<2, true>(grid, a, s);
        }
        // one workgroup per tile of 16 rows, up to 32 queries
        if (sample || !a.whole_best || a.Q > 32 || grid != a.n_tiles) return hipErrorInvalidValue;
        return a.Q <= 16 ? launch_small_f32<1>(grid, a, s) : launch_small_f32<2>(grid, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace kbi
