// The scan of the whole-store and the dense plan for batches of up to 32 or 64 queries (gfx950 only): the queries stay in LDS, every
// wavefront streams rows of its own.
//
// Such a call reads the rows once and does little with them, so it is as long as the stream of the rows, its start and what
// interrupts it.  One workgroup a compute unit holds the queries (whole rows of them); each of its wavefronts takes tiles
// of 16 or 32 rows through a private ring of 128-byte pieces of every row.  No wavefront waits for another once the queries are
// there, the row's tags and 1/|k| come with the stream, and while one wavefront searches its products the others' loads go on.
// The tiled kernel meets a barrier every piece, reads the queries again for every tile and joins its wavefronts' groups through LDS.
// A call with the tiled kernel's plan | with this one, us (bytes of rows over the second: TB/s):
//   1,000,003 x 1024 bf16 rows, 1 query, masked    322 | 305 (6.7)     200,000 x 512 bf16, 64 queries    69.5 | 53.5 (3.8)
//   300,007 x 384 f32 rows (split), 20 queries     98 | 93 (5.0)    200,000 x 512 fp8, 64 queries     60.5 | 36.9 (2.8)
// What is left: the launches and the selection (about 12 us), the first rows' way in (2), and with many queries or short rows the
// search of the products, 1 us for 32 rows and 32 queries of each wavefront.
#pragma once
#include "kb_epilogue.hpp"
#include "kb_internal.hpp"
#include "kb_norm.hpp"
#include "kb_scan.hpp"

namespace kbi {

struct StreamArgs {
    const void *keys, *queries;
    const float *inv_norm;
    const uint64_t *tags, *qmask;       // nullptr when no filter is applied
    float *best;                        // whole-store plan: [Q][groups], see WholePlan; dense plan: [Q][stride] products
    u32x4 *pair;
    int32_t n, d, Q;
    int32_t units, waves;               // tiles; wavefronts that share them (tile t belongs to wavefront t % waves)
    int32_t per_group, groups;          // tiles of a group; groups, or the dense plan's stride
    int32_t query_stride;               // bytes from query to query in LDS, a multiple of 256
    int32_t side_slots;                 // tiles whose side data can be in flight or in use
    int32_t blocks;                     // workgroups per query block
    uint64_t *gate;                     // f32 rows: as in ScanArgs; split ones: the word to clear
};

constexpr int STREAM_RING_16 = 4, STREAM_RING_32 = 3;     // pieces in a wavefront's ring, by the rows of a tile
constexpr int STREAM_LDS = 160 * 1024;

template <int KT_, int TR_, int NST_, int NQ_> struct StreamCfg {
    static constexpr int KT = KT_, TR = TR_, NST = NST_;
    static constexpr int NQ = NQ_, TQ = NQ * 32;     // blocks of 32 queries that a wavefront multiplies its rows with
    static constexpr bool SPLIT = KT == KB_F32_SPLIT;
    static constexpr bool PAIRED = KT == KB_FP8_Q8 || SPLIT;     // a matrix step takes 64 bytes of a row
    static constexpr int STEPS = PAIRED ? 2 : 4;
    static constexpr int KEY_BYTES = KeyTraits<KT>::KEY_BYTES, BMUL = KeyTraits<KT>::QRY_BYTES / KEY_BYTES;
    static constexpr int RB = 128, LOADS = TR * RB / 1024, CHUNK = TR * RB;
    static constexpr int SIDE = TR * 12;             // 1/|k| and tag of a tile's rows
    static_assert(LOADS * (NST - 1) < 60, "vmcnt is a 6-bit counter");
};

// Knowledge-base row at place `pos` of wavefront w's tile in a layer of c tiles (layer jt holds the tiles jt * waves .. of the
// store's rows from jt * waves * TR on): rows dealt to the tiles one by one, so that rows rise with the places of a group and
// neighbours, which may be alike, are in groups of their own (three of a query's best in one group cost a rescoring of it).
// The distance of a tile's rows is odd (see whole_row; a few tiles have nothing to gain from it).
// Dealt in runs of four, a tile's rows lie closer: 0 to 4 % faster on stores of 17,000 to 330,000 rows in no order, 11 % on larger ones of short rows (700,000 x 128 bf16
// 53.3 us one by one, 48.0), and slower by far on stores of similar neighbours: 90,000 x 512, 16 queries, k 32, runs of 16 26.1 us one by one, 47.7;
// 200,000 x 512 43.9, 79.7; pairs of rows 26.6 and 45.8 (runs of 4: 30.8).
__host__ __device__ inline int32_t stream_step(int32_t c) { return c <= 64 ? 0 : (c & 1) != 0 ? 2 : 1; }
__host__ __device__ inline int32_t stream_row(int32_t base, int32_t w, int32_t c, int32_t step, int pos)
{
    int32_t t = w + pos * step;              // (pos < 32)
    t -= t >= c ? c : 0;
    return base + pos * c + t;
}
// Row at a place of a group (past the store's end: none).
constexpr int STREAM_GROUP_TILE = 32;        // rows of a tile where groups are kept
__host__ __device__ inline int64_t stream_group_row(int32_t units, int32_t waves, int32_t per_group, uint32_t group, uint32_t place)
{
    const uint32_t first = group / (uint32_t)waves, w = group - first * (uint32_t)waves;
    const int32_t layer = (int32_t)first * per_group + (int32_t)(place / (uint32_t)STREAM_GROUP_TILE);
    const int32_t left = units - layer * waves, c = left < waves ? left : waves;
    return (int32_t)w < c ? stream_row(layer * waves * STREAM_GROUP_TILE, (int32_t)w, c, stream_step(c), (int)(place % (uint32_t)STREAM_GROUP_TILE)) : (int64_t)0x7fffffff;
}

// Waits for a piece of a ring behind which `younger` pieces have been asked for, up to MOST of them: it has landed once at most
// their loads are outstanding.  (What else is under way is younger still or counted too strictly.)
template <int LOADS, int MOST> __device__ inline void wait_landed(int younger)
{
    if (MOST <= 0 || younger >= MOST) __builtin_amdgcn_s_waitcnt(waitcnt_vm(MOST > 0 ? LOADS * MOST : 0));
    else if constexpr (MOST > 0) wait_landed<LOADS, MOST - 1>(younger);
}

// The 16-byte fragments of one matrix step: 32 bytes of a row (fp8 x fp8 and f32: 64).
template <class C> struct StreamStep {
    u32x4 a[C::PAIRED ? 2 : 1], b[C::NQ][C::PAIRED || C::BMUL == 2 ? 2 : 1];
};

template <class C, bool DENSE, bool NT> __global__ __launch_bounds__(512, 2) void kb_stream_kernel(StreamArgs p)
{
    constexpr int TR = C::TR, NST = C::NST, NQ = C::NQ, TQ = C::TQ, LOADS = C::LOADS, RB = C::RB, STEPS = C::STEPS;
    constexpr bool SPLIT = C::SPLIT;
    static_assert(DENSE || TR == STREAM_GROUP_TILE, "groups of whole tiles");
    if constexpr (C::KT == KB_F32) {
        if (*p.gate == 0) return;
    }
    if constexpr (SPLIT) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *p.gate = 0;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, lrow = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)blockDim.x >> 6;
    const int qb = DENSE ? blockIdx.x / p.blocks : 0, block = DENSE ? blockIdx.x % p.blocks : blockIdx.x, q0 = qb * TQ;
    const int nq = p.Q - q0 < TQ ? p.Q - q0 : TQ;
    // neighbouring tiles on different compute units of one XCD: their rows' tags and lengths share cache lines
    const int rank = (p.blocks & 7) == 0 ? (block & 7) * (p.blocks >> 3) + (block >> 3) : block;
    const int w = wave * p.blocks + rank;
    const int my_tiles = w < p.waves ? (p.units - w + p.waves - 1) / p.waves : 0;
    const uint32_t row_bytes = (uint32_t)p.d * C::KEY_BYTES;
    const int NC = (int)(row_bytes + RB - 1) / RB;
    const bool odd_tail = C::KEY_BYTES == 1 && (row_bytes & (RB - 1)) != 0;     // the last piece is half a line
    const int total = my_tiles * NC;
    const bool filter = p.qmask != nullptr;
    const int resident = (p.Q < TQ ? p.Q : TQ) * p.query_stride;

    // ---- the wavefront's stream ----
    unsigned char *ring = smem + resident + wave * (NST * C::CHUNK);
    unsigned char *side0 = smem + resident + nw * (NST * C::CHUNK) + wave * p.side_slots * C::SIDE;
    const unsigned char *src[LOADS];
    int ld_layer = 0, ld_c = 0, ld_slot = 0, ld_side = 0;
    // lane -> row and piece of a load instruction's eight rows: the piece's number within the line is swizzled as in the tiled kernel,
    // the same for every second instruction
    auto row_of = [&](int layer, int pos) {
        if constexpr (DENSE) return (layer * p.waves + w) * TR + pos;
        const int left = p.units - layer * p.waves, c = left < p.waves ? left : p.waves;
        return stream_row(layer * p.waves * TR, w, c, stream_step(c), pos);
    };
    auto piece_of = [&](int j) { return (uint32_t)((lane & 7) ^ swizzle<8>(8 * j + (lane >> 3))); };
    // what goes out before the first piece of a tile: the addresses of its rows, their 1/|k| and tags
    auto issue_tile = [&]() {
        const int last = p.n - 1;
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int row = row_of(ld_layer, 8 * j + (lane >> 3));
            src[j] = static_cast<const unsigned char *>(p.keys) + (uint64_t)(uint32_t)(row < last ? row : last) * row_bytes + piece_of(j) * 16;
        }
        unsigned char *side = side0 + ld_side * C::SIDE;
        if (lane < TR) {
            const int row = row_of(ld_layer, lane);
            __builtin_amdgcn_global_load_lds((const void *)(p.inv_norm + (row < last ? row : last)), (lds_ptr)side, 4, 0, 0);
        }
        if (filter && lane < 2 * TR) {
            const int row = row_of(ld_layer, lane >> 1);
            __builtin_amdgcn_global_load_lds((const void *)(reinterpret_cast<const uint32_t *>(p.tags) + 2 * (size_t)(uint32_t)(row < last ? row : last) + (lane & 1)), (lds_ptr)(side + TR * 4), 4, 0, 0);
        }
        ld_side = ld_side + 1 == p.side_slots ? 0 : ld_side + 1;
    };
    auto issue_load = [&](int j) {
        const unsigned char *at = src[j];
        // (the upper half of half a line is not there: its lanes fetch the lower one again)
        if (C::KEY_BYTES == 1 && odd_tail && ld_c + 1 == NC) at -= (piece_of(j) & 4u) * 16;
        __builtin_amdgcn_global_load_lds((const void *)at, (lds_ptr)(ring + ld_slot * C::CHUNK + j * 1024), 16, 0, NT ? LOAD_NT : 0);
        src[j] += RB;
    };
    auto issue_end = [&]() {
        ld_slot = ld_slot + 1 == NST ? 0 : ld_slot + 1;
        if (++ld_c == NC) {
            ld_c = 0;
            ++ld_layer;
        }
    };
    auto issue = [&]() {
        if (ld_c == 0) issue_tile();
#pragma unroll
        for (int j = 0; j < LOADS; ++j) issue_load(j);
        issue_end();
    };
    if (total > 0) issue();
    // ---- queries to LDS: 16-byte pieces, swizzled over 16 of them by the row (whole rows lie a multiple of 256 bytes apart) ----
    {
        // (a wavefront takes rows of its own)
        const uint32_t qrow = row_bytes * C::BMUL;
        for (int r = wave; r < nq; r += nw) {
            const unsigned char *from = static_cast<const unsigned char *>(p.queries) + (size_t)(q0 + r) * qrow;
            for (int o = 0; o < p.query_stride; o += 1024) {
                const uint32_t at = (uint32_t)((o >> 4) + lane) ^ (uint32_t)(r & 15);
                if (at * 16 < qrow) __builtin_amdgcn_global_load_lds((const void *)(from + at * 16), (lds_ptr)(smem + r * p.query_stride + o), 16, 0, 0);
            }
        }
    }
    asm volatile("" ::: "memory");
#pragma unroll 1
    for (int s = 1; s < NST; ++s)
        if (s < total) issue();
    // the queries and the first piece were asked for before the others
    wait_landed<LOADS, NST - 1>(total - 1);
    if constexpr (SPLIT) {
        // The queries are kept as the two f16 values of each element, eight of the one and then eight of the other: each wavefront turns
        // the rows it has asked for.  (Their lengths are summed up as everywhere, piece by piece.)
        const int pieces = (int)row_bytes / 16;
        for (int r = wave; r < nq; r += nw) {
            unsigned char *row = smem + r * p.query_stride;
            float sum = 0.f;
            for (int i = lane; i < pieces; i += 64) sum += piece_sum_squares<KB_F32>(*reinterpret_cast<const u32x4 *>(row + ((i ^ (r & 15)) << 4)));
            const float scale = f32_row_scale(inv_norm_of(wave_sum(sum)));
            for (int i = 2 * lane; i < pieces; i += 128) {
                u32x4 *first = reinterpret_cast<u32x4 *>(row + ((i ^ (r & 15)) << 4)), *second = reinterpret_cast<u32x4 *>(row + (((i | 1) ^ (r & 15)) << 4));
                const typename Mma<KB_F32_SPLIT>::PrepA x = Mma<KB_F32_SPLIT>::prepare(*first, *second, scale);
                *first = __builtin_bit_cast(u32x4, x.h);
                *second = __builtin_bit_cast(u32x4, x.l);
            }
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());
    }
    bare_barrier();
    if (total == 0) return;

    uint64_t qm[NQ];
    const unsigned char *sQ[NQ];
    uint32_t qx[NQ];
#pragma unroll
    for (int jb = 0; jb < NQ; ++jb) {
        const int qcol = q0 + jb * 32 + lrow < p.Q ? jb * 32 + lrow : nq - 1;        // padding columns repeat the last query
        qm[jb] = 0;
        if (filter) {
            qm[jb] = p.qmask[q0 + qcol];
            asm volatile("" : "+v"(qm[jb]));        // (waited for here, not between the pieces)
        }
        sQ[jb] = smem + qcol * p.query_stride;
        qx[jb] = (uint32_t)(((C::PAIRED || C::BMUL == 2 ? 2 * half : half) ^ (qcol & 15)) << 4);
    }
    const int arow = lrow & (TR - 1);
    const uint32_t ax = (uint32_t)(arow * RB) | (uint32_t)(((C::PAIRED ? 2 * half : half) ^ swizzle<8>(arow)) << 4);
    StreamStep<C> step[STEPS];
    auto read_step = [&](int k, const unsigned char *sA, uint32_t qc) {      // step k of the piece at sA, whose query bytes begin at qc
        const uint32_t ak = (uint32_t)(k * (RB / STEPS)), qk = qc + (uint32_t)(k * (RB / STEPS) * C::BMUL);
        step[k].a[0] = *reinterpret_cast<const u32x4 *>(sA + (ax ^ ak));
        if constexpr (C::PAIRED) step[k].a[1] = *reinterpret_cast<const u32x4 *>(sA + (ax ^ ak ^ 16u));
#pragma unroll
        for (int jb = 0; jb < NQ; ++jb) {
            step[k].b[jb][0] = *reinterpret_cast<const u32x4 *>(sQ[jb] + (qk ^ qx[jb]));
            if constexpr (C::PAIRED || C::BMUL == 2) step[k].b[jb][1] = *reinterpret_cast<const u32x4 *>(sQ[jb] + (qk ^ qx[jb] ^ 16u));
        }
    };

    // split f32: the scale of the lane's row, and the tile's 1/|k| in LDS as the products have them (once the tile's first piece is there)
    float key_scale = 1.f;
    auto scale_tile = [&](int at) {
        if constexpr (SPLIT) {
            float *inv = reinterpret_cast<float *>(side0 + at * C::SIDE);
            const float raw = inv[arow];
            key_scale = f32_row_scale(raw);
            if (lane < TR) inv[lane] = f32_scaled_inv(raw);
        }
    };
    f32x16 acc[1][NQ];
    auto multiply = [&](int k) {
#pragma unroll
        for (int jb = 0; jb < NQ; ++jb) {
            if constexpr (SPLIT) {
                typename Mma<C::KT>::PrepA b;
                b.h = __builtin_bit_cast(f16x8, step[k].b[jb][0]);
                b.l = __builtin_bit_cast(f16x8, step[k].b[jb][1]);
                Mma<C::KT>::run(acc[0][jb], Mma<C::KT>::prepare(step[k].a[0], step[k].a[1], key_scale), b);
            } else if constexpr (C::PAIRED) {
                typename Mma<C::KT>::PrepA a;
                a.lo = step[k].a[0];
                a.hi = step[k].a[1];
                Mma<C::KT>::run(acc[0][jb], a, step[k].b[jb][0], step[k].b[jb][1]);
            } else {
                Mma<C::KT>::run(acc[0][jb], Mma<C::KT>::prepare(step[k].a[0]), step[k].b[jb][0], step[k].b[jb][C::BMUL - 1]);
            }
        }
    };
    auto clear = [&]() {
#pragma unroll
        for (int jb = 0; jb < NQ; ++jb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[0][jb][i] = SPLIT ? SPLIT_START : 0.f;
    };
    clear();
#pragma unroll
    for (int k = 0; k < STEPS; ++k) read_step(k, ring, 0u);
    scale_tile(0);
    TopThree kept[NQ];        // (of the group, once it has a tile)
    int c = 0, layer = 0, in_group = 0, slot = 0, side_slot = 0;
    // Piece g is in registers when its turn comes, the fragments of piece g + 1 follow step by step, and the loads of piece g + NST
    // go into the slot that piece g has left, one after every matrix instruction: none of the three waits for another.
    for (int g = 0; g < total; ++g) {
        wait_landed<LOADS, NST - 2>(total - 2 - g);          // piece g + 1
        __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());        // piece g has been read
        asm volatile("" ::: "memory");
        const bool more = g + NST < total;
        if (more && ld_c == 0) issue_tile();
        const int next_c = c + 1 == NC ? 0 : c + 1;
        slot = slot + 1 == NST ? 0 : slot + 1;
        const unsigned char *sA = ring + slot * C::CHUNK;
        const uint32_t qc = (uint32_t)next_c * (RB * C::BMUL);
        const bool whole_piece = !(odd_tail && next_c == 0);        // (of piece g)
#pragma unroll
        for (int k = 0; k < STEPS; ++k) {
            if (C::KEY_BYTES != 1 || k < STEPS / 2 || whole_piece) multiply(k);
            __builtin_amdgcn_sched_barrier(0);
            read_step(k, sA, qc);       // (behind the last piece: what is in the slot, for nobody)
            if (more) {
#pragma unroll
                for (int j = k * LOADS / STEPS; j < (k + 1) * LOADS / STEPS; ++j) issue_load(j);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (more) issue_end();
        c = next_c;
        if (c != 0) continue;

        // ---- the tile's products ----
        const unsigned char *side = side0 + side_slot * C::SIDE;
        side_slot = side_slot + 1 == p.side_slots ? 0 : side_slot + 1;
        const EpiSide sd{reinterpret_cast<const float *>(side), reinterpret_cast<const uint64_t *>(side + TR * 4), nullptr, nullptr, nullptr, nullptr};
        if constexpr (DENSE) {
            const int row0 = (layer * p.waves + w) * TR;
#pragma unroll
            for (int run = 0; run < TR / 8; ++run) {
                const int rl = 4 * half + 8 * run;
                const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
                const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool ok = row0 + rl + e < p.n && !row_removed(ik[e]) && (!filter || (sd.tag[rl + e] & qm[0]) != 0);
                    v[e] = ok ? acc[0][0][4 * run + e] * ik[e] : -__builtin_inff();
                }
                if (q0 + lrow < p.Q) *reinterpret_cast<f32x4 *>(p.best + (size_t)(q0 + lrow) * p.groups + row0 + rl) = v;
            }
        } else {
            const uint32_t dead = (uint32_t)__builtin_amdgcn_ballot_w64(row_removed(sd.invk[lrow]) || row_of(layer, lrow) >= p.n);
            const uint32_t place0 = (uint32_t)(in_group * TR);
            const bool ends = in_group + 1 == p.per_group || g + 1 == total;
            const size_t group = (size_t)(layer / p.per_group) * (uint32_t)p.waves + (uint32_t)w;
#pragma unroll
            for (int jb = 0; jb < NQ; ++jb) {
                TopThree t = whole_column<1, NQ>(acc, jb, sd, filter, qm[jb], 0, half, dead);
                t = join(t, across_halves(t));
                if (__builtin_expect(unclear(t), 0)) {
                    t = whole_column_in_order<NATURAL_ORDER, 1, NQ>(acc, jb, sd, filter, qm[jb], 0, half, dead);
                    t = join_in_order<NATURAL_ORDER>(t, across_halves(t));
                }
                if (in_group > 0) {
                    t.rows += place0 | place0 << 8 | ((t.rows >> 16 & WHOLE_THIRD) != 0 ? place0 << 16 : 0u);
                    const TopThree both = join(kept[jb], t);
                    kept[jb] = __builtin_expect(unclear(both), 0) ? join_in_order<NATURAL_ORDER>(kept[jb], t) : both;
                } else kept[jb] = t;
                const int query = q0 + jb * 32 + lrow;
                if (ends && half == 0 && query < p.Q) {
                    const size_t at = (size_t)query * p.groups + group;
                    p.best[at] = kept[jb].first;
                    p.pair[at] = u32x4{as_u32(kept[jb].second), as_u32(kept[jb].third), kept[jb].rows, 0u};
                }
            }
            in_group = ends ? 0 : in_group + 1;
        }
        ++layer;
        if (g + 1 < total) scale_tile(side_slot);
        clear();
    }
}

template <class C, bool DENSE, bool NT> hipError_t launch_stream_variant(const StreamPlan &p, const StreamArgs &a, hipStream_t s)
{
    static LdsAllowed allowed;
    auto *fn = &kb_stream_kernel<C, DENSE, NT>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(fn), allowed, STREAM_LDS); e != hipSuccess) return e;
    hipExtLaunchKernelGGL(fn, dim3((unsigned)(p.blocks * p.nqb)), dim3(64u * (unsigned)p.waves_per_block), (unsigned)p.lds, s, scan_timing.start, scan_timing.stop, 0, a);
    return hipGetLastError();
}
template <int KT> hipError_t launch_stream(const StreamPlan &p, bool dense, bool once, const StreamArgs &a, hipStream_t s)
{
    if constexpr (KT == KB_F32_SPLIT || KT == KB_F32) {
        if (dense || p.tq != 32) return hipErrorInvalidValue;        // (no such plan)
    } else {
        if (dense) return launch_stream_variant<StreamCfg<KT, 16, STREAM_RING_16, 1>, true, false>(p, a, s);
        if (p.tq == 64) {
            if (once) return launch_stream_variant<StreamCfg<KT, 32, STREAM_RING_32, 2>, false, true>(p, a, s);
            return launch_stream_variant<StreamCfg<KT, 32, STREAM_RING_32, 2>, false, false>(p, a, s);
        }
    }
    if (once) return launch_stream_variant<StreamCfg<KT, 32, STREAM_RING_32, 1>, false, true>(p, a, s);
    return launch_stream_variant<StreamCfg<KT, 32, STREAM_RING_32, 1>, false, false>(p, a, s);
}
}  // namespace kbi
