// Epilogues shared by the scan kernels: what happens to a wave's accumulator blocks once an item's
// contraction is complete.  In the 32x32 accumulator layout lane (lrow, half) of a block holds query
// column lrow and key rows 8*(i/4) + 4*half + (i%4), i = 0..15.
#pragma once
#include "kb_internal.hpp"
#include <utility>

namespace kbi {

struct EpiSide {               // side data of the item, in LDS
    const float *invk;         // [TK]  1/|k| of the tile's rows
    const uint64_t *tag;       // [TK]
    const float *thrp;         // [TQ]  pre-filter on dot * inv_k
    const float *invq;         // [TQ]
    const uint64_t *thr64;     // [TQ]  candidate words below this cannot be in the result (read by the weighted selection only)
    const uint64_t *qmask;     // [TQ]
    const float *lgain = nullptr;   // [TK]  ln(gain) of the tile's rows (weighted random selection only)
    const uint32_t *row = nullptr;  // [TK]  rows of the store behind those of the tile (sampling pass of the tiled kernel)
};

__device__ inline float select16(const f32x16 &a, int i)
{
    float v = a[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) v = (i == e) ? a[e] : v;
    return v;
}

// The records a wavefront has collected in its private region go to the per-query candidate lists: one lane per
// record claims a slot of the record's (query, segment) with a device-wide atomic and stores the candidate word
// there; a full segment flags the query (it is then resolved exhaustively).  Called when the region is nearly full
// and when the wavefront ends, by all its lanes.  The region was written by this wavefront's own global stores: they
// are waited for, and read back past the vector L1 (agent scope), which may hold lines from an earlier call here.
__device__ inline void flush_records(const ScanArgs &p, Record *region, uint32_t &wave_cnt, uint32_t region_id)
{
    if (wave_cnt == 0) return;
    __builtin_amdgcn_s_waitcnt(0x0070 | 0x0F00);        // vmcnt(0): the stores of the records
    const uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const uint32_t seg_cap = (uint32_t)p.cand_cap / CAND_SEGMENTS;
    for (uint32_t i = lane; i < wave_cnt; i += 64) {
        const uint64_t cw = __hip_atomic_load(&region[i].cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t q = __hip_atomic_load(&region[i].query, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t seg = candidate_segment(candidate_index(cw));
        const uint32_t slot = atomicAdd(&p.cnt[q * CAND_SEGMENTS + seg], 1u);
        if (slot < seg_cap)
            p.cand[(size_t)q * p.cand_cap + seg * seg_cap + slot] = cw;
        else
            p.flag[q] = 1u;
    }
    if (lane == 0)
        atomicAdd(reinterpret_cast<unsigned long long *>(p.stats + STAT_WORDS + region_id % STAT_PARTIALS), (unsigned long long)wave_cnt);
    wave_cnt = 0;
}

// Main pass.  Per block: a bound test (largest dot times largest 1/|k| of the lane's 16 rows against the
// query's pre-filter) costs one max-reduction and decides whether any lane has to look closer; lanes that
// do build the 16-bit mask of elements passing the exact pre-filter (sign bit of fma(dot, inv_k, -thrp),
// collected with one v_alignbit each).  Survivors are rare (a handful per wave and item), and a wave spends
// their cost with its matrix core idle, so as little as possible is done for them here: every lane with a
// survivor picks its own element (a 16-way select, no wave-uniform walk and no exchange between lanes), checks
// the tag predicate (the one test that can thin the records out by orders of magnitude), drops removed rows and
// appends (dot * inv_k, row, query) to the wave's private record region (no atomics: slot = the wave's running count +
// the lane's rank among the appending lanes; flush_records moves a full region to the per-query lists).  The
// second product of the final score, the exact threshold test and the ordering are left to the kernel that
// selects from the lists, which needs nothing but the query's 1/|q| for them: the pre-filter admits an element
// whenever its final score can reach the threshold (and almost only then), so the lists hold what they would hold
// after an exact test here.
struct EpiRows {               // 1/|k| of the 16 key rows a lane holds in one 32-row block
    float ik[16];
    float ikmax;
    int rl0;                   // tile-local row of element 0
};

__device__ inline EpiRows load_rows(const EpiSide &sd, int rl0)
{
    EpiRows r;
    const f32x4 ik0 = *reinterpret_cast<const f32x4 *>(sd.invk + rl0);
    const f32x4 ik1 = *reinterpret_cast<const f32x4 *>(sd.invk + rl0 + 8);
    const f32x4 ik2 = *reinterpret_cast<const f32x4 *>(sd.invk + rl0 + 16);
    const f32x4 ik3 = *reinterpret_cast<const f32x4 *>(sd.invk + rl0 + 24);
    const float ik[16] = {ik0.x, ik0.y, ik0.z, ik0.w, ik1.x, ik1.y, ik1.z, ik1.w,
                          ik2.x, ik2.y, ik2.z, ik2.w, ik3.x, ik3.y, ik3.z, ik3.w};
    r.ikmax = ik[0];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        r.ik[i] = ik[i];
        r.ikmax = __builtin_fmaxf(r.ikmax, ik[i]);
    }
    r.rl0 = rl0;
    return r;
}

// EXACT: the block test takes the largest dot * inv_k of the lane's elements itself (16 products) instead of the
// product of the two maxima.  For stores whose rows have norms of one size (normalised bf16 or f32 rows) the
// cheap bound is as good; for fp8 codes, whose norms differ by a factor of two from row to row, it lets nine
// blocks in ten through where two in ten hold a survivor.
// (MAPPED: the main pass may leave rows out, see main_row)
template <bool EXACT, bool MAPPED>
__device__ inline void main_block(const f32x16 &a, const EpiRows &rw, float tp, uint64_t qm, uint32_t query, const EpiSide &sd, bool filter,
                                  int64_t row0, const ScanArgs &p, Record *region, uint32_t &wave_cnt, uint32_t region_id)
{
    bool maybe;
    if constexpr (EXACT) {
        float smax = a[0] * rw.ik[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) smax = __builtin_fmaxf(smax, a[i] * rw.ik[i]);
        maybe = !(smax < tp);       // (the survivors' mask below repeats the products as fused ones: never stricter than this)
    } else {
        float amax = a[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) amax = __builtin_fmaxf(amax, a[i]);
        // some element can reach the pre-filter only if amax * ikmax does (thrp > 0); otherwise look closer
        maybe = !(__builtin_fmaf(amax, rw.ikmax, -tp) < 0.f) || !(tp > 0.f);
    }
    if (__builtin_amdgcn_ballot_w64(maybe) == 0) return;
    uint32_t fail = 0;
    if (maybe) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            fail = __builtin_amdgcn_alignbit(fail, as_u32(__builtin_fmaf(a[i], rw.ik[i], -tp)), 31);
    }
    uint32_t pass = maybe ? (~fail & 0xffffu) : 0u;     // element i sits at bit 15 - i
    while (__builtin_amdgcn_ballot_w64(pass != 0) != 0) {
        const bool has = pass != 0;
        const int b = 31 - __builtin_clz(has ? pass : 1u);
        pass &= ~(1u << b);
        const int i = 15 - b;
        const int rl = rw.rl0 + 8 * (i >> 2) + (i & 3);
        const uint64_t tg = filter ? sd.tag[rl] : 0ull;         // (in flight during the select)
        const float ikv = sd.invk[rl];
        const float dot = select16(a, i);
        const int64_t place = row0 + rl;
        bool ok = has && place < p.n_keys && !row_removed(ikv);
        const uint32_t row = MAPPED ? main_row(p, (uint32_t)place) : (uint32_t)place;
        if (filter) ok = ok && (tg & qm) != 0;
        // slot in the wave's own record region: running count + rank among the lanes that append (up to 64 of
        // them: the region is emptied first when fewer slots are left)
        const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
        if (okm != 0 && wave_cnt + 64 > (uint32_t)p.region_cap) flush_records(p, region, wave_cnt, region_id);
        if (ok) {
            const uint32_t pos = wave_cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(okm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)okm, 0u));
            Record rec;
            rec.cand = pack_raw_candidate(dot * ikv, row);       // final_score's first product
            rec.query = query;
            rec.pad = 0;
            region[pos] = rec;
        }
        wave_cnt += (uint32_t)__builtin_popcountll(okm);
    }
}

template <int IB, int JB, bool EXACT = false, bool MAPPED = false>
__device__ inline void main_epilogue(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0,
                                     int half, int64_t row0, int q0, const ScanArgs &p, Record *region, uint32_t &wave_cnt, uint32_t region_id)
{
    float thrp[JB];
    uint64_t qm[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        thrp[jb] = sd.thrp[ql0 + jb * 32];
        qm[jb] = filter ? sd.qmask[ql0 + jb * 32] : 0ull;
    }
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        const EpiRows rw = load_rows(sd, wave_row0 + ib * 32 + 4 * half);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb)
            main_block<EXACT, MAPPED>(acc[ib][jb], rw, thrp[jb], qm[jb], (uint32_t)(q0 + ql0 + jb * 32), sd, filter, row0, p, region, wave_cnt, region_id);
    }
}

// Sampling pass: per lane and query column, one qualifying entry of the lane's rows with (nearly) the largest
// s1 = dot * inv_k, stored as the candidate word of s1.  The final score is a non-decreasing function of s1 (one
// more fp32 product with 1/|q| >= 0), which the threshold kernel applies: the sampling pass itself needs no
// per-query value but the mask word.  Any qualifying entry with its exact s1 is a valid sample.
//
// Every element is looked at here, so the search is kept to a few instructions per element: the bits of s1 are read
// as a signed integer (order_key below), the element's number within the lane (5 bits) replaces its low bits, entries
// that fail the tag filter become the smallest integer, and a running integer maximum leaves the number of an
// element whose s1 is within 2^-18 relative of the largest (when that is not negative); that element's exact s1 is
// then recomputed.  Removed
// rows and the repeated rows of a partial tile are not told apart in the search: when one of them wins, its lane
// records no sample for this group of rows, which is always valid (and rare).  Side data
// of the rows is read as 16-byte pieces, four rows at a time.  (Registers are scarce here, with 128 accumulators
// live, and a spilled register costs these kernels dearly: its reload queues behind the stream loads in flight.)
constexpr int32_t SAMPLE_NONE = (int32_t)0x80000000;
// The integer the search compares: the bits of the float as they are.  Non-negative floats keep their order, every
// negative one lies below them, and among negative ones the order is reversed, which costs nothing: a group whose
// best product is negative then records another of its entries, and any qualifying entry with its exact product is a
// valid sample (only the thresholds of queries with fewer than k positive groups could be lower than necessary).
__device__ inline int32_t order_key(float x) { return (int32_t)as_u32(x); }

// one 32x32 block: the best key of the lane's 16 elements joins `best`
__device__ inline void sample_block(const f32x16 &a, int rl0, int id0, const EpiSide &sd, bool filter, uint32_t qm_lo, uint32_t qm_hi,
                                    int32_t &best)
{
#pragma unroll
    for (int run = 0; run < 4; ++run) {             // four runs of four rows: 16 bytes of 1/|k|, 32 bytes of tags
        const int rl = rl0 + 8 * run;
        const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
        const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
        u32x4 tg[2] = {};
        if (filter) {
            tg[0] = *reinterpret_cast<const u32x4 *>(sd.tag + rl);
            tg[1] = *reinterpret_cast<const u32x4 *>(sd.tag + rl + 2);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * run + e;
            int32_t key = (order_key(a[i] * ik[e]) & ~31) | (id0 + i);
            if (filter) {
                const u32x4 t = tg[e >> 1];
                const uint32_t lo = (e & 1) ? t.z : t.x, hi = (e & 1) ? t.w : t.y;
                key = ((lo & qm_lo) | (hi & qm_hi)) != 0 ? key : SAMPLE_NONE;
            }
            best = key > best ? key : best;
        }
    }
}

// The same search with few registers: four elements at a time, their side data read from LDS when it is needed.  For the kernels that keep a software pipeline's fragments live across the
// epilogue and have no registers to spare: there the version above spills, and loses more than it gains.
__device__ inline void sample_block_lean(const f32x16 &a, int rl0, int id0, const EpiSide &sd, bool filter, uint64_t qm, int32_t &best)
{
#pragma unroll
    for (int run = 0; run < 4; ++run) {         // four runs of four rows: one 16-byte read of 1/|k| each
        const int rl = rl0 + 8 * run;
        const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
        const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * run + e;
            int32_t key = (order_key(a[i] * ik[e]) & ~31) | (id0 + i);
            if (filter) key = (sd.tag[rl + e] & qm) != 0 ? key : SAMPLE_NONE;
            best = key > best ? key : best;
        }
    }
}

// store_row: row of the store behind a row of the tile.
template <int IB, int JB, bool LEAN, class F>
__device__ inline void sample_epilogue(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0,
                                       int half, int64_t row0, int q0, const ScanArgs &p, int64_t slot, F store_row)
{
    static_assert(IB * 16 <= 32, "element numbers take five bits");
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int ql = ql0 + jb * 32;
        const uint64_t qm = filter ? sd.qmask[ql] : 0ull;
        int32_t best = SAMPLE_NONE;
#pragma unroll
        for (int ib = 0; ib < IB; ++ib) {
            // the side data is read again for every column: kept from one column to the next it would take a
            // hundred registers that the kernels with a software pipeline do not have
            asm volatile("" ::: "memory");
            if constexpr (LEAN) sample_block_lean(acc[ib][jb], wave_row0 + ib * 32 + 4 * half, ib * 16, sd, filter, qm, best);
            else sample_block(acc[ib][jb], wave_row0 + ib * 32 + 4 * half, ib * 16, sd, filter, (uint32_t)qm, (uint32_t)(qm >> 32), best);
        }
        if (q0 + ql >= p.Q) continue;
        uint64_t cw = 0ull;
        if (best != SAMPLE_NONE) {
            const int e = best & 31, ib = e >> 4, i = e & 15;
            const int rl = wave_row0 + ib * 32 + 4 * half + 8 * (i >> 2) + (i & 3);
            float dot = select16(acc[0][jb], i);
            if (IB > 1 && ib == 1) dot = select16(acc[IB - 1][jb], i);
            const float ikv = sd.invk[rl];
            // a removed row, or a row past the end of the knowledge base (the repeated last row of a partial tile): no sample
            if (!row_removed(ikv) && row0 + rl < p.n_keys)
                cw = pack_candidate(dot * ikv, store_row(rl));     // dot * inv_k exactly as final_score's first product
        }
        p.samp[sample_slot_index(slot, p.sample_group_shift, p.qpad, q0 + ql)] = cw;
    }
}
// The same where the main pass leaves the sampled rows out: everything of a group that can reach the threshold has to be known, so
// the search keeps the best three (floats, as in the whole-store plan's search below, which order negative products too), the
// first two are recomputed exactly and the third bounds the rest.  Removed rows (dead: bit r is row r of the wave's 64) and, in the
// tail of a sample that is whole tiles, repeated ones do not take part.  The side data of four rows serves all columns.
// 2^20 x 1024 bf16 rows, 256 masked queries, a tile of 256 rows for every compute unit: the pass takes 49.6 us, 43.4 with the best
// of a group alone; the main pass, 1/16 shorter for it, 473 us instead of 499.
template <int JB, bool FILTER>
__device__ inline void sample_search(const f32x16 (&acc)[2][JB], const EpiSide &sd, int wave_row0, int half, const uint64_t (&qm)[JB], uint64_t dead, float none,
                                     float (&m1)[JB], float (&m2)[JB], float (&m3)[JB])
{
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) {
#pragma unroll
        for (int run = 0; run < 4; ++run) {
            int rl = wave_row0 + ib * 32 + 4 * half + 8 * run;
            asm volatile("" : "+v"(rl));        // (side data of all rows at once would take a hundred registers)
            const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
            const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
            u32x4 t0 = {}, t1 = {};
            if constexpr (FILTER) {
                t0 = *reinterpret_cast<const u32x4 *>(sd.tag + rl);
                t1 = *reinterpret_cast<const u32x4 *>(sd.tag + rl + 2);
            }
            const uint32_t lo[4] = {t0.x, t0.z, t1.x, t1.z}, hi[4] = {t0.y, t0.w, t1.y, t1.w};
            const uint32_t dead4 = dead != 0 ? (uint32_t)(dead >> (ib * 32 + 8 * run)) >> (4 * half) : 0u;      // (uniform condition)
#pragma unroll
            for (int jb = 0; jb < JB; ++jb) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = acc[ib][jb][4 * run + e] * ik[e];
                    if constexpr (FILTER) v[e] = ((lo[e] & (uint32_t)qm[jb]) | (hi[e] & (uint32_t)(qm[jb] >> 32))) != 0 ? v[e] : none;
                }
                if (dead != 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (dead4 >> e & 1u) != 0 ? none : v[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float f = as_f32((as_u32(v[e]) & ~31u) | (uint32_t)(ib * 16 + 4 * run + e));
                    m3[jb] = __builtin_amdgcn_fmed3f(m2[jb], m3[jb], f);
                    m2[jb] = __builtin_amdgcn_fmed3f(m1[jb], m2[jb], f);
                    m1[jb] = __builtin_fmaxf(m1[jb], f);
                }
            }
        }
    }
}
template <int JB>
__device__ inline void sample_epilogue_more(const f32x16 (&acc)[2][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0, int half, int64_t row0, int q0,
                                            const ScanArgs &p, int64_t slot, int64_t tile_run, int tk)
{
    const float none = as_f32(0xff7fffe0u);        // the lowest finite value but for its low bits
    float m1[JB], m2[JB], m3[JB];
    uint64_t qm[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        m1[jb] = m2[jb] = m3[jb] = none;
        qm[jb] = filter ? sd.qmask[ql0 + jb * 32] : 0ull;
    }
    uint64_t dead;
    {
        const int lane = threadIdx.x & 63;
        dead = __builtin_amdgcn_ballot_w64(row_removed(sd.invk[wave_row0 + lane]) || row0 + wave_row0 + lane >= p.n_keys);
    }
    if (filter) sample_search<JB, true>(acc, sd, wave_row0, half, qm, dead, none, m1, m2, m3);
    else sample_search<JB, false>(acc, sd, wave_row0, half, qm, dead, none, m1, m2, m3);
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int ql = ql0 + jb * 32;
        float value[2];
        int rl[2], place[2];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const float m = w == 0 ? m1[jb] : m2[jb];
            const int e = (int)(as_u32(m) & 31u), i = e & 15;
            place[w] = e;
            rl[w] = wave_row0 + (e >> 4) * 32 + 4 * half + 8 * (i >> 2) + (i & 3);
            const float dot = e < 16 ? select16(acc[0][jb], i) : select16(acc[1][jb], i);
            value[w] = dot * sd.invk[rl[w]];
        }
        if (q0 + ql >= p.Q) continue;
        const bool any = m1[jb] > none, two = m2[jb] > none;
        // (the search's order is that of the values but for their low bits: either may be the larger one)
        const bool swap = two && value[1] > value[0];
        const size_t at = sample_slot_index(slot, p.sample_group_shift, p.qpad, q0 + ql);
        p.samp[at] = any ? pack_candidate(swap ? value[1] : value[0], sample_index<true>(p, tile_run, row0, tk, swap ? rl[1] : rl[0])) : 0ull;
        const uint32_t b3 = as_u32(m3[jb]);
        const uint32_t others = m3[jb] > none ? score_to_ordered(as_f32((int32_t)b3 < 0 ? b3 & ~31u : b3 | 31u)) : 0u;
        p.samp_more[at] = two ? pack_second(swap ? value[0] : value[1], others, (uint32_t)(swap ? place[0] : place[1])) : 0ull;
    }
}

// ------------------------------------------------------------------------------------------------
// Whole-store plan: per query and group of rows the two best qualifying products, exact, and the third or a bound on it.
// ------------------------------------------------------------------------------------------------
struct TopThree {
    float first, second;       // products of the two best rows; -inf where there is none
    float third;               // no other row of the group has a larger product
    uint32_t rows;             // places in the tile, as in the group's entry (see WholePlan)
};
// The same of the rows of both arguments; the third is a bound.
__device__ inline TopThree join(const TopThree &a, const TopThree &b)
{
    const bool swap = b.first > a.first;
    const TopThree x = swap ? b : a, y = swap ? a : b;
    const bool keep = x.second >= y.first;
    TopThree r;
    r.first = x.first;
    r.second = keep ? x.second : y.first;
    r.rows = keep ? x.rows & 0xffffu : (x.rows & 255u) | (y.rows << 8 & 0xff00u);
    r.third = __builtin_fmaxf(__builtin_fmaxf(x.third, y.third), keep ? y.first : __builtin_fmaxf(x.second, y.second));
    return r;
}
__device__ inline TopThree other_half(const TopThree &t, int lanes)
{
    TopThree o;
    o.first = __shfl_xor(t.first, lanes, 64);
    o.second = __shfl_xor(t.second, lanes, 64);
    o.third = __shfl_xor(t.third, lanes, 64);
    o.rows = (uint32_t)__shfl_xor((int)t.rows, lanes, 64);
    return o;
}
// ... of the lane 32 places away, without the round trip through LDS that a shuffle is
__device__ inline uint32_t across(uint32_t x)
{
    typedef uint32_t u32x2_ __attribute__((ext_vector_type(2)));
    const u32x2_ r = __builtin_amdgcn_permlane32_swap(x, x, false, false);        // {lower half twice, upper half twice}
    return (threadIdx.x & 32) != 0 ? r.x : r.y;
}
__device__ inline TopThree across_halves(const TopThree &t)
{
    return TopThree{as_f32(across(as_u32(t.first))), as_f32(across(as_u32(t.second))), as_f32(across(as_u32(t.third))), across(t.rows)};
}
// Whether, in some lane, what is not named could be as good as the second row (uniform).
__device__ inline bool unclear(const TopThree &t)
{
    return __builtin_amdgcn_ballot_w64(t.third >= t.second && t.third > -__builtin_inff()) != 0;
}

// Does product a at order number oa come before b at ob?
__device__ inline bool comes_before(float a, uint32_t oa, float b, uint32_t ob) { return a > b || (a == b && oa < ob); }
// Units in the last place by which x is below `top`, less one (a large number where it is not); a row is near below 2.
__device__ inline uint32_t gap_below(float top, float x)
{
    auto ordered = [](uint32_t u) { return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u); };      // (score_to_ordered without a condition)
    return ordered(as_u32(top + 0.0f)) - ordered(as_u32(x + 0.0f)) - 1u;       // (one zero)
}
__device__ inline uint32_t least(uint32_t a, uint32_t b) { return a < b ? a : b; }

// join for rows in the order of the result.  Each argument names its first three, or its first two and a bound below the
// second; so does the result, as a bound that reaches the third place belongs to an argument whose two rows are the first
// two.  (A bound wins against an equal product: the row behind it may have the lower index.)
template <int TK> __device__ inline TopThree join_in_order(TopThree a, TopThree b)
{
    auto sorted = [](TopThree t) {        // two equal products that a join without order left as they came
        const uint32_t p = t.rows & 255u, q = t.rows >> 8 & 255u;
        if (t.first == t.second && whole_order<TK>(p) > whole_order<TK>(q)) t.rows = (t.rows & ~0xffffu) | q | p << 8;
        return t;
    };
    a = sorted(a);
    b = sorted(b);
    auto order = [](const TopThree &t, int w) { return whole_order<TK>(t.rows >> (8 * w) & 255u); };
    const bool swap = comes_before(b.first, order(b, 0), a.first, order(a, 0));
    const TopThree x = swap ? b : a, y = swap ? a : b;
    const bool keep = comes_before(x.second, order(x, 1), y.first, order(y, 0));
    const uint32_t x3 = x.rows >> 16 & WHOLE_THIRD;
    const bool bound = keep && x3 == 0u && x.third >= y.first;
    const bool third_x = keep ? bound || (x3 != 0u && comes_before(x.third, whole_order<TK>(x3 - 1u), y.first, order(y, 0)))
                              : comes_before(x.second, order(x, 1), y.second, order(y, 1));
    TopThree r;
    r.first = x.first;
    r.second = keep ? x.second : y.first;
    r.third = keep ? (third_x ? x.third : y.first) : (third_x ? x.second : y.second);
    const uint32_t place = keep ? (third_x ? x3 - 1u : y.rows & 255u) : ((third_x ? x.rows : y.rows) >> 8 & 255u);
    r.rows = (keep ? x.rows & 0xffffu : (x.rows & 255u) | (y.rows << 8 & 0xff00u)) | (bound ? 0u : (place + 1u) << 16);
    const float third = r.third;
    auto gap = [third](const TopThree &t) { return least(least(gap_below(third, t.first), gap_below(third, t.second)), gap_below(third, t.third)); };
    auto near = [third](const TopThree &t) { return t.third == third ? t.rows & WHOLE_NEAR : 0u; };
    r.rows |= near(x) | near(y) | (least(gap(x), gap(y)) < 2u ? WHOLE_NEAR : 0u);
    return r;
}

// The products of the lane's 16 elements of block (ib, jb), `none` in the place of rows that do not count.  rl0: tile-local
// row of the first; dead: bit r set = row r of the wave's 32 * IB is removed or past the end.
__device__ inline void whole_products(const f32x16 &a, const EpiSide &sd, bool filter, uint64_t qm, int rl0, int half, int ib, uint64_t dead, float none,
                                      float (&v)[16])
{
#pragma unroll
    for (int run = 0; run < 4; ++run) {
        const int rl = rl0 + 8 * run;
        const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
        const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * run + e] = a[4 * run + e] * ik[e];
        if (filter) {
            const u32x4 t0 = *reinterpret_cast<const u32x4 *>(sd.tag + rl), t1 = *reinterpret_cast<const u32x4 *>(sd.tag + rl + 2);
            const uint32_t lo[4] = {t0.x, t0.z, t1.x, t1.z}, hi[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * run + e] = ((lo[e] & (uint32_t)qm) | (hi[e] & (uint32_t)(qm >> 32))) != 0 ? v[4 * run + e] : none;
        }
    }
    if (dead != 0) {            // (uniform)
        const uint32_t dead32 = (uint32_t)(dead >> (32 * ib)) >> (4 * half);
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = (dead32 >> (8 * (i >> 2) + (i & 3)) & 1u) ? none : v[i];
    }
}

// One wave column: the lane's 16 * IB elements.  As in the sampling search the element's number replaces the product's
// low five bits, here with the product left a float: one maximum and two medians per element keep the largest three
// in order.  The first two are then recomputed exactly; the third, its low bits at their largest, bounds the rest.
template <int IB, int JB>
__device__ inline TopThree whole_column(const f32x16 (&acc)[IB][JB], int jb, const EpiSide &sd, bool filter, uint64_t qm, int wave_row0, int half,
                                        uint64_t dead)
{
    const float none = as_f32(0xff7fffe0u);        // the lowest finite value but for its low bits
    float m1 = none, m2 = none, m3 = none;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        float v[16];
        whole_products(acc[ib][jb], sd, filter, qm, wave_row0 + ib * 32 + 4 * half, half, ib, dead, none, v);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float f = as_f32((as_u32(v[i]) & ~31u) | (uint32_t)(ib * 16 + i));       // (never above `none` where v is)
            m3 = __builtin_amdgcn_fmed3f(m2, m3, f);
            m2 = __builtin_amdgcn_fmed3f(m1, m2, f);
            m1 = __builtin_fmaxf(m1, f);
        }
    }
    TopThree t;
    const uint32_t b3 = as_u32(m3);
    t.third = m3 > none ? as_f32((int32_t)b3 < 0 ? b3 & ~31u : b3 | 31u) : -__builtin_inff();
    t.rows = 0;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const float m = w == 0 ? m1 : m2;
        const int e = (int)(as_u32(m) & 31u), ib = e >> 4, i = e & 15;
        const int rl = wave_row0 + (IB > 1 ? ib * 32 : 0) + 4 * half + 8 * (i >> 2) + (i & 3);
        float dot = select16(acc[0][jb], i);
        if (IB > 1 && ib == 1) dot = select16(acc[IB - 1][jb], i);
        const float exact = m > none ? dot * sd.invk[rl] : -__builtin_inff();
        (w == 0 ? t.first : t.second) = exact;
        t.rows |= (uint32_t)rl << (8 * w);
    }
    if (t.second > t.first) {       // (equal but for the bits that held the numbers)
        const float f = t.first;
        t.first = t.second;
        t.second = f;
        t.rows = (t.rows >> 8) | (t.rows & 255u) << 8;
    }
    return t;
}

// The same with the first three in the order of the result: the elements are taken by rising row, one that is larger than
// a place's moves in.  For the few columns where the search above leaves the third unclear, one in ten thousand of a store
// without equal rows; so it is written for few registers (with those of a search over arrays, eight more to 64, calls of
// 65 to 128 queries and of fp8 queries were 3 to 5 % slower).
template <int TK, int IB, int JB>
__device__ inline TopThree whole_column_in_order(const f32x16 (&acc)[IB][JB], int jb, const EpiSide &sd, bool filter, uint64_t qm, int wave_row0, int half,
                                                 uint64_t dead)
{
    static_assert(TK == 128 || IB == 1, "order of the elements");
    constexpr float NONE = -__builtin_inff();
    TopThree t = {NONE, NONE, NONE, 0u};
    float below = NONE;         // the largest product below the third
    int p1 = 0, p2 = 0, p3 = 0;
    int rl0 = wave_row0 + 4 * half;
    asm volatile("" : "+v"(rl0));       // (the products are formed again: kept from the search they would cost it registers)
    uint32_t out_of_it = 0;     // bit ib * 16 + i: element i of block ib does not count
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        const uint32_t d = (uint32_t)(dead >> (32 * ib)) >> (4 * half);
        out_of_it |= ((d & 15u) | (d >> 4 & 0xf0u) | (d >> 8 & 0xf00u) | (d >> 12 & 0xf000u)) << (16 * ib);
    }
    if (filter) {
#pragma unroll
        for (int e = 0; e < 16 * IB; ++e) {
            const uint64_t hit = sd.tag[rl0 + (e >> 4) * 32 + 8 * (e >> 2 & 3) + (e & 3)] & qm;
            out_of_it |= hit != 0 ? 0u : 1u << e;
            if (e % 4 == 3) asm volatile("" : "+v"(out_of_it));
        }
    }
#pragma unroll
    for (int n = 0; n < 16 * IB; ++n) {
        // by rising whole_order: rows 32 places apart follow each other in a tile of 128, 16 places apart in one of 64
        const int ib = TK == 64 ? 0 : n % IB, i = TK == 64 ? (n >> 1) | (n & 1) << 3 : n / IB, at = ib * 32 + 8 * (i >> 2) + (i & 3);
        float f = acc[ib][jb][i] * sd.invk[rl0 + at];
        f = (out_of_it >> (ib * 16 + i) & 1u) != 0 ? NONE : f;
        const bool g1 = f > t.first, g2 = f > t.second, g3 = f > t.third;
        const float out = g3 ? t.third : f;
        t.third = g2 ? t.second : g3 ? f : t.third;
        p3 = g2 ? p2 : g3 ? rl0 + at : p3;
        t.second = g1 ? t.first : g2 ? f : t.second;
        p2 = g1 ? p1 : g2 ? rl0 + at : p2;
        t.first = g1 ? f : t.first;
        p1 = g1 ? rl0 + at : p1;
        below = out < t.third ? __builtin_fmaxf(below, out) : below;
        // (here and now: moved to the end, the places would keep the conditions of all elements, which spill)
        if (n % 2 == 1) asm volatile("" : "+v"(p1), "+v"(p2), "+v"(p3), "+v"(below));
    }
    t.rows = (uint32_t)p1 | (uint32_t)p2 << 8 | (uint32_t)(p3 + 1) << 16 | (gap_below(t.third, below) < 2u ? WHOLE_NEAR : 0u);
    return t;
}

// All waves of the workgroup call this, converged.  `exchange`: (WM - 1) * TQ entries in LDS.
template <int TK, int IB, int JB, int WM, int TQ>
__device__ inline void whole_epilogue(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wm, int ql0, int half, int64_t tile,
                                      int q0, const ScanArgs &p, uint64_t dead, u32x4 *exchange)
{
    TopThree t[JB];
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const uint64_t qm = filter ? sd.qmask[ql0 + jb * 32] : 0ull;
        const TopThree own = whole_column<IB, JB>(acc, jb, sd, filter, qm, wm * IB * 32, half, dead);
        t[jb] = join(own, other_half(own, 32));
        if (__builtin_expect(unclear(t[jb]), 0)) {
            const TopThree o = whole_column_in_order<TK, IB, JB>(acc, jb, sd, filter, qm, wm * IB * 32, half, dead);
            t[jb] = join_in_order<TK>(o, other_half(o, 32));
        }
        if (!p.whole_fine && wm > 0 && half == 0) exchange[(wm - 1) * TQ + ql0 + jb * 32] = u32x4{as_u32(t[jb].first), as_u32(t[jb].second), as_u32(t[jb].third), t[jb].rows};
    }
    const int64_t group = p.whole_fine ? tile * WM + wm : tile;
    if (!p.whole_fine) {
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (wm != 0) return;
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int ql = ql0 + jb * 32, q = q0 + ql;
        if (!p.whole_fine) {
            auto of_wave = [&](int w) {
                const u32x4 x = exchange[w * TQ + ql];
                return TopThree{as_f32(x[0]), as_f32(x[1]), as_f32(x[2]), x[3]};
            };
            const TopThree own = t[jb];
            for (int w = 0; w < WM - 1; ++w) t[jb] = join(t[jb], of_wave(w));
            if (__builtin_expect(unclear(t[jb]), 0)) {
                t[jb] = own;
                for (int w = 0; w < WM - 1; ++w) t[jb] = join_in_order<TK>(t[jb], of_wave(w));
            }
        }
        if (half == 0 && q < p.Q) {
            const size_t at = (size_t)q * p.whole_groups + group;
            p.whole_best[at] = t[jb].first;
            p.whole_pair[at] = u32x4{as_u32(t[jb].second), as_u32(t[jb].third), t[jb].rows, 0u};
        }
    }
}

// Dense plan: every product, -inf where the row does not qualify.  A lane stores four neighbouring rows of its query at a
// time; the rows past the last one up to the tile's end are there too.
__device__ inline void dense_store(float (&v)[4], const float (&ik)[4], const EpiSide &sd, bool filter, uint64_t qm, int rl, int64_t row0, int q, const ScanArgs &p)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const bool ok = row0 + rl + e < p.n_keys && !row_removed(ik[e]) && (!filter || (sd.tag[rl + e] & qm) != 0);
        v[e] = ok ? v[e] : -__builtin_inff();
    }
    if (q < p.Q) *reinterpret_cast<f32x4 *>(p.dense + (size_t)q * p.dense_stride + row0 + rl) = f32x4{v[0], v[1], v[2], v[3]};
}
template <int IB, int JB>
__device__ inline void dense_epilogue(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0, int half, int64_t row0, int q0,
                                      const ScanArgs &p)
{
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
        const int ql = ql0 + jb * 32;
        const uint64_t qm = filter ? sd.qmask[ql] : 0ull;
#pragma unroll
        for (int ib = 0; ib < IB; ++ib)
#pragma unroll
            for (int run = 0; run < 4; ++run) {
                const int rl = wave_row0 + ib * 32 + 4 * half + 8 * run;
                const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl);
                const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w};
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[ib][jb][4 * run + e] * ik[e];
                dense_store(v, ik, sd, filter, qm, rl, row0, q0 + ql, p);
            }
    }
}

// ------------------------------------------------------------------------------------------------
// Weighted random selection: the same two epilogues on keys = score / T + ln(gain) + Gumbel noise.
// ------------------------------------------------------------------------------------------------

// Philox4x32 with 10 rounds (Salmon, Moraes, Dror, Shaw, SC'11) on the counter (c0, c1, 0, 0).  The weighted selection's
// main pass is bound by the vector instructions of this function, so they are counted: a round is two 32 x 32 -> 64 bit
// multiplies (v_mad_u64_u32, which issues at the rate of a 32-bit one) and two three-operand exclusive-ors (v_bitop3_b32),
// 41 instructions a call where separate halves and two-operand ones took 74.  2^20 x 1024 rows, 256 queries: 0.722 -> 0.655 ms.
// (Two operations a pair less in the bound below and one less in the comparison changed nothing: at that point the clock
// that the device grants sets the time.)
__device__ inline uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1, uint32_t (&out)[4])
{
    uint32_t c2 = 0u, c3 = 0u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u, p1 = (uint64_t)c2 * 0xCD9E8D57u;
        c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        c1 = (uint32_t)p1;
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c3 = (uint32_t)p0;
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// Standard Gumbel variate from one generator word: U = (upper 23 bits + 1/2) / 2^23 (exact in fp32), G = -ln(-ln U).
// Both logarithms are the hardware's base-2 logarithm times ln 2: U and -ln U are normal numbers (2^-24 <= U < 1,
// 6e-8 <= -ln U <= 16.7), so the library logarithm's handling of denormals and its extended-precision product (three
// quarters of this function's instructions) buy nothing.  Over all 2^23 values of U the result is within 1.7e-6 of
// the exact variate and non-decreasing in U.
__device__ inline float gumbel_of_word(uint32_t w)
{
    constexpr float LN2 = 0.6931471805599453f;
    const float u = __builtin_fmaf((float)(w >> 9), 0x1p-23f, 0x1p-24f);
    const float l1 = __builtin_amdgcn_logf(u) * LN2;
    return -(__builtin_amdgcn_logf(-l1) * LN2);
}

// Key of one (query, entry) pair.  Entries 4j .. 4j+3 share one generator call (counter (j, query, 0, 0)); the word
// is picked by entry % 4.  "+ 0.0f" as in final_score: equal keys have equal bit patterns.
__device__ inline float draw_key(float score, float log_gain, float gumbel, float inv_t)
{
    return (__builtin_fmaf(score, inv_t, log_gain) + gumbel) + 0.0f;
}
__device__ inline float draw_key_of(float score, float log_gain, const DrawArgs &dr, uint32_t query, int64_t row)
{
    uint32_t w[4];
    philox4x32_10((uint32_t)(row >> 2), query, dr.seed_lo, dr.seed_hi, w);
    const uint32_t word = (row & 3) == 0 ? w[0] : (row & 3) == 1 ? w[1] : (row & 3) == 2 ? w[2] : w[3];
    return draw_key(score, log_gain, gumbel_of_word(word), dr.inv_t);
}
__device__ inline float draw_key_of(float score, const DrawArgs &dr, uint32_t query, int64_t row)
{
    return draw_key_of(score, dr.log_gain[row], dr, query, row);
}

// Keys of the 16 elements a lane holds in one block (four runs of four consecutive rows: four generator calls).
__device__ inline void block_keys(const f32x16 &a, const EpiRows &rw, float iq, const ScanArgs &p, uint32_t query, int64_t row0,
                                  const EpiSide &sd, float (&key)[16])
{
    const DrawArgs &dr = p.draw;
#pragma unroll
    for (int run = 0; run < 4; ++run) {
        const int64_t first = row0 + rw.rl0 + 8 * run;         // a multiple of 4
        uint32_t w[4];
        philox4x32_10((uint32_t)(first >> 2), query, dr.seed_lo, dr.seed_hi, w);
        const f32x4 lg = *reinterpret_cast<const f32x4 *>(sd.lgain + rw.rl0 + 8 * run);
        const float lgs[4] = {lg.x, lg.y, lg.z, lg.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * run + e;
            key[i] = draw_key(final_score(a[i], rw.ik[i], iq), lgs[e], gumbel_of_word(w[e]), dr.inv_t);
        }
    }
}

// The largest generator word (its upper 23 bits, as an integer) with which an element whose noise-free part is at
// most xmax still has a key below the threshold key tp; -1 if there is none.  The noise is a non-decreasing function
// of those bits and the two additions of draw_key are monotone, so every element of the block with bits at or below
// the returned value fails "key >= tp" however its own key rounds.  The value is found from the inverse of the
// Gumbel transform with a margin (fast exponentials, 2 % on the inner one, two steps on the integer) and then checked
// with the very operations of draw_key; a value that fails the check is replaced by a more careful one, then by -1.
__device__ inline int noise_floor(float xmax, float tp)
{
    if (!(tp > -__builtin_inff())) return -1;
    float t = __expf(xmax - tp) * 1.02f;       // e^-c, c = the noise an element at xmax needs
    int m = -1;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        const float mf = __builtin_fmaf(__expf(-t), 0x1p23f, -2.0f);
        const int cand = mf >= 0.f ? (int)__builtin_fminf(mf, 8388607.f) : -1;
        if (cand < 0) break;
        const float key = (xmax + gumbel_of_word((uint32_t)cand << 9)) + 0.0f;
        if (key < tp) {
            m = cand;
            break;
        }
        t *= 8.f;
    }
    return m;
}

// Main pass on keys.  Computing a key costs a generator call per four elements and two logarithms per element; the
// test against the query's threshold key does not need them: with the largest noise-free part of the lane's 16
// elements, noise_floor gives the generator word below which no element of the block can pass, and the per-element
// test is one integer compare on the generator's output.  What passes (the elements whose key can reach the
// threshold, and as many again) is handled like the survivors of the score pass, each lane walking its own
// elements, with the exact key and the exact tests.
__device__ inline void main_block_draw(const f32x16 &a, const EpiRows &rw, float tp, int ql, const EpiSide &sd, bool filter,
                                       int64_t row0, int q0, const ScanArgs &p, Record *region, uint32_t &wave_cnt, uint32_t region_id)
{
    const DrawArgs &dr = p.draw;
    const float iq = sd.invq[ql];
    const uint32_t query = dr.first_query + (uint32_t)(q0 + ql);
    float xmax = -__builtin_inff();
#pragma unroll
    for (int run = 0; run < 4; ++run) {
        const f32x4 lg = *reinterpret_cast<const f32x4 *>(sd.lgain + rw.rl0 + 8 * run);
        const float lgs[4] = {lg.x, lg.y, lg.z, lg.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            xmax = __builtin_fmaxf(xmax, __builtin_fmaf(final_score(a[4 * run + e], rw.ik[4 * run + e], iq), dr.inv_t, lgs[e]));
    }
    const int floor_m = noise_floor(xmax, tp);
    const uint32_t floor_w = floor_m < 0 ? 0u : ((uint32_t)floor_m << 9) | 0x1ffu;
    uint32_t pass = 0;
#pragma unroll
    for (int run = 0; run < 4; ++run) {
        uint32_t w[4];
        philox4x32_10((uint32_t)((row0 + rw.rl0 + 8 * run) >> 2), query, dr.seed_lo, dr.seed_hi, w);
#pragma unroll
        for (int e = 0; e < 4; ++e) pass = (pass << 1) | (w[e] > floor_w ? 1u : 0u);       // element i at bit 15 - i
    }
    if (floor_m < 0) pass = 0xffffu;
    if (__builtin_amdgcn_ballot_w64(pass != 0) == 0) return;
    const uint64_t t64 = sd.thr64[ql];
    const uint64_t qm = filter ? sd.qmask[ql] : 0ull;
    do {
        const bool has = pass != 0;
        const int b = 31 - __builtin_clz(has ? pass : 1u);
        pass &= ~(1u << b);
        const int i = 15 - b;
        const int rl = rw.rl0 + 8 * (i >> 2) + (i & 3);
        const int64_t row = row0 + rl;
        const float ik = sd.invk[rl];
        const float kv = draw_key_of(final_score(select16(a, i), ik, iq), sd.lgain[rl], dr, query, row);
        const uint64_t cw = pack_candidate(kv, (uint32_t)row);
        bool ok = has && row < p.n_keys && kv > -__builtin_inff() && cw >= t64 && !row_removed(ik);
        if (filter) ok = ok && (sd.tag[rl] & qm) != 0;
        const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
        if (okm != 0 && wave_cnt + 64 > (uint32_t)p.region_cap) flush_records(p, region, wave_cnt, region_id);
        if (ok) {
            const uint32_t pos = wave_cnt + __builtin_amdgcn_mbcnt_hi((uint32_t)(okm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)okm, 0u));
            Record rec;
            rec.cand = cw;
            rec.query = (uint32_t)(q0 + ql);
            rec.pad = 0;
            region[pos] = rec;
        }
        wave_cnt += (uint32_t)__builtin_popcountll(okm);
    } while (__builtin_amdgcn_ballot_w64(pass != 0) != 0);
}

template <int IB, int JB>
__device__ inline void main_epilogue_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0,
                                          int half, int64_t row0, int q0, const ScanArgs &p, Record *region, uint32_t &wave_cnt, uint32_t region_id)
{
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        int rl0 = wave_row0 + ib * 32 + 4 * half;
        EpiRows rw = load_rows(sd, rl0);
#pragma unroll
        for (int jb = 0; jb < JB; ++jb) {
            if (IB * JB >= 8 && jb > 0) {       // (128 accumulators: the rows' 1/|k| are read again rather than kept, or registers spill)
                asm volatile("" : "+v"(rl0));
                rw = load_rows(sd, rl0);
            }
            main_block_draw(acc[ib][jb], rw, sd.thrp[ql0 + jb * 32], ql0 + jb * 32, sd, filter, row0, q0, p, region, wave_cnt, region_id);
        }
    }
}

// Dense plan on keys.
template <int IB, int JB, int JBX>
__device__ inline void dense_column_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0, int half, int64_t row0, int q0,
                                         const ScanArgs &p)
{
    const int ql = ql0 + JBX * 32;
    const uint64_t qm = filter ? sd.qmask[ql] : 0ull;
    const float iq = sd.invq[ql];
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        int rl0 = wave_row0 + ib * 32 + 4 * half;
        asm volatile("" : "+v"(rl0));       // (see sample_column_draw)
        const EpiRows rw = load_rows(sd, rl0);
        float key[16];
        block_keys(acc[ib][JBX], rw, iq, p, p.draw.first_query + (uint32_t)(q0 + ql), row0, sd, key);
#pragma unroll
        for (int run = 0; run < 4; ++run) {
            float v[4] = {key[4 * run], key[4 * run + 1], key[4 * run + 2], key[4 * run + 3]};
            const float ik[4] = {rw.ik[4 * run], rw.ik[4 * run + 1], rw.ik[4 * run + 2], rw.ik[4 * run + 3]};
            dense_store(v, ik, sd, filter, qm, rl0 + 8 * run, row0, q0 + ql, p);
        }
    }
}
template <int IB, int JB, int... JBX>
__device__ inline void dense_epilogue_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0, int half, int64_t row0, int q0,
                                           const ScanArgs &p, std::integer_sequence<int, JBX...>)
{
    (dense_column_draw<IB, JB, JBX>(acc, sd, filter, wave_row0, ql0, half, row0, q0, p), ...);
}

// Sampling pass on keys: per lane and query column the qualifying entry with the largest key.  One function per
// query column of the wave's tile, expanded at compile time: as a loop over the columns the body (eight generator
// calls and 32 keys per column) is too large to be unrolled, and the accumulators, indexed by a loop counter, would
// live in scratch memory.
template <int IB, int JB, int JBX>
__device__ inline void sample_column_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0,
                                          int half, int64_t row0, int q0, const ScanArgs &p, int64_t slot)
{
    const int ql = ql0 + JBX * 32;
    const float iq = sd.invq[ql];
    const uint64_t qm = filter ? sd.qmask[ql] : 0ull;
    const uint32_t query = p.draw.first_query + (uint32_t)(q0 + ql);
    float best = -__builtin_inff();
    int best_e = 0;
#pragma unroll
    for (int ib = 0; ib < IB; ++ib) {
        // (the row number is opaque per block: otherwise the side data and the scattered-row arithmetic of all the
        // wave's rows, which do not depend on the column, are kept in registers across the columns and spilled)
        int rl0 = wave_row0 + ib * 32 + 4 * half;
        asm volatile("" : "+v"(rl0));
#pragma unroll
        for (int run = 0; run < 4; ++run) {         // (four rows at a time, one generator call: few registers)
            int rl = rl0 + 8 * run;
            asm volatile("" : "+v"(rl), "+v"(best), "+v"(best_e));
            const f32x4 ik4 = *reinterpret_cast<const f32x4 *>(sd.invk + rl), lg4 = *reinterpret_cast<const f32x4 *>(sd.lgain + rl);
            const float ik[4] = {ik4.x, ik4.y, ik4.z, ik4.w}, lg[4] = {lg4.x, lg4.y, lg4.z, lg4.w};
            uint32_t w[4];
            philox4x32_10(sd.row[rl] >> 2, query, p.draw.seed_lo, p.draw.seed_hi, w);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool ok = row0 + rl + e < p.n_keys && !row_removed(ik[e]);
                if (filter) ok = ok && (sd.tag[rl + e] & qm) != 0;
                const float key = draw_key(final_score(acc[ib][JBX][4 * run + e], ik[e], iq), lg[e], gumbel_of_word(w[e]), p.draw.inv_t);
                const float f = ok ? key : -__builtin_inff();
                best_e = f > best ? ib * 16 + 4 * run + e : best_e;
                best = __builtin_fmaxf(best, f);
            }
        }
    }
    if (q0 + ql < p.Q) {
        const size_t at = sample_slot_index(slot, p.sample_group_shift, p.qpad, q0 + ql);
        p.samp[at] = best > -__builtin_inff() ? pack_candidate(best, sd.row[wave_row0 + (best_e >> 4) * 32 + 4 * half + 8 * (best_e >> 2 & 3) + (best_e & 3)]) : 0ull;
    }
}

template <int IB, int JB, int... JBX>
__device__ inline void sample_columns_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0, int half, int64_t row0,
                                           int q0, const ScanArgs &p, int64_t slot, std::integer_sequence<int, JBX...>)
{
    (sample_column_draw<IB, JB, JBX>(acc, sd, filter, wave_row0, ql0, half, row0, q0, p, slot), ...);
}

template <int IB, int JB>
__device__ inline void sample_epilogue_draw(const f32x16 (&acc)[IB][JB], const EpiSide &sd, bool filter, int wave_row0, int ql0,
                                            int half, int64_t row0, int q0, const ScanArgs &p, int64_t slot)
{
    sample_columns_draw<IB, JB>(acc, sd, filter, wave_row0, ql0, half, row0, q0, p, slot, std::make_integer_sequence<int, JB>{});
}

}  // namespace kbi
