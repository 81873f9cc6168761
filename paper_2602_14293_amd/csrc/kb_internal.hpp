// Internal declarations shared by the translation units of libkb (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <atomic>

#include "kb.h"

// The handle: host-side bookkeeping over caller-owned device storage.
struct kb {
    int32_t d;
    kb_dtype_t dtype;
    int64_t capacity, n, n_normalized;
    void *keys;
    float *row_scale, *inv_norm;
    uint64_t *tags;
    int64_t tune_sample_keys, tune_config, tune_wg_per_cu, tune_no_small_path;
    hipEvent_t *prof_events;   // 2 * prof_max events while profiling, else nullptr
    int prof_max, prof_used;
    int prof_stride, prof_seen;   // every prof_stride-th scan launch of a profiling session is timed
};

namespace kbi {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Bit reinterpretation of scalars passed BY VALUE.  (__builtin_bit_cast applied directly to a vector
// element such as v[e] or f.y has been seen to read element 0 instead; never do that.)
__host__ __device__ inline float as_f32(uint32_t x) { return __builtin_bit_cast(float, x); }
__host__ __device__ inline uint32_t as_u32(float x) { return __builtin_bit_cast(uint32_t, x); }

// A candidate is one 64-bit sortable word: larger word = earlier in the result order
// (score descending, index ascending).  0 is never a valid candidate ("empty").
//   high 32 bits: the fp32 score mapped monotonically onto unsigned integers
//   low  32 bits: ~index  (index < 2^31, so a smaller index gives a larger word)
__host__ __device__ inline uint32_t score_to_ordered(float s)
{
    uint32_t u = __builtin_bit_cast(uint32_t, s);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__host__ __device__ inline float ordered_to_score(uint32_t o)
{
    uint32_t u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
    return __builtin_bit_cast(float, u);
}
__host__ __device__ inline uint64_t pack_candidate(float score, uint32_t index)
{
    return ((uint64_t)score_to_ordered(score) << 32) | (uint32_t)(~index);
}
__host__ __device__ inline uint32_t candidate_index(uint64_t c) { return ~(uint32_t)c; }
// What the main pass of a scan leaves in the candidate lists of a plain query: the bits of dot * inv_k (the first
// product of final_score) instead of the ordered score, which the kernel that selects from the lists derives with the
// query's 1/|q|; the same low word.
__host__ __device__ inline uint64_t pack_raw_candidate(float dot_inv_k, uint32_t index)
{
    return ((uint64_t)__builtin_bit_cast(uint32_t, dot_inv_k) << 32) | (uint32_t)(~index);
}
__host__ __device__ inline float raw_candidate_product(uint64_t c) { return __builtin_bit_cast(float, (uint32_t)(c >> 32)); }
__host__ __device__ inline float candidate_score(uint64_t c) { return ordered_to_score((uint32_t)(c >> 32)); }

// The fp32 score every kernel of the library computes from an fp32 dot product.
// "+ 0.0f" turns -0.0 into +0.0 so that equal scores have equal bit patterns.
__device__ inline float final_score(float dot, float inv_k, float inv_q) { return (dot * inv_k) * inv_q + 0.0f; }

// A removed entry keeps its row and its index but is never a candidate again: kb_remove sets the sign bit of its
// 1/|k| (which is never negative otherwise; a zero row's 0 becomes -0).
constexpr uint32_t REMOVED_BIT = 0x80000000u;
__host__ __device__ inline bool row_removed(float inv_k) { return (as_u32(inv_k) & REMOVED_BIT) != 0; }

// Kernel-side name of f32 rows and queries that go to the matrix cores as two f16 values an element (see Mma<KB_F32_SPLIT>): large calls,
// see split_f32.
constexpr int KB_F32_SPLIT = 4;
// They are scaled by a power of two that brings the row's
// length to [2^7, 2^8]: the largest f16 value is far away, and what is lost below the smallest one is 2^-32 of the length.  The
// scale comes from 1/|x| alone, so every kernel has the same; a row without a length (zero, or past the largest float) is taken as zeros.
//
// These scores only say which rows are scored again by the f32 instruction, and whether those can be all that count (see restated_suffice).
// For that they must be near the f32 ones, which lengths between 2^-48 and 2^62 ensure: no product of two such rows leaves the
// range of floats, and what falls out of it below is nothing beside the length.  A row of another length has a score above all others
// instead, so that it is among those that are scored again; a query of another length is left to the f32 instruction.
__host__ __device__ inline bool f32_ordinary(float inv)
{
    const uint32_t e = as_u32(inv) >> 23 & 255u;
    return e >= 127u - 62u && e <= 127u + 48u;
}
__host__ __device__ inline float f32_row_scale(float inv) { return as_f32(f32_ordinary(inv) ? (as_u32(inv) & 0x7f800000u) + (8u << 23) : 0u); }
// 1/|x| of the scaled row: the same digits, so dot products of scaled rows end in the score of the rows as they are.  (The removed bit stays.)
// The products of a row without scale are all SPLIT_START, which this takes to 2^107.
__host__ __device__ inline float f32_scaled_inv(float inv)
{
    const uint32_t u = as_u32(inv), other = (u & 0x7f800000u) != 0u ? (u & 0x80000000u) | 254u << 23 : u;
    return as_f32(f32_ordinary(inv) ? (u & 0x807fffffu) | 119u << 23 : other);
}
// What their sums begin with: 2^-34 of the product of two scaled lengths, so it is far below the rounding of one product.
constexpr float SPLIT_START = 0x1p-20f;
constexpr int SPLIT_MAX_SPARE = 32;         // entries selected beyond the k wanted (see split_spare)
// The most by which a row's split score and its f32 score differ, lengths as above, u = 2^-24 and in units of the two lengths' product (which
// no partial sum exceeds):
//   the f32 chain: one rounding an element, of at most u each                                               d u
//   the f16 instruction, three for 16 elements: products are exact, adding one loses at most 2 u              6 d u
//     (how it rounds is not documented; measured over random operands of any spread, an instruction loses
//     up to 6.3 u of the magnitudes it adds, where this has 32)
//   the elements: h + l is within 2^-22 of an element, for both rows, and l l is left out                    12 u
//   1/|x| are the same; two roundings in each score; 1/|x| is within d u / 4 of the length                     8 u
// (d u below 2^-9; what is left over is room for the products of these.)
__host__ __device__ inline float split_error(int d) { return (7.5f * (float)d + 64.f) * 0x1p-24f; }
// 1/|x| as the kernels of a key type use it
template <int KT> __device__ inline float used_inv(float inv) { return KT == KB_F32_SPLIT ? f32_scaled_inv(inv) : inv; }

// Kernel-side name of "fp8 keys with fp8 queries" where a kernel template is selected by key type: the keys are
// KB_FP8_E4M3 either way, but both operands go to the fp8 matrix instruction as they are stored.
constexpr int KB_FP8_Q8 = 3;

// Sampling pass whose rows the main pass leaves out: what is known of a group of 32 rows besides its best.  The second best
// row's value as an ordered score | the upper 27 bits, rounded up, of an ordered score that no other row is above | the second's
// place, element e of the lane's 32.  0: the group has one row at most.
__host__ __device__ inline uint64_t pack_second(float value, uint32_t others, uint32_t place)
{
    const uint32_t up = others == 0u ? 0u : others > 0xffffffe0u ? 0x07ffffffu : (others + 31u) >> 5;
    return ((uint64_t)score_to_ordered(value) << 32) | up << 5 | place;
}
// ... the bound on the others (0: there are none; a value between two ordered scores is as good as the upper one)
__host__ __device__ inline uint32_t others_bound(uint64_t second) { return (uint32_t)second & ~31u; }

struct Record {  // one candidate that passed the threshold filter of the scan
    uint64_t cand;
    uint32_t query;
    uint32_t pad;
};

// A query's candidate list is CAND_SEGMENTS segments with a counter each, so that the slot-claiming atomics of one
// query are spread over that many addresses instead of serialising on one.  A candidate's segment comes from its
// row number: a query's candidates spread over all segments even when they sit in a few neighbouring tiles (rows
// grouped by cluster) and were found by a few workgroups; consecutive rows take the segments in turn.
constexpr int CAND_SEGMENTS = 16;
__host__ __device__ inline uint32_t candidate_segment(uint32_t row) { return (row ^ (row >> 4) ^ (row >> 8)) % CAND_SEGMENTS; }
// Diagnostics at the start of the workspace: STAT_WORDS words (candidates, exhaustive queries, sample keys, scan
// workgroups), then the candidate count as STAT_PARTIALS partial sums (one hot address would serialise).
constexpr int STAT_WORDS = 4;
constexpr int STAT_PARTIALS = 64;
// ... and a word that is not shown: whether a query of split f32 rows needs the f32 instruction (see restated_suffice).
constexpr int STAT_GATE = STAT_WORDS + STAT_PARTIALS;
// Records a scan wavefront collects before it moves them to the per-query lists (it also does so when it ends).
constexpr int REGION_CAP = 128;

// Workspace layout (offsets in bytes from a 256-byte aligned base).
struct Plan {
    int32_t Q, k, tq, nqb, qpad;        // queries, tile width in queries, query blocks, padded count
    int32_t config;                     // scan tile configuration id
    int family;                         // which kernel family the configuration belongs to (ConfigInfo::family)
    int32_t tk;                         // keys per tile
    int32_t groups_per_tile;            // sample groups per key tile
    int32_t sample_config, sample_family, sample_wgpc, sample_tk;   // the sampling pass may use another scan configuration (and tile height)
    int64_t sample_tiles;               // key tiles (of the sampling configuration) scored by the sampling pass (0 = none)
    int64_t sample_keys;                // rows they cover
    int32_t sample_slots;               // sample_tiles * groups_per_tile, per query
    int32_t grid;                       // workgroups of the main scan
    int32_t region_cap;                 // records a scan wavefront collects before it moves them to the lists
    int32_t regions;                    // grid * wavefronts per workgroup
    int32_t cand_cap;                   // candidates per query the final sort can take (power of two)
    bool once;                              // the main pass leaves out what the sampling pass scored
    int64_t main_rows;                      // rows of the main pass
    size_t off_samp_more;
    size_t off_fb_done, off_fb_lists;       // exhaustive path: per-query arrival counters, per-(query, part) partial lists
    int32_t fb_parts;                      // parts the rows are split into when a query takes the exhaustive path
    size_t off_invq, off_thr64, off_thrp, off_cnt, off_flag, off_stats, off_qmask, off_samp, off_regions,
        off_cand, off_lgain, total;
};

// The whole-store plan: a small or middling store, or a handful of queries, where the sampling pass, the thresholds
// and the candidate lists cost more than they save.  Two launches: the tiled scan leaves, per query and group of rows
// (the rows of a wave, or of a key tile), the two best products and a bound on all others; one workgroup per query finds the
// k-th best of the groups' best and takes what reaches it, scoring a group again only when a further row of it might.
// A group's entry is four words: the second best product; the third best one or a bound on it; the places of these rows
// in the tile (or the group, see StreamPlan), first | second << 8 | (third + 1) << 16, where 0 means that the third is only a bound; 0.  -inf where there is no row.
//
// What is not named is strictly worse than the second row if the third is a bound.  Where it could not be told from the
// second (equal rows, most of all), the scan names the third as well, the rows taken in the order of the result: by
// product, then by index.  So a group is scored again only if two rows of it are better than the k-th result, which is
// at most k / 2 groups, however many rows are alike.  One thing is left: products a unit or two in the last place apart
// can round to equal scores, and then the lower index wins.  WHOLE_NEAR says that such a row may be among those not named.
constexpr uint32_t WHOLE_NEAR = 1u << 25;
constexpr uint32_t WHOLE_THIRD = 511u;      // ... after the shift: the third's place + 1, of up to 256 rows
constexpr int WHOLE_MAX_GROUPS = 4096;      // a thread of the selecting workgroup (256) keeps 16 of them
// The scan with the queries in LDS (kb_stream.hpp): tiles of `tr` rows, dealt to `waves` wavefronts; a group is `per_group` tiles of one of them.
struct StreamPlan {
    int32_t tr, tq, pieces_in_ring, waves_per_block, blocks, nqb;       // blocks: per query block
    int32_t units, waves, per_group, side_slots, query_stride;
    int32_t lds;
};
struct WholePlan {
    bool stream;                        // the first launch is kb_stream_kernel; tk is the tile's rows, config says nothing
    StreamPlan st;
    int32_t config, tk, tq, nqb, grid;
    int32_t groups, group_rows, fine;
    int32_t k_groups;                   // groups as the rules for k count them
    size_t off_best, off_pair, off_invq, total;      // (off_invq: split f32 rows and the tiled kernel)
};

// The dense plan: a store of some thousand rows.  The tiled scan writes the product (the key, in the weighted selection) of
// every row and query, one workgroup per query selects from its row of them.
constexpr int DENSE_THREADS = 256;
constexpr int64_t DENSE_MAX_ROWS = 16384;   // a thread of the selecting workgroup keeps 64 of them
struct DensePlan {
    bool stream;
    StreamPlan st;
    int32_t config, tk, tq, nqb, grid, stride;      // stride: values per query, a multiple of the tile's rows and of what a load of the selection takes
    size_t off_values, off_invq, off_lgain, off_unused, total;      // (off_invq on: the weighted selection only)
};

// Weighted random selection (Section 3, Optimization Selector: its top-k is a random draw whose weights are the
// entries' predicted gains): entries are ranked by key = score / T + ln(gain) + Gumbel noise instead of by
// score, which draws k entries without replacement with probability proportional to gain * exp(score / T).
struct DrawArgs {
    const float *log_gain;    // [rows padded to a multiple of 256]: ln(gain), -inf for entries that are never drawn
    float inv_t;              // 1 / temperature
    uint32_t seed_lo, seed_hi;
    uint32_t first_query;     // the noise of query row r is that of global query number first_query + r
    int32_t enabled;
};

// Load policy of key rows that are read once, as the last operand of a direct-to-LDS load: non-temporal.
constexpr int LOAD_NT = 2;

struct ScanArgs {
    const void *keys;
    const float *inv_norm;
    const uint64_t *tags;     // nullptr when no filter is applied
    const void *queries;
    const uint64_t *qmask;    // nullptr when no filter is applied
    const uint64_t *qmask_pad; // [qpad] copy of qmask padded with zero words (library workspace)
    const float *invq;        // [qpad] (split f32: q < Q)
    int32_t split;            // f32 rows go to the matrix cores as two f16 values an element
    const uint64_t *gate;     // f32 rows: the launch does nothing where this word is zero; nullptr: it always runs
    const uint64_t *thr64;    // [qpad] candidate words below this cannot be in the result
    const float *thrp;        // [qpad] conservative pre-filter on dot * inv_k
    uint64_t *samp;           // sampling pass output [sample tiles][qpad][groups per tile]: see sample_slot_index
    uint64_t *samp_more;      // ... and the group's second best row with a bound on the others (see pack_second); nullptr: not wanted
    Record *regions;          // [grid * waves per workgroup][region_cap]: one private region per wavefront
    uint64_t *cand;           // [qpad][cand_cap] per-query candidate lists, CAND_SEGMENTS segments each
    uint32_t *cnt;            // [qpad][CAND_SEGMENTS] entries claimed in each segment (zero before the launch)
    uint32_t *flag;           // [qpad] set to 1 when a query lost a candidate to a full list
    uint64_t *stats;          // diagnostics (see STAT_WORDS)
    int64_t n_keys;           // rows to scan: [0, n_keys)
    int64_t n_tiles;          // key tiles to scan: logical tile t is rows [t * tile_stride * TK, +TK)
    int32_t tile_stride;      // 1 for the main pass; a sampling pass takes every tile_stride-th tile ...
    uint64_t row_mul;         // ... or, when nonzero, scatters its rows in runs of 2^row_run_shift (see sample_row)
    int64_t sample_runs;      // runs that the scatter goes over
    double row_inv_runs;      // 1 / sample_runs
    float row_ratio;          // row_mul / sample_runs
    int32_t row_run_shift;
    uint32_t skip_mul;        // the main pass leaves out what the sampling pass scored: see main_row (0: it does not)
    double skip_inv;          // 2^32 / skip_mul
    uint32_t mixed_rows;      // rows whose order is mixed (see mixed)
    int32_t d, Q, nqb, qpad, sample_slots, sample_group_shift, region_cap, cand_cap;
    DrawArgs draw;
    int32_t keys_once;        // the launch reads keys that no cache holds and nobody reads again: see stream_keys
    // Whole-store plan (see WholePlan): the best two of every group of rows, nothing is filtered.  nullptr otherwise.
    float *whole_best;        // [Q][groups]: product of the best row of the group
    u32x4 *whole_pair;        // [Q][groups]: the rest of the group's entry
    int32_t whole_groups, whole_fine;       // fine: a group is the rows of one wave, not of the tile
    float *dense;             // dense plan: [Q][dense_stride] products or keys, -inf in the place of what does not qualify.  nullptr otherwise
    int32_t dense_stride;
};

// Key row behind row r of logical tile `tile` in a sampling pass.  With row_mul the sample is scattered in runs of
// R = 2^row_run_shift rows: run j of the sample is run (j * row_mul) mod (n_keys / R) of the knowledge base (row_mul
// coprime to the number of runs and about 0.618 of it: one to one, consecutive runs far apart).  Every group of
// rows whose maximum the sampling epilogue keeps then mixes rows from all over the knowledge base, so the
// threshold stays tight when the rows are grouped by cluster.  R = 1 for the plain retrieval; the weighted
// selection takes runs of four, which keep what it shares between neighbouring rows (one generator call, one
// 16-byte load of gains).  Without row_mul the tile is tile_stride tiles further on and rows past the end repeat
// the last row.
//
// Where the main pass leaves the sample out (skip_mul, see main_row), the scatter goes over the rows that are left out instead of
// all, and row m of those is sampled_row(m).  (SKIP: kernels that sample for such a main pass, row by row.)
//
// The map is linear, so a workgroup maps the first run of its tile once (sample_tile_run: exact 64-bit arithmetic with
// a quotient estimated in double precision; a 64-bit division would be a software routine of some hundred
// instructions) and every row of the tile from that (sample_row: the product of a run number below 256 with row_mul
// has a quotient below 256, which single precision estimates to within one).
// The division of the store between the two passes: with U rows, S of them sampled and M = U - S left, the main pass's row m (m < M)
// is row m + floor(m a / 2^32) of the store with a = skip_mul = ceil(2^32 S / M): the multiple steps over one row whenever the quotient
// grows, evenly, S times up to M.
// One multiplication a row, and the rows of a tile stay neighbours.  Stores of 2^20 rows would have every sampled row at the same
// place of each 32 KiB, in a few of the memory's channels (sampling pass 55 us, 46 with 1,000,003 rows), so both passes count the
// rows in an order in which each block of 16 is turned by the number of the block.
__device__ inline uint32_t mixed(const ScanArgs &p, uint32_t row) { return row < p.mixed_rows ? row ^ (row >> 4 & 15u) : row; }
__device__ inline uint32_t main_row(const ScanArgs &p, uint32_t row) { return mixed(p, row + __umulhi(row, p.skip_mul)); }
// no row from `row` on is below this (nor in the tile that begins there)
__device__ inline uint32_t main_base(const ScanArgs &p, uint32_t row) { return (row + __umulhi(row, p.skip_mul)) & ~15u; }
// Row j (0 <= j < S) of those stepped over: it follows the first m whose quotient is j + 1.  (The estimate in double precision is
// off by one at most.)
__device__ inline int64_t sampled_row(const ScanArgs &p, int64_t j)
{
    const uint32_t want = (uint32_t)j + 1u;
    const double x = (double)want * p.skip_inv;
    uint32_t m = x > 1.0 ? (uint32_t)x - 1u : 0u;
#pragma unroll
    for (int i = 0; i < 3; ++i) m += __umulhi(m, p.skip_mul) < want ? 1u : 0u;
    return (int64_t)mixed(p, m + (uint32_t)j);
}
__device__ inline int64_t mulmod_runs(const ScanArgs &p, int64_t run)      // (run * row_mul) mod runs, run < runs < 2^31
{
    const int64_t runs = p.sample_runs, prod = run * (int64_t)p.row_mul;
    int64_t r = prod - (int64_t)((double)prod * p.row_inv_runs) * runs;
    r += r < 0 ? runs : 0;
    r -= r >= runs ? runs : 0;
    return r;
}
__device__ inline int64_t sample_tile_run(const ScanArgs &p, int64_t tile, int tk)     // mapped run of the tile's first row
{
    return p.row_mul ? mulmod_runs(p, (tile * tk) >> p.row_run_shift) : 0;
}
template <bool SKIP> __device__ inline int64_t sample_row(const ScanArgs &p, int64_t tile_run, int64_t tile, int tk, int r)     // 0 <= r < tk <= 256
{
    if (p.row_mul) {
        const int sh = p.row_run_shift;
        const int64_t runs = p.sample_runs;
        const uint32_t lr = (uint32_t)r >> sh;                                          // run within the tile
        const uint32_t q = (uint32_t)((float)lr * p.row_ratio);                         // floor(lr * row_mul / runs), or one off
        int64_t m = (int64_t)((uint64_t)lr * p.row_mul) - (int64_t)((uint64_t)q * (uint64_t)runs);
        m += m < 0 ? runs : 0;
        m -= m >= runs ? runs : 0;
        m += tile_run;
        m -= m >= runs ? runs : 0;
        if (SKIP) return sampled_row(p, m);
        return (m << sh) + (r & ((1 << sh) - 1));
    }
    const int64_t row = tile * p.tile_stride * tk + r;
    return row < p.n_keys ? row : p.n_keys - 1;
}
// first row number the sampling epilogues count from: logical when the rows are scattered
__device__ inline int64_t sample_row0(const ScanArgs &p, int64_t tile, int tk) { return p.row_mul ? tile * tk : tile * p.tile_stride * tk; }
// knowledge-base row of tile-local row rl of a sampling pass whose epilogue counts rows from row0 = sample_row0()
template <bool SKIP> __device__ inline uint32_t sample_index(const ScanArgs &p, int64_t tile_run, int64_t row0, int tk, int rl)
{
    return (uint32_t)(p.row_mul ? sample_row<SKIP>(p, tile_run, 0, tk, rl) : row0 + rl);
}

// Knowledge-base row at place `pos` of a tile of the whole-store plan (>= n_keys: none).  The rows of a tile are not
// neighbours: where rows are grouped by cluster, a query's best entries are, and a group of neighbours would hold more
// of them than the two it can name.  The store is cut into runs of R = 2^shift rows; every tile takes one run of each
// `tiles` consecutive ones, and the rows of a run are a quarter (R = 4) of the tile apart.  Which one moves on by one or
// two from place to place, so that the distance between a tile's runs is an odd number of them: at 2048 tiles of 128
// rows a fixed place made it a power of two, and the scan took 120 us where 115 % of the rows took 131 (bf16, d = 1024).
__host__ __device__ constexpr int whole_run_shift(int tk) { return tk >= 64 ? 2 : 0; }
__host__ __device__ inline int64_t whole_row(int32_t tile, int32_t tiles, int tk, int pos)
{
    const int shift = whole_run_shift(tk), per = tk >> shift, j = pos & (per - 1);        // runs in a tile, which of them
    int32_t t = tile + j * (2 - (tiles & 1 ? 0 : 1));
    if (tiles > 2 * 128) t -= t >= tiles ? tiles : 0;        // (j < 128)
    else t %= tiles;
    return (((int64_t)j * tiles + t) << shift) + (shift ? pos / per : 0);
}
// A number below tk that rises with the row at a place.
constexpr int NATURAL_ORDER = 256;      // groups whose rows rise with the places
template <int TK> __host__ __device__ inline uint32_t whole_order(uint32_t place)
{
    if (TK == NATURAL_ORDER) return place;
    constexpr int SHIFT = whole_run_shift(TK);
    return ((place << SHIFT) | (place / (uint32_t)(TK >> SHIFT))) & (uint32_t)(TK - 1);
}

// Where sample `slot` (= tile * groups + group) of query q lives.  The groups of one tile are adjacent (64 bytes per
// query for eight groups) and the queries of a tile follow each other: a sampling wavefront stores words 64 bytes apart
// inside one 16 KiB run instead of 16 KiB apart, and the threshold kernel reads a query's samples 64 bytes at a time.
__host__ __device__ inline size_t sample_slot_index(int64_t slot, int group_shift, int qpad, int q)      // groups = 2^group_shift
{
    return ((((size_t)slot >> group_shift) * qpad + q) << group_shift) + ((size_t)slot & ((1u << group_shift) - 1));
}

// A kernel that uses more than 64 KiB of dynamic LDS must be allowed to, once per device (the attribute belongs to the
// device's copy of the kernel).  `done` holds one bit per device ordinal; callers keep one such word per kernel.
// Two threads that race here both set the attribute, which is harmless.
typedef std::atomic<uint64_t> LdsAllowed;
inline hipError_t allow_dynamic_lds(const void *kernel, LdsAllowed &done, size_t bytes)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (dev >= 0 && dev < 64) ? 1ull << dev : 0ull;       // beyond 64 devices: set it on every call
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
}

// Kernel timing for roofline reports (kb_profile_begin): while `start` is set, the next scan launch of this thread
// carries the two events on its own dispatch packet (hipExtLaunchKernelGGL), so that their difference is the
// kernel's duration and no extra packets sit between it and its neighbours (events recorded around a launch cost
// about 7 us each).
struct ScanTiming {
    hipEvent_t start = nullptr, stop = nullptr;
};
extern thread_local ScanTiming scan_timing;

// Launchers, one translation unit per key dtype.  `sample` selects the sampling epilogue.
hipError_t launch_scan_f32(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_f32_split(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_bf16(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_fp8(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_sp_bf16(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_wide_bf16(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_wide_fp8(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_sp_fp8(int config, bool sample, int grid, const ScanArgs &a, hipStream_t s);
struct StreamArgs;
hipError_t launch_stream_f32(const StreamPlan &p, bool split, bool once, const StreamArgs &a, hipStream_t s);
hipError_t launch_stream_bf16(const StreamPlan &p, bool dense, bool once, const StreamArgs &a, hipStream_t s);
hipError_t launch_stream_fp8(const StreamPlan &p, bool q8, bool dense, bool once, const StreamArgs &a, hipStream_t s);

// Shortest key row (bytes) of the kernel with a software pipeline of 64-byte pieces and rings of ns chunks: see SPCfg::AUX_COPIES.
constexpr int pipelined_min_row_bytes(int ns, bool interleaved) { return 64 * (ns == 3 ? (interleaved ? 2 : 3) : interleaved ? ns : ns + 1); }

// Static description of a scan configuration (host side planning).
struct ConfigInfo {
    int tk, tq, threads, groups_per_tile, wg_per_cu;
    int min_row_bytes;      // smallest key row (bytes) the configuration's pipeline is valid for
    int family;             // 0: kb_scan.hpp, 3: kb_scan_sp.hpp, 4: kb_scan_wide.hpp
};
bool scan_config_info(int key_dtype, int config, ConfigInfo *out);   // false if the id does not exist
int scan_config_for(int key_dtype, int Q, int d, int64_t n);         // automatic choice for n rows

}  // namespace kbi
