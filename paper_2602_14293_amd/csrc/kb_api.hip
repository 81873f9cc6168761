// libkb: C ABI, host-side planning, and the small kernels around the scan (gfx950 only).
//
//   kb_normalize : row_norm_kernel            (row L2 norms as a side scale)
//   kb_query     : scan kernel, sampling pass (kb_scan.hpp)
//                  threshold_kernel           (k-th best group maximum per query; query norms, counters reset; what the sample
//                                              itself adds to the lists where the main pass leaves its rows out)
//                  [prep_kernel               (query norms, counters reset: when no sampling pass runs)]
//                  scan kernel, main pass     (kb_scan.hpp; its wavefronts move their records to per-query lists)
//                  finalize_kernel            (top k of each query's list by radix selection; or the
//                                              exhaustive per-query scan when a list overflowed)
//                  or, smaller stores and batches: a scan that keeps the best of every group or every product
//                  (kb_stream.hpp, kb_scan.hpp), whole_select_kernel or dense_select_kernel
//   kb_append    : append_kernel              (rows, scales and tags; a single copy by the runtime)
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>

#include "kb_configs.hpp"
#include "kb_internal.hpp"
#include "kb_scan.hpp"
#include "kb_norm.hpp"
#include "kb_stream.hpp"

using namespace kbi;


namespace kbi {

thread_local ScanTiming scan_timing;

bool scan_config_info(int key_dtype, int config, ConfigInfo *out)
{
#define X(ID, KT, TK, TQ, WM, WN, RBA, NSTAGE, WGPC)                          \
    if (key_dtype == KT && config == ID) {                                    \
        *out = ConfigInfo{TK, TQ, 64 * WM * WN, WM * 2, WGPC, RBA, 0};    \
        return true;                                                          \
    }
    KB_SCAN_CONFIGS_BF16(X)
    KB_SCAN_CONFIGS_F32(X)
    KB_SCAN_CONFIGS_FP8(X)
    KB_SCAN_WHOLE_CONFIGS_BF16(X)
    KB_SCAN_WHOLE_CONFIGS_FP8(X)
#undef X
    if (key_dtype == KB_F32 && config == SMALL_F32_CONFIG) {
        *out = ConfigInfo{16, 32, 64, 2, 4, 128, 0};
        return true;
    }
#define X(ID, KT, TK, TQ, WM, WN, RBA, NSTAGE, WGPC)                          \
    if (key_dtype == KB_FP8_E4M3 && config == ID) {                           \
        *out = ConfigInfo{TK, TQ, 64 * WM * WN, WM * 2, WGPC, RBA, 0};    \
        return true;                                                          \
    }
    KB_SCAN_CONFIGS_FP8_Q8(X)
    KB_SCAN_DENSE_CONFIGS_FP8_Q8(X)
#undef X
#define XS(ID, KT, TQ, NSA, NSB)                                              \
    if (key_dtype == KT && config == ID) {                                    \
        *out = ConfigInfo{256, TQ, 512, 8, 1, pipelined_min_row_bytes(NSA > NSB ? NSA : NSB, INTERLEAVED), 3}; \
        return true;                                                          \
    }
    {
        constexpr bool INTERLEAVED = true;
        KB_SCAN_SP_CONFIGS_BF16_IL(XS)
        KB_SCAN_SP_CONFIGS_FP8_Q8(XS)
    }
    {
        constexpr bool INTERLEAVED = false;
        KB_SCAN_SP_CONFIGS_FP8(XS)
    }
#undef XS
#define XW(ID, KT, TQ)                                                        \
    if (key_dtype == KT && config == ID) {                                    \
        *out = ConfigInfo{256, TQ, 512, 8, 1, 512, 4};                        \
        return true;                                                          \
    }
    KB_SCAN_WIDE_CONFIGS_BF16(XW)
    KB_SCAN_WIDE_CONFIGS_FP8_Q8(XW)
#undef XW
#define XW(ID, KT, TQ)                                                        \
    if (key_dtype == KT && config == ID) {                                    \
        *out = ConfigInfo{256, TQ, 512, 8, 1, 256, 4};                        \
        return true;                                                          \
    }
    KB_SCAN_WIDE_CONFIGS_FP8(XW)
#undef XW
    return false;
}

constexpr int F32_SQUARE_CONFIG = 26;  // f32 rows: tiles of 64 x 64
constexpr int FP8_WIDE_CONFIG = 22;    // fp8 keys with bf16 queries: the full-line kernel (rows of a multiple of 128 bytes, 256 at least)
constexpr int64_t WIDE128_MIN_ROWS = 4 * 65536;     // rows from which the 128-query full-line kernel is the faster one (measured: 2^18)

// What a plan gives up for less memory, step by step: a call whose workspace is too small for the fastest plan is served by the
// first that fits.
enum Thrift {
    AMPLE,              // nothing
    SCORED_TWICE,       // the main pass scores the sampled rows again: no second word per sampled group, no sample in whole rounds
    LEAST               // ... and the tiled kernel (f32: its 128-row tiles) where another is faster on rows too short for deep rings
};

// Rows too short for rings of four: the pipelined kernel's tiles of 256 rows pay once there are enough of them for the compute units.  Time of
// the tiled kernel's call over that of the pipelined one's: fp8 keys of 192 elements with bf16 queries, 24,134 rows 0.75, 18,106 rows and 945
// queries 0.88, 33,063 rows 1.00, 39,161 1.15; with fp8 queries 107 items (27,424 rows of 128, 256 queries) 0.96, 130 items 1.2 to 1.3
constexpr int64_t SHORT_ROWS_MIN_ROWS = 32768, SHORT_ROWS_MIN_ITEMS = 112;

int scan_config_for(int key_dtype, int Q, int d, int64_t n, Thrift thrift)
{
    const bool least = thrift == LEAST;
    if (key_dtype == KB_BF16 && Q > 128 && d * 2 >= 512) return 18;
    // 33 to 128 queries: the full-line kernel once a workgroup has several tiles to stream (its ring takes longer to fill)
    if (key_dtype == KB_BF16 && Q > 32 && d * 2 >= 512 && n >= WIDE128_MIN_ROWS) return 19;
    if (key_dtype == KB_BF16 && Q > 128 && d * 2 >= 384) return 17;      // (rows of 256 bytes: see kb_configs.hpp)
    if (key_dtype == KB_FP8_E4M3 && Q > 128 && d >= (least || n < SHORT_ROWS_MIN_ROWS ? 256 : 192)) return d >= 256 && d % 128 == 0 ? FP8_WIDE_CONFIG : 4;
    // below that size a query is bound by the latency of its launches: tiles of 64 rows (twice the workgroups, half the
    // chunks each) finish sooner: 62 against 71 us per call on 65,536 rows of 768 bf16 values with 64 queries
    // (and 64 against 70 us with 128 queries)
    if (key_dtype == KB_BF16 && Q > 32 && Q <= 128 && n < WIDE128_MIN_ROWS) return Q <= 64 ? 12 : 16;
    if (key_dtype == KB_F32 && Q > 32 && Q <= 64 && !least) return F32_SQUARE_CONFIG;
    return Q <= 32 ? 1 : Q <= 128 ? 2 : 3;
}

}  // namespace kbi

namespace {

constexpr int DEVICE_CUS = 256;        // compute units of an MI355X: the scan grids are sized for them (a device with fewer runs the same grid in turns)
constexpr int MAX_REGION_CAP = 8192;   // records a scan wavefront collects at most before it moves them to the lists
constexpr int MAX_SAMPLE_SLOTS = 8192; // threshold_kernel sorts this many 64-bit words in LDS (64 KiB)
constexpr int MAX_CAND_CAP = 8192;     // finalize_kernel likewise
constexpr int MIN_CAND_CAP = 1024;
constexpr int FALLBACK_PARTS = 32;    // workgroups that share the rows of a query on the exhaustive path
constexpr size_t WS_ALIGN = 256;
constexpr int FP8_QUERY_CONFIG = 5;    // scan configuration of fp8 keys with fp8 queries (kb_configs.hpp)
constexpr int FP8_QUERY_SHORT_CONFIG = 27;    // ... rows of 128 and 192 bytes
constexpr int FP8_QUERY_WIDE_CONFIG = 20;     // ... with 128-byte row pieces: rows of a multiple of 128 bytes, 512 at least
constexpr int FP8_QUERY_TILED_CONFIG = 6;     // ... the tiled kernel: 6, 7, 8 for query blocks of 64, 128, 256; every row length
constexpr int FP8_STREAM_CONFIG = 23;         // fp8 keys with bf16 queries: the tiled kernel with whole lines, up to 32 queries
constexpr int FP8_QUERY_STREAM_CONFIG = 24;   // ... the tiled kernel with whole lines, up to 32 queries
constexpr int FP8_QUERY_SMALL_CONFIG = 25;    // ... with tiles of 32 x 32, the dense plan
bool is_fp8_query_config(int config)
{
    return config == FP8_QUERY_CONFIG || config == FP8_QUERY_SHORT_CONFIG || config == FP8_QUERY_STREAM_CONFIG || config == FP8_QUERY_WIDE_CONFIG || (config >= FP8_QUERY_TILED_CONFIG && config <= FP8_QUERY_TILED_CONFIG + 2);
}

bool is_whole_config(int config) { return (config >= 13 && config <= 15) || config == 21 || config == FP8_QUERY_SMALL_CONFIG; }      // no pipeline with a sampling pass runs them

int key_bytes(kb_dtype_t t) { return t == KB_F32 ? 4 : t == KB_BF16 ? 2 : 1; }
int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t pow2_ceil(int64_t x)
{
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}
size_t align_up(size_t x) { return (x + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN; }

// Multiplier of the sampling pass's scatter j -> (j * m) mod n over the n runs of rows: about n / golden ratio, so
// that consecutive j land far apart and fill the range evenly, and coprime to n, so that the map is one to one.
// 0 (no scatter) when there are too few runs.
uint64_t scatter_multiplier(int64_t n)
{
    if (n < 3) return 0;
    uint64_t m = (uint64_t)((double)n * 0.6180339887498949) | 1u;
    for (;; m += 2) {
        uint64_t a = m, b = (uint64_t)n;
        while (b) {
            const uint64_t t = a % b;
            a = b;
            b = t;
        }
        if (a == 1) return m % (uint64_t)n;
    }
}

// Whether a scan's key loads carry the non-temporal policy: the store does not fit the Infinity Cache (256 MiB), so the next
// call will find too little of it there, and no second query block of this launch reads the rows again.  A stream that leaves
// the caches alone is the faster one: 1,000,003 x 1024 bf16 rows and one query 358 -> 321 us, 2^20 rows and 128 queries 425 ->
// 396, 256 queries 588 -> 570.  With a store that fits and is asked again it loses (100 MB and 64 queries 28.1 -> 29.2 us),
// with two query blocks too (2,500,001 x 512 fp8 rows, 500 queries: 684 -> 708 us), and with half lines by a tenth.
// Where the line lies, against cached loads, on one store asked again and again | on three in turn (bf16, 1024 elements):
//   20 queries   260 MiB 1.06 | 0.91    288 MiB 1.00 | 0.93    320 MiB 0.91 | 0.92
//   256 queries  260 MiB 1.07 | 0.98    288 MiB 1.00 | 0.98    320 MiB 0.99 | 0.97    (100, rows of 512: 1.07, 1.05, 1.00 | 1.00, 0.98, 0.98)
// fp8 rows and few queries, where whole lines come with it: 0.96 | 0.82 at 260 MiB already.
bool stream_keys(const kb *h, int64_t n, int32_t Q, int nqb)
{
    const int64_t limit = (int64_t)(Q > 32 ? 320 : h->dtype == KB_FP8_E4M3 ? 256 : 288) << 20;
    return nqb == 1 && n * h->d * key_bytes(h->dtype) > limit;
}

// ------------------------------------------------------------------------------------------------
// Planning: which kernels a query runs, how large its buffers are, where they live in the workspace.
// ------------------------------------------------------------------------------------------------
struct Choice {                 // kernels of a query over n rows
    int config;
    ConfigInfo ci;
    int sample_config;          // the sampling pass may run another configuration (same tile, bit-identical scores)
    ConfigInfo sci;
};

bool choose_kernels(const kb *h, int64_t n, int32_t Q, bool draw, bool q8, Thrift thrift, Choice *out)
{
    Choice c;
    const int generic = Q <= 32 ? 1 : Q <= 128 ? 2 : 3;        // the tiled kernel: every dtype, every row length
    const size_t row_bytes = (size_t)h->d * key_bytes(h->dtype);
    // fp8 rows beyond the caches, few queries: the tiled kernel with 128-byte row pieces (the others take 64 bytes, half a
    // cache line, of an fp8 row at a time).  1,000,000 x 512 rows: one query 119.5 -> 100.9 us, 20 queries 121 -> 108.6
    const bool whole_line_rows = row_bytes % 128 == 0;
    if (q8) {       // fp8 queries: only the kernels built on the fp8 matrix instruction take them
        if (h->dtype != KB_FP8_E4M3) return false;
        const int generic8 = Q <= 64 ? FP8_QUERY_TILED_CONFIG : Q <= 128 ? FP8_QUERY_TILED_CONFIG + 1 : FP8_QUERY_TILED_CONFIG + 2;
        // large batches: the pipelined kernels (256-query blocks); smaller ones would pad their query columns there
        const bool few_items = row_bytes < 256 && ceil_div(n, 256) * ceil_div(Q, 256) < SHORT_ROWS_MIN_ITEMS;
        c.config = Q <= 128 || few_items || (thrift == LEAST && row_bytes < 384) ? generic8 : (row_bytes % 128 == 0 && row_bytes >= 512) ? FP8_QUERY_WIDE_CONFIG
                                  : row_bytes >= 256 ? FP8_QUERY_CONFIG : FP8_QUERY_SHORT_CONFIG;
        if (Q <= 32 && whole_line_rows && stream_keys(h, n, Q, 1)) c.config = FP8_QUERY_STREAM_CONFIG;
        if (is_fp8_query_config((int)h->tune_config)) c.config = (int)h->tune_config;         // another one can be asked for
        if (!scan_config_info(h->dtype, c.config, &c.ci)) return false;
        // the weighted random selection exists in the tiled kernel only, and rows may be too short for a pipelined kernel
        if ((draw && c.ci.family != 0) || row_bytes < (size_t)c.ci.min_row_bytes ||
            (!whole_line_rows && (c.config == FP8_QUERY_STREAM_CONFIG || c.config == FP8_QUERY_WIDE_CONFIG))) {
            c.config = generic8;
            if (!scan_config_info(h->dtype, c.config, &c.ci)) return false;
        }
    } else {
        c.config = h->tune_config > 0 ? (int)h->tune_config : scan_config_for(h->dtype, Q, h->d, n, thrift);
        if (h->tune_config == 0 && h->dtype == KB_FP8_E4M3 && Q <= 32 && whole_line_rows && stream_keys(h, n, Q, 1)) c.config = FP8_STREAM_CONFIG;
        if (!scan_config_info(h->dtype, c.config, &c.ci)) return false;
        // fall back where a (forced) configuration does not apply: the weighted random selection exists in the
        // tiled kernel and in the main pass of the bf16 full-line kernel, rows may be too short for a pipelined kernel,
        // and the fp8-query kernels read fp8 queries
        const bool draws = c.ci.family == 0 || (c.ci.family == 4 && h->dtype == KB_BF16);
        if ((draw && !draws) || row_bytes < (size_t)c.ci.min_row_bytes || (!whole_line_rows && (c.config == FP8_STREAM_CONFIG || c.config == FP8_WIDE_CONFIG)) || (h->dtype == KB_FP8_E4M3 && is_fp8_query_config(c.config))) {
            c.config = generic;
            if (!scan_config_info(h->dtype, c.config, &c.ci)) return false;
        }
    }
    c.sci = c.ci;
    c.sample_config = c.config;
    if (q8 && c.ci.family == 4) {       // with fp8 queries the full-line kernel is a main pass only
        c.sample_config = FP8_QUERY_CONFIG;
        if (!scan_config_info(h->dtype, c.sample_config, &c.sci) || c.sci.tq != c.ci.tq || c.sci.tk != c.ci.tk) return false;
    }
    if (draw && c.ci.family == 4) {     // the full-line kernel on keys is a main pass only: the tiled kernel with the same query blocks samples
        c.sample_config = c.ci.tq == 128 ? 2 : 3;
        if (!scan_config_info(h->dtype, c.sample_config, &c.sci) || c.sci.tq != c.ci.tq || c.sci.family != 0) return false;
    }
    *out = c;
    return true;
}

// Key tiles the sampling pass scores when the knowledge base has nt tiles: max(k, 8) / 512 of them (1/64 of the
// rows up to k = 8, 1/16 at k = 32, 1/4 at k = 128), at least two samples per wanted result, at most what the
// threshold kernel sorts and half of the tiles.  A sampling pass of few tiles is bound by the latency of one tile, not
// by its bytes: as long as the sample stays small (FREE_SAMPLE_BYTES of keys, a quarter of the tiles) it takes as many
// tiles as the device runs side by side, which costs no time and thins the candidates of the main pass.
// 0 = no sampling pass (every entry is a candidate).  Depends on the row count through nt only, and never falls as
// nt grows (`floor` switched off).
constexpr int64_t FREE_SAMPLE_BYTES = 32 << 20;
int64_t sample_tiles_for(const kb *h, const ConfigInfo &sci, int64_t nt, int32_t Q, int32_t k, bool whole_rounds, bool floor)
{
    if (nt < 8) return 0;
    const int64_t kk = k > 8 ? k : 8;
    int64_t st = h->tune_sample_keys > 0 ? ceil_div(h->tune_sample_keys, sci.tk) : ceil_div(nt * kk, 512);
    const int64_t want = ceil_div(2 * (int64_t)k, sci.groups_per_tile);
    if (st < want) st = want;
    if (h->tune_sample_keys <= 0) {
        const int64_t nqb = ceil_div(Q, sci.tq);
        int64_t free_tiles = (int64_t)DEVICE_CUS * sci.wg_per_cu / nqb;
        const int64_t by_bytes = FREE_SAMPLE_BYTES / ((int64_t)sci.tk * h->d * key_bytes(h->dtype));
        if (free_tiles > by_bytes) free_tiles = by_bytes;
        if (free_tiles > nt / 4) free_tiles = nt / 4;
        if (st < free_tiles) st = free_tiles;
        // a sample that the main pass leaves out costs nothing as long as both are whole rounds of the compute units (down by a
        // quarter at most, with samples enough for k, and not where a round is more than a quarter of the store; the quotient drops the
        // part of a tile, which of few tiles is much, and with more than 256 query blocks may be all of them)
        if (whole_rounds) {
            const int64_t rounded = ceil_div(3 * st * nqb, 4 * DEVICE_CUS) * DEVICE_CUS / nqb;
            const bool down = floor && 4 * rounded >= 3 * st - st / 16 && rounded * sci.groups_per_tile >= k;
            if (rounded > st ? rounded <= nt / 4 || !floor : down) st = rounded;
        }
    }
    if (st > MAX_SAMPLE_SLOTS / sci.groups_per_tile) st = MAX_SAMPLE_SLOTS / sci.groups_per_tile;
    if (st > nt / 2) st = nt / 2;
    if (floor && st * sci.groups_per_tile < k) st = 0;
    return st;
}

// Kernels whose main pass can leave the sampled rows out (their sample is then whole rounds of the compute units).  Not the weighted
// selection, whose sample goes in runs of four neighbours: where a query's best rows are some thousand neighbours every run of theirs makes a
// group to score again (600,000 x 768 rows in runs of 1000 similar ones, 100 queries, k = 100: 394 us a call, 537 with the rows left out, 117 of
// them in the threshold kernel; rows in no order 451 and 408; 2^20 x 1024 rows, 256 queries, k = 32 738 and 715).
bool leaves_sample_out(const Choice &c) { return c.ci.family == 4 && c.sci.family == 4; }

int32_t cand_cap_for(int64_t expect, bool sampled)
{
    int64_t cc = pow2_ceil(sampled ? 8 * expect : expect);
    if (cc < MIN_CAND_CAP) cc = MIN_CAND_CAP;
    if (cc > MAX_CAND_CAP) cc = MAX_CAND_CAP;
    return (int32_t)cc;
}

// Sizes of the workspace arrays.  The layout is a function of these alone and its total grows with each of them.
struct Sizes {
    int32_t k, qpad, regions, sample_slots, more_slots, cand_cap;
    int64_t region_records;     // scan wavefronts * region_cap
    int64_t lgain_rows;
};

void lay_out(const Sizes &z, Plan *p)
{
    size_t off = 0;
    p->off_stats = off;       off = align_up(off + sizeof(uint64_t) * (STAT_WORDS + STAT_PARTIALS));   // always first: kb_query_counters reads it
    p->off_invq = off;        off = align_up(off + sizeof(float) * z.qpad);
    p->off_thr64 = off;       off = align_up(off + sizeof(uint64_t) * z.qpad);
    p->off_thrp = off;        off = align_up(off + sizeof(float) * z.qpad);
    p->off_cnt = off;         off = align_up(off + sizeof(uint32_t) * z.qpad * CAND_SEGMENTS);
    p->off_flag = off;        off = align_up(off + sizeof(uint32_t) * z.qpad);
    p->fb_parts = z.cand_cap / KB_K_MAX < FALLBACK_PARTS ? z.cand_cap / KB_K_MAX : FALLBACK_PARTS;     // parts * k words fit the LDS buffer
    p->off_fb_done = off;     off = align_up(off + sizeof(uint32_t) * z.qpad);
    p->off_fb_lists = off;    off = align_up(off + sizeof(uint64_t) * (size_t)z.qpad * p->fb_parts * z.k);
    p->off_qmask = off;       off = align_up(off + sizeof(uint64_t) * z.qpad);
    p->off_samp = off;        off = align_up(off + sizeof(uint64_t) * (size_t)z.qpad * (z.sample_slots > 0 ? z.sample_slots : 1));
    p->off_samp_more = off;   off = align_up(off + sizeof(uint64_t) * (size_t)z.qpad * z.more_slots);
    p->off_regions = off;     off = align_up(off + sizeof(Record) * (size_t)z.region_records);
    p->off_cand = off;        off = align_up(off + sizeof(uint64_t) * (size_t)z.qpad * z.cand_cap);
    p->off_lgain = off;       off = align_up(off + sizeof(float) * (size_t)z.lgain_rows);   // ln(gain), padded past the last tile
    p->total = off;
}

double cubed(int32_t k) { return (double)k * k * k; }

// The plan of a query over n rows with the kernels `c`.  Apart from the ln(gain) array it depends on n through the
// number of key tiles only, which is what lets kb_query_workspace_bytes bound it over all row counts.
void plan_for(const kb *h, const Choice &c, int64_t n, int32_t Q, int32_t k, bool draw, Thrift thrift, Plan *out, Sizes *sizes)
{
    Plan p;
    memset(&p, 0, sizeof p);
    const ConfigInfo &ci = c.ci, &sci = c.sci;
    p.Q = Q;
    p.k = k;
    p.config = c.config;
    p.family = ci.family;
    p.tk = ci.tk;
    p.tq = ci.tq;
    p.groups_per_tile = ci.groups_per_tile;
    p.nqb = (int32_t)ceil_div(Q, ci.tq);
    p.qpad = p.nqb * ci.tq;
    p.sample_config = c.sample_config;
    p.sample_family = sci.family;
    p.sample_wgpc = sci.wg_per_cu;
    if (n < 1) n = 1;
    const int64_t nt = ceil_div(n, ci.tk), nts = ceil_div(n, sci.tk);     // key tiles of the main pass, of the sampling pass

    // Where the full-line kernel runs the main pass, that pass can leave the sampled rows out: see main_row.  (Not where the sample is
    // whole tiles: the full-line kernel addresses scattered rows in 32 bits, in units of 16 bytes, up to 64 GiB of keys.)  What it
    // takes costs a call 3 to 10 us, a 50th of the main pass at most; what it gives is whole rounds of the compute units.  Time of the
    // call with the sampled rows scored twice over this one's, 166 random calls of 17,000 to 1,300,000 rows and 33 to 1200 queries:
    //   no round saved                       0.83 to 0.98    (97,373 x 256 bf16 rows, 256 queries, 381 items or 286: 52.5 us, 59.9)
    //   one of 25 rounds and more            0.97 to 1.01
    //   rows of 256 elements (128 queries    0.96 to 1.05    (321,757 rows, 742 queries, 15 rounds or 13: 218 us, 223)
    //   a block: of 512)
    //   else                                 0.99 to 1.15
    // And k must be small for the groups, or most of them are scored again (k^3 = 31 groups^2: 85 us, 135).
    // A handle that asks for a configuration gets it with all that belongs to it.
    const int64_t plain_st = sample_tiles_for(h, sci, nts, Q, k, false, true);
    int64_t st = sample_tiles_for(h, sci, nts, Q, k, leaves_sample_out(c), true);
    bool leaves_out = leaves_sample_out(c) && thrift == AMPLE;
    if (leaves_out && !h->tune_config) {
        const int64_t round = (int64_t)DEVICE_CUS * ci.wg_per_cu, rounds = ceil_div(nt * p.nqb, round), groups = st * sci.groups_per_tile;
        const int64_t saved = rounds - ceil_div(ceil_div(n - st * sci.tk, ci.tk) * p.nqb, round);
        leaves_out = saved > 0 && 24 * saved >= rounds && h->d * ci.tq >= 384 * 256 && cubed(k) <= (double)groups * groups;
    }
    if (leaves_out) leaves_out = st > 0 && 2 * st * sci.tk < n && (uint64_t)n * h->d * key_bytes(h->dtype) < ((uint64_t)1 << 36);
    if (!leaves_out) st = plain_st;
    p.sample_tk = sci.tk;
    p.sample_tiles = st;
    p.sample_slots = (int32_t)(st * sci.groups_per_tile);
    p.sample_keys = st * sci.tk;
    p.once = leaves_out;
    p.main_rows = p.once ? n - p.sample_keys : n;
    // candidates per query.  (Where k is small the k-th best of the sample scatters widely, and lists that were large enough for the sample
    // before it was rounded down run over now and then: 1,284,972 x 256 rows, 850 queries, k = 2, a query in 1000, 6.2 ms for a call of 0.6.)
    const int64_t expect = st > 0 ? ceil_div((int64_t)k * nts, k < 4 ? st : plain_st) : nt * ci.tk;
    p.cand_cap = cand_cap_for(expect, st > 0);

    const int wgpc = h->tune_wg_per_cu > 0 ? (int)h->tune_wg_per_cu : ci.wg_per_cu;
    const int64_t items = nt * p.nqb, main_items = ceil_div(p.main_rows, ci.tk) * p.nqb;
    const int64_t grid = items < (int64_t)DEVICE_CUS * wgpc ? items : (int64_t)DEVICE_CUS * wgpc;
    p.grid = (int32_t)(main_items < grid ? main_items : grid);
    const int waves = ci.threads / 64;
    p.regions = (int32_t)(grid * waves);
    // Records a scan wavefront collects before it moves them to the per-query lists.  With a sampling pass few pairs
    // pass the filter (a wavefront sees some tens in a whole scan).  Without one every scored pair is a record: room
    // for the pairs of the wavefront's part of its workgroup's items, within limits.
    int64_t rc = REGION_CAP;
    if (st == 0) {
        rc = pow2_ceil(ceil_div(items, grid) * ci.tk * ci.tq / waves);
        if (rc < REGION_CAP) rc = REGION_CAP;
        if (rc > MAX_REGION_CAP) rc = MAX_REGION_CAP;
    }
    p.region_cap = (int32_t)rc;

    Sizes z;
    z.k = k;
    z.qpad = p.qpad;
    z.regions = p.regions;
    z.sample_slots = p.sample_slots;
    z.more_slots = leaves_out ? p.sample_slots : 0;
    z.cand_cap = p.cand_cap;
    z.region_records = (int64_t)p.regions * rc;
    z.lgain_rows = draw ? ceil_div(n, 256) * 256 + 256 : 0;      // the weighted random selection only
    lay_out(z, &p);
    *out = p;
    if (sizes) *sizes = z;
}

// The whole-store plan, where it applies (the knobs ask for a particular scan pipeline).  It saves the latency of a
// sampling pass, a threshold kernel and the candidate lists, 10 to 20 us per call, and pays for it in the scan's epilogue,
// which keeps the best three of every group where the pipeline's only tests a bound: about 1.3 us per tile and
// workgroup.  Measured against the pipeline on stores of 256 and 1024 elements a row, masked and not: up to three tiles
// for every resident workgroup 1.05 to 1.8 times as fast, with up to 32 queries still 1.0 to 1.3 times at five, with more
// 0.9 to 1.05 times at four; at ten it loses (0.85 to 1.05).
// With the queries in LDS (kb_stream.hpp) a tile costs less, and rows dealt one by one leave no group to score again where similar rows are
// neighbours: up to sixteen tiles a wavefront, for up to 64 queries (those past 32: two_blocks_stream).  Time of the pipeline over this plan's (runs of 1, 4, 16, 64 and 1000 similar rows, k 4 to 96):
//   400,000 x 256 bf16, 8 queries      1.26 to 1.47 (58 us, 44)      400,000 x 1024, 1 query     1.11 to 1.29 (151 us, 135)
//   700,000 x 512 bf16, 20 queries     1.10 to 1.39 (138 us, 122)    1,000,003 x 1024, 1 query   1.04 to 1.22 (332 us, 317)
//   1,000,003 x 256 bf16, 32 queries   1.11 to 1.38 (108 us, 95)     900,000 x 512 fp8, 8        1.10 to 1.35 (100 us, 90)
//   700,000 x 320 fp8 x 8, 20 queries  1.21 to 1.86 (60 us, 49)     320,000 x 128 bf16, 64         1.33 to 2.10 (47 us, 34)
//   1,000,003 x 256 bf16, 40 queries   1.16 to 1.50 (115 us, 99)    700,000 x 512 fp8, 48          1.45 to 1.62 (133 us, 91)
// (4096 groups of 256 rows hold one row more.  That store, the size of the large shared ones here, keeps the plan with a sampling pass that callers of
// kb_query_plan know for it: 1.02 to 1.2 times as long, bf16 x 1024 and 1 query 334 us, 315 with this plan.)
constexpr int64_t WHOLE_MAX_ROWS_STREAM = (1 << 20) - 1;
constexpr int64_t WHOLE_MAX_ROWS_FEW = 5 * 128 * 2 * DEVICE_CUS, WHOLE_MAX_ROWS = 3 * 128 * 2 * DEVICE_CUS;     // up to 32 queries; up to 128
// More than 128 queries: every product costs the epilogue the same, while the pipeline's scan gets better with larger query
// blocks and pays 30 us of latencies once.  Time of the pipeline over this plan's, k = 16, rows of 256 | 768 elements:
//            just inside                                            outside
//   bf16     65,536 x 256: 1.37 | 1.28    16,000 x 1024: 1.23 | 1.18    65,536 x 400: 0.96 | 0.89    131,072 x 160: 0.96 | 0.97
//   fp8      65,536 x 512: 1.43 | 1.33    32,000 x 1024: 1.33 | 1.27    131,072 x 400: 0.99 | 0.99
//   fp8 x 8  65,536 x 512: 1.84 | 1.16    131,072 x 256: 1.73 | 1.23    65,536 x 1024: 1.71 | 0.89   (rows of 256: no pipelined kernel)
//   f32      65,536 x 1024: 1.14 | 1.16   131,072 x 512: 1.14 | 1.06    131,072 x 1024: 1.02 | 1.05
constexpr int WHOLE_MAX_QUERIES = 4096;
// Those are calls whose last block of 128 queries is full; bf16 rows pay for the padding (130,055 x 1024 rows, 129 queries: 0.87), so
// that it counts.  Where the kernel of the pipeline has the matrix cores' rate and this one has not, long rows lose as well: bf16 | fp8 x 8
//   2^24 products  2048: 1.09 to 1.12 | 1.53    4096: 0.95 to 1.04 | 1.13    8192: 0.88 to 0.90 | 0.95
//   2^25 products  1024:      -       | 1.18    2048:      -       | 0.97    4096:      -       | 0.86 to 0.98
//   10,000,000     2048: 1.27         | 1.46    4096: 1.01         | 1.09    8192: 0.88         | 0.97
//   2^23 products  8192: 1.16 to 1.52 | 1.47   16384: 1.12         | 1.34
// (fp8 rows with bf16 queries 1.10 and more at 2^25 products of up to 16,384 elements, f32 1.03 and more)
int64_t whole_max_rows(const kb *h, int32_t Q, bool q8)
{
    if (Q <= 64) return WHOLE_MAX_ROWS_STREAM;
    if (Q <= 128) return WHOLE_MAX_ROWS;
    const int64_t columns = h->dtype == KB_BF16 ? ceil_div(Q, 128) * 128 : Q;
    int64_t pairs = (int64_t)1 << (h->dtype == KB_BF16 ? 24 : h->dtype == KB_F32 ? 26 : 25);
    if (h->dtype == KB_BF16 || q8) pairs = std::min(pairs, std::max((int64_t)1 << 23, ((int64_t)1 << 35) / h->d));
    return std::min(WHOLE_MAX_ROWS, pairs / columns);
}
constexpr int64_t WHOLE_SMALL_TILE_ROWS = 128 * DEVICE_CUS / 2;      // up to 32 queries: tiles of 16 or 32 rows up to here
// Calls on f32 rows whose scan takes two f16 values an element (Mma<KB_F32_SPLIT>).  They select a few entries more than k by the split
// products; the launch that selects scores these again by the f32 instruction's chain (restate) and knows from the bound on the difference
// (split_error) whether another row could belong to the best k.  Where it could, it scores all rows again that are near enough, up to some 200.  Where
// they are more, for any query, two more launches do the call's scan and selection with the f32 instruction: they are always there and
// leave at once otherwise.  So results don't depend on the path.  us a call, f32 instruction | split, half of the queries near rows that are copies of one:
//   300,007 x 384, Q 20, k 10    no copies 98 | 93    30 102 | 105    100 99 | 120    1000 105 | 207     60,000 x 768, Q 128, k 16    120 | 90   115 | 98   115 | 114   135 | 244
//   600,000 x 128, Q 20, k 32    91 | 72    92 | 72    92 | 91    99 | 166    150,000 2256 | 265         400,000 x 512, Q 200, k 32    932 | 473   930 | 467   932 | 486   923 | 1316
// That takes a call some 8 us with few queries (the rows of the selected entries in LDS at once; more with k) and 10 to 15 with many, so it is for
// calls whose scan is long enough.  us a call, f32 instruction | split:
//   up to 32 queries (kb_stream.hpp, eight wavefronts)     300,007 x 384, Q 20  97.8 | 93.3    200,000 x 768, Q 16  126 | 119     300,000 x 768, Q 18  181 | 166
//     past the rows that the tiled kernel's whole-store plan takes   450,000 x 128, Q 32  75.5 | 64.8    600,000 x 128, Q 16  85.3 | 70.7     1,000,000 x 256, Q 32  208 | 176
//     under the limits   250,000 x 256  62.4 | 65.4   150,000 x 512  63.3 | 65.7   120,000 x 768  77.2 | 79.1   250,000 x 384, k 30  82.0 | 84.3   300,000 x 1024, all rows on the same few channels  231 | 243
//   up to 64 (tiled kernel, 64 x 64)    400,000 x 512  273 | 260    1,000,000 x 256, Q 48  343 | 324    600,000 x 1024  769 | 724     under the limit  70,000 x 1024  107 | 109    300,000 x 256, k 30  131 | 138
//   more     60,000 x 768, Q 128   118 | 98.8     179,009 x 576, Q 115  248 | 177     150,000 x 256, Q 500  414 | 248     400,000 x 512, Q 200, k 128  1105 | 594
//     rows of all selected entries past 400 KB, few keys    20,000 x 1024, Q 300, k 128  395 | 417    30,000 x 1024, Q 512, k 128  410 | 454    50,000 x 768, Q 100, k 128  173 | 171    60,000 x 1024, Q 300, k 128  639 | 589
// (The instances of 128 x 256 tiles keep 9 and 4 registers in scratch memory.  With 128 x 128 tiles, which keep none, 150,000 x 256 and 500 queries take
// 260 us, not 240, 400,000 x 512 and 200 702, not 567.)
constexpr int RESTATE_LDS = 96 * 1024;
constexpr int64_t SPLIT_MIN_MULTIPLICATIONS = (int64_t)1 << 32;
// Entries that are selected beyond k.  The scores of rows in no order have a deviation of 1 / sqrt(d), and near the k-th best, some five
// deviations up, the number of rows falls by a factor e every fifth of one: about 5 k sqrt(d) split_error(d) rows are too close to the k-th.  Four
// times the root of that and three beyond it are not enough for a query in some ten thousand.  More than SPLIT_MAX_SPARE: not split.
int32_t split_spare(int32_t d, int32_t k)
{
    const double close = 5.0 * k * sqrt((double)d) * split_error(d);
    return (int32_t)std::min(1e6, ceil(close + 4.0 * sqrt(close) + 3.0));
}
bool split_f32(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw)
{
    if (h->dtype != KB_F32 || draw || h->tune_config) return false;
    const int32_t spare = split_spare(h->d, k);
    if (spare > SPLIT_MAX_SPARE) return false;
    const int64_t bytes = n * h->d * 4, again_bytes = (int64_t)(k + spare + 1) * (h->d + 4) * 4;
    if (Q > 32) return n * Q * h->d >= (Q <= 64 ? 2 : 1) * SPLIT_MIN_MULTIPLICATIONS && (again_bytes <= 400 << 10 || n >= 3 << 14);
    return bytes >= (n > WHOLE_MAX_ROWS_FEW ? 192 : 400) << 20 && k <= 32 && h->d < 1024 && again_bytes <= RESTATE_LDS && n <= WHOLE_MAX_ROWS_STREAM && Q * ceil_div(h->d, 64) * 256 <= 56 * 1024;
}
// The scan with the queries in LDS (kb_stream.hpp), where they fit beside the rings of four wavefronts and up.
// `most_groups`: no more groups than that.
// Batches of 33 to 64 queries (a wavefront multiplies its rows with two blocks of them) against the tiled kernel's plans: the whole-store
// plan up to WHOLE_MAX_ROWS, the pipeline past it.  us a call, tiled | this:
//   fp8 rows, bf16 queries   5000 x 256 14.4 | 12.0    17,000 x 768 19.5 | 15.9    90,000 x 512 32.4 | 26.5    131,000 x 768 49.7 | 44.1
//                            200,000 x 512 60.5 | 36.9    700,000 x 512 135 | 105    1,000,000 x 64 55.0 | 63.2, x 256 109 | 95.1
//   fp8 rows, fp8 queries    30,000 x 768 15.5 | 17.2    120,000 x 256 19.5 | 20.8    140,000 x 768 43.0 | 36.6    200,000 x 512 50.1 | 34.7
//                            320,000 x 128 36.3 | 35.1   420,000 x 128 32.3 | 33.7    700,000 x 512 107 | 85.6    1,000,000 x 768 187 | 138, x 64 44.8 | 59.9
//   bf16                     30,000 x 768 18.8 | 24.1    45,000 x 256 15.8 | 15.5     90,000 x 512 32.8 | 31.4    120,000 x 256 25.9 | 24.0
//                            131,000 x 768, five wavefronts 56.5 | 57.9               200,000 x 512 69.0 | 52.5    420,000 x 128 51.0 | 39.4    1,000,000 x 256 119 | 109
//   and, one store for both: bf16 65,536 x 768, 40 queries, whose eight tiles a compute unit seven wavefronts take in two rounds 0.87 of the speed; 1,000,000 x 768
//   and 1024, where groups of 256 rows leave four of seven wavefronts 0.97; rows of 128 bytes in the largest stores, where every product meets its mask and those of
//   the pipeline only if they pass: masked | not   bf16 x 64  700,000 rows 0.94 | 1.08    1,000,000 0.88 to 0.93 | 1.03 to 1.07    fp8 x 128  800,000 0.98 | 1.10    1,000,000 0.95 | 1.06
// What loses: tiles so few that the tiled kernel has more wavefronts a compute unit; rows so short that the search of the products is what takes the
// time in stores of many.  (In between tiled fp8 x fp8 scans need no conversions, and the pipeline they give way to begins at 131,072 rows.)
bool two_blocks_stream(const kb *h, int64_t n, bool q8, int32_t waves_per_block)
{
    const int64_t row_bytes = (int64_t)h->d * key_bytes(h->dtype), eight_tiles = 32 * 8 * DEVICE_CUS;
    if (row_bytes == 128 && !q8 && n > (h->dtype == KB_BF16 ? 768 : 896) << 10) return false;
    if (h->dtype == KB_BF16) {
        if (waves_per_block < 8 && n > 896 << 10) return false;
        return n > WHOLE_MAX_ROWS || (waves_per_block >= 7 && n > eight_tiles) || (waves_per_block == 8 && n == eight_tiles);
    }
    if (n > WHOLE_MAX_ROWS_FEW && h->d < (q8 ? 256 : 128)) return false;
    return !q8 || n > WHOLE_MAX_GROUPS * 32;
}
// Up to 32 queries, the whole-store plan: this scan against the plan without it, one store for both.  us a call, without | with:
//   rows of a multiple of 4 KB: a piece of every row lies on the same few channels, and the wavefronts, which begin together, are at one piece
//     bf16 x 2048, 1 query    40,000 rows 46.7 | 44.4    60,000 58.8 | 60.6    100,000 89.1 | 98.1    200,000 136 | 196    400,000 310 | 329
//     bf16 x 4096, 8 queries  40,000 rows 75.7 | 73.9    60,000 94.5 | 124     fp8 x 4096  50,000 62.2 | 60.1    60,000 69.6 | 79.4
//   rows of 64 bytes in large stores: the search of the products is longer than their stream (8 masked queries)
//     fp8    150,000 rows: 0.95 of the speed, 260,000: 0.94    340,000 31.5 | 24.9    600,000 35.4 | 33.8    1,000,000 39.6 | 47.2
//     fp8 x fp8    150,000 rows: 1.18    340,000 29.7 | 24.0    600,000 34.3 | 32.8    1,000,000 40.5 | 45.0
//   few tiles a compute unit: long rows are a chain of loads of a wavefront's, and where queries are so long that fewer than eight wavefronts have
//   room, so is a last round of few tiles.  Time without over with it, by tiles a compute unit:
//     bf16 x 1024 to 1536, 8 masked queries   2.1 1.02    2.3-4 0.94 to 0.99    4.1-5 1.0 to 1.16    more 0.95 to 1.1     (1 query, 20: 0.98 to 1.03 at 2.3-4)
//     bf16 x 1536, 32 queries, five wavefronts  2-4 0.83 to 0.96    4.1 1.22    4.6 1.12    5.5-8 0.90 to 0.96    8.5-9.4 1.09, 1.04    10-11.6 0.93    12-32 1.0 to 1.12
//     bf16 x 1024, 32 queries, seven            2-4 0.86 to 0.99    4.1 1.08    4.6-7 0.95 to 1.01    8 0.93    8.5-11 0.97 to 1.03    12-32 1.02 to 1.22
//     fp8 x 1280, 8 to 32 queries               2-5 1.02 to 1.09    5.5-8 0.94 to 0.98  (x 1024: 0.96 to 1.0, x 2048: 1.0 to 1.1)      more 1.03 to 1.2
//     fp8 x 1536, 32 queries, five              2-4 0.96 to 1.07    4.1 1.08    4.6 0.99    5.5-7 0.83 to 0.90    8 0.99     8.5-9.4 1.24, 1.14    10-11 0.99    12-32 1.02 to 1.13
//     fp8 x 2048, 20 queries, six               2-5 1.03 to 1.15    6.2-8 0.94 to 0.96                  8.5-16 1.09 to 1.2
//   and, of these, the largest stores, where groups of 256 rows leave four or five wavefronts: fp8 1,000,000 x 1024, 32 queries 180 | 196 (bf16 323 | 311).
// (fp8 x fp8 gains in all of these.)  Elsewhere 0.96 to 1.15; what loses there are masked calls on bf16 rows of 1.5 to 2 KB, 45,000 to 95,000 of them.
bool one_block_stream(const kb *h, int64_t n, bool q8, const StreamPlan &p)
{
    const int64_t row_bytes = (int64_t)h->d * key_bytes(h->dtype), tiles = ceil_div(p.units, DEVICE_CUS), w = p.waves_per_block;
    if (row_bytes % 4096 == 0 && n > 48 << 10) return false;
    if (row_bytes == 64 && (n > 640 << 10 || (!q8 && n > WHOLE_MAX_GROUPS * 32 && n <= WHOLE_MAX_ROWS_FEW))) return false;
    if (q8) return true;
    if (n > WHOLE_MAX_ROWS_FEW) return h->dtype == KB_BF16 || w == 8 || n <= 896 << 10;
    if (h->dtype == KB_BF16 && row_bytes >= 2048 && tiles > 2 && tiles <= 4 && (w < 8 || n > 18 << 10)) return false;
    if (h->dtype == KB_FP8_E4M3 && row_bytes >= 1024 && row_bytes < 2048 && tiles > 5 && tiles <= 8) return false;
    return w == 8 || (!(tiles > w && tiles <= 8) && !(tiles > 2 * w && tiles <= 12));
}
bool make_stream_plan(const kb *h, int64_t n, int32_t Q, bool q8, bool split, bool dense, int64_t most_groups, StreamPlan *out)
{
    if ((h->dtype == KB_F32 && !split) || Q > (split ? 32 : dense ? INT32_MAX : 64)) return false;
    StreamPlan p;
    p.tq = dense || Q <= 32 ? 32 : 64;
    const int64_t row_bytes = (int64_t)h->d * key_bytes(h->dtype), pieces = ceil_div(row_bytes, 128);
    const int64_t query_bytes = row_bytes * (h->dtype == KB_FP8_E4M3 && !q8 ? 2 : 1);
    const int64_t stride = ceil_div(query_bytes, 256) * 256, resident = std::min<int64_t>(Q, p.tq) * stride;
    p.nqb = (int32_t)ceil_div(Q, p.tq);
    p.blocks = DEVICE_CUS / p.nqb < 1 ? 1 : DEVICE_CUS / p.nqb;
    p.tr = dense ? 16 : 32;
    p.units = (int32_t)ceil_div(n, p.tr);
    if (p.blocks > p.units) p.blocks = p.units;
    p.pieces_in_ring = p.tr == 16 ? STREAM_RING_16 : STREAM_RING_32;
    p.side_slots = (int32_t)(1 + ceil_div(p.pieces_in_ring, pieces));       // (a piece is asked for that many before its turn)
    p.query_stride = (int32_t)stride;
    // (the most wavefronts whose rings have room and whose groups come out at no more than 256 rows)
    for (p.waves_per_block = 8; p.waves_per_block >= 4; --p.waves_per_block) {
        const int64_t lds = resident + (int64_t)p.waves_per_block * (p.pieces_in_ring * p.tr * 128 + p.side_slots * p.tr * 12) + 256;
        if (lds > STREAM_LDS) continue;
        p.lds = (int32_t)lds;
        p.waves = (int32_t)std::min<int64_t>({p.units, (int64_t)p.blocks * p.waves_per_block, most_groups});
        const int64_t layers = ceil_div(p.units, p.waves), room = dense ? layers : std::max<int64_t>(1, most_groups / p.waves);
        p.per_group = (int32_t)ceil_div(layers, room);
        if (!dense && p.per_group * p.tr > 256) continue;
        *out = p;
        return dense || (Q <= 32 ? one_block_stream(h, n, q8, p) : two_blocks_stream(h, n, q8, p.waves_per_block));
    }
    return false;
}
int stream_groups(const StreamPlan &p)
{
    const int64_t layers = ceil_div(p.units, p.waves), full = (layers - 1) / p.per_group;       // groups of a wavefront but for the last
    return (int)(full * p.waves + std::min<int64_t>(p.waves, p.units - full * p.per_group * p.waves));
}

constexpr size_t WHOLE_OFF_BEST = (sizeof(uint64_t) * (STAT_WORDS + STAT_PARTIALS) + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN;       // the diagnostics come first, as always
size_t whole_bytes(int32_t Q, int32_t groups, size_t *off_pair)
{
    *off_pair = WHOLE_OFF_BEST + align_up(sizeof(float) * (size_t)Q * groups);
    return *off_pair + align_up(sizeof(u32x4) * (size_t)Q * groups);
}
// (k: entries wanted; split f32 rows select a few more)
bool make_whole_plan(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw, bool q8, bool split, Thrift thrift, WholePlan *out)
{
    if (draw || h->tune_no_small_path || h->tune_config || h->tune_sample_keys || h->tune_wg_per_cu) return false;
    if (n < 1 || Q > WHOLE_MAX_QUERIES || n > whole_max_rows(h, Q, q8) || (q8 && h->dtype != KB_FP8_E4M3)) return false;
    WholePlan p;
    p.stream = make_stream_plan(h, n, Q, q8, split, false, thrift == LEAST ? ceil_div(n, 128) : WHOLE_MAX_GROUPS, &p.st);
    if (!p.stream && n > (Q <= 32 ? WHOLE_MAX_ROWS_FEW : WHOLE_MAX_ROWS)) return false;
    if (q8) p.config = Q <= 64 ? FP8_QUERY_TILED_CONFIG : FP8_QUERY_TILED_CONFIG + 1;
    else if (h->dtype == KB_BF16) p.config = Q <= 32 ? 1 : Q <= 64 ? (n >= 128 * 2 * DEVICE_CUS ? 14 : 12) : n >= 128 * 2 * DEVICE_CUS && h->d >= 512 ? 21 : 16;    // (14: once every resident workgroup gets a tile)
    else if (h->dtype == KB_F32 && Q > 32 && thrift != LEAST) p.config = Q <= 64 || ceil_div(n, 128) * ceil_div(Q, 128) <= DEVICE_CUS ? F32_SQUARE_CONFIG : 2;
    else p.config = Q <= 32 ? 1 : 2;
    if (h->dtype == KB_FP8_E4M3 && Q <= 32 && h->d % 128 == 0 && stream_keys(h, n, Q, 1)) p.config = q8 ? FP8_QUERY_STREAM_CONFIG : FP8_STREAM_CONFIG;
    // tiles of 32 rows while those of 128 would leave compute units without one; f32: of 16 while they run side by side (16,000 x
    // 768 rows, 20 queries: 40 us, 27 with tiles of 64 x 64; at 8000 rows 25 against 26)
    if (p.config == 1 && n <= WHOLE_SMALL_TILE_ROWS)
        p.config = h->dtype != KB_F32 ? 13 : Q <= 16 || n <= WHOLE_SMALL_TILE_ROWS / 2 || thrift == LEAST ? SMALL_F32_CONFIG : F32_SQUARE_CONFIG;
    ConfigInfo ci;
    if (!scan_config_info(h->dtype, p.config, &ci)) return false;
    p.tk = ci.tk;
    p.tq = ci.tq;
    p.nqb = (int32_t)ceil_div(Q, ci.tq);
    const int64_t tiles = ceil_div(n, ci.tk);
    // a group is the rows of one wave while there are few of them (groups_per_tile counts both lane halves of its waves)
    const int fine_rows = 2 * ci.tk / ci.groups_per_tile;
    p.fine = tiles * (ci.tk / fine_rows) <= WHOLE_MAX_GROUPS;
    p.group_rows = p.fine ? fine_rows : ci.tk;
    static_assert(WHOLE_MAX_ROWS_FEW / 128 <= WHOLE_MAX_GROUPS && WHOLE_MAX_ROWS / 64 <= WHOLE_MAX_GROUPS, "whole tiles: 128 rows, or 64 with more than 32 queries");
    p.groups = (int32_t)(tiles * (ci.tk / p.group_rows));
    p.k_groups = p.groups;
    if (p.stream) {
        p.tk = p.st.tr;
        p.tq = p.st.tq;
        p.nqb = 1;
        p.fine = 0;
        p.group_rows = p.st.per_group * p.st.tr;
        p.groups = stream_groups(p.st);
        p.k_groups = (int32_t)std::min<int64_t>(p.groups, ceil_div(n, p.st.per_group > 1 ? 128 : q8 ? 64 : 32));
    }
    // Groups with three of a query's k best are scored again, k^3 / 6 / groups^2 of them if rows come in no order, up to k / 2 where
    // similar rows are neighbours.  That costs a call one step of the selecting workgroups or several, each as long as a row's loads.
    // Time of the pipeline over this plan's at k^3 / groups^2 of 0.12 to 4, stores of 5000 to 131,072 rows in runs of 4 to 64
    // similar ones, lowest | tenth | median of some 40 calls each:
    //                            up to 32 queries                                                  more
    //   groups of 16 or 32 rows  bf16 768: 1.21 1.25 1.40    1024: 0.96 1.15 1.50    2048: 0.69    256: 0.95 1.12 1.40    768: 0.75
    //                            fp8 1024: 1.04 1.38 1.80    2048: 0.95 1.39 1.78    4096: 0.88    -
    //                            f32  256: 1.16 1.31 1.57     512: 0.55 1.02 1.51   1024: 0.61     128: 1.18 1.42 1.90    768: 0.82
    //   groups of 64 rows        fp8 x 8 256: 0.99 1.06 1.25  768: 0.66 0.81 1.00                  fp8 768: 0.68, f32 768: 0.60
    //   whole tiles              0.18 to 0.42                                                      0.24 to 0.73
    // One in fifty queries is the limit where that loses.
    // f32, tiles of 64 rows, too many to be halved into groups: four neighbours share a group.  The pipeline from before had tiles of 128 as this
    // plan had; now, with 64 in both, time of the pipeline over this plan's, 140,000 x 768 rows and 64 queries in no order | runs of 4 | 32:
    // k = 16 1.06 | 0.80 | 0.69 (256 elements 1.28 | 1.00 | 0.91), 24 1.07 | 0.71 | 0.64, 40 1.08 | 0.59 | 0.53, 80 1.16 | 0.46 | 0.40
    if (p.config == F32_SQUARE_CONFIG && !p.fine && k > 16) return false;
    const size_t row_bytes = (size_t)h->d * key_bytes(h->dtype);
    const bool cheap = p.group_rows <= 32 && !(p.stream && q8) && row_bytes <= (Q > 32 ? 512 : h->dtype == KB_F32 ? 1024 : 1536);
    if (cubed(k) > (cheap ? 4.0 : 0.12) * (double)p.k_groups * p.k_groups) return false;
    const int64_t items = tiles * p.nqb, most = (int64_t)DEVICE_CUS * ci.wg_per_cu;
    p.grid = p.stream ? p.st.blocks : (int32_t)(items < most ? items : most);
    p.off_best = WHOLE_OFF_BEST;
    p.off_invq = whole_bytes(Q, p.groups, &p.off_pair);
    p.total = p.off_invq + (split && !p.stream ? align_up(sizeof(float) * (size_t)Q) : 0);
    *out = p;
    return true;
}

// The dense plan, where it applies.  Time in us of this plan | the whole-store plan | neither (1000 x 768 bf16 rows unless said):
//   256 queries, k 8      14 | 23 | 192        k 32    14 | 36 | 194       k 128   17 |  -  | 200
//   8 queries, k 128      16 |  -  | 28        4000 rows, 128 queries, k 32    16 | 24 | 37        f32, 64 queries, k 8   21 | 40 | 126
//   8000 rows, 128 queries, k 8    21 | 18 | 32        k 32    22 | 22 | 34        k 128   26 | 49 | 43
//   16,000 rows, 128 queries, k 8   28 | 19 | 33       k 32    29 | 25 | 35        k 128   33 | 34 | 52
// (the weighted selection, 256 queries, k 32: 1000 rows 18 | - | 228, 16,000 rows 38 | - | 114).  At 16,000 rows and 1024 queries
// it is level with the pipeline.
constexpr int64_t DENSE_MAX_PAIRS = (int64_t)1 << 23;
constexpr int64_t DENSE_FIRST_ROWS = 4096;                 // up to here the dense plan is never the slower one
bool dense_is_better(int64_t n, int32_t k, const WholePlan &w) { return n <= DENSE_FIRST_ROWS || cubed(k) > 0.5 * (double)w.k_groups * w.k_groups; }
bool make_dense_plan(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw, bool q8, DensePlan *out)
{
    if (h->tune_no_small_path || h->tune_config || h->tune_sample_keys || h->tune_wg_per_cu) return false;
    if (n < 1 || n > DENSE_MAX_ROWS || n * Q > DENSE_MAX_PAIRS || (q8 && h->dtype != KB_FP8_E4M3)) return false;
    DensePlan p;
    // the smallest tiles while they all run at once; then those that read the rows and queries less often
    // (f32, tiles of 16 x 32: two of them a compute unit; 2000 x 768 rows, 256 queries 39 us, 512 queries with tiles of 64 x 64 29)
    const int64_t tiles32 = ceil_div(n, 32) * ceil_div(Q, 32);
    const bool small = tiles32 <= (h->dtype == KB_F32 ? DEVICE_CUS : 2 * DEVICE_CUS);
    if (q8) p.config = small ? FP8_QUERY_SMALL_CONFIG : Q <= 64 ? FP8_QUERY_TILED_CONFIG : FP8_QUERY_TILED_CONFIG + 1;
    else if (h->dtype == KB_F32) p.config = small && !draw ? SMALL_F32_CONFIG : F32_SQUARE_CONFIG;
    else if (h->dtype == KB_BF16) p.config = small ? 13 : Q <= 64 ? 12 : 16;
    else p.config = small ? 13 : Q <= 32 ? 1 : 2;
    ConfigInfo ci;
    if (!scan_config_info(h->dtype, p.config, &ci)) return false;
    p.tk = ci.tk;
    p.tq = p.config == SMALL_F32_CONFIG && Q <= 16 ? 16 : ci.tq;
    p.nqb = (int32_t)ceil_div(Q, p.tq);
    const int64_t items = ceil_div(n, ci.tk) * p.nqb, most = (int64_t)DEVICE_CUS * ci.wg_per_cu;
    p.grid = (int32_t)(items < most || p.config == SMALL_F32_CONFIG ? items : most);
    p.stream = small && !draw && make_stream_plan(h, n, Q, q8, false, true, WHOLE_MAX_GROUPS, &p.st);
    if (p.stream) p.grid = p.st.blocks * p.st.nqb;
    p.stride = (int32_t)(ceil_div(n, 128) * 128);
    p.off_values = align_up(sizeof(uint64_t) * (STAT_WORDS + STAT_PARTIALS));       // the diagnostics come first, as always
    p.off_invq = p.off_values + align_up(sizeof(float) * (size_t)Q * p.stride);
    const int64_t qpad = (int64_t)p.nqb * p.tq;
    p.off_lgain = p.off_invq + (draw ? align_up(sizeof(float) * qpad) : 0);
    p.off_unused = p.off_lgain + (draw ? align_up(sizeof(float) * (ceil_div(n, 256) * 256 + 256)) : 0);
    p.total = p.off_unused + (draw ? align_up((size_t)qpad * (2 * sizeof(uint64_t) + (3 + CAND_SEGMENTS) * sizeof(uint32_t))) : 0);    // (what prep_kernel writes for the pipeline)
    *out = p;
    return true;
}

// Pure function of (handle settings, row count n, Q, k): which kernels run on what, and where everything lives
// in the workspace.
bool make_plan(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw, bool q8, Thrift thrift, Plan *out)
{
    Choice c;
    if (!choose_kernels(h, n, Q, draw, q8, thrift, &c)) return false;
    plan_for(h, c, n, Q, k, draw, thrift, out, nullptr);
    return true;
}

void max_into(Sizes &m, const Sizes &z)
{
    m.k = z.k;
    if (z.qpad > m.qpad) m.qpad = z.qpad;
    if (z.regions > m.regions) m.regions = z.regions;
    if (z.sample_slots > m.sample_slots) m.sample_slots = z.sample_slots;
    if (z.more_slots > m.more_slots) m.more_slots = z.more_slots;
    if (z.cand_cap > m.cand_cap) m.cand_cap = z.cand_cap;
    if (z.region_records > m.region_records) m.region_records = z.region_records;
    if (z.lgain_rows > m.lgain_rows) m.lgain_rows = z.lgain_rows;
}

// Upper bound of the Sizes of plan_for(h, c, n, ...) over every n in [1, capacity].  nt counts the key tiles of the
// sampling configuration (its tiles may be lower than the main pass's; both counts are constant between multiples of
// the lower tile height).
//   Up to EXACT_TILES key tiles the plans are enumerated (one per pair of tile counts; this range contains every case
//   without a sampling pass: sample_tiles_for gives at least min(2k / groups, nt / 2) tiles, which is k samples once
//   nt >= 256).
//   Beyond, with st = sample_tiles_for(nt) > 0 and expect = ceil(k nt / st):
//     st = ceil(nt max(k, 8) / 512), or raised to 2k / groups:  expect <= 512
//     st = nt / 2 (rounded down):                               expect <= 2k + 1 <= 257
//     st = MAX_SAMPLE_SLOTS / groups:                           expect grows with nt, largest at the capacity
//   (with the "sample_keys" knob st does not follow nt: the largest candidate capacity is assumed), so cand_cap is
//   bounded; the number of scan wavefronts and sample_slots do not fall as nt grows, and region_cap is REGION_CAP.
constexpr int64_t EXACT_TILES = 256;
void bound_sizes(const kb *h, const Choice &c, int32_t Q, int32_t k, bool draw, Sizes &m)
{
    const ConfigInfo &ci = c.ci, &sci = c.sci;
    const int64_t step = ci.tk < sci.tk ? ci.tk : sci.tk;
    const int64_t cap_nt = ceil_div(h->capacity, sci.tk);
    Plan p;
    Sizes z;
    for (int64_t n = step; n < h->capacity + step && ceil_div(n, sci.tk) <= EXACT_TILES; n += step) {
        plan_for(h, c, n, Q, k, draw, AMPLE, &p, &z);
        max_into(m, z);
    }
    plan_for(h, c, h->capacity, Q, k, draw, AMPLE, &p, &z);       // the ln(gain) array, and the largest grid
    max_into(m, z);
    if (cap_nt <= EXACT_TILES) return;
    int64_t expect = 512;
    const int64_t at_cap = ceil_div((int64_t)k * cap_nt * sci.groups_per_tile, MAX_SAMPLE_SLOTS);
    if (at_cap > expect) expect = at_cap;
    z.cand_cap = h->tune_sample_keys > 0 ? MAX_CAND_CAP : cand_cap_for(expect, true);
    z.sample_slots = (int32_t)(sample_tiles_for(h, sci, cap_nt, Q, k, leaves_sample_out(c), false) * sci.groups_per_tile);
    z.more_slots = leaves_sample_out(c) ? z.sample_slots : 0;
    z.region_records = (int64_t)z.regions * REGION_CAP;
    max_into(m, z);
}

// ------------------------------------------------------------------------------------------------
// row norms (see kb_norm.hpp)
// ------------------------------------------------------------------------------------------------
template <int DT> __global__ __launch_bounds__(256) void row_norm_kernel(const void *keys, int64_t begin, int64_t end, int d, float *inv_norm)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = begin + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= end) return;
    const float inv = row_inv_norm<DT>(keys, row, d * (DT == KB_F32 ? 4 : DT == KB_BF16 ? 2 : 1), lane);
    if (lane == 0) inv_norm[row] = inv;
}

// ------------------------------------------------------------------------------------------------
// append: rows, scales and tags to the tail of the store in one launch.  Blocks of a few thousand rows are what is appended, and there the
// calls cost the host more than the copies cost the device: for 4000 x 320 fp8 rows with scales and tags three copies by the runtime take
// the host 8.5 us, this launch with the checks of its addresses 4.5.  Bound by memory on blocks that are large: four blocks of 16384 x 1024
// bf16 rows, each appended, normalized and asked about, 225 us with copies by the runtime and 215 like this.
// Each thread moves APPEND_PIECES pieces of 16 bytes of the rows, all in flight, read past the cache (the store's lines are what the
// normalization reads next; 1.006 of cached loads); the last workgroups move one word of scale or tag a thread.
// ------------------------------------------------------------------------------------------------
struct AppendArgs {
    const u32x4 *rows;
    u32x4 *rows_to;             // nullptr: in place
    const uint32_t *scale;
    uint32_t *scale_to;
    const uint64_t *tags;
    uint64_t *tags_to;
    int64_t pieces, n;
    int32_t row_blocks;
};
constexpr int APPEND_PIECES = 4;
__global__ __launch_bounds__(256) void append_kernel(AppendArgs a)
{
    if ((int)blockIdx.x < a.row_blocks) {
        const int64_t at = (int64_t)blockIdx.x * (256 * APPEND_PIECES) + threadIdx.x;
        u32x4 v[APPEND_PIECES];
#pragma unroll
        for (int u = 0; u < APPEND_PIECES; ++u)
            if (at + u * 256 < a.pieces) v[u] = __builtin_nontemporal_load(a.rows + at + u * 256);
#pragma unroll
        for (int u = 0; u < APPEND_PIECES; ++u)
            if (at + u * 256 < a.pieces) a.rows_to[at + u * 256] = v[u];
        return;
    }
    const int64_t i = (int64_t)(blockIdx.x - a.row_blocks) * 256 + threadIdx.x;
    if (i >= a.n) return;
    if (a.scale_to) a.scale_to[i] = a.scale[i];
    if (a.tags_to) a.tags_to[i] = a.tags[i];
}

// ------------------------------------------------------------------------------------------------
// weighted random selection: ln(gain) per entry, -inf for entries without weight and for the padding
// ------------------------------------------------------------------------------------------------
struct GainArgs {
    const float *gain;          // nullptr: no weighted selection
    float *log_gain;
    int64_t n, n_padded;
    int blocks;                 // workgroups of 256 entries
};
__device__ inline void log_gain_block(const GainArgs &g, int block)
{
    const int64_t i = (int64_t)block * 256 + threadIdx.x;
    if (i >= g.n_padded) return;
    float v = -__builtin_inff();
    if (i < g.n) {
        const float x = g.gain[i];
        if (x > 0.f) v = logf(x);
    }
    g.log_gain[i] = v;
}

// ------------------------------------------------------------------------------------------------
// prep: query norms + reset of the per-call counters; for the weighted selection its last workgroups form ln(gain), which
// as a launch of its own cost a call 5 us
// ------------------------------------------------------------------------------------------------
template <int QT> __global__ __launch_bounds__(256) void prep_kernel(const void *queries, int Q, int qpad, int d, float *invq, uint64_t *thr64, float *thrp,
                                                                       uint32_t *cnt, uint32_t *flag, uint64_t *stats, uint64_t sample_keys,
                                                                       const uint64_t *qmask, uint64_t *qmask_pad, int grid, uint32_t *fb_done, GainArgs g)
{
    const int prep_blocks = (int)gridDim.x - g.blocks;
    if ((int)blockIdx.x >= prep_blocks) {
        log_gain_block(g, (int)blockIdx.x - prep_blocks);
        return;
    }
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t < qpad) fb_done[t] = 0;
    if (t < qpad) {     // padding queries (t >= Q) can never pass the filter of the scan
        thr64[t] = t < Q ? 0ull : ~0ull;
        thrp[t] = t < Q ? -__builtin_inff() : __builtin_inff();
        for (int sg = 0; sg < CAND_SEGMENTS; ++sg) cnt[t * CAND_SEGMENTS + sg] = 0;
        flag[t] = 0;
        qmask_pad[t] = (qmask && t < Q) ? qmask[t] : 0ull;
    }
    if (t <= STAT_GATE) stats[t] = t == 2 ? sample_keys : t == 3 ? (uint64_t)grid : 0ull;
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row < qpad) {
        const float inv = row < Q ? row_inv_norm<QT>(queries, row, d * (QT == KB_F32 ? 4 : QT == KB_BF16 ? 2 : 1), lane) : 0.f;
        if (lane == 0) invq[row] = inv;
    }
}

// ------------------------------------------------------------------------------------------------
// A full sort is a chain of dependent LDS round trips (one per stage) and costs tens of microseconds for a
// few thousand words.  Selection needs far fewer: a most-significant-digit radix search for the k-th
// largest word (8-bit digits, starting at the highest bit in which the words' upper halves differ; each pass is
// one histogram with LDS atomics and one wavefront-wide scan), then the survivors are compacted
// and ordered by counting, for each, how many survivors are larger.  The selection runs in kernels whose whole
// length is a few microseconds, so its own fixed costs count: the reductions and scans across lanes are
// data-parallel-primitive moves (a shuffle is an LDS round trip each), the wavefronts exchange their partial
// results through LDS without atomics, and a pass has two barriers.  Zero words are padding: they are
// never selected, and if fewer than k words are nonzero the result is zero-padded.
constexpr int SELECT_MAX = KB_K_MAX + SPLIT_MAX_SPARE;        // entries that a call selects at most
struct SelectScratch {
    uint64_t sel[SELECT_MAX];
    uint32_t hist[256];
    uint32_t part[16][4];  // per wavefront: its nonzero words, AND and OR of their upper halves
    uint32_t ctl[8];       // 1 selected, 2 digit found, 3 still needed, 4 words in that bin
};

__device__ inline uint64_t shr64(uint64_t v, int s) { return s >= 64 ? 0ull : v >> s; }

// Cross-lane steps as data-parallel-primitive moves (one vector instruction each, no LDS round trip): `x` of the lane
// `shr` places down its row of 16, or lane 15 / 31 of the rows before (row_bcast), or `idle` where there is none.
template <int CTRL, int ROW_MASK> __device__ inline uint32_t dpp_or(uint32_t idle, uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)idle, (int)x, CTRL, ROW_MASK, 0xf, false);
}
// Inclusive scans over the 64 lanes of a (fully active) wavefront; lane 63 ends up with the total.
__device__ inline uint32_t wave_scan_add(uint32_t x)
{
    x += dpp_or<0x111, 0xf>(0u, x);
    x += dpp_or<0x112, 0xf>(0u, x);
    x += dpp_or<0x114, 0xf>(0u, x);
    x += dpp_or<0x118, 0xf>(0u, x);
    x += dpp_or<0x142, 0xa>(0u, x);
    x += dpp_or<0x143, 0xc>(0u, x);
    return x;
}
__device__ inline uint32_t wave_scan_and(uint32_t x)
{
    x &= dpp_or<0x111, 0xf>(~0u, x);
    x &= dpp_or<0x112, 0xf>(~0u, x);
    x &= dpp_or<0x114, 0xf>(~0u, x);
    x &= dpp_or<0x118, 0xf>(~0u, x);
    x &= dpp_or<0x142, 0xa>(~0u, x);
    x &= dpp_or<0x143, 0xc>(~0u, x);
    return x;
}
__device__ inline uint32_t wave_scan_or(uint32_t x)
{
    x |= dpp_or<0x111, 0xf>(0u, x);
    x |= dpp_or<0x112, 0xf>(0u, x);
    x |= dpp_or<0x114, 0xf>(0u, x);
    x |= dpp_or<0x118, 0xf>(0u, x);
    x |= dpp_or<0x142, 0xa>(0u, x);
    x |= dpp_or<0x143, 0xc>(0u, x);
    return x;
}

__device__ inline float wave_scan_min(float x)
{
    constexpr uint32_t IDLE = 0x7f800000u;      // +inf
    x = __builtin_fminf(x, as_f32(dpp_or<0x111, 0xf>(IDLE, as_u32(x))));
    x = __builtin_fminf(x, as_f32(dpp_or<0x112, 0xf>(IDLE, as_u32(x))));
    x = __builtin_fminf(x, as_f32(dpp_or<0x114, 0xf>(IDLE, as_u32(x))));
    x = __builtin_fminf(x, as_f32(dpp_or<0x118, 0xf>(IDLE, as_u32(x))));
    x = __builtin_fminf(x, as_f32(dpp_or<0x142, 0xa>(IDLE, as_u32(x))));
    x = __builtin_fminf(x, as_f32(dpp_or<0x143, 0xc>(IDLE, as_u32(x))));
    return x;
}
__device__ inline float wave_scan_max(float x) { return -wave_scan_min(-x); }

// buf[0..n) in, buf[0..k) out (the rest of buf is left as it was).  All threads of the workgroup call it (at most 16
// wavefronts), converged.
__device__ inline void select_topk_desc(uint64_t *buf, int n, int k, SelectScratch *sc, int tid, int nthreads)
{
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthreads >> 6;
    // ---- how many words there are, and the highest bit in which their upper halves differ ----
    {
        uint32_t cnt = 0, ahi = ~0u, ohi = 0u;
        for (int i = tid; i < n; i += nthreads) {
            const uint64_t e = buf[i];
            if (e != 0) {
                ++cnt;
                ahi &= (uint32_t)(e >> 32);
                ohi |= (uint32_t)(e >> 32);
            }
        }
        cnt = wave_scan_add(cnt);
        ahi = wave_scan_and(ahi);
        ohi = wave_scan_or(ohi);
        if (lane == 63) {
            sc->part[wave][0] = cnt;
            sc->part[wave][1] = ahi;
            sc->part[wave][2] = ohi;
        }
        for (int i = tid; i < 256; i += nthreads) sc->hist[i] = 0u;
        if (tid == 0) sc->ctl[1] = 0u;
    }
    __syncthreads();
    uint32_t nz, all_and, all_or;
    {
        // every wavefront adds the wavefronts' parts up for itself: lanes 0..15 take one each, lane 15 gets the totals
        const int w = lane & 15;
        const bool have = w < nwaves;
        uint32_t c = have ? sc->part[w][0] : 0u, a = have ? sc->part[w][1] : ~0u, o = have ? sc->part[w][2] : 0u;
        c += dpp_or<0x111, 0xf>(0u, c);
        c += dpp_or<0x112, 0xf>(0u, c);
        c += dpp_or<0x114, 0xf>(0u, c);
        c += dpp_or<0x118, 0xf>(0u, c);
        a &= dpp_or<0x111, 0xf>(~0u, a);
        a &= dpp_or<0x112, 0xf>(~0u, a);
        a &= dpp_or<0x114, 0xf>(~0u, a);
        a &= dpp_or<0x118, 0xf>(~0u, a);
        o |= dpp_or<0x111, 0xf>(0u, o);
        o |= dpp_or<0x112, 0xf>(0u, o);
        o |= dpp_or<0x114, 0xf>(0u, o);
        o |= dpp_or<0x118, 0xf>(0u, o);
        nz = (uint32_t)__builtin_amdgcn_readlane((int)c, 15);
        all_and = (uint32_t)__builtin_amdgcn_readlane((int)a, 15);
        all_or = (uint32_t)__builtin_amdgcn_readlane((int)o, 15);
    }
    // selected words: nonzero and (word >> shift) >= pref
    int shift = 0;
    uint64_t pref = 1;
    if ((int)nz > k) {
        const uint32_t diff = all_and ^ all_or;
        int hi = diff ? 64 - __builtin_clz(diff) : 32;       // bits [hi, 64) are decided and equal pref
        pref = hi >= 64 ? 0ull : (uint64_t)(all_or >> (hi - 32));
        if (diff == 0) {        // equal scores: what the row numbers share would be counted into one bin each, one word after the other
            uint32_t alo = ~0u, olo = 0u;
            for (int i = tid; i < n; i += nthreads) {
                const uint64_t e = buf[i];
                alo &= e != 0 ? (uint32_t)e : ~0u;
                olo |= (uint32_t)e;
            }
            alo = wave_scan_and(alo);
            olo = wave_scan_or(olo);
            __syncthreads();            // (the parts above have been read)
            if (lane == 63) {
                sc->part[wave][1] = alo;
                sc->part[wave][2] = olo;
            }
            __syncthreads();
            for (int w = 0; w < nwaves; ++w) {
                alo &= sc->part[w][1];
                olo |= sc->part[w][2];
            }
            alo = (uint32_t)__builtin_amdgcn_readlane((int)alo, 63);
            olo = (uint32_t)__builtin_amdgcn_readlane((int)olo, 63);
            hi = alo != olo ? 32 - __builtin_clz(alo ^ olo) : 0;
            pref = ((uint64_t)all_or << 32 | olo) >> hi;
        }
        uint32_t need = (uint32_t)k;
        for (int pass = 0; pass < 9 && hi > 0; ++pass) {
            const int width = hi < 8 ? hi : 8, lo = hi - width;
            for (int i = tid; i < n; i += nthreads) {
                const uint64_t e = buf[i];
                if (e != 0 && shr64(e, hi) == pref) atomicAdd(&sc->hist[(uint32_t)(e >> lo) & ((1u << width) - 1u)], 1u);
            }
            __syncthreads();
            if (tid < 64) {
                // lane l owns bins 4 (63 - l) .. + 3, so the scan over the lanes counts the words in higher bins; it
                // clears its bins for the next pass
                const int base = 4 * (63 - lane);
                const uint32_t c0 = sc->hist[base], c1 = sc->hist[base + 1], c2 = sc->hist[base + 2], c3 = sc->hist[base + 3];
                sc->hist[base] = 0u;
                sc->hist[base + 1] = 0u;
                sc->hist[base + 2] = 0u;
                sc->hist[base + 3] = 0u;
                const uint32_t mine = c0 + c1 + c2 + c3;
                const uint32_t incl = wave_scan_add(mine);
                uint32_t above = incl - mine;
                if (incl >= need && above < need) {
                    const uint32_t c[4] = {c0, c1, c2, c3};
                    int bin = 0;
                    uint32_t in_bin = 0;
#pragma unroll
                    for (int j = 3; j >= 0; --j) {
                        if (in_bin == 0 && above + c[j] >= need) {
                            bin = base + j;
                            in_bin = c[j];
                        } else if (in_bin == 0) {
                            above += c[j];
                        }
                    }
                    sc->ctl[2] = (uint32_t)bin;
                    sc->ctl[3] = need - above;
                    sc->ctl[4] = in_bin;
                }
            }
            __syncthreads();
            pref = (width < 64 ? pref << width : 0ull) | sc->ctl[2];
            need = sc->ctl[3];
            hi = lo;
            if (sc->ctl[4] == need) break;       // the whole bin belongs to the result
        }
        shift = hi;
    }
    for (int i = tid; i < n; i += nthreads) {
        const uint64_t e = buf[i];
        if (e != 0 && shr64(e, shift) >= pref) {
            const uint32_t slot = atomicAdd(&sc->ctl[1], 1u);
            if (slot < (uint32_t)SELECT_MAX) sc->sel[slot] = e;
        }
    }
    __syncthreads();
    const int m = (int)sc->ctl[1] < k ? (int)sc->ctl[1] : k;
    for (int t = tid; t < k; t += nthreads) {
        if (t < m) {
            const uint64_t e = sc->sel[t];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < m; ++j) rank += sc->sel[j] > e;
            buf[rank] = e;
        } else {
            buf[t] = 0ull;
        }
    }
    __syncthreads();
}

template <int KT, int UNR> __device__ f32x16 score_rows(const void *keys, const void *queries, int d, int64_t my_row, int q, float key_scale = 1.f, float query_scale = 1.f);
constexpr int KT_FP8_Q8 = 3;        // stands for fp8 keys with fp8 queries (one fp8 matrix instruction per 64-byte chunk, as in the scan)

// k-th best group maximum of the sampling pass = a lower bound of the k-th best score (k distinct
// entries reach it).  Also derives the conservative pre-filter on dot * inv_k used by the main pass:
// whenever fp32((dot*inv_k) * inv_q) >= s_thr holds, dot*inv_k >= thrp holds (2^-20 relative slack
// covers the three fp32 roundings involved).
//
// Two modes.  KEYS (weighted random selection; prep_kernel has run): the samples are candidate words of keys and the
// k-th best word is the threshold as it is.  Otherwise the kernel also does what prep_kernel does (the query's
// 1/|q|, its counters, flag and padded mask word; one workgroup per PADDED query), so that a plain query has one
// launch less, and the samples are words of s1 = dot * inv_k, which the sampling pass can form without 1/|q|.  The final
// score f(s1) = fp32(s1 * inv_q) + 0 never falls as s1 grows, so the k sampled entries with the largest words all
// have a score >= S = f(s1 of the k-th); those of them whose score equals S have an index <= the largest such
// index, and the threshold word is (S, that index): k distinct entries reach it.
struct ThresholdArgs {
    const uint64_t *samp;       // see sample_slot_index
    const void *queries;
    const uint64_t *qmask;      // or nullptr
    float *invq, *thrp;
    uint64_t *thr64, *qmask_pad, *stats;
    uint32_t *cnt, *flag, *fb_done;
    uint64_t sample_keys;
    int32_t slots, group_shift, k, Q, qpad, d, grid;
    // where the main pass leaves the sampled rows out:
    const uint64_t *more;       // ScanArgs::samp_more
    uint64_t *cand;             // the candidate lists
    int32_t cand_cap, tile_rows;
    ScanArgs scan;              // of the sampling pass
};
// A load whose value nobody needs: the line is in the L2 for whoever asks next.
__device__ inline void touch(const unsigned char *at)
{
    uint32_t v = *reinterpret_cast<const volatile uint32_t *>(at);
    asm volatile("" : : "v"(v));
}
constexpr int THRESHOLD_AGAIN = 1024;       // groups that are scored again, a query

// KT: type of the keys where the main pass leaves the sampled rows out (never with fp8 queries or KEYS), -1 otherwise.  The kernel
// then also lists the sample's own candidates: the best and the second row of a group where they reach the threshold; groups whose
// bound on the others does too (k^3 / (6 slots^2) of them on a store in no order, one query in a thousand) are scored again
// with the instruction sequence of the scan, 32 rows a wavefront.
template <int QT, bool KEYS, int KT, int PER = 2> __global__ __launch_bounds__(1024) void threshold_kernel(ThresholdArgs a)
{
    constexpr bool ONCE = KT >= 0;
    static_assert(!(ONCE && KEYS));
    constexpr int SEGS = ONCE ? CAND_SEGMENTS : 1;
    __shared__ uint32_t sh_seg[SEGS], sh_again, sh_lost;
    __shared__ uint16_t sh_group[ONCE ? THRESHOLD_AGAIN : 1];
    if constexpr (ONCE) {
        if (threadIdx.x < CAND_SEGMENTS) sh_seg[threadIdx.x] = 0;
        if (threadIdx.x == 0) sh_again = sh_lost = 0;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint64_t *buf = reinterpret_cast<uint64_t *>(smem_raw);
    const int q = blockIdx.x, tid = threadIdx.x, slots = a.slots, k = a.k;
    SelectScratch *sc = reinterpret_cast<SelectScratch *>(smem_raw + sizeof(uint64_t) * (slots > k ? slots : k));
    __shared__ float sh_iq;
    __shared__ uint32_t sh_low;
    __shared__ bool sh_endless;         // the query's squared length is past the largest float
    // Everything the kernel reads from global memory is asked for before anything waits: the query's mask word, the
    // first two samples of every thread and (first wavefront) the query row are one memory round trip, not three.
    const int bd = (int)blockDim.x;
    uint64_t mask_word = 0ull, words[PER];
    if (!KEYS && tid == 0 && a.qmask && q < a.Q) mask_word = a.qmask[q];
    if (KEYS || q < a.Q) {
#pragma unroll
        for (int u = 0; u < PER; ++u) words[u] = tid + u * bd < slots ? a.samp[sample_slot_index(tid + u * bd, a.group_shift, a.qpad, q)] : 0ull;
    }
    if constexpr (!KEYS) {
        if (tid < CAND_SEGMENTS) a.cnt[q * CAND_SEGMENTS + tid] = 0;
        if (tid == 0) {
            a.flag[q] = 0;
            a.fb_done[q] = 0;
            a.qmask_pad[q] = mask_word;
            sh_low = 0xffffffffu;
        }
        if (q == 0 && tid < STAT_WORDS + STAT_PARTIALS) a.stats[tid] = tid == 2 ? a.sample_keys : tid == 3 ? (uint64_t)a.grid : 0ull;
        if (q >= a.Q) {         // a padding query can never pass the filter of the scan
            if (tid == 0) {
                a.invq[q] = 0.f;
                a.thr64[q] = ~0ull;
                a.thrp[q] = __builtin_inff();
            }
            return;
        }
        if (tid < 64) {
            const float square_sum = row_square_sum<QT>(a.queries, q, a.d * bytes_of(QT), tid), inv = inv_norm_of(square_sum);
            if (tid == 0) {
                a.invq[q] = inv;
                sh_iq = used_inv<QT>(inv);
                sh_endless = square_sum == __builtin_inff();
            }
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (tid + u * bd < slots) buf[tid + u * bd] = words[u];
    for (int i = tid + PER * bd; i < slots; i += bd) buf[i] = a.samp[sample_slot_index(i, a.group_shift, a.qpad, q)];
    __syncthreads();
    select_topk_desc(buf, slots, k, sc, tid, bd);
    uint64_t t = k <= slots ? buf[k - 1] : 0ull;
    const float iq = KEYS ? a.invq[q] : sh_iq;
    if constexpr (!KEYS) {
        if (t != 0) {
            const float s = candidate_score(t) * iq + 0.0f;
            if (tid < k && candidate_score(buf[tid]) * iq + 0.0f == s) atomicMin(&sh_low, (uint32_t)buf[tid]);
            __syncthreads();
            t = ((uint64_t)score_to_ordered(s) << 32) | sh_low;
        }
    }
    float tp = -__builtin_inff();
    if (KEYS) {
        // keys are compared as they are: a word at or above t has a key at or above t's key
        if (t != 0) tp = candidate_score(t);
    } else if (t != 0 && iq > 0.f) {
        const float x = candidate_score(t) / iq;
        tp = x - fabsf(x) * 0x1p-20f - 1e-30f;
    }
    if (tid == 0) {
        a.thr64[q] = t;
        a.thrp[q] = tp;
    }
    if constexpr (ONCE) {
        const uint32_t seg_cap = (uint32_t)a.cand_cap / CAND_SEGMENTS;
        uint64_t *list = a.cand + (size_t)q * a.cand_cap;
        auto append = [&](uint64_t word) {
            const uint32_t seg = candidate_segment(candidate_index(word)), at = atomicAdd(&sh_seg[seg], 1u);
            if (at < seg_cap) list[seg * seg_cap + at] = word;
            else sh_lost = 1u;
        };
        // the sample's slot i: its group's lane half holds element e of 32 at this row of the tile
        auto row_of = [&](int slot, int e) {
            const int tile = slot >> a.group_shift, group = slot & ((1 << a.group_shift) - 1);
            const int rl = (group >> 1) * 64 + 4 * (group & 1) + (e >> 4) * 32 + 8 * ((e & 15) >> 2) + (e & 3);
            return (uint32_t)sample_row<true>(a.scan, sample_tile_run(a.scan, tile, a.tile_rows), tile, a.tile_rows, rl);
        };
        // (what is known of a group besides its best is read only where it can reach the threshold: the search tells values apart
        // but for their low five bits)
        auto look = [&](int i, uint64_t w) {
            if (w == 0) return;
            const float best = candidate_score(w);
            const uint32_t bits = as_u32(best);
            if (!(as_f32((int32_t)bits < 0 ? bits & ~31u : bits | 31u) >= tp)) return;
            if (best >= tp) append(pack_raw_candidate(best, candidate_index(w)));
            const uint64_t more = a.more[sample_slot_index(i, a.group_shift, a.qpad, q)];
            if (more == 0) return;
            const float second = ordered_to_score((uint32_t)(more >> 32));
            if (second >= tp) append(pack_raw_candidate(second, row_of(i, (int)(more & 31u))));
            if (others_bound(more) != 0u && ordered_to_score(others_bound(more)) >= tp) {
                const uint32_t n = atomicAdd(&sh_again, 1u);
                if (n < THRESHOLD_AGAIN) sh_group[n] = (uint16_t)i;
            }
        };
#pragma unroll
        for (int u = 0; u < PER; ++u) look(tid + u * bd, words[u]);
        for (int i = tid + PER * bd; i < slots; i += bd) look(i, a.samp[sample_slot_index(i, a.group_shift, a.qpad, q)]);
        __syncthreads();
        const uint32_t again = sh_again;
        if (again > 0 && again <= THRESHOLD_AGAIN) {
            const ScanArgs &p = a.scan;
            const int lane = tid & 63, lrow = lane & 31, half = lane >> 5;
            const uint64_t qm = p.qmask ? p.qmask[q] : 0ull;
            // The rows of a group are asked for by all wavefronts before one of them scores it, piece after piece: a call in two has
            // such a group, and the kernel is as long as its slowest query.
            for (uint32_t j = 0; j < again && j < 2; ++j) {
                const unsigned char *at = static_cast<const unsigned char *>(p.keys) + (size_t)row_of(sh_group[j], tid & 31) * ((size_t)a.d * (KT == KB_BF16 ? 2 : 1));
                for (int b = tid >> 5; b * 128 < a.d * (KT == KB_BF16 ? 2 : 1); b += bd >> 5) touch(at + (size_t)b * 128);
            }
            for (uint32_t j = (uint32_t)(tid >> 6); j < again; j += (uint32_t)(bd >> 6)) {
                const int slot = sh_group[j];
                const uint32_t row = row_of(slot, lrow);
                const size_t at = sample_slot_index(slot, a.group_shift, a.qpad, q);
                const uint32_t known = candidate_index(a.samp[at]), second = row_of(slot, (int)(a.more[at] & 31u));
                const f32x16 acc = score_rows<ONCE ? KT : 0, KT == KB_FP8_E4M3 ? 4 : 8>(p.keys, a.queries, a.d, row, q);
                const float dot = select16(acc, lrow & 15);
                const int64_t mine = __shfl((int)row, 8 * ((lrow & 15) >> 2) + 4 * half + (lrow & 3), 64);      // whose product lanes 0..15 of each half hold
                const float ik = p.inv_norm[mine];
                bool ok = lrow < 16 && !row_removed(ik) && known != (uint32_t)mine && second != (uint32_t)mine;
                if (p.qmask) ok = ok && (p.tags[mine] & qm) != 0;
                if (ok && dot * ik >= tp) append(pack_raw_candidate(dot * ik, (uint32_t)mine));
            }
            __syncthreads();
        }
        if (tid < CAND_SEGMENTS) a.cnt[q * CAND_SEGMENTS + tid] = sh_seg[tid] < seg_cap ? sh_seg[tid] : seg_cap;
        // The sample's search does not know infinite products, which only a query of endless length has on finite rows: it goes the
        // exhaustive way, unless its mask lets nothing through.  (A zero query's products are zeros, one with a NaN has nothing to list.)
        const bool unknown = sh_endless && (!a.qmask || mask_word != 0);       // (thread 0 holds the mask word)
        if (tid == 0 && (sh_lost != 0 || again > THRESHOLD_AGAIN || unknown)) a.flag[q] = 1u;
    }
}

// ------------------------------------------------------------------------------------------------
// finalize: select each query's best k in order; a query whose list overflowed is resolved by an
// exhaustive scan of all keys (shared by fb_parts workgroups) that uses the same MFMA sequence per output
// element as the scan kernel, so both paths produce bit-identical scores.
// ------------------------------------------------------------------------------------------------
struct FinalArgs {
    const void *keys;
    const float *inv_norm;
    const uint64_t *tags;
    const void *queries;
    const uint64_t *qmask;
    const float *invq;
    const uint64_t *cand;
    uint32_t *cnt;
    const uint32_t *flag;
    uint64_t *stats;
    int32_t *out_index;
    float *out_score;
    int64_t n_keys;
    int32_t d, k, cand_cap;
    DrawArgs draw;
    uint32_t *fb_done;        // [Q] arrivals of the parts of an exhaustive scan (zero before the launch)
    uint64_t *fb_lists;       // [Q][fb_parts][k] their partial results
    int32_t fb_parts;
    uint64_t *thr64;          // [Q] threshold words of the scan
    float *thrp;              // ... and the bounds that go with them
    int32_t again;            // the launch behind one on split f32 rows: the queries that this one left to it, if any
    int32_t raw;              // the lists hold dot * inv_k products (plain queries), not finished candidate words
    int32_t k_out, more_lds;  // as in WholeSelectArgs
    int32_t more_at;          // offset of these bytes in the dynamic LDS
};

typedef int i32x8 __attribute__((ext_vector_type(8)));
// 32 dot products of one query by one wavefront, accumulated exactly as the scan kernels do: lane (lrow, half) supplies
// row my_row for lrow and gets, in element i, the product of the row that lane 8 (i / 4) + 4 half + i % 4 supplied
// (every column holds the same query).
// (split f32: the scales of that row and of the query)
template <int KT, int UNR> __device__ inline f32x16 score_rows(const void *keys, const void *queries, int d, int64_t my_row, int q, float key_scale, float query_scale)
{
    constexpr bool Q8 = KT == KT_FP8_Q8;
    constexpr int KTT = Q8 ? (int)KB_FP8_E4M3 : KT;
    constexpr int KEY_BYTES = KeyTraits<KTT>::KEY_BYTES, QRY_BYTES = Q8 ? 1 : KeyTraits<KTT>::QRY_BYTES, BMUL = QRY_BYTES / KEY_BYTES;
    const int half = (threadIdx.x & 63) >> 5;
    const size_t key_row_bytes = (size_t)d * KEY_BYTES;
    const unsigned char *qrow = static_cast<const unsigned char *>(queries) + (size_t)q * d * QRY_BYTES;
    const int n_groups = (int)(key_row_bytes / (Q8 || KT == KB_F32_SPLIT ? 64 : 32));
    const unsigned char *krow = static_cast<const unsigned char *>(keys) + (size_t)my_row * key_row_bytes + half * 16;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = KT == KB_F32_SPLIT ? SPLIT_START : 0.f;
    // The loads of UNR groups go out before their matrix instructions (the order of the accumulation does not
    // change): one memory round trip per UNR groups instead of one per group.
    if constexpr (KT == KB_F32_SPLIT) {
        const unsigned char *kp = krow + half * 16, *qp = qrow + half * 32;
        auto at = [](const unsigned char *base, int g, int piece) { return *reinterpret_cast<const u32x4 *>(base + (size_t)g * 64 + piece * 16); };
        auto step = [&](const u32x4 &a0, const u32x4 &a1, const u32x4 &b0, const u32x4 &b1) {
            Mma<KT>::run(acc, Mma<KT>::prepare(a0, a1, key_scale), Mma<KT>::prepare(b0, b1, query_scale));
        };
        int g = 0;
        for (; g + UNR <= n_groups; g += UNR) {
            u32x4 a0[UNR], a1[UNR], b0[UNR], b1[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                a0[u] = at(kp, g + u, 0);
                a1[u] = at(kp, g + u, 1);
                b0[u] = at(qp, g + u, 0);
                b1[u] = at(qp, g + u, 1);
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) step(a0[u], a1[u], b0[u], b1[u]);
        }
        for (; g < n_groups; ++g) step(at(kp, g, 0), at(kp, g, 1), at(qp, g, 0), at(qp, g, 1));
    } else if constexpr (Q8) {
        // one fp8 matrix instruction per 64-byte chunk: lane half h supplies bytes [32h, 32h+32) of its key row
        // and of the query row, the operand layout the scan uses, so both paths give the same bits
        const unsigned char *kp = krow + half * 16;
        auto step = [&](const u32x4 &a0, const u32x4 &a1, const u32x4 &b0, const u32x4 &b1) {
            const i32x8 av = {(int)a0[0], (int)a0[1], (int)a0[2], (int)a0[3], (int)a1[0], (int)a1[1], (int)a1[2], (int)a1[3]};
            const i32x8 bv = {(int)b0[0], (int)b0[1], (int)b0[2], (int)b0[3], (int)b1[0], (int)b1[1], (int)b1[2], (int)b1[3]};
            acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc, 0, 0, 0, 0, 0, 0);
        };
        int g = 0;
        for (; g + UNR <= n_groups; g += UNR) {
            u32x4 a0[UNR], a1[UNR], b0[UNR], b1[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                a0[u] = *reinterpret_cast<const u32x4 *>(kp + (size_t)(g + u) * 64);
                a1[u] = *reinterpret_cast<const u32x4 *>(kp + (size_t)(g + u) * 64 + 16);
                b0[u] = *reinterpret_cast<const u32x4 *>(qrow + (size_t)(g + u) * 64 + half * 32);
                b1[u] = *reinterpret_cast<const u32x4 *>(qrow + (size_t)(g + u) * 64 + half * 32 + 16);
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) step(a0[u], a1[u], b0[u], b1[u]);
        }
        for (; g < n_groups; ++g)
            step(*reinterpret_cast<const u32x4 *>(kp + (size_t)g * 64), *reinterpret_cast<const u32x4 *>(kp + (size_t)g * 64 + 16),
                 *reinterpret_cast<const u32x4 *>(qrow + (size_t)g * 64 + half * 32), *reinterpret_cast<const u32x4 *>(qrow + (size_t)g * 64 + half * 32 + 16));
    } else {
        const unsigned char *qbase = qrow + half * 16 * BMUL;
        int g = 0;
        for (; g + UNR <= n_groups; g += UNR) {
            u32x4 av[UNR], b0[UNR], b1[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                av[u] = *reinterpret_cast<const u32x4 *>(krow + (size_t)(g + u) * 32);
                const unsigned char *qp = qbase + (size_t)(g + u) * 32 * BMUL;
                b0[u] = *reinterpret_cast<const u32x4 *>(qp);
                b1[u] = BMUL == 2 ? *reinterpret_cast<const u32x4 *>(qp + 16) : b0[u];
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u) Mma<KTT>::run(acc, Mma<KTT>::prepare(av[u]), b0[u], b1[u]);
        }
        for (; g < n_groups; ++g) {
            const u32x4 av = *reinterpret_cast<const u32x4 *>(krow + (size_t)g * 32);
            const unsigned char *qp = qbase + (size_t)g * 32 * BMUL;
            const u32x4 b0 = *reinterpret_cast<const u32x4 *>(qp);
            const u32x4 b1 = BMUL == 2 ? *reinterpret_cast<const u32x4 *>(qp + 16) : b0;
            Mma<KTT>::run(acc, Mma<KTT>::prepare(av), b0, b1);
        }
    }
    return acc;
}

template <int KT> __device__ inline float key_scale_of(const float *inv_norm, int64_t row) { return KT == KB_F32_SPLIT ? f32_row_scale(inv_norm[row]) : 1.f; }
template <int KT> __device__ void exhaustive_query(const FinalArgs &a, int q, uint64_t *buf, uint32_t *ctl, SelectScratch *sc, int64_t row_begin,
                                                   int64_t row_end, const float *inv_q = nullptr)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, half = lane >> 5;
    const int cap = a.cand_cap;
    const bool filter = a.qmask != nullptr;
    const uint64_t qm = filter ? a.qmask[q] : 0;
    const float iq = inv_q ? *inv_q : a.invq[q];
    uint64_t *thr_local = reinterpret_cast<uint64_t *>(ctl + 2);   // ctl[0] = count, ctl[2..3] = threshold word
    if (tid == 0) {
        ctl[0] = 0;
        *thr_local = 0;
    }
    __syncthreads();
    for (int64_t row0 = row_begin; row0 < row_end; row0 += 128) {
        int64_t my_row = row0 + wave * 32 + lrow;
        if (my_row >= row_end) my_row = row_end - 1;
        const f32x16 acc = score_rows<KT, KT == KB_F32 || KT == KB_BF16 ? 16 : 8>(a.keys, a.queries, a.d, my_row, q);    // (16 where a group is two register quadruples, 8 where it is three or four)
        // every column holds the same query; lanes 0..15 of each half own one row each
        float v = acc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) v = (lrow == i) ? acc[i] : v;
        if (lrow < 16) {
            const int64_t row = row0 + wave * 32 + 8 * (lrow >> 2) + 4 * half + (lrow & 3);
            if (row < row_end && !row_removed(a.inv_norm[row]) && (!filter || (a.tags[row] & qm) != 0)) {
                float value = final_score(v, a.inv_norm[row], iq);
                if (a.draw.enabled) value = draw_key_of(value, a.draw, a.draw.first_query + (uint32_t)q, row);
                const uint64_t cw = pack_candidate(value, (uint32_t)row);
                if (cw > *thr_local && value > -__builtin_inff()) {
                    const uint32_t pos = atomicAdd(&ctl[0], 1u);
                    buf[pos] = cw;      // pos < cap: at most 128 appends between compactions
                }
            }
        }
        __syncthreads();
        const uint32_t n = ctl[0];
        if (n + 128 > (uint32_t)cap) {      // uniform: compact to the best k (sorted into buf[0..k))
            select_topk_desc(buf, (int)n, a.k, sc, tid, 256);
            if (tid == 0) {
                ctl[0] = n < (uint32_t)a.k ? n : (uint32_t)a.k;
                *thr_local = n >= (uint32_t)a.k ? buf[a.k - 1] : 0ull;
            }
            __syncthreads();
        }
    }
    select_topk_desc(buf, (int)ctl[0], a.k, sc, tid, 256);      // buf[0..k): the result in order, zero words where there is none
}

// ------------------------------------------------------------------------------------------------
// Whole-store plan, second launch: one workgroup per query selects from what the scan left of every group of rows.
//
// The k-th largest of the groups' best scores bounds the k-th best score from below (k distinct rows reach it).  It is
// found by counting the best scores in equal bins between the smallest and the largest: scores near the top of a store
// are sparse, so one pass of the counting leaves a handful of groups beyond the k wanted ones; only when many groups
// share the deciding bin is that bin divided again.  Of the groups that reach the bound two or three rows are known.
// Where a row that is not could reach it as well, the group is scored again, with the instruction sequence of the scan.  If
// that is more than one step of the workgroup, the k-th best of all known rows is found first, and only groups
// where such a row might come before that stay: at most about k / 2 (see WholePlan).
// 16,384 equal bf16 rows of 1024 elements and 8 queries, where every group ties: 24 us a call; when every group whose third
// row ties was scored again, 1502.  Everything that decides is a comparison of final scores, a non-decreasing function
// of the products, or of candidate words, which order equal scores by index.
// ------------------------------------------------------------------------------------------------
struct WholeSelectArgs {
    const void *keys, *queries;
    const float *inv_norm;
    const uint64_t *tags, *qmask;       // nullptr when no filter is applied
    const float *best;                  // ScanArgs::whole_best, whole_pair
    const u32x4 *pair;
    int32_t *out_index;
    float *out_score;
    uint64_t *stats;
    int64_t n_keys;
    int32_t k, d, groups, group_rows, tile_rows, tiles, grid;
    int32_t k_out;                      // results wanted, where k is a few more (split f32)
    uint64_t *gate;                     // split f32: the word that says whether the f32 instruction is needed; f32: as in ScanArgs
    int32_t more_lds;                   // bytes of dynamic LDS
    int32_t waves, per_group;        // StreamPlan (tiles: its units), where the scan was kb_stream_kernel
};
// 256 threads hold the groups: the kernel's length is a dozen barriers, which more wavefronts only make longer (64 queries
// x 2048 groups: 7.6 us with 256 threads, 8.2 with 1024)
constexpr int WHOLE_THREADS = 256;
constexpr int WHOLE_BINS = 256;          // four a lane of the wavefront that adds them up
constexpr int WHOLE_CAP = 4096;         // words gathered before they are cut down to the best k

// The k-th largest of the values that the threads of a workgroup of 256 hold, as a bound from below: counted in equal bins
// between the smallest and the largest value; only when many share the deciding bin is that bin divided again.
// -inf stands for no value.
struct KthBound {
    float lo, hi, scale;
    int bin_min;
    bool all;                   // fewer than k values: no bound, every value counts
    uint32_t reach;             // values that reach it (where `all` is not set: k at least)
    __device__ int bin_of(float f) const        // (never falls as f grows)
    {
        const int b = (int)((f - lo) * scale);
        return b < 0 ? 0 : b < WHOLE_BINS - 1 ? b : WHOLE_BINS - 1;
    }
    __device__ bool passes(float f) const { return all || f > hi || (f >= lo && bin_of(f) >= bin_min); }
};
struct KthScratch {
    __attribute__((aligned(16))) uint32_t hist[WHOLE_BINS];         // zero before the call, and after it
    float lo[2][WHOLE_THREADS / 64], hi[2][WHOLE_THREADS / 64];
    uint32_t bin, above, ge;
};
// v[u], u < rounds, are this thread's values (rounds uniform), lo and hi the smallest and largest of them.  All threads call it, converged.
template <int PER> __device__ __forceinline__ KthBound bound_kth(const float (&v)[PER], int rounds, float lo, float hi, uint32_t need, KthScratch &sh)
{
    constexpr float NONE = -__builtin_inff();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    KthBound r;
    r.lo = lo;
    r.hi = hi;
    r.scale = 0.f;
    r.bin_min = 0;
    r.all = false;
    r.reach = 0;
    // smallest and largest over the workgroup of what each thread has found (called converged, `turn` alternating)
    auto reduce_range = [&](float &lo, float &hi, int turn) {
        lo = wave_scan_min(lo);
        hi = wave_scan_max(hi);
        if (lane == 63) {
            sh.lo[turn][wave] = lo;
            sh.hi[turn][wave] = hi;
        }
        __syncthreads();
        lo = sh.lo[turn][0];
        hi = sh.hi[turn][0];
        for (int w = 1; w < WHOLE_THREADS / 64; ++w) {
            lo = __builtin_fminf(lo, sh.lo[turn][w]);
            hi = __builtin_fmaxf(hi, sh.hi[turn][w]);
        }
    };
    reduce_range(r.lo, r.hi, 0);
#pragma unroll 1
    for (int round = 0; round < 4 && r.hi >= r.lo; ++round) {
        r.scale = r.hi > r.lo ? (float)WHOLE_BINS / (r.hi - r.lo) : 0.f;
        if (!(r.scale < __builtin_inff())) r.scale = 0.f;
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (u < rounds && v[u] >= r.lo && v[u] <= r.hi) atomicAdd(&sh.hist[r.bin_of(v[u])], 1u);
        __syncthreads();
        if (tid < 64) {         // lane l owns bins 4 (63 - l) .. + 3: the scan over the lanes counts the higher bins
            u32x4 *h = reinterpret_cast<u32x4 *>(sh.hist) + (63 - lane);
            const u32x4 c = *h;
            *h = u32x4{0u, 0u, 0u, 0u};     // (for the next round)
            const uint32_t mine = c[0] + c[1] + c[2] + c[3];
            const uint32_t incl = wave_scan_add(mine);
            uint32_t above = incl - mine;
            if ((above < need && incl >= need) || (lane == 63 && incl < need)) {
                int b = 0;
                bool found = false;
                uint32_t ge = incl;
#pragma unroll
                for (int j = 3; j >= 0; --j) {
                    if (!found && above + c[j] >= need) {
                        found = true;
                        b = 4 * (63 - lane) + j;
                        ge = above + c[j];
                    } else if (!found) {
                        above += c[j];
                    }
                }
                sh.bin = (uint32_t)b;
                sh.above = above;
                sh.ge = ge;
            }
        }
        __syncthreads();
        r.bin_min = (int)sh.bin;
        const uint32_t ge = sh.ge;
        r.all = ge < need;
        if (ge <= 256u + need || r.scale == 0.f) {
            r.reach += ge;
            break;
        }
        // many share the deciding bin: its own range next
        need -= sh.above;
        r.reach += sh.above;
        float lo2 = __builtin_inff(), hi2 = NONE;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (v[u] >= r.lo && v[u] <= r.hi && r.bin_of(v[u]) == r.bin_min) {
                lo2 = __builtin_fminf(lo2, v[u]);
                hi2 = __builtin_fmaxf(hi2, v[u]);
            }
        }
        reduce_range(lo2, hi2, (round + 1) & 1);
        if (round == 3) r.reach += ge - sh.above;
        r.lo = lo2;
        r.hi = hi2;
        r.scale = 0.f;
        r.bin_min = 0;
    }
    return r;
}

// Split f32: the scores of the m rows in `words` as every other kernel has them for f32 rows, in place of those that selected them.  A dot
// product is v_mfma_f32_32x32x2f32's chain (0 4 1 5 2 6 3 7 of every eight elements) on the vector units, which has the same bits;
// the rows come through LDS a few columns at a time (stage: stage_bytes, 16-byte aligned).  256 threads, converged.
// So f32 scores don't depend on how many queries or rows a call has, nor does the order of those selected.
__device__ inline void restate(uint64_t *words, int m, const void *keys, const float *inv_norm, const void *query, int d, float inv_q, float *stage, int stage_bytes)
{
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int floats = stage_bytes / 4, batch = min(m, floats / 36 - 1);        // rows at a time, so that 32 columns fit (stage_bytes >= 8 KB)
    float dot = 0.f;
    for (int r0 = 0; r0 < m; r0 += batch) {
        const int rows = min(batch, m - r0), room = floats / (rows + 1) - 4;              // floats of a row at a time, four more against bank conflicts
        const int cols = room >= d ? d : room & ~31, stride = cols + 4;                   // (d is a multiple of 32)
        for (int c0 = 0; c0 < d; c0 += cols) {
            const int n = (d - c0 < cols ? d - c0 : cols) / 4;
            __syncthreads();
            for (int r = wave; r <= rows; r += 4) {
                const uint32_t row = r < rows ? candidate_index(words[r0 + r]) : 0u;
                const float *from = r < rows ? static_cast<const float *>(keys) + (size_t)__builtin_amdgcn_readfirstlane(row) * d : static_cast<const float *>(query);
                for (int at = 0; at < n; at += 64)
                    if (at + lane < n) __builtin_amdgcn_global_load_lds((const void *)(from + c0 + 4 * (at + lane)), (lds_ptr)(stage + r * stride + 4 * at), 16, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(0x0070 | 0x0F00);        // vmcnt(0)
            __syncthreads();
            if (tid >= r0 && tid < r0 + rows) {
                const f32x4 *a = reinterpret_cast<const f32x4 *>(stage + (tid - r0) * stride), *b = reinterpret_cast<const f32x4 *>(stage + rows * stride);
#pragma unroll 4
                for (int i = 0; i < n; i += 2) {
                    const f32x4 a0 = a[i], a1 = a[i + 1], b0 = b[i], b1 = b[i + 1];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        dot = __builtin_fmaf(a0[e], b0[e], dot);
                        dot = __builtin_fmaf(a1[e], b1[e], dot);
                    }
                }
            }
        }
    }
    __syncthreads();
    if (tid < m) {
        const uint32_t row = candidate_index(words[tid]);
        const float value = final_score(dot, inv_norm[row], inv_q);
        words[tid] = value > -__builtin_inff() ? pack_candidate(value, row) : 0ull;
    }
    __syncthreads();
}
// LDS for these rows beside what the selecting kernels have (their own buffers, in several rounds, where more queries than compute units would wait
// for each other)
int restate_lds(int32_t Q) { return Q > DEVICE_CUS ? 0 : RESTATE_LDS; }
// ... the place of thread tid's word among them, and the best k of them to the query's place in the output.
__device__ inline int restated_rank(const uint64_t *words, int m)
{
    const int tid = threadIdx.x;
    const uint64_t e = tid < m ? words[tid] : 0ull;
    int rank = 0;
#pragma unroll 8
    for (int j = 0; j < m; ++j) rank += words[j] > e || (e == 0ull && j < tid);       // (words without a score come last, as nothing)
    return rank;
}
__device__ inline void write_restated(const uint64_t *words, int m, int rank, int q, int k, int32_t *out_index, float *out_score)
{
    const int tid = threadIdx.x;
    const uint64_t e = tid < m ? words[tid] : 0ull;
    if (tid < m && rank < k) {
        out_index[(size_t)q * k + rank] = e ? (int32_t)candidate_index(e) : -1;
        out_score[(size_t)q * k + rank] = e ? candidate_score(e) : -__builtin_inff();
    }
    if (tid >= m && tid < k) {
        out_index[(size_t)q * k + tid] = -1;
        out_score[(size_t)q * k + tid] = -__builtin_inff();
    }
}
// Are the k best of the m rows that were scored again the query's results?  They are
//   if fewer than the `selected` rows asked for were there, as then all that qualify are among them;
//   if the k-th best f32 score lies above the lowest split score `last` of the selected rows by more than the two can differ: no row that was
//   not selected has a higher split score, so none has an f32 score that comes near (rows of extraordinary length have higher ones than all
//   others, and a row whose f32 products overflow has no f32 score);
//   if the query is zero: all scores are, and the rows were selected by their index.
// A query whose length is not ordinary, or not a number, is left to the f32 instruction.
__device__ inline bool restated_suffice(int m, int selected, float last, uint64_t kth, float square_sum, int d)
{
    if (square_sum == 0.f) return m < selected || kth != 0ull;
    if (!f32_ordinary(inv_norm_of(square_sum))) return false;
    return m < selected || (kth != 0ull && candidate_score(kth) > last + split_error(d));
}
// Where they are not, the rows whose split score is no further than that below the k-th f32 score are all that count.  If they are known and no
// more than these, they are scored again as well: a handful of copies of a row take a call 10 us longer and not the f32 instruction's scan.
constexpr int RESTATE_AGAIN = 256;

// The best k of the `have` words of `buf` go to sc->sel (256 threads, converged); returns how many there are.
__device__ __forceinline__ int best_to_scratch(uint64_t *buf, uint32_t have, int k, SelectScratch *sc)
{
    const int tid = threadIdx.x, m = (int)have < k ? (int)have : k;
    if (have <= 128u) {
        const uint64_t e = tid < (int)have ? buf[tid] : 0ull;
        int rank = 0;
#pragma unroll 8
        for (int j = 0; j < (int)have; ++j) rank += buf[j] > e;
        if (tid < (int)have && rank < k) sc->sel[rank] = e;
    } else {
        __syncthreads();
        select_topk_desc(buf, (int)have, k, sc, tid, WHOLE_THREADS);
        if (tid < m) sc->sel[tid] = buf[tid];
    }
    __syncthreads();
    return m;
}

// The best k of the `have` words of `buf`, in order, to a query's place in the output (256 threads, converged).
__device__ __forceinline__ void write_best(uint64_t *buf, uint32_t have, int q, int k, int32_t *out_index, float *out_score, SelectScratch *sc)
{
    const int tid = threadIdx.x;
    // the result in order: few words place themselves by counting the larger ones, many are cut down first
    const int m = (int)have < k ? (int)have : k;
    if (have <= 128u) {
        if (tid < (int)have) {
            const uint64_t e = buf[tid];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < (int)have; ++j) rank += buf[j] > e;
            if (rank < k) {
                out_index[(size_t)q * k + rank] = (int32_t)candidate_index(e);
                out_score[(size_t)q * k + rank] = candidate_score(e);
            }
        }
    } else {
        __syncthreads();
        select_topk_desc(buf, (int)have, k, sc, tid, WHOLE_THREADS);
        if (tid < m) {
            out_index[(size_t)q * k + tid] = (int32_t)candidate_index(buf[tid]);
            out_score[(size_t)q * k + tid] = candidate_score(buf[tid]);
        }
    }
    if (tid >= m && tid < k) {          // fewer than k qualify
        out_index[(size_t)q * k + tid] = -1;
        out_score[(size_t)q * k + tid] = -__builtin_inff();
    }
}

// PER: groups a thread holds.  (The kernel is a few microseconds long: instructions that a small store skips are fetched all the same.)
template <int KT, int PER, bool STREAM> __global__ __launch_bounds__(WHOLE_THREADS) void whole_select_kernel(WholeSelectArgs a)
{
    static_assert(PER * WHOLE_THREADS <= WHOLE_MAX_GROUPS);
    constexpr int QT = queries_of(KT);
    extern __shared__ __attribute__((aligned(16))) unsigned char more_lds[];        // split f32: see restate_lds
    __shared__ __attribute__((aligned(16))) uint64_t buf[WHOLE_CAP];
    __shared__ KthScratch kth;
    __shared__ uint16_t list[WHOLE_MAX_GROUPS], again[WHOLE_MAX_GROUPS];        // groups that reach the bound; with what is not known of them
    __shared__ SelectScratch sc;
    __shared__ float sh_iq, sh_square;
    __shared__ uint32_t sh_cnt, sh_listed, sh_again;
    __shared__ uint64_t sh_thr, sh_kth;
    if constexpr (KT == KB_F32) {
        if (a.gate != nullptr && *a.gate == 0) return;
    }
    constexpr int nt = WHOLE_THREADS, nw = nt / 64;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, k = a.k, groups = a.groups;
    constexpr float NONE = -__builtin_inff();
    const float *best = a.best + (size_t)q * groups;
    const u32x4 *pair = a.pair + (size_t)q * groups;
    // this thread's groups: tid, tid + nt, ...; their loads go out first
    const int rounds = (groups + nt - 1) / nt;
    float v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u)
        v[u] = u < rounds && tid + u * nt < groups ? best[tid + u * nt] : NONE;
    const uint64_t qm = a.qmask ? a.qmask[q] : 0ull;
    if (q == 0 && tid < STAT_WORDS + STAT_PARTIALS) a.stats[tid] = tid == 3 ? (uint64_t)a.grid : 0ull;
    if (tid < 64) {
        const float square_sum = row_square_sum<QT>(a.queries, q, a.d * bytes_of(QT), tid);
        if (tid == 0) {
            sh_iq = used_inv<KT>(inv_norm_of(square_sum));
            sh_square = square_sum;
            sh_cnt = sh_listed = sh_again = 0;
            sh_thr = sh_kth = 0;
        }
    }
    for (int i = tid; i < WHOLE_BINS; i += nt) kth.hist[i] = 0u;
    __syncthreads();
    if constexpr (KT == KB_F32_SPLIT) {        // (all scores of a zero query tie, so every group would be scored again)
        if (!f32_ordinary(inv_norm_of(sh_square))) {
            if (tid == 0) *a.gate = 1;
            return;
        }
    }
    const float iq = sh_iq;
    // score that no row behind a group's product exceeds (infinite products, of a query too long for its length to be a number, have
    // none themselves but stand for finite ones too)
    auto score_bound = [&](float product) { return __builtin_amdgcn_fmed3f(product, -0x1.fffffep127f, 0x1.fffffep127f) * iq + 0.0f; };
    float lo = __builtin_inff(), hi = NONE;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (v[u] > NONE) {
            v[u] = score_bound(v[u]);
            lo = __builtin_fminf(lo, v[u]);
            hi = __builtin_fmaxf(hi, v[u]);
        }
    }
    const KthBound bound = bound_kth(v, rounds, lo, hi, (uint32_t)k, kth);
    auto passes = [&](float f) { return bound.passes(f); };

    // row at a place of the tile of group g (the groups of a tile follow each other)
    const uint32_t per_tile = STREAM ? 1u : (uint32_t)a.tile_rows / (uint32_t)a.group_rows;
    auto row_at = [&](uint32_t g, uint32_t place) {
        if constexpr (STREAM) return (uint32_t)stream_group_row(a.tiles, a.waves, a.per_group, g, place);
        else return (uint32_t)whole_row((int32_t)(g / per_tile), a.tiles, a.tile_rows, (int)place);
    };
    auto first_place = [&](uint32_t g) { return STREAM ? 0u : g % per_tile * (uint32_t)a.group_rows; };
    auto append = [&](float product, uint32_t row) {
        const float f = product * iq + 0.0f;
        const uint64_t cw = pack_candidate(f, row);
        if (f > NONE && passes(f) && cw > sh_thr) buf[atomicAdd(&sh_cnt, 1u)] = cw;
    };
    // Cuts the `have` words gathered down to the best k and takes the k-th as the threshold (called converged, nobody
    // appending).
    auto cut = [&](uint32_t have) {
        select_topk_desc(buf, (int)have, k, &sc, tid, nt);
        if (tid == 0) {
            sh_cnt = have < (uint32_t)k ? have : (uint32_t)k;
            sh_thr = have >= (uint32_t)k ? buf[k - 1] : 0ull;
        }
        __syncthreads();
    };
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (u < rounds && v[u] > NONE && passes(v[u])) list[atomicAdd(&sh_listed, 1u)] = (uint16_t)(tid + u * nt);
    __syncthreads();
    const uint32_t listed = sh_listed;
    uint32_t have = 0;
    for (uint32_t j0 = 0; j0 < listed; j0 += (uint32_t)nt) {        // one group a thread: the rows known
        if (have + 3 * (uint32_t)nt > (uint32_t)WHOLE_CAP) cut(have);
        const uint32_t j = j0 + (uint32_t)tid;
        if (j < listed) {
            const uint32_t g = list[j];
            const u32x4 x = pair[g];
            append(best[g], row_at(g, x[2] & 255u));
            append(as_f32(x[0]), row_at(g, x[2] >> 8 & 255u));
            const uint32_t third = x[2] >> 16 & WHOLE_THIRD;
            if (third != 0u) append(as_f32(x[1]), row_at(g, third - 1u));
            if (as_f32(x[1]) > NONE && passes(score_bound(as_f32(x[1])))) again[atomicAdd(&sh_again, 1u)] = (uint16_t)g;
        }
        __syncthreads();
        have = sh_cnt;
        if (j0 + (uint32_t)nt < listed) __syncthreads();         // (everyone has the count that the next step moves on)
    }
    const uint32_t asked = listed > 0 ? sh_again : 0u;
    const uint32_t per = ((uint32_t)a.group_rows + 31) / 32;            // pieces of 32 rows, one a wavefront at a time
    uint32_t tasks = asked * per;
    const uint16_t *to_score = again;
    if (tasks > (uint32_t)nw) {         // more than one step of the workgroup: it pays to look again (a single one takes as long)
        __syncthreads();
        if (tid == 0) sh_listed = 0;
        if (have > (uint32_t)nt) {
            cut(have);
        } else {                    // few words: the one with k - 1 larger ones is the k-th
            const uint64_t e = tid < (int)have ? buf[tid] : 0ull;
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < (int)have; ++j) rank += buf[j] > e;
            if (tid < (int)have && rank == k - 1) sh_thr = e;
            __syncthreads();
        }
        // those of which a row that is not known could come before the k-th of those that are
        for (uint32_t j = (uint32_t)tid; j < asked; j += (uint32_t)nt) {
            const uint32_t g = again[j];
            const u32x4 x = pair[g];
            const float third = as_f32(x[1]), f = score_bound(third);
            const uint32_t place = x[2] >> 16 & WHOLE_THIRD;
            uint64_t most = pack_candidate(f, row_at(g, first_place(g)));       // (the group's lowest row)
            if (place != 0u) {          // known: the others' scores are lower, or equal at higher rows unless the rounding hides a difference
                const float below = ordered_to_score(score_to_ordered(third + 0.0f) - ((x[2] & WHOLE_NEAR) != 0u ? 1u : 3u));
                if (below * iq + 0.0f < f) most = pack_candidate(f, row_at(g, place - 1u));
            }
            if (most > sh_thr) list[atomicAdd(&sh_listed, 1u)] = (uint16_t)g;
        }
        __syncthreads();
        have = sh_cnt;
        tasks = sh_listed * per;
        to_score = list;
    }
    for (uint32_t t0 = 0; t0 < tasks; t0 += (uint32_t)nw) {
        __syncthreads();
        if (have + 32 * (uint32_t)nw > (uint32_t)WHOLE_CAP) cut(have);
        const uint32_t t = t0 + (uint32_t)wave;
        if (t < tasks) {
            const uint32_t g = to_score[t / per], in_group = t % per * 32, place0 = first_place(g) + in_group, known = pair[g][2];
            const int lrow = lane & 31, half = lane >> 5;
            const int64_t at = row_at(g, place0 + lrow), mine = at < a.n_keys ? at : a.n_keys - 1;      // (a place past a group of 16 is some other row)
            const f32x16 acc = score_rows<KT, KT == KB_F32 || KT == KB_BF16 ? 16 : 8>(a.keys, a.queries, a.d, mine, q, key_scale_of<KT>(a.inv_norm, mine), KT == KB_F32_SPLIT ? f32_row_scale(inv_norm_of(sh_square)) : 1.f);
            const float dot = select16(acc, lrow & 15);
            const uint32_t rel = 8 * ((lrow & 15) >> 2) + 4 * half + (lrow & 3), place = place0 + rel;
            const int64_t row = row_at(g, place);
            const bool listed_before = place == (known & 255u) || place == (known >> 8 & 255u) || place + 1u == (known >> 16 & WHOLE_THIRD);
            if (lrow < 16 && in_group + rel < (uint32_t)a.group_rows && row < a.n_keys && !listed_before) {
                const float ik = used_inv<KT>(a.inv_norm[row]);
                if (!row_removed(ik) && (!a.qmask || (a.tags[row] & qm) != 0)) append(dot * ik, (uint32_t)row);
            }
        }
        __syncthreads();
        have = sh_cnt;
    }
    if constexpr (KT == KB_F32_SPLIT) {
        const int m = best_to_scratch(buf, have, k, &sc);
        const float last = m == k ? candidate_score(sc.sel[k - 1]) : NONE, inv = inv_norm_of(sh_square);
        const float *query = static_cast<const float *>(a.queries) + (size_t)q * a.d;
        float *stage = a.more_lds ? reinterpret_cast<float *>(more_lds) : reinterpret_cast<float *>(buf + RESTATE_AGAIN);
        const int stage_bytes = a.more_lds ? a.more_lds : (int)(sizeof buf - sizeof(uint64_t) * RESTATE_AGAIN);
        restate(sc.sel, m, a.keys, a.inv_norm, query, a.d, inv, stage, stage_bytes);
        int rank = restated_rank(sc.sel, m);
        if (tid < m && rank == a.k_out - 1) sh_kth = sc.sel[tid];
        __syncthreads();
        bool done = restated_suffice(m, k, last, sh_kth, sh_square, a.d);       // (uniform)
        if (done) {
            write_restated(sc.sel, m, rank, q, a.k_out, a.out_index, a.out_score);
        } else if (sh_kth != 0ull) {
            const float reach = candidate_score(sh_kth) - split_error(a.d);
            if (tid == 0) sh_cnt = sh_again = 0;
            __syncthreads();
            auto put = [&](float product, uint32_t row) {
                const float f = product * iq + 0.0f;
                if (!(f >= reach)) return;
                const uint32_t at = atomicAdd(&sh_cnt, 1u);
                if (at < (uint32_t)RESTATE_AGAIN) buf[at] = pack_candidate(f, row);
            };
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                if (!(u < rounds && v[u] >= reach)) continue;
                const uint32_t g = (uint32_t)(tid + u * nt);
                const u32x4 x = pair[g];
                put(best[g], row_at(g, x[2] & 255u));
                put(as_f32(x[0]), row_at(g, x[2] >> 8 & 255u));
                if (as_f32(x[1]) > NONE && score_bound(as_f32(x[1])) >= reach) sh_again = 1;        // (a row that is not known may be one of them)
            }
            __syncthreads();
            const uint32_t n = sh_cnt;
            done = sh_again == 0 && n <= (uint32_t)RESTATE_AGAIN;
            if (done) {
                restate(buf, (int)n, a.keys, a.inv_norm, query, a.d, inv, stage, stage_bytes);
                rank = restated_rank(buf, (int)n);
                write_restated(buf, (int)n, rank, q, a.k_out, a.out_index, a.out_score);
            }
        }
        if (tid == 0 && !done) *a.gate = 1;
    } else write_best(buf, have, q, k, a.out_index, a.out_score, &sc);
}

// Dense plan, second launch: one workgroup per query selects from the products (KEYS: the keys of the weighted selection)
// of all rows.  PIECES: four values each that a thread holds.
struct DenseSelectArgs {
    const float *values;        // ScanArgs::dense
    const void *queries;
    int32_t *out_index;
    float *out_score;
    uint64_t *stats;
    int32_t k, d, n, stride, grid;
};
template <int QT, bool KEYS, int PIECES> __global__ __launch_bounds__(DENSE_THREADS) void dense_select_kernel(DenseSelectArgs a)
{
    static_assert(DENSE_THREADS == WHOLE_THREADS && PIECES * 4 * DENSE_THREADS <= DENSE_MAX_ROWS);
    constexpr int PER = 4 * PIECES;
    constexpr float NONE = -__builtin_inff();
    __shared__ __attribute__((aligned(16))) uint64_t buf[WHOLE_CAP];
    __shared__ KthScratch kth;
    __shared__ SelectScratch sc;
    __shared__ float sh_iq;
    __shared__ uint32_t sh_cnt;
    __shared__ uint64_t sh_thr;
    const int q = blockIdx.x, tid = threadIdx.x, k = a.k;
    const f32x4 *values = reinterpret_cast<const f32x4 *>(a.values + (size_t)q * a.stride);
    const int pieces = (a.n + 3) / 4, rounds = (pieces + DENSE_THREADS - 1) / DENSE_THREADS;      // (rounds <= PIECES; the scan has filled the last piece)
    float v[PER];
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const f32x4 x = tid + u * DENSE_THREADS < pieces ? values[tid + u * DENSE_THREADS] : f32x4{NONE, NONE, NONE, NONE};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * u + e] = x[e];
    }
    if (q == 0 && tid < STAT_WORDS + STAT_PARTIALS) a.stats[tid] = tid == 3 ? (uint64_t)a.grid : 0ull;
    if (!KEYS && tid < 64) {
        const float inv = row_inv_norm<QT>(a.queries, q, a.d * bytes_of(QT), tid);
        if (tid == 0) sh_iq = inv;
    }
    if (tid == 0) {
        sh_cnt = 0;
        sh_thr = 0;
    }
    for (int i = tid; i < WHOLE_BINS; i += DENSE_THREADS) kth.hist[i] = 0u;
    __syncthreads();
    const float iq = KEYS ? 0.f : sh_iq;
    float lo = __builtin_inff(), hi = NONE;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (v[u] > NONE) {
            if (!KEYS) v[u] = v[u] * iq + 0.0f;
            lo = __builtin_fminf(lo, v[u]);
            hi = __builtin_fmaxf(hi, v[u]);
        }
    }
    const KthBound bound = bound_kth(v, 4 * rounds, lo, hi, (uint32_t)k, kth);
    // the rows that reach it
    uint32_t have = 0;
    if (bound.reach <= (uint32_t)WHOLE_CAP) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (u < 4 * rounds && v[u] > NONE && bound.passes(v[u]))
                buf[atomicAdd(&sh_cnt, 1u)] = pack_candidate(v[u], (uint32_t)(4 * (tid + u / 4 * DENSE_THREADS) + u % 4));
        __syncthreads();
        have = sh_cnt;
    } else {        // equal values, most of all: read again, the buffer cut down to the best k whenever it is full
        for (int u = 0; u < rounds; ++u) {
            if (have + 4 * DENSE_THREADS > (uint32_t)WHOLE_CAP) {
                select_topk_desc(buf, (int)have, k, &sc, tid, DENSE_THREADS);
                if (tid == 0) {
                    sh_cnt = have < (uint32_t)k ? have : (uint32_t)k;
                    sh_thr = have >= (uint32_t)k ? buf[k - 1] : 0ull;
                }
                __syncthreads();
            }
            const int piece = tid + u * DENSE_THREADS;
            const f32x4 x = piece < pieces ? values[piece] : f32x4{NONE, NONE, NONE, NONE};
            const float val[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = KEYS || !(val[e] > NONE) ? val[e] : val[e] * sh_iq + 0.0f;
                const uint64_t cw = pack_candidate(w, (uint32_t)(4 * piece + e));
                if (w > NONE && bound.passes(w) && cw > sh_thr) buf[atomicAdd(&sh_cnt, 1u)] = cw;
            }
            __syncthreads();
            have = sh_cnt;
            __syncthreads();
        }
    }
    write_best(buf, have, q, k, a.out_index, a.out_score, &sc);
}

// Split f32, a list's rows: buf[0..a.k) are the best by the split products, in order.  best_again(word): the best SELECT_MAX of those
// that are not below the word, to buf in order.
template <class AGAIN> __device__ __forceinline__ void finish_split(const FinalArgs &a, int q, uint64_t *buf, SelectScratch *sc, unsigned char *smem_raw, uint64_t t64, AGAIN best_again)
{
    __shared__ float sh_square;
    __shared__ uint64_t sh_kth;
    const int tid = threadIdx.x;
    const float *query = static_cast<const float *>(a.queries) + (size_t)q * a.d;
    float *stage = reinterpret_cast<float *>(a.more_lds ? smem_raw + a.more_at : smem_raw);
    const int stage_bytes = a.more_lds ? a.more_lds : a.cand_cap * 8;
    if (tid < 64) {
        const float square_sum = row_square_sum<KB_F32>(a.queries, q, a.d * 4, tid);
        if (tid == 0) {
            sh_square = square_sum;
            sh_kth = 0;
        }
    }
    int rank = 0;
    float last = 0.f, inv = 0.f;
    auto again = [&](int most) {        // scores the best `most` of buf again; returns how many there are
        const uint64_t cw = tid < most ? buf[tid] : 0ull;
        if (tid < most) sc->sel[tid] = cw;
        const int m = __syncthreads_count(cw != 0ull);          // (the words without an entry come last)
        last = m == most ? candidate_score(sc->sel[most - 1]) : 0.f;
        inv = inv_norm_of(sh_square);
        restate(sc->sel, m, a.keys, a.inv_norm, query, a.d, inv, stage, stage_bytes);
        rank = restated_rank(sc->sel, m);
        if (tid < m && rank == a.k_out - 1) sh_kth = sc->sel[tid];
        __syncthreads();
        return m;
    };
    int m = again(a.k);
    bool done = restated_suffice(m, a.k, last, sh_kth, sh_square, a.d);       // (uniform)
    if (!done && sh_kth != 0ull && f32_ordinary(inv)) {
        const float reach = candidate_score(sh_kth) - split_error(a.d);
        const uint64_t word = (uint64_t)score_to_ordered(reach) << 32;
        if (word > t64) {       // the list has them all
            __syncthreads();
            best_again(word);
            m = again(SELECT_MAX);
            done = m < SELECT_MAX;
        }
    }
    if (done) write_restated(sc->sel, m, rank, q, a.k_out, a.out_index, a.out_score);
    if (tid == 0) {
        // what the scan behind this launch lists: nothing, or what reaches the k-th best f32 word known
        const float x = inv > 0.f && sh_kth != 0ull ? candidate_score(sh_kth) / inv : -__builtin_inff();
        a.thr64[q] = done ? ~0ull : sh_kth;
        a.thrp[q] = done ? __builtin_inff() : x - fabsf(x) * 0x1p-20f - 1e-30f;
        if (!done) a.stats[STAT_GATE] = 1;
    }
    if (tid < CAND_SEGMENTS) a.cnt[(size_t)q * CAND_SEGMENTS + tid] = 0;        // (everyone has read them)
}

template <int KT> __global__ __launch_bounds__(256) void finalize_kernel(FinalArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint64_t *buf = reinterpret_cast<uint64_t *>(smem_raw);
    uint32_t *ctl = reinterpret_cast<uint32_t *>(smem_raw + sizeof(uint64_t) * a.cand_cap);
    SelectScratch *sc = reinterpret_cast<SelectScratch *>(smem_raw + sizeof(uint64_t) * a.cand_cap + 16);
    const int q = blockIdx.x, part = blockIdx.y, tid = threadIdx.x;
    if constexpr (KT == KB_F32) {
        if (a.again && (a.stats[STAT_GATE] == 0 || (a.flag[q] == 0 && a.thr64[q] == ~0ull))) return;
    }
    // (the segment counters are asked for together with the flag: one memory round trip instead of two on the path
    // of every query; the parts that turn out to have nothing to do have read 64 bytes in vain)
    uint32_t seg_cnt[CAND_SEGMENTS];
    {
        const u32x4 *cp = reinterpret_cast<const u32x4 *>(a.cnt + (size_t)q * CAND_SEGMENTS);
#pragma unroll
        for (int v = 0; v < CAND_SEGMENTS / 4; ++v) {
            const u32x4 c4 = cp[v];
            seg_cnt[4 * v] = c4[0];
            seg_cnt[4 * v + 1] = c4[1];
            seg_cnt[4 * v + 2] = c4[2];
            seg_cnt[4 * v + 3] = c4[3];
        }
    }
    const bool flagged = a.flag[q] != 0 && a.n_keys > 0;
    if (!flagged && part != 0) return;
    if constexpr (KT == KB_F32_SPLIT) {
        if (flagged) {          // (the scan behind this launch has nothing to do for this query: the exhaustive one is that of f32 rows)
            if (tid < CAND_SEGMENTS) a.cnt[(size_t)q * CAND_SEGMENTS + tid] = 0;
            if (tid == 0) {
                a.thr64[q] = ~0ull;
                a.thrp[q] = __builtin_inff();
                a.stats[STAT_GATE] = 1;
            }
            return;
        }
    }
    if (KT != KB_F32_SPLIT && flagged) {
        // The grid has fb_parts workgroups per query; for a flagged query each scans its share of the rows and leaves
        // its best k as a sorted list, and the one that arrives last merges the lists.  (One workgroup alone would
        // read the whole knowledge base at the speed of a single compute unit.)
        const int64_t len = ((a.n_keys + a.fb_parts - 1) / a.fb_parts + 127) / 128 * 128;
        const int64_t begin = (int64_t)part * len, end = begin + len < a.n_keys ? begin + len : a.n_keys;
        uint64_t *mine = a.fb_lists + ((size_t)q * a.fb_parts + part) * a.k;
        if (begin < end) exhaustive_query<KT == KB_F32_SPLIT ? (int)KB_F32 : KT>(a, q, buf, ctl, sc, begin, end);
        if (tid < a.k) mine[tid] = begin < end ? buf[tid] : 0ull;
        __threadfence();                // the list is visible device-wide before the arrival is counted
        __syncthreads();
        if (tid == 0) ctl[1] = atomicAdd(&a.fb_done[q], 1u);
        __syncthreads();
        if (ctl[1] != (uint32_t)a.fb_parts - 1) return;
        __threadfence();
        const int n = a.fb_parts * a.k;                                  // <= cand_cap words
        const uint64_t *lists = a.fb_lists + (size_t)q * a.fb_parts * a.k;
        for (int i = tid; i < n; i += 256) buf[i] = __builtin_nontemporal_load(lists + i);
        __syncthreads();
        select_topk_desc(buf, n, a.k, sc, tid, 256);
        if (tid == 0) atomicAdd(reinterpret_cast<unsigned long long *>(a.stats + 1), 1ull);
    } else {
        // gather the query's segments into one contiguous list
        const uint32_t seg_cap = (uint32_t)a.cand_cap / CAND_SEGMENTS;
        uint32_t seg_n[CAND_SEGMENTS], seg_off[CAND_SEGMENTS], n = 0;
#pragma unroll
        for (int sg = 0; sg < CAND_SEGMENTS; ++sg) {
            uint32_t c = a.n_keys > 0 ? seg_cnt[sg] : 0;
            seg_n[sg] = c < seg_cap ? c : seg_cap;
            seg_off[sg] = n;
            n += seg_n[sg];
        }
        // Thread t takes positions t, t + 256, ... of the gathered list, four at a time: their loads are in flight
        // together, where a loop over the segments would wait for one segment's words before asking for the next.
        // A plain scan leaves (dot * inv_k, row) of live rows: each candidate is finished here as the scan's exact test
        // would have: the final score from the same three fp32 operations every kernel uses, nothing below the
        // threshold word.  What fails becomes a zero word, which sorts last.
        const float iq = used_inv<KT>(a.invq[q]);
        const uint64_t t64 = a.raw ? a.thr64[q] : 0ull;
        const uint64_t *lists = a.cand + (size_t)q * a.cand_cap;
        auto gather = [&](uint64_t least) {
            for (uint32_t j0 = tid; j0 < n; j0 += 4 * 256) {
                uint64_t w[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t j = j0 + u * 256;
                    uint32_t sg = 0, off = 0;
#pragma unroll
                    for (int s2 = 1; s2 < CAND_SEGMENTS; ++s2) {
                        const bool past = j >= seg_off[s2];
                        sg += past ? 1u : 0u;
                        off = past ? seg_off[s2] : off;
                    }
                    w[u] = j < n ? lists[sg * seg_cap + (j - off)] : 0ull;
                }
                if (a.raw) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint64_t c = pack_candidate(raw_candidate_product(w[u]) * iq + 0.0f, candidate_index(w[u]));
                        w[u] = (w[u] != 0ull && c >= least) ? c : 0ull;
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j0 + u * 256 < n) buf[j0 + u * 256] = w[u];
            }
            __syncthreads();
        };
        gather(t64);
        select_topk_desc(buf, (int)n, a.k, sc, tid, 256);
        if constexpr (KT == KB_F32_SPLIT) {
            finish_split(a, q, buf, sc, smem_raw, t64, [&](uint64_t least) {
                gather(least);
                select_topk_desc(buf, (int)n, SELECT_MAX, sc, tid, 256);
            });
            return;
        }
    }
    if (tid < a.k) {
        const uint64_t cw = tid < a.cand_cap ? buf[tid] : 0ull;
        a.out_index[(size_t)q * a.k + tid] = cw ? (int32_t)candidate_index(cw) : -1;
        a.out_score[(size_t)q * a.k + tid] = cw ? candidate_score(cw) : -__builtin_inff();
    }
}

// ------------------------------------------------------------------------------------------------
// Two-stage retrieval, second stage: exact top-k of one query over the rows of the clusters it probes.
// ------------------------------------------------------------------------------------------------
constexpr int PROBE_CAP = 1024;        // LDS candidate buffer of a partial scan (words); k <= 128 fits eight times
constexpr int PROBE_MAX = 64;          // clusters a query can probe: one list of 128 words each is MAX_CAND_CAP words, what the merge takes

// A wavefront's stream of 32 key rows and the query row through its own ring of chunks in LDS: every chunk is RB bytes of
// each row, loaded directly to LDS whole cache lines at a time (fp8: half lines, rows are multiples of 64 bytes), swizzled
// as in the tiled scan.  No wavefront waits for another.
template <int KT> struct ProbeRing {
    static constexpr bool Q8 = KT == KT_FP8_Q8;
    static constexpr int KTT = Q8 ? (int)KB_FP8_E4M3 : KT;
    static constexpr int KEY_BYTES = KeyTraits<KTT>::KEY_BYTES, QRY_BYTES = Q8 ? 1 : KeyTraits<KTT>::QRY_BYTES, BMUL = QRY_BYTES / KEY_BYTES;
    static constexpr int RB = KEY_BYTES == 1 ? 64 : 128, PPR = RB / 16;
    static constexpr int LOADS = 32 * RB / 1024;                        // load instructions for the keys of a chunk; one more for the query
    static constexpr int CHUNK = 32 * RB + 256;                         // ... whose bytes follow the keys' (RB * BMUL of 256)
    static constexpr int DEPTH = KEY_BYTES == 1 ? 14 : 8;
    static constexpr int BYTES = DEPTH * CHUNK;
    static_assert((LOADS + 1) * (DEPTH - 2) < 64 && RB * BMUL <= 256, "vmcnt is a 6-bit counter");
};

// score_rows with the rows taken through the ring (the same instruction sequence per element).
template <int KT> __device__ inline f32x16 score_rows_ring(const void *keys, const void *queries, int d, int64_t row_begin, int64_t row_end, int q,
                                                           unsigned char *ring)
{
    typedef ProbeRing<KT> R;
    typedef __attribute__((address_space(3))) void *lds_ptr;
    const int lane = threadIdx.x & 63, lrow = lane & 31, half = lane >> 5;
    const size_t row_bytes = (size_t)d * R::KEY_BYTES;
    const int NC = (int)(row_bytes / R::RB);
    const unsigned char *src[R::LOADS];
#pragma unroll
    for (int j = 0; j < R::LOADS; ++j) {
        const int r = j * (64 / R::PPR) + lane / R::PPR;
        const int64_t row = row_begin + r < row_end ? row_begin + r : row_end - 1;
        src[j] = static_cast<const unsigned char *>(keys) + (size_t)row * row_bytes + (((lane % R::PPR) ^ swizzle<R::PPR>(r)) * 16);
    }
    const unsigned char *qsrc = static_cast<const unsigned char *>(queries) + (size_t)q * d * R::QRY_BYTES + lane * 16;
    int issued = 0, slot = 0;
    auto issue = [&]() {
        unsigned char *dst = ring + slot * R::CHUNK;
#pragma unroll
        for (int j = 0; j < R::LOADS; ++j)
            __builtin_amdgcn_global_load_lds((const void *)(src[j] + (size_t)issued * R::RB), (lds_ptr)(dst + j * 1024), 16, 0, 0);
        if (lane < R::RB * R::BMUL / 16)
            __builtin_amdgcn_global_load_lds((const void *)(qsrc + (size_t)issued * R::RB * R::BMUL), (lds_ptr)(dst + 32 * R::RB), 16, 0, 0);
        ++issued;
        slot = slot + 1 == R::DEPTH ? 0 : slot + 1;
    };
    __builtin_amdgcn_s_waitcnt(waitcnt_lgkm0());        // (the ring's last readers: an earlier call of this wavefront)
    asm volatile("" ::: "memory");
    for (int s = 0; s < R::DEPTH - 1 && s < NC; ++s) issue();
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    int stage = 0;
    const int sw = swizzle<R::PPR>(lrow);
    for (int c = 0; c < NC; ++c) {
        if (c + (R::DEPTH - 2) < NC) __builtin_amdgcn_s_waitcnt(waitcnt_vm((R::LOADS + 1) * (R::DEPTH - 2)));
        else __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        asm volatile("" ::: "memory");
        const unsigned char *sA = ring + stage * R::CHUNK + lrow * R::RB, *sB = ring + stage * R::CHUNK + 32 * R::RB;
        if constexpr (R::Q8) {
            const u32x4 a0 = *reinterpret_cast<const u32x4 *>(sA + (((2 * half) ^ sw) << 4)), a1 = *reinterpret_cast<const u32x4 *>(sA + (((2 * half + 1) ^ sw) << 4));
            const u32x4 b0 = *reinterpret_cast<const u32x4 *>(sB + half * 32), b1 = *reinterpret_cast<const u32x4 *>(sB + half * 32 + 16);
            typename Mma<KB_FP8_Q8>::PrepA a;
            a.lo = a0;
            a.hi = a1;
            Mma<KB_FP8_Q8>::run(acc, a, b0, b1);
        } else {
#pragma unroll
            for (int g = 0; g < R::RB / 32; ++g) {
                const u32x4 a = *reinterpret_cast<const u32x4 *>(sA + (((2 * g + half) ^ sw) << 4));
                const u32x4 b0 = *reinterpret_cast<const u32x4 *>(sB + (g * 2 + half) * 16 * R::BMUL);
                const u32x4 b1 = R::BMUL == 2 ? *reinterpret_cast<const u32x4 *>(sB + (g * 2 + half) * 32 + 16) : b0;
                Mma<R::KTT>::run(acc, Mma<R::KTT>::prepare(a), b0, b1);
            }
        }
        stage = stage + 1 == R::DEPTH ? 0 : stage + 1;
        asm volatile("" ::: "memory");      // (the slot of the chunk before: its fragments went into matrix instructions issued by now)
        if (c + (R::DEPTH - 1) < NC) issue();
    }
    return acc;
}

constexpr int PROBE_WAVES = 2;              // scoring wavefronts of a block, 32 rows each at a time; one more forms 1/|q| meanwhile
constexpr int PROBE_THREADS = 64 * (PROBE_WAVES + 1);
template <int KT> size_t probe_scan_lds() { return (size_t)PROBE_WAVES * ProbeRing<KT>::BYTES + PROBE_CAP * 8 + sizeof(SelectScratch); }

// Block (p, s, q): part s of `splits` of the rows of cluster probe[q][p], scored exactly as the scan kernels score
// (same MFMA sequence per element), best k written as a sorted list of candidate words (zero = no entry).
// Every block computes 1/|q| of its query itself (one wavefront, the row-norm routine every path uses: the same bits),
// which saves the launch that would do it once per query.  Such a call is bound by the latency of its loads: seven chunks
// of 128 bytes of each of a wavefront's 32 rows are in flight at once (fp8: thirteen of 64).  8 queries, four clusters of about 1000 rows of 1024
// bf16 values each (65 MB): 20.7 us, 32.7 us with fragments loaded to registers, a quarter of a row at a time and each
// lane from a row of its own.
template <int KT> __global__ __launch_bounds__(PROBE_THREADS) void probe_scan_kernel(FinalArgs a, const int64_t *cluster_offsets, int n_clusters,
                                                                                        const int32_t *probe, int nprobe, int splits, uint64_t *lists)
{
    constexpr int QT = queries_of(KT);
    constexpr int THREADS = PROBE_THREADS, STEP = 32 * PROBE_WAVES;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint64_t *buf = reinterpret_cast<uint64_t *>(smem_raw + PROBE_WAVES * ProbeRing<KT>::BYTES);
    SelectScratch *sc = reinterpret_cast<SelectScratch *>(smem_raw + PROBE_WAVES * ProbeRing<KT>::BYTES + PROBE_CAP * 8);
    __shared__ uint32_t count;
    __shared__ uint64_t thr_local;
    __shared__ float inv_q;
    const int p = blockIdx.x, s = blockIdx.y, q = blockIdx.z, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, half = lane >> 5;
    uint64_t *out = lists + ((size_t)q * nprobe * splits + (size_t)p * splits + s) * a.k;
    const int c = probe[(size_t)q * nprobe + p];
    bool first = true;          // a cluster named twice is scanned once (the merge takes distinct entries)
    for (int e = 0; e < p; ++e) first = first && probe[(size_t)q * nprobe + e] != c;
    int64_t begin = 0, end = 0;
    if (first && c >= 0 && c < n_clusters) {
        const int64_t cb = cluster_offsets[c], ce = cluster_offsets[c + 1];
        if (cb >= 0 && ce <= a.n_keys && cb < ce) {
            const int64_t len = ((ce - cb + splits - 1) / splits + STEP - 1) / STEP * STEP;    // whole steps
            begin = cb + (int64_t)s * len;
            end = begin + len < ce ? begin + len : ce;
        }
    }
    if (begin >= end) {         // workgroup-uniform
        for (int i = tid; i < a.k; i += THREADS) out[i] = 0ull;
        return;
    }
    if (tid == 0) {
        count = 0;
        thr_local = 0;
    }
    const uint64_t qm = a.qmask ? a.qmask[q] : 0;
    for (int64_t row0 = begin; row0 < end; row0 += STEP) {
        const int64_t base = row0 + wave * 32;
        const int64_t row = base + 8 * ((lrow & 15) >> 2) + 4 * half + (lrow & 3);      // lanes 0..15 of each half own one row each
        const int64_t at = row < end ? row : end - 1;
        const float ik = a.inv_norm[at];
        const uint64_t tag = a.qmask ? a.tags[at] : 0;
        float dot = 0.f;
        if (wave < PROBE_WAVES && base < end) dot = select16(score_rows_ring<KT>(a.keys, a.queries, a.d, base, end, q, smem_raw + wave * ProbeRing<KT>::BYTES), lrow & 15);
        if (row0 == begin) {
            if (wave == PROBE_WAVES) {
                const float inv = row_inv_norm<QT>(a.queries, q, a.d * bytes_of(QT), lane);
                if (lane == 0) inv_q = inv;
            }
            __syncthreads();
        }
        if (wave < PROBE_WAVES && lrow < 16 && row < end && !row_removed(ik) && (!a.qmask || (tag & qm) != 0)) {
            const float value = final_score(dot, ik, inv_q);
            const uint64_t cw = pack_candidate(value, (uint32_t)row);
            if (cw > thr_local && value > -__builtin_inff()) buf[atomicAdd(&count, 1u)] = cw;      // < PROBE_CAP: at most STEP appends between compactions
        }
        __syncthreads();
        const uint32_t n = count;
        if (n + STEP > (uint32_t)PROBE_CAP) {      // uniform: compact to the best k (sorted into buf[0..k))
            select_topk_desc(buf, (int)n, a.k, sc, tid, THREADS);
            if (tid == 0) {
                count = n < (uint32_t)a.k ? n : (uint32_t)a.k;
                thr_local = n >= (uint32_t)a.k ? buf[a.k - 1] : 0ull;
            }
        }
        __syncthreads();        // (everyone has read the count that the next step moves on)
    }
    const int n = (int)count;
    if (n <= THREADS) {         // a block of one or two steps: every word finds its place by counting the larger ones
        if (tid < n) {
            const uint64_t e = buf[tid];
            int rank = 0;
#pragma unroll 8
            for (int j = 0; j < n; ++j) rank += buf[j] > e;
            if (rank < a.k) out[rank] = e;
        }
        for (int i = n + tid; i < a.k; i += THREADS) out[i] = 0ull;
        return;
    }
    select_topk_desc(buf, n, a.k, sc, tid, THREADS);
    for (int i = tid; i < a.k; i += THREADS) out[i] = buf[i];
}

// A small knowledge base, block (s, q): part s of the rows, as above but with fragments loaded to registers.  It takes the
// calls whose k is large for the number of rows, which the whole-store plan leaves, where they bring memory for the lists of
// the parts but not for the products of the dense plan (1000 x 768 bf16 rows, 8 queries, k = 128: 28 us, the dense plan 16).
// stats: the diagnostics of a query that took this path: no candidates, no sampling, one workgroup per block.
template <int KT> __global__ __launch_bounds__(256) void small_scan_kernel(FinalArgs a, uint64_t *lists, uint64_t *stats)
{
    constexpr int QT = queries_of(KT);
    __shared__ __attribute__((aligned(16))) uint64_t buf[PROBE_CAP];
    __shared__ uint32_t ctl[4];
    __shared__ SelectScratch sc;
    __shared__ float inv_q;
    const int s = blockIdx.x, parts = gridDim.x, q = blockIdx.y, tid = threadIdx.x;
    if (s == 0 && q == 0 && tid < STAT_WORDS + STAT_PARTIALS) stats[tid] = tid == 3 ? (uint64_t)gridDim.x * gridDim.y : 0ull;
    uint64_t *out = lists + ((size_t)q * parts + s) * a.k;
    const int64_t len = ((a.n_keys + parts - 1) / parts + 127) / 128 * 128;    // whole steps of the scorer
    const int64_t begin = (int64_t)s * len, end = begin + len < a.n_keys ? begin + len : a.n_keys;
    if (begin >= end) {         // workgroup-uniform
        if (tid < a.k) out[tid] = 0ull;
        return;
    }
    if (tid < 64) {
        const float inv = row_inv_norm<QT>(a.queries, q, a.d * bytes_of(QT), tid);
        if (tid == 0) inv_q = inv;
    }
    __syncthreads();
    exhaustive_query<KT>(a, q, buf, ctl, &sc, begin, end, &inv_q);
    if (tid < a.k) out[tid] = buf[tid];
}

__global__ __launch_bounds__(1024) void probe_merge_kernel(const uint64_t *lists, int n_lists, int k, int32_t *out_index, float *out_score)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    uint64_t *buf = reinterpret_cast<uint64_t *>(smem_raw);
    const int n = n_lists * k, q = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    SelectScratch *sc = reinterpret_cast<SelectScratch *>(smem_raw + sizeof(uint64_t) * (size_t)(n > k ? n : k) + 16);
    for (int i = tid; i < n; i += nt) buf[i] = lists[(size_t)q * n + i];
    __syncthreads();
    select_topk_desc(buf, n, k, sc, tid, nt);
    if (tid < k) {
        const uint64_t cw = buf[tid];
        out_index[(size_t)q * k + tid] = cw ? (int32_t)candidate_index(cw) : -1;
        out_score[(size_t)q * k + tid] = cw ? candidate_score(cw) : -__builtin_inff();
    }
}

template <int KT> hipError_t launch_probe_scan(const dim3 &grid, const FinalArgs &f, const int64_t *cluster_offsets_dev, int32_t n_clusters,
                                               const int32_t *probe_dev, int32_t nprobe, int splits, uint64_t *lists, hipStream_t s)
{
    static_assert(2 * (PROBE_WAVES * ProbeRing<KT>::BYTES + PROBE_CAP * 8 + sizeof(SelectScratch) + 64) <= 160 * 1024, "two blocks share a compute unit");
    static LdsAllowed allowed;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&probe_scan_kernel<KT>), allowed, probe_scan_lds<KT>()); e != hipSuccess) return e;
    hipLaunchKernelGGL(probe_scan_kernel<KT>, grid, dim3(PROBE_THREADS), probe_scan_lds<KT>(), s, f, cluster_offsets_dev, n_clusters, probe_dev, nprobe, splits, lists);
    return hipGetLastError();
}
template <int KT> auto threshold_once(int slots) -> void (*)(ThresholdArgs)
{
    return slots <= 2048 ? &threshold_kernel<KB_BF16, false, KT, 2> : &threshold_kernel<KB_BF16, false, KT, 8>;
}
template <int KT, bool STREAM> auto whole_select(int groups) -> void (*)(WholeSelectArgs)
{
    return groups <= 4 * WHOLE_THREADS ? &whole_select_kernel<KT, 4, STREAM> : groups <= 8 * WHOLE_THREADS ? &whole_select_kernel<KT, 8, STREAM> : &whole_select_kernel<KT, 16, STREAM>;
}
template <bool STREAM> auto whole_select_for(int kt, int groups) -> void (*)(WholeSelectArgs)
{
    return kt == KB_F32 ? whole_select<KB_F32, STREAM>(groups) : kt == KB_F32_SPLIT ? whole_select<KB_F32_SPLIT, STREAM>(groups) : kt == KB_BF16 ? whole_select<KB_BF16, STREAM>(groups)
         : kt == KB_FP8_E4M3 ? whole_select<KB_FP8_E4M3, STREAM>(groups) : whole_select<KT_FP8_Q8, STREAM>(groups);
}
template <int QT, bool KEYS> void launch_dense_select(const DenseSelectArgs &t, int32_t Q, hipStream_t s)
{
    void (*fn)(DenseSelectArgs) = t.n <= 4096 ? &dense_select_kernel<QT, KEYS, 4> : t.n <= 8192 ? &dense_select_kernel<QT, KEYS, 8> : &dense_select_kernel<QT, KEYS, 16>;
    hipLaunchKernelGGL(fn, dim3(Q), dim3(DENSE_THREADS), 0, s, t);
}

hipError_t launch_scan(kb_dtype_t dt, int config, int family, bool sample, int grid, const ScanArgs &a, hipStream_t s)
{
    if (family == 4)
        return dt == KB_BF16 ? launch_scan_wide_bf16(config, sample, grid, a, s)
               : dt == KB_FP8_E4M3 ? launch_scan_wide_fp8(config, sample, grid, a, s) : hipErrorInvalidValue;
    if (family == 3)
        return dt == KB_BF16 ? launch_scan_sp_bf16(config, sample, grid, a, s)
               : dt == KB_FP8_E4M3 ? launch_scan_sp_fp8(config, sample, grid, a, s) : hipErrorInvalidValue;
    switch (dt) {
    case KB_F32: return a.split ? launch_scan_f32_split(config, sample, grid, a, s) : launch_scan_f32(config, sample, grid, a, s);
    case KB_BF16: return launch_scan_bf16(config, sample, grid, a, s);
    default: return launch_scan_fp8(config, sample, grid, a, s);
    }
}

bool valid_dtype(int t) { return t == KB_F32 || t == KB_BF16 || t == KB_FP8_E4M3; }

}  // namespace

// ------------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------------
extern "C" {

kb_status_t kb_create(kb_t **out, int32_t d, kb_dtype_t key_dtype, int64_t capacity, void *keys_dev, float *row_scale_dev,
                      float *inv_norm_dev, uint64_t *tags_dev)
{
    if (!out) return KB_ERR_NULL;
    *out = nullptr;
    if (!valid_dtype((int)key_dtype)) return KB_ERR_DTYPE;
    if (!keys_dev || !inv_norm_dev) return KB_ERR_NULL;
    if (key_dtype == KB_FP8_E4M3 && !row_scale_dev) return KB_ERR_NULL;
    if (key_dtype != KB_FP8_E4M3 && row_scale_dev) return KB_ERR_INVALID_ARG;
    const int granule = key_dtype == KB_F32 ? 32 : 64;
    if (d <= 0 || d % granule != 0 || d > 16384) return KB_ERR_INVALID_ARG;
    if (capacity < 1 || capacity >= ((int64_t)1 << 31)) return KB_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(keys_dev) & 15) != 0) return KB_ERR_INVALID_ARG;
    kb *h = new (std::nothrow) kb();
    if (!h) return KB_ERR_INVALID_ARG;
    h->d = d;
    h->dtype = key_dtype;
    h->capacity = capacity;
    h->n = h->n_normalized = 0;
    h->keys = keys_dev;
    h->row_scale = row_scale_dev;
    h->inv_norm = inv_norm_dev;
    h->tags = tags_dev;
    h->tune_sample_keys = h->tune_config = h->tune_wg_per_cu = h->tune_no_small_path = 0;
    h->prof_events = nullptr;
    h->prof_max = h->prof_used = 0;
    h->prof_stride = 1;
    h->prof_seen = 0;
    *out = h;
    return KB_OK;
}

// Whether these bytes are memory of the present device, aligned and all within one allocation: a kernel moves them as a copy by the runtime would.
static bool within_reach(const void *at, size_t alignment, size_t bytes)
{
    if ((reinterpret_cast<uintptr_t>(at) & (alignment - 1)) != 0) return false;
    hipPointerAttribute_t attr;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    int dev = -1;
    if (hipPointerGetAttributes(&attr, at) != hipSuccess || attr.type != hipMemoryTypeDevice || hipGetDevice(&dev) != hipSuccess || attr.device != dev ||
        hipMemGetAddressRange(&base, &size, const_cast<void *>(at)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const size_t before = (size_t)(static_cast<const unsigned char *>(at) - static_cast<const unsigned char *>(base));
    return before <= size && bytes <= size - before;
}

kb_status_t kb_append(kb_t *kb, const void *rows_dev, const float *row_scale_dev, const uint64_t *tags_dev, int64_t n,
                      void *hip_stream, int64_t *first_index_out)
{
    if (!kb) return KB_ERR_NULL;
    if (n < 0) return KB_ERR_INVALID_ARG;
    if (n == 0) {
        if (first_index_out) *first_index_out = kb->n;
        return KB_OK;
    }
    if (!rows_dev) return KB_ERR_NULL;
    if (kb->dtype == KB_FP8_E4M3 && !row_scale_dev) return KB_ERR_NULL;
    if (kb->tags && !tags_dev) return KB_ERR_NULL;
    if (kb->n + n > kb->capacity) return KB_ERR_CAPACITY;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const size_t row_bytes = (size_t)kb->d * key_bytes(kb->dtype);
    void *dst = static_cast<unsigned char *>(kb->keys) + (size_t)kb->n * row_bytes;
    float *scale_to = kb->dtype == KB_FP8_E4M3 && kb->row_scale + kb->n != row_scale_dev ? kb->row_scale + kb->n : nullptr;
    uint64_t *tags_to = kb->tags && kb->tags + kb->n != tags_dev ? kb->tags + kb->n : nullptr;
    const bool rows_move = dst != rows_dev;
    // One launch instead of two or three copies where the kernel can reach both sides: memory of this device, as a whole, words at their own
    // alignment.  (The runtime copies the rest, or refuses it.  A single copy stays with it: it takes the host 1 to 2 us less than the checks and
    // the launch do.  741 x 768 f32 rows appended, normalized and asked about three times: 81 us, 87 with this kernel.)
    auto reached = [](const void *to, const void *from, size_t alignment, size_t bytes) {
        return within_reach(to, alignment, bytes) && within_reach(from, alignment, bytes);
    };
    const bool several = (int)rows_move + (scale_to != nullptr) + (tags_to != nullptr) > 1;
    // (not with an error of the caller's pending, which the checks and the launch would take for theirs: a copy says itself how it went)
    const bool direct = several && hipPeekAtLastError() == hipSuccess && (!rows_move || reached(dst, rows_dev, 16, row_bytes * n)) && (!scale_to || reached(scale_to, row_scale_dev, 4, sizeof(float) * n)) &&
                        (!tags_to || reached(tags_to, tags_dev, 8, sizeof(uint64_t) * n));
    if (direct) {
        AppendArgs a;
        a.rows = static_cast<const u32x4 *>(rows_dev);
        a.rows_to = static_cast<u32x4 *>(dst);
        a.scale = reinterpret_cast<const uint32_t *>(row_scale_dev);
        a.scale_to = reinterpret_cast<uint32_t *>(scale_to);
        a.tags = tags_dev;
        a.tags_to = tags_to;
        a.pieces = rows_move ? (int64_t)(row_bytes / 16) * n : 0;
        a.n = scale_to || tags_to ? n : 0;
        a.row_blocks = (int32_t)ceil_div(a.pieces, 256 * APPEND_PIECES);
        const int64_t blocks = a.row_blocks + ceil_div(a.n, 256);
        if (blocks > 0) {
            hipLaunchKernelGGL(append_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
            if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
        }
    } else {
        if (rows_move && hipMemcpyAsync(dst, rows_dev, row_bytes * n, hipMemcpyDeviceToDevice, s) != hipSuccess) return KB_ERR_DEVICE;
        if (scale_to && hipMemcpyAsync(scale_to, row_scale_dev, sizeof(float) * n, hipMemcpyDeviceToDevice, s) != hipSuccess) return KB_ERR_DEVICE;
        if (tags_to && hipMemcpyAsync(tags_to, tags_dev, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, s) != hipSuccess) return KB_ERR_DEVICE;
    }
    if (first_index_out) *first_index_out = kb->n;
    kb->n += n;
    return KB_OK;
}

kb_status_t kb_normalize(kb_t *kb, void *hip_stream)
{
    if (!kb) return KB_ERR_NULL;
    const int64_t begin = kb->n_normalized, end = kb->n;
    if (end <= begin) return KB_OK;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const unsigned grid = (unsigned)ceil_div(end - begin, 4);
    switch (kb->dtype) {
    case KB_F32: hipLaunchKernelGGL(row_norm_kernel<KB_F32>, dim3(grid), dim3(256), 0, s, kb->keys, begin, end, kb->d, kb->inv_norm); break;
    case KB_BF16: hipLaunchKernelGGL(row_norm_kernel<KB_BF16>, dim3(grid), dim3(256), 0, s, kb->keys, begin, end, kb->d, kb->inv_norm); break;
    default: hipLaunchKernelGGL(row_norm_kernel<KB_FP8_E4M3>, dim3(grid), dim3(256), 0, s, kb->keys, begin, end, kb->d, kb->inv_norm); break;
    }
    if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    kb->n_normalized = end;
    return KB_OK;
}

// ------------------------------------------------------------------------------------------------
// Two-stage retrieval, second stage (host side)
// ------------------------------------------------------------------------------------------------
namespace {

// Parts a cluster's rows are split into, so that a small batch still fills the device, as far as the merge can take the
// partial lists: a function of (Q, nprobe, k) only.
int probe_splits(int Q, int k, int nprobe)
{
    int64_t s = (4 * (int64_t)DEVICE_CUS + (int64_t)Q * nprobe - 1) / ((int64_t)Q * nprobe);
    if (s > 16) s = 16;
    if (s > MAX_CAND_CAP / k / nprobe) s = MAX_CAND_CAP / k / nprobe;
    return s < 1 ? 1 : (int)s;
}

struct ProbePlan {
    int splits;
    size_t off_lists, total;
};

// `few`: no more than 64 lists per query.  Enough for the same results, in less memory where k is small; a call that brings
// only that much runs so.
bool make_probe_plan(int32_t Q, int32_t k, int32_t nprobe, ProbePlan *out, bool few = false)
{
    if (Q < 1 || Q > 65535 || k < 1 || k > KB_K_MAX || nprobe < 1 || nprobe > PROBE_MAX) return false;
    ProbePlan p;
    p.splits = probe_splits(Q, few ? KB_K_MAX : k, nprobe);
    p.off_lists = 0;
    p.total = p.off_lists + align_up((size_t)Q * nprobe * p.splits * k * 8);
    *out = p;
    return true;
}


// The merge of a query's sorted lists, the second launch of the two paths below.
kb_status_t launch_merge(const uint64_t *lists, int n_lists, int32_t Q, int32_t k, int32_t *indices_out_dev, float *scores_out_dev, hipStream_t s)
{
    const int n = n_lists * k, threads = n > 1024 ? 1024 : n > 512 ? 512 : 256;
    const size_t merge_lds = sizeof(uint64_t) * (size_t)(n > k ? n : k) + 16 + sizeof(SelectScratch);
    static LdsAllowed merge_allowed;
    if (allow_dynamic_lds(reinterpret_cast<const void *>(&probe_merge_kernel), merge_allowed, MAX_CAND_CAP * 8 + 16 + sizeof(SelectScratch)) != hipSuccess)
        return KB_ERR_DEVICE;
    hipLaunchKernelGGL(probe_merge_kernel, dim3(Q), dim3(threads), merge_lds, s, lists, n_lists, k, indices_out_dev, scores_out_dev);
    return hipGetLastError() == hipSuccess ? KB_OK : KB_ERR_DEVICE;
}

FinalArgs list_scan_args(const kb *h, const void *queries_dev, const uint64_t *qmask_dev, int32_t k)
{
    FinalArgs f;
    memset(&f, 0, sizeof f);
    f.keys = h->keys;
    f.inv_norm = h->inv_norm;
    f.tags = h->tags;
    f.queries = queries_dev;
    f.qmask = qmask_dev;
    f.n_keys = h->n;
    f.d = h->d;
    f.k = k;
    f.cand_cap = PROBE_CAP;
    return f;
}

// The two launches behind kb_query_probe.
kb_status_t launch_probe(kb *h, const void *queries_dev, bool q8, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                         const int64_t *cluster_offsets_dev, int32_t n_clusters, const int32_t *probe_dev, int32_t nprobe, int splits,
                         uint64_t *lists, int32_t *indices_out_dev, float *scores_out_dev, hipStream_t s)
{
    const FinalArgs f = list_scan_args(h, queries_dev, qmask_dev, k);
    const dim3 grid(nprobe, splits, Q);
    hipError_t e;
    switch (q8 ? KT_FP8_Q8 : (int)h->dtype) {
    case KB_F32: e = launch_probe_scan<KB_F32>(grid, f, cluster_offsets_dev, n_clusters, probe_dev, nprobe, splits, lists, s); break;
    case KB_BF16: e = launch_probe_scan<KB_BF16>(grid, f, cluster_offsets_dev, n_clusters, probe_dev, nprobe, splits, lists, s); break;
    case KB_FP8_E4M3: e = launch_probe_scan<KB_FP8_E4M3>(grid, f, cluster_offsets_dev, n_clusters, probe_dev, nprobe, splits, lists, s); break;
    default: e = launch_probe_scan<KT_FP8_Q8>(grid, f, cluster_offsets_dev, n_clusters, probe_dev, nprobe, splits, lists, s); break;
    }
    return e == hipSuccess ? launch_merge(lists, nprobe * splits, Q, k, indices_out_dev, scores_out_dev, s) : KB_ERR_DEVICE;
}

// kb_query on a small knowledge base that the whole-store plan leaves, with too little memory for the dense plan: two launches.
kb_status_t launch_small(kb *h, const void *queries_dev, bool q8, int32_t Q, const uint64_t *qmask_dev, int32_t k, int parts, uint64_t *lists,
                         uint64_t *stats, int32_t *indices_out_dev, float *scores_out_dev, hipStream_t s)
{
    const FinalArgs f = list_scan_args(h, queries_dev, qmask_dev, k);
    const dim3 grid(parts, Q);
    const bool timed = h->prof_events && h->prof_used < h->prof_max && h->prof_seen++ % h->prof_stride == h->prof_stride / 2;     // the scoring kernel stands for the scan
    if (timed && hipEventRecord(h->prof_events[2 * h->prof_used], s) != hipSuccess) return KB_ERR_DEVICE;
    switch (q8 ? KT_FP8_Q8 : (int)h->dtype) {
    case KB_F32: hipLaunchKernelGGL(small_scan_kernel<KB_F32>, grid, dim3(256), 0, s, f, lists, stats); break;
    case KB_BF16: hipLaunchKernelGGL(small_scan_kernel<KB_BF16>, grid, dim3(256), 0, s, f, lists, stats); break;
    case KB_FP8_E4M3: hipLaunchKernelGGL(small_scan_kernel<KB_FP8_E4M3>, grid, dim3(256), 0, s, f, lists, stats); break;
    default: hipLaunchKernelGGL(small_scan_kernel<KT_FP8_Q8>, grid, dim3(256), 0, s, f, lists, stats); break;
    }
    if (timed) {
        if (hipEventRecord(h->prof_events[2 * h->prof_used + 1], s) != hipSuccess) return KB_ERR_DEVICE;
        ++h->prof_used;
    }
    return hipGetLastError() == hipSuccess ? launch_merge(lists, parts, Q, k, indices_out_dev, scores_out_dev, s) : KB_ERR_DEVICE;
}

// A small knowledge base in parts of 128 or 256 rows (one or two steps of the scorer): no
// sampling pass, no candidate lists.  Same scores, same order: results do not depend on which path ran.
constexpr int64_t SMALL_ROWS = 16384;
constexpr int SMALL_BLOCKS = 1024;
int small_path_parts(const kb *h, int64_t n, int32_t Q, bool draw)
{
    if (draw || h->tune_no_small_path || h->tune_config || h->tune_sample_keys || h->tune_wg_per_cu) return 0;
    if (n < 1 || n > SMALL_ROWS || Q > 65535) return 0;
    int64_t parts = (n + 127) / 128;       // one step of the scorer per part up to 8192 rows, two beyond
    if (parts > PROBE_MAX) parts = PROBE_MAX;
    return parts * Q <= SMALL_BLOCKS ? (int)parts : 0;
}

struct SmallPlan {
    size_t off_lists, total;
};
SmallPlan make_small_plan(int32_t Q, int32_t k, int parts)
{
    SmallPlan p;
    p.off_lists = align_up(sizeof(uint64_t) * (STAT_WORDS + STAT_PARTIALS));      // the diagnostics come first, as always
    p.total = p.off_lists + align_up((size_t)Q * parts * k * 8);
    return p;
}

// query norms, counters and (weighted random selection) ln(gain)
void launch_prep(const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, int32_t qpad, int32_t d, float *invq, uint64_t *thr64, float *thrp, uint32_t *cnt,
                 uint32_t *flag, uint64_t *stats, uint64_t sample_keys, const uint64_t *qmask_dev, uint64_t *qmask_pad, int32_t grid, uint32_t *fb_done,
                 const GainArgs &ga, hipStream_t s)
{
    const int n_init = qpad > STAT_GATE + 1 ? qpad : STAT_GATE + 1;
    const int blocks_rows = (int)ceil_div(qpad, 4), blocks_init = (int)ceil_div(n_init, 256);
    const unsigned blocks = (blocks_rows > blocks_init ? blocks_rows : blocks_init) + ga.blocks;
    auto *fn = q_dtype == KB_F32 ? &prep_kernel<KB_F32> : q_dtype == KB_FP8_E4M3 ? &prep_kernel<KB_FP8_E4M3> : &prep_kernel<KB_BF16>;
    hipLaunchKernelGGL(fn, dim3(blocks), dim3(256), 0, s, queries_dev, Q, qpad, d, invq, thr64, thrp, cnt, flag, stats, sample_keys, qmask_dev, qmask_pad, grid, fb_done, ga);
}

hipError_t launch_stream_scan(const kb *h, const StreamPlan &p, const void *queries_dev, bool q8, bool split, int32_t Q, const uint64_t *qmask_dev, float *best, u32x4 *pair, int32_t groups,
                              bool dense, bool once, uint64_t *gate, hipStream_t s)
{
    StreamArgs a;
    a.keys = h->keys;
    a.queries = queries_dev;
    a.inv_norm = h->inv_norm;
    a.tags = qmask_dev ? h->tags : nullptr;
    a.qmask = qmask_dev;
    a.best = best;
    a.pair = pair;
    a.n = (int32_t)h->n;
    a.d = h->d;
    a.Q = Q;
    a.units = p.units;
    a.waves = p.waves;
    a.per_group = p.per_group;
    a.groups = groups;
    a.query_stride = p.query_stride;
    a.side_slots = p.side_slots;
    a.blocks = p.blocks;
    a.gate = gate;
    return h->dtype == KB_F32 ? launch_stream_f32(p, split, once, a, s) : h->dtype == KB_BF16 ? launch_stream_bf16(p, dense, once, a, s) : launch_stream_fp8(p, q8, dense, once, a, s);
}

// The tiled scan of split f32 rows needs the queries' scales, which come from 1/|q|.  (The gate's word is cleared here: nothing of the call has run.)
__global__ __launch_bounds__(256) void query_inv_kernel(const void *queries, int Q, int d, float *out, uint64_t *gate)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *gate = 0;
    const int row = blockIdx.x * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= Q) return;
    const float inv = row_inv_norm<KB_F32>(queries, row, d * 4, lane);
    if (lane == 0) out[row] = inv;
}

// kb_query by the whole-store plan: two launches (split f32 rows: two more that do nothing as a rule, and one before the tiled scan).
kb_status_t launch_whole(kb *h, const WholePlan &p, const void *queries_dev, bool q8, int32_t Q, const uint64_t *qmask_dev, int32_t k, int32_t k_out,
                         bool split, int32_t *indices_out_dev, float *scores_out_dev, unsigned char *ws, hipStream_t s)
{
    ScanArgs a;
    memset(&a, 0, sizeof a);
    a.keys = h->keys;
    a.inv_norm = h->inv_norm;
    a.tags = qmask_dev ? h->tags : nullptr;
    a.queries = queries_dev;
    a.qmask = qmask_dev;
    a.n_keys = h->n;
    a.n_tiles = ceil_div(h->n, p.tk);
    a.tile_stride = 1;
    a.d = h->d;
    a.Q = Q;
    a.nqb = p.nqb;
    a.qpad = p.nqb * p.tq;
    a.keys_once = stream_keys(h, h->n, Q, p.nqb);
    a.whole_best = reinterpret_cast<float *>(ws + p.off_best);
    a.whole_pair = reinterpret_cast<u32x4 *>(ws + p.off_pair);
    a.whole_groups = p.groups;
    a.whole_fine = p.fine;
    uint64_t *gate = reinterpret_cast<uint64_t *>(ws) + STAT_GATE;
    if (split && !p.stream) {
        float *invq = reinterpret_cast<float *>(ws + p.off_invq);
        a.invq = invq;
        a.split = 1;
        hipLaunchKernelGGL(query_inv_kernel, dim3((unsigned)ceil_div(Q, 4)), dim3(256), 0, s, queries_dev, Q, h->d, invq, gate);
        if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    }
    const bool timed = h->prof_events && h->prof_used < h->prof_max && h->prof_seen++ % h->prof_stride == h->prof_stride / 2;
    if (timed) {
        scan_timing.start = h->prof_events[2 * h->prof_used];
        scan_timing.stop = h->prof_events[2 * h->prof_used + 1];
    }
    const hipError_t launched = p.stream ? launch_stream_scan(h, p.st, queries_dev, q8, split, Q, qmask_dev, a.whole_best, a.whole_pair, p.groups, false, a.keys_once != 0, split ? gate : nullptr, s)
                                         : launch_scan(h->dtype, p.config, 0, false, p.grid, a, s);
    scan_timing = ScanTiming();
    if (launched != hipSuccess) return KB_ERR_DEVICE;
    if (timed) ++h->prof_used;

    WholeSelectArgs t;
    t.waves = p.stream ? p.st.waves : 0;
    t.per_group = p.stream ? p.st.per_group : 1;
    t.keys = a.keys;
    t.queries = queries_dev;
    t.inv_norm = a.inv_norm;
    t.tags = a.tags;
    t.qmask = qmask_dev;
    t.best = a.whole_best;
    t.pair = a.whole_pair;
    t.out_index = indices_out_dev;
    t.out_score = scores_out_dev;
    t.stats = reinterpret_cast<uint64_t *>(ws);
    t.n_keys = h->n;
    t.k = k;
    t.k_out = k_out;
    t.d = h->d;
    t.groups = p.groups;
    t.group_rows = p.group_rows;
    t.tile_rows = p.tk;
    t.tiles = p.stream ? p.st.units : (int32_t)a.n_tiles;
    t.grid = p.grid;
    const int kt = q8 ? KT_FP8_Q8 : split ? KB_F32_SPLIT : (int)h->dtype;
    auto *fn = p.stream ? whole_select_for<true>(kt, p.groups) : whole_select_for<false>(kt, p.groups);
    t.gate = split ? gate : nullptr;
    t.more_lds = split ? restate_lds(Q) : 0;
    static LdsAllowed allowed[6];
    if (t.more_lds > 0 && allow_dynamic_lds(reinterpret_cast<const void *>(fn), allowed[(p.stream ? 3 : 0) + (p.groups <= 4 * WHOLE_THREADS ? 0 : p.groups <= 8 * WHOLE_THREADS ? 1 : 2)], RESTATE_LDS) != hipSuccess)
        return KB_ERR_DEVICE;
    hipLaunchKernelGGL(fn, dim3(Q), dim3(WHOLE_THREADS), t.more_lds, s, t);
    if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    if (split) {        // the same with the f32 instruction, where a query needs it
        a.split = 0;
        a.gate = gate;
        const hipError_t again = p.stream ? launch_stream_scan(h, p.st, queries_dev, q8, false, Q, qmask_dev, a.whole_best, a.whole_pair, p.groups, false, a.keys_once != 0, gate, s)
                                          : launch_scan(h->dtype, p.config, 0, false, p.grid, a, s);
        if (again != hipSuccess) return KB_ERR_DEVICE;
        t.k = k_out;
        t.more_lds = 0;
        hipLaunchKernelGGL(p.stream ? whole_select_for<true>(KB_F32, p.groups) : whole_select_for<false>(KB_F32, p.groups), dim3(Q), dim3(WHOLE_THREADS), 0, s, t);
        if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    }
    return KB_OK;
}

// kb_query and kb_query_sampled by the dense plan: two launches, three with the weighted selection (its scan needs 1/|q| and ln(gain)).
kb_status_t launch_dense(kb *h, const DensePlan &p, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                         DrawArgs dr, GainArgs ga, int32_t *indices_out_dev, float *scores_out_dev, unsigned char *ws, hipStream_t s)
{
    ScanArgs a;
    memset(&a, 0, sizeof a);
    a.keys = h->keys;
    a.inv_norm = h->inv_norm;
    a.tags = qmask_dev ? h->tags : nullptr;
    a.queries = queries_dev;
    a.qmask = qmask_dev;
    a.n_keys = h->n;
    a.n_tiles = ceil_div(h->n, p.tk);
    a.tile_stride = 1;
    a.d = h->d;
    a.Q = Q;
    a.nqb = p.nqb;
    a.qpad = p.nqb * p.tq;
    a.dense = reinterpret_cast<float *>(ws + p.off_values);
    a.dense_stride = p.stride;
    uint64_t *stats = reinterpret_cast<uint64_t *>(ws);
    if (dr.enabled) {
        float *invq = reinterpret_cast<float *>(ws + p.off_invq);
        uint64_t *u64 = reinterpret_cast<uint64_t *>(ws + p.off_unused);
        float *thrp = reinterpret_cast<float *>(u64 + 2 * (size_t)a.qpad);
        uint32_t *u32 = reinterpret_cast<uint32_t *>(thrp + a.qpad);
        ga.log_gain = reinterpret_cast<float *>(ws + p.off_lgain);
        dr.log_gain = ga.log_gain;
        a.invq = invq;
        a.draw = dr;
        launch_prep(queries_dev, q_dtype, Q, a.qpad, h->d, invq, u64, thrp, u32, u32 + (size_t)a.qpad * CAND_SEGMENTS, stats, 0, qmask_dev, u64 + a.qpad, p.grid,
                    u32 + (size_t)a.qpad * (CAND_SEGMENTS + 1), ga, s);
        if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    }
    const bool timed = h->prof_events && h->prof_used < h->prof_max && h->prof_seen++ % h->prof_stride == h->prof_stride / 2;
    if (timed) {
        scan_timing.start = h->prof_events[2 * h->prof_used];
        scan_timing.stop = h->prof_events[2 * h->prof_used + 1];
    }
    const hipError_t launched = p.stream ? launch_stream_scan(h, p.st, queries_dev, q_dtype == KB_FP8_E4M3, false, Q, qmask_dev, a.dense, nullptr, p.stride, true, false, nullptr, s)
                                         : launch_scan(h->dtype, p.config, 0, false, p.grid, a, s);
    scan_timing = ScanTiming();
    if (launched != hipSuccess) return KB_ERR_DEVICE;
    if (timed) ++h->prof_used;

    DenseSelectArgs t;
    t.values = a.dense;
    t.queries = queries_dev;
    t.out_index = indices_out_dev;
    t.out_score = scores_out_dev;
    t.stats = stats;
    t.k = k;
    t.d = h->d;
    t.n = (int32_t)h->n;
    t.stride = p.stride;
    t.grid = p.grid;
    if (dr.enabled) launch_dense_select<KB_F32, true>(t, Q, s);        // (the keys are finished)
    else if (q_dtype == KB_F32) launch_dense_select<KB_F32, false>(t, Q, s);
    else if (q_dtype == KB_BF16) launch_dense_select<KB_BF16, false>(t, Q, s);
    else launch_dense_select<KB_FP8_E4M3, false>(t, Q, s);
    return hipGetLastError() == hipSuccess ? KB_OK : KB_ERR_DEVICE;
}

}  // namespace

size_t kb_query_workspace_bytes(const kb_t *kb, int32_t Q, int32_t k)
{
    if (!kb || Q < 1 || k < 1 || k > KB_K_MAX) return 0;
    // Every combination of kernels a query on this handle can run, each bounded over all row counts.  The choice depends on
    // the kind of query and, through limits of which a handle's type and batch meet at most one for every kind, on the row count
    // (WIDE128_MIN_ROWS for bf16 rows, stream_keys and SHORT_ROWS_MIN_* for fp8 rows): its two sides are those of 1 and of the capacity.
    Sizes m;
    memset(&m, 0, sizeof m);
    bool any = false;
    const int32_t selected = kb->dtype == KB_F32 && split_spare(kb->d, k) <= SPLIT_MAX_SPARE ? k + split_spare(kb->d, k) : k;
    const int64_t ns[2] = {1, kb->capacity};
    // (the weighted selection first: with the same kernels its plan has everything that the plain one has)
    Choice seen[8];
    int n_seen = 0;
    for (int64_t n : ns)
        for (const int kind : {1, 0, 3, 2}) {      // weighted random selection, plain, both with fp8 queries
            Choice c;
            if (!choose_kernels(kb, n, Q, (kind & 1) != 0, (kind & 2) != 0, AMPLE, &c)) continue;
            bool again = false;
            for (int i = 0; i < n_seen; ++i) again = again || (seen[i].config == c.config && seen[i].sample_config == c.sample_config);
            if (again) continue;
            seen[n_seen++] = c;
            bound_sizes(kb, c, Q, selected, (kind & 1) != 0, m);
            any = true;
        }
    if (!any) return 0;
    Plan p;
    lay_out(m, &p);
    size_t total = p.total;
    // a store scored in parts: the most parts that its rows and the limit on workgroups allow
    const int64_t parts = std::min<int64_t>({PROBE_MAX, SMALL_BLOCKS / Q, ceil_div(kb->capacity, 128)});
    if (parts > 0) total = std::max(total, make_small_plan(Q, k, (int)parts).total);
    // the whole-store plan: grows with its groups, so with the rows up to where the groups get coarser and to the most it takes
    size_t unused;
    for (int q8 = 0; q8 < 2; ++q8) {
        const int64_t whole_rows = std::min(kb->capacity, whole_max_rows(kb, Q, q8 != 0));
        const int64_t f32_square = DEVICE_CUS / ceil_div(Q, 128) * 128;        // rows up to which f32 batches past 64 queries have the lower tiles
        // (7, 6, 5 wavefronts a compute unit: the last rows that those of the scan with the queries in LDS take a tile at a time; then groups of two)
        const int64_t most[] = {WHOLE_SMALL_TILE_ROWS, f32_square, WHOLE_MAX_GROUPS * 32, WHOLE_MAX_GROUPS * 64, whole_rows,
                                2 * 7 * DEVICE_CUS * 32, 2 * 6 * DEVICE_CUS * 32, 3 * 5 * DEVICE_CUS * 32};
        for (int64_t n : most) {
            WholePlan wp;
            if (make_whole_plan(kb, std::min(n, whole_rows), Q, k, false, q8 != 0, false, AMPLE, &wp)) total = std::max(total, wp.total + (kb->dtype == KB_F32 ? align_up(sizeof(float) * (size_t)Q) : 0));
        }
        // (the scan with the queries in LDS: never more groups than these)
        if (Q <= 32) total = std::max(total, whole_bytes(Q, (int32_t)std::min<int64_t>(WHOLE_MAX_GROUPS, ceil_div(whole_rows, 16)), &unused));
    }
    // the dense plan: grows with the rows
    for (int kind = 0; kind < 4; ++kind) {
        DensePlan dp;
        if (make_dense_plan(kb, std::min({kb->capacity, DENSE_MAX_ROWS, DENSE_MAX_PAIRS / Q}), Q, k, (kind & 1) != 0, (kind & 2) != 0, &dp))
            total = std::max(total, dp.total);
    }
    return total;
}

namespace {

// What a call does that brings workspace_bytes: the best plan that fits.
// (a store that can be scored in parts takes no call that brings less than their lists, whichever plan it then runs)
struct Route {
    enum Kind { PIPELINE = 0, WHOLE = 1, DENSE = 2, PARTS = 3 } kind;
    Plan pipeline;
    WholePlan whole;
    DensePlan dense;
    SmallPlan small;
    int parts;
    size_t bytes;
    bool split;                 // see split_f32
    int32_t k;                  // entries that are selected
};
kb_status_t choose_route_for(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw, bool q8, bool split, size_t workspace_bytes, Route *r)
{
    r->k = split ? k + split_spare(h->d, k) : k;
    r->split = split;
    const auto whole_fits = [&](Thrift thrift) { return make_whole_plan(h, n, Q, k, draw, q8, split, thrift, &r->whole) && r->whole.total <= workspace_bytes; };
    const bool whole = whole_fits(AMPLE);
    r->parts = small_path_parts(h, n, Q, draw);
    if (r->parts) r->small = make_small_plan(Q, k, r->parts);
    const bool lists = !r->parts || workspace_bytes >= r->small.total;
    const bool dense = !split && (whole || lists) && make_dense_plan(h, n, Q, k, draw, q8, &r->dense) && r->dense.total <= workspace_bytes;
    if (dense && !(whole && !dense_is_better(n, k, r->whole))) {
        r->kind = Route::DENSE;
        r->bytes = !whole && r->parts ? std::max(r->dense.total, r->small.total) : r->dense.total;
    } else if (whole || (r->parts && whole_fits(LEAST))) {
        r->kind = Route::WHOLE;
        r->bytes = r->whole.total;
    } else if (r->parts) {
        r->kind = Route::PARTS;
        r->bytes = r->small.total;
        if (!lists) return KB_ERR_WORKSPACE;
    } else {
        for (const Thrift thrift : {AMPLE, SCORED_TWICE, LEAST}) {
            r->kind = Route::PIPELINE;
            if (!make_plan(h, n, Q, r->k, draw, q8, thrift, &r->pipeline)) return KB_ERR_INVALID_ARG;
            r->bytes = r->pipeline.total;
            if (r->bytes <= workspace_bytes) break;
            if (thrift == AMPLE && whole_fits(LEAST)) {
                r->kind = Route::WHOLE;
                r->bytes = r->whole.total;
                break;
            }
        }
        if (workspace_bytes < r->bytes) return KB_ERR_WORKSPACE;
    }
    return KB_OK;
}
kb_status_t choose_route(const kb *h, int64_t n, int32_t Q, int32_t k, bool draw, bool q8, size_t workspace_bytes, Route *r)
{
    // (a call that brings no more than the f32 instruction takes, runs with it; so do stores small enough for the dense plan that it is the better one for)
    if (split_f32(h, n, Q, k, draw) && choose_route_for(h, n, Q, k, draw, q8, true, workspace_bytes, r) == KB_OK &&
        (r->kind == Route::WHOLE ? Q > 32 ? n > DENSE_MAX_ROWS || !dense_is_better(n, k, r->whole) : r->whole.stream : r->kind == Route::PIPELINE && Q > 32 && n > DENSE_MAX_ROWS))
        return KB_OK;
    return choose_route_for(h, n, Q, k, draw, q8, false, workspace_bytes, r);
}

}  // namespace

size_t kb_query_plan_bytes(const kb_t *kb, int64_t n, int32_t Q, int32_t k, int32_t kind)
{
    if (!kb || n < 0 || n > kb->capacity || Q < 1 || k < 1 || k > KB_K_MAX || kind < 0 || kind > 3) return 0;
    const bool draw = (kind & 1) != 0, q8 = (kind & 2) != 0;
    if (q8 && kb->dtype != KB_FP8_E4M3) return 0;
    Route r;
    return choose_route(kb, n, Q, k, draw, q8, SIZE_MAX, &r) == KB_OK ? r.bytes : 0;
}

kb_status_t kb_query_plan(const kb_t *kb, int64_t n, int32_t Q, int32_t k, int32_t kind, size_t workspace_bytes, int64_t *out)
{
    if (!kb || !out) return KB_ERR_NULL;
    if (n < 0 || n > kb->capacity || Q < 1 || k < 1 || k > KB_K_MAX || kind < 0 || kind > 3) return KB_ERR_INVALID_ARG;
    const bool draw = (kind & 1) != 0, q8 = (kind & 2) != 0;
    if (q8 && kb->dtype != KB_FP8_E4M3) return KB_ERR_DTYPE;
    Route r;
    if (const kb_status_t e = choose_route(kb, n, Q, k, draw, q8, workspace_bytes, &r); e != KB_OK) return e;
    const bool pipeline = r.kind == Route::PIPELINE;
    out[0] = r.kind;
    out[1] = (int64_t)r.bytes;
    out[2] = pipeline && n > 0 ? r.pipeline.sample_keys : 0;
    out[3] = pipeline && n > 0 ? r.pipeline.main_rows : n;
    return KB_OK;
}

// kb_query and kb_query_sampled: the same pipeline; `gain_dev` != nullptr selects the weighted random selection.
static kb_status_t run_query(kb_t *kb, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                             const float *gain_dev, float temperature, uint64_t seed, int32_t first_query,
                             int32_t *indices_out_dev, float *scores_out_dev, void *workspace_dev, size_t workspace_bytes,
                             void *hip_stream)
{
    const bool draw = gain_dev != nullptr;
    if (!kb || !queries_dev || !indices_out_dev || !scores_out_dev) return KB_ERR_NULL;
    if (!valid_dtype((int)q_dtype)) return KB_ERR_DTYPE;
    const kb_dtype_t want_q = kb->dtype == KB_F32 ? KB_F32 : KB_BF16;
    const bool q8 = kb->dtype == KB_FP8_E4M3 && q_dtype == KB_FP8_E4M3;     // fp8 queries against fp8 keys
    if (q_dtype != want_q && !q8) return KB_ERR_DTYPE;
    if (Q < 1 || k < 1 || k > KB_K_MAX) return KB_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(queries_dev) & 15) != 0) return KB_ERR_INVALID_ARG;
    if (qmask_dev && !kb->tags) return KB_ERR_NO_TAGS;
    if (kb->n_normalized != kb->n) return KB_ERR_NOT_NORMALIZED;
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & (WS_ALIGN - 1)) != 0) return KB_ERR_WORKSPACE;
    DrawArgs dr;
    memset(&dr, 0, sizeof dr);
    GainArgs ga;
    memset(&ga, 0, sizeof ga);
    if (draw) {
        dr.inv_t = 1.0f / temperature;
        dr.seed_lo = (uint32_t)seed;
        dr.seed_hi = (uint32_t)(seed >> 32);
        dr.first_query = (uint32_t)first_query;
        dr.enabled = 1;
        ga.gain = gain_dev;
        ga.n = kb->n;
        ga.n_padded = ceil_div(kb->n > 0 ? kb->n : 1, 256) * 256 + 256;
        ga.blocks = (int)ceil_div(ga.n_padded, 256);
    }

    Route r;
    if (const kb_status_t e = choose_route(kb, kb->n, Q, k, draw, q8, workspace_bytes, &r); e != KB_OK) return e;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    unsigned char *ws = static_cast<unsigned char *>(workspace_dev);
    if (r.kind == Route::DENSE) return launch_dense(kb, r.dense, queries_dev, q_dtype, Q, qmask_dev, k, dr, ga, indices_out_dev, scores_out_dev, ws, s);
    if (r.kind == Route::WHOLE) return launch_whole(kb, r.whole, queries_dev, q8, Q, qmask_dev, r.k, k, r.split, indices_out_dev, scores_out_dev, ws, s);
    if (r.kind == Route::PARTS)
        return launch_small(kb, queries_dev, q8, Q, qmask_dev, k, r.parts, reinterpret_cast<uint64_t *>(ws + r.small.off_lists), reinterpret_cast<uint64_t *>(ws),
                            indices_out_dev, scores_out_dev, s);
    const Plan &p = r.pipeline;
    float *invq = reinterpret_cast<float *>(ws + p.off_invq);
    uint64_t *thr64 = reinterpret_cast<uint64_t *>(ws + p.off_thr64);
    float *thrp = reinterpret_cast<float *>(ws + p.off_thrp);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(ws + p.off_cnt);
    uint32_t *flag = reinterpret_cast<uint32_t *>(ws + p.off_flag);
    uint32_t *fb_done = reinterpret_cast<uint32_t *>(ws + p.off_fb_done);
    uint64_t *stats = reinterpret_cast<uint64_t *>(ws + p.off_stats);
    uint64_t *qmask_pad = reinterpret_cast<uint64_t *>(ws + p.off_qmask);
    uint64_t *samp = reinterpret_cast<uint64_t *>(ws + p.off_samp);
    Record *regions = reinterpret_cast<Record *>(ws + p.off_regions);
    uint64_t *cand = reinterpret_cast<uint64_t *>(ws + p.off_cand);
    float *log_gain = reinterpret_cast<float *>(ws + p.off_lgain);

    dr.log_gain = ga.log_gain = log_gain;

    // Query norms and per-call counters: the threshold kernel sets them when there is a sampling pass on scores;
    // otherwise (no sampling pass, or the weighted random selection and split f32 rows, whose sampling pass needs 1/|q|) this launch does.
    const bool sampled = kb->n > 0 && p.sample_tiles > 0, split = r.split;
    if (!sampled || draw || split) {
        launch_prep(queries_dev, q_dtype, Q, p.qpad, kb->d, invq, thr64, thrp, cnt, flag, stats, (uint64_t)p.sample_keys, qmask_dev, qmask_pad, p.grid, fb_done, ga, s);
        if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    }

    ScanArgs a;
    if (kb->n > 0) {
        a.keys = kb->keys;
        a.inv_norm = kb->inv_norm;
        a.tags = qmask_dev ? kb->tags : nullptr;
        a.queries = queries_dev;
        a.qmask = qmask_dev;
        a.qmask_pad = qmask_pad;
        a.invq = invq;
        a.split = split;
        a.gate = nullptr;
        a.thr64 = thr64;
        a.thrp = thrp;
        a.samp = samp;
        a.regions = regions;
        a.cand = cand;
        a.cnt = cnt;
        a.stats = stats;
        a.cand_cap = p.cand_cap;
        a.flag = flag;
        a.n_keys = kb->n;
        a.d = kb->d;
        a.Q = Q;
        a.nqb = p.nqb;
        a.qpad = p.qpad;
        a.sample_slots = p.sample_slots;
        a.sample_group_shift = 0;        // groups per tile of the sampling configuration: a power of two
        while (p.sample_tiles > 0 && ((int64_t)p.sample_tiles << (a.sample_group_shift + 1)) <= p.sample_slots) ++a.sample_group_shift;
        a.region_cap = p.region_cap;
        a.draw = dr;
        a.keys_once = stream_keys(kb, kb->n, Q, p.nqb);
        a.whole_best = nullptr;
        a.whole_pair = nullptr;
        a.whole_groups = a.whole_fine = 0;
        a.dense = nullptr;
        a.dense_stride = 0;
        a.tile_stride = 1;
        a.row_mul = 0;
        a.row_run_shift = 0;
        a.row_inv_runs = 0.0;
        a.row_ratio = 0.f;
        a.sample_runs = 1;
        a.skip_mul = 0;
        a.skip_inv = 0.0;
        a.mixed_rows = 0;
        a.samp_more = nullptr;
        if (p.sample_tiles > 0) {
            // the sample is spread evenly over the knowledge base: a prefix says nothing about later rows when
            // the rows are grouped (by state, by cluster, by age)
            a.n_tiles = p.sample_tiles;
            a.tile_stride = (int32_t)(ceil_div(kb->n, p.sample_tk) / p.sample_tiles);
            // ... row by row where the kernel can gather (the two-phase and register-tile kernels load whole tiles:
            // they take every tile_stride-th tile instead)
            a.row_run_shift = draw ? 2 : 0;
            a.sample_runs = kb->n >> a.row_run_shift;
            if (p.once) {
                a.sample_runs = p.sample_keys;
                a.skip_mul = (uint32_t)ceil_div(p.sample_keys << 32, p.main_rows);
                a.skip_inv = 4294967296.0 / (double)a.skip_mul;
                a.mixed_rows = (uint32_t)kb->n & ~255u;
                a.samp_more = reinterpret_cast<uint64_t *>(ws + p.off_samp_more);
            }
            a.row_mul = scatter_multiplier(a.sample_runs);
            // (the full-line kernel addresses scattered rows in 32 bits, in units of 16 bytes: up to 64 GiB of keys)
            if (p.sample_family == 4 && (uint64_t)kb->n * kb->d * key_bytes(kb->dtype) >= ((uint64_t)1 << 36)) a.row_mul = 0;
            if (a.sample_runs < 1) a.sample_runs = 1;
            a.row_inv_runs = 1.0 / (double)a.sample_runs;
            a.row_ratio = (float)((double)a.row_mul / (double)a.sample_runs);
            int64_t sgrid = p.sample_tiles * p.nqb;
            const int64_t smax = (int64_t)DEVICE_CUS * p.sample_wgpc;
            if (sgrid > smax && p.sample_family != 4) sgrid = smax;        // (the full-line kernel samples one item per workgroup)
            if (launch_scan(kb->dtype, p.sample_config, p.sample_family, true, (int)sgrid, a, s) != hipSuccess) return KB_ERR_DEVICE;
            const int thr_threads = p.sample_slots > 1024 ? 1024 : p.sample_slots > 512 ? 512 : 256;
            const size_t thr_lds = sizeof(uint64_t) * (p.sample_slots > r.k ? p.sample_slots : r.k) + sizeof(SelectScratch);
            ThresholdArgs t;
            t.samp = samp;
            t.queries = queries_dev;
            t.qmask = qmask_dev;
            t.invq = invq;
            t.thrp = thrp;
            t.thr64 = thr64;
            t.qmask_pad = qmask_pad;
            t.stats = stats;
            t.cnt = cnt;
            t.flag = flag;
            t.fb_done = fb_done;
            t.sample_keys = (uint64_t)p.sample_keys;
            t.slots = p.sample_slots;
            t.group_shift = a.sample_group_shift;
            t.k = r.k;
            t.Q = Q;
            t.qpad = p.qpad;
            t.d = kb->d;
            t.grid = p.grid;
            t.more = a.samp_more;
            t.cand = cand;
            t.cand_cap = p.cand_cap;
            t.tile_rows = p.sample_tk;
            t.scan = a;
            static LdsAllowed thr_allowed[9];
            const int thr_kind = split ? 8 : p.once ? (kb->dtype == KB_BF16 ? 4 : 5) + (p.sample_slots > 2048 ? 2 : 0) : draw ? 3 : (int)q_dtype;
            void (*thr_fn)(ThresholdArgs) = p.once ? (kb->dtype == KB_BF16 ? threshold_once<KB_BF16>(p.sample_slots) : threshold_once<KB_FP8_E4M3>(p.sample_slots))
                                          : draw ? &threshold_kernel<KB_F32, true, -1>
                                          : split ? &threshold_kernel<KB_F32_SPLIT, false, -1>
                                          : q_dtype == KB_F32 ? &threshold_kernel<KB_F32, false, -1>
                                          : q_dtype == KB_BF16 ? &threshold_kernel<KB_BF16, false, -1> : &threshold_kernel<KB_FP8_E4M3, false, -1>;
            if (allow_dynamic_lds(reinterpret_cast<const void *>(thr_fn), thr_allowed[thr_kind], MAX_SAMPLE_SLOTS * 8 + sizeof(SelectScratch)) != hipSuccess)
                return KB_ERR_DEVICE;
            hipLaunchKernelGGL(thr_fn, dim3(draw ? Q : p.qpad), dim3(thr_threads), thr_lds, s, t);
            if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
        }
        a.n_keys = p.main_rows;
        a.n_tiles = ceil_div(a.n_keys, p.tk);
        a.tile_stride = 1;
        a.row_mul = 0;
        const bool timed = kb->prof_events && kb->prof_used < kb->prof_max && kb->prof_seen++ % kb->prof_stride == kb->prof_stride / 2;
        if (timed) {
            scan_timing.start = kb->prof_events[2 * kb->prof_used];
            scan_timing.stop = kb->prof_events[2 * kb->prof_used + 1];
        }
        const hipError_t launched = launch_scan(kb->dtype, p.config, p.family, false, p.grid, a, s);
        scan_timing = ScanTiming();
        if (launched != hipSuccess) return KB_ERR_DEVICE;
        if (timed) ++kb->prof_used;
    }

    FinalArgs f;
    f.keys = kb->keys;
    f.inv_norm = kb->inv_norm;
    f.tags = qmask_dev ? kb->tags : nullptr;
    f.queries = queries_dev;
    f.qmask = qmask_dev;
    f.invq = invq;
    f.cand = cand;
    f.cnt = cnt;
    f.flag = flag;
    f.stats = stats;
    f.out_index = indices_out_dev;
    f.out_score = scores_out_dev;
    f.n_keys = kb->n;
    f.d = kb->d;
    f.k = r.k;
    f.k_out = k;
    f.cand_cap = p.cand_cap;
    f.draw = dr;
    f.fb_done = fb_done;
    f.fb_lists = reinterpret_cast<uint64_t *>(ws + p.off_fb_lists);
    f.fb_parts = p.fb_parts;
    f.thr64 = thr64;
    f.thrp = thrp;
    f.again = 0;
    f.raw = draw ? 0 : 1;
    constexpr size_t FIN_LDS_MAX = ((size_t)MAX_CAND_CAP * 8 + 16 + sizeof(SelectScratch) + 15) / 16 * 16;
    const size_t fin_base = ((size_t)p.cand_cap * 8 + 16 + sizeof(SelectScratch) + 15) / 16 * 16;
    f.more_at = (int32_t)fin_base;
    f.more_lds = split ? std::min(restate_lds(Q), (int)(MAX_CAND_CAP * 8 + RESTATE_LDS / 2 - fin_base)) : 0;
    const size_t fin_lds = fin_base + f.more_lds;
    static LdsAllowed fin_allowed[5];
    const int fin_kind = q8 ? KT_FP8_Q8 : split ? KB_F32_SPLIT : (int)kb->dtype;
    const void *fin_fn = fin_kind == KB_F32_SPLIT ? reinterpret_cast<const void *>(&finalize_kernel<KB_F32_SPLIT>)
                       : fin_kind == KB_F32 ? reinterpret_cast<const void *>(&finalize_kernel<KB_F32>)
                       : fin_kind == KB_BF16 ? reinterpret_cast<const void *>(&finalize_kernel<KB_BF16>)
                       : fin_kind == KB_FP8_E4M3 ? reinterpret_cast<const void *>(&finalize_kernel<KB_FP8_E4M3>)
                                                 : reinterpret_cast<const void *>(&finalize_kernel<KT_FP8_Q8>);
    if (allow_dynamic_lds(fin_fn, fin_allowed[fin_kind], FIN_LDS_MAX + (split ? RESTATE_LDS / 2 : 0)) != hipSuccess) return KB_ERR_DEVICE;
    switch (fin_kind) {
    case KB_F32_SPLIT: hipLaunchKernelGGL(finalize_kernel<KB_F32_SPLIT>, dim3(Q), dim3(256), fin_lds, s, f); break;
    case KB_F32: hipLaunchKernelGGL(finalize_kernel<KB_F32>, dim3(Q, p.fb_parts), dim3(256), fin_lds, s, f); break;
    case KB_BF16: hipLaunchKernelGGL(finalize_kernel<KB_BF16>, dim3(Q, p.fb_parts), dim3(256), fin_lds, s, f); break;
    case KB_FP8_E4M3: hipLaunchKernelGGL(finalize_kernel<KB_FP8_E4M3>, dim3(Q, p.fb_parts), dim3(256), fin_lds, s, f); break;
    default: hipLaunchKernelGGL(finalize_kernel<KT_FP8_Q8>, dim3(Q, p.fb_parts), dim3(256), fin_lds, s, f); break;
    }
    if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    if (split) {        // the same with the f32 instruction, where a query needs it
        a.split = 0;
        a.gate = stats + STAT_GATE;
        if (launch_scan(kb->dtype, p.config, p.family, false, p.grid, a, s) != hipSuccess) return KB_ERR_DEVICE;
        f.k = k;
        f.again = 1;
        static LdsAllowed again_allowed;
        if (allow_dynamic_lds(reinterpret_cast<const void *>(&finalize_kernel<KB_F32>), again_allowed, FIN_LDS_MAX) != hipSuccess) return KB_ERR_DEVICE;
        hipLaunchKernelGGL(finalize_kernel<KB_F32>, dim3(Q, p.fb_parts), dim3(256), fin_base, s, f);
        if (hipGetLastError() != hipSuccess) return KB_ERR_DEVICE;
    }
    return KB_OK;
}

kb_status_t kb_query(kb_t *kb, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                     int32_t *indices_out_dev, float *scores_out_dev, void *workspace_dev, size_t workspace_bytes,
                     void *hip_stream)
{
    return run_query(kb, queries_dev, q_dtype, Q, qmask_dev, k, nullptr, 1.0f, 0, 0, indices_out_dev, scores_out_dev, workspace_dev,
                     workspace_bytes, hip_stream);
}

// The library's own scratch memory for kb_query_static: one array per device, in device memory for as long as the
// process lives.  In host code the name `scratch` only stands for the symbol; its device address is asked for once
// per device (hipGetSymbolAddress, with that device current) and kept in scratch_address[].
static __device__ __align__(256) unsigned char scratch[KB_STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
static std::atomic<void *> scratch_address[MAX_DEVICES];

kb_status_t kb_query_static(kb_t *kb, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                            int32_t *indices_out_dev, float *scores_out_dev, void *hip_stream)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return KB_ERR_DEVICE;
    void *ptr = scratch_address[dev].load(std::memory_order_acquire);
    if (!ptr) {     // first call on this device (two threads racing here get the same address)
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KB_ERR_DEVICE;
        scratch_address[dev].store(ptr, std::memory_order_release);
    }
    // run_query checks the plan of this call against the size of the array and returns KB_ERR_WORKSPACE beyond it
    return run_query(kb, queries_dev, q_dtype, Q, qmask_dev, k, nullptr, 1.0f, 0, 0, indices_out_dev, scores_out_dev, ptr,
                     KB_STATIC_SCRATCH_BYTES, hip_stream);
}

kb_status_t kb_query_sampled(kb_t *kb, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                             const float *gain_dev, float temperature, uint64_t seed, int32_t first_query,
                             int32_t *indices_out_dev, float *keys_out_dev, void *workspace_dev, size_t workspace_bytes,
                             void *hip_stream)
{
    if (!gain_dev) return KB_ERR_NULL;
    if (!(temperature > 0.0f) || !(temperature < __builtin_inff()) || first_query < 0) return KB_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(gain_dev) & 3) != 0) return KB_ERR_INVALID_ARG;
    return run_query(kb, queries_dev, q_dtype, Q, qmask_dev, k, gain_dev, temperature, seed, first_query, indices_out_dev, keys_out_dev,
                     workspace_dev, workspace_bytes, hip_stream);
}

size_t kb_query_probe_workspace_bytes(const kb_t *kb, int32_t Q, int32_t k, int32_t nprobe)
{
    ProbePlan p;
    return kb && make_probe_plan(Q, k, nprobe, &p) ? p.total : 0;
}

kb_status_t kb_query_probe(kb_t *kb, const void *queries_dev, kb_dtype_t q_dtype, int32_t Q, const uint64_t *qmask_dev, int32_t k,
                           const int64_t *cluster_offsets_dev, int32_t n_clusters, const int32_t *probe_dev, int32_t nprobe,
                           int32_t *indices_out_dev, float *scores_out_dev, void *workspace_dev, size_t workspace_bytes, void *hip_stream)
{
    if (!kb || !queries_dev || !cluster_offsets_dev || !probe_dev || !indices_out_dev || !scores_out_dev) return KB_ERR_NULL;
    if (!valid_dtype((int)q_dtype)) return KB_ERR_DTYPE;
    const kb_dtype_t want_q = kb->dtype == KB_F32 ? KB_F32 : KB_BF16;
    const bool q8 = kb->dtype == KB_FP8_E4M3 && q_dtype == KB_FP8_E4M3;
    if (q_dtype != want_q && !q8) return KB_ERR_DTYPE;
    ProbePlan p;
    if (n_clusters < 1 || !make_probe_plan(Q, k, nprobe, &p)) return KB_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(queries_dev) & 15) != 0 || (reinterpret_cast<uintptr_t>(cluster_offsets_dev) & 7) != 0 ||
        (reinterpret_cast<uintptr_t>(probe_dev) & 3) != 0)
        return KB_ERR_INVALID_ARG;
    if (qmask_dev && !kb->tags) return KB_ERR_NO_TAGS;
    if (kb->n_normalized != kb->n) return KB_ERR_NOT_NORMALIZED;
    if (workspace_bytes < p.total) make_probe_plan(Q, k, nprobe, &p, true);
    if (!workspace_dev || (reinterpret_cast<uintptr_t>(workspace_dev) & (WS_ALIGN - 1)) != 0 || workspace_bytes < p.total) return KB_ERR_WORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    unsigned char *ws = static_cast<unsigned char *>(workspace_dev);
    uint64_t *lists = reinterpret_cast<uint64_t *>(ws + p.off_lists);
    return launch_probe(kb, queries_dev, q8, Q, qmask_dev, k, cluster_offsets_dev, n_clusters, probe_dev, nprobe, p.splits, lists, indices_out_dev,
                        scores_out_dev, s);
}

kb_status_t kb_query_counters(const kb_t *kb, const void *workspace_dev, int64_t *out, void *hip_stream)
{
    if (!kb || !workspace_dev || !out) return KB_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (hipStreamSynchronize(s) != hipSuccess) return KB_ERR_DEVICE;
    uint64_t host[STAT_WORDS + STAT_PARTIALS];
    if (hipMemcpy(host, workspace_dev, sizeof host, hipMemcpyDeviceToHost) != hipSuccess) return KB_ERR_DEVICE;
    for (int i = 0; i < STAT_WORDS; ++i) out[i] = (int64_t)host[i];
    for (int i = 0; i < STAT_PARTIALS; ++i) out[0] += (int64_t)host[STAT_WORDS + i];
    return KB_OK;
}

namespace {
// out[0]: values m of the generator word's upper 23 bits whose variate is below that of m - 1; out[1]: values looked at
__global__ __launch_bounds__(256) void draw_noise_check_kernel(unsigned long long *out)
{
    const uint32_t m = blockIdx.x * 256u + threadIdx.x;      // < 2^23
    const bool falls = m > 0 && gumbel_of_word(m << 9) < gumbel_of_word((m - 1) << 9);
    const unsigned long long bad = __builtin_amdgcn_ballot_w64(falls);
    if ((threadIdx.x & 63) == 0) {
        if (bad) atomicAdd(out, (unsigned long long)__builtin_popcountll(bad));
        atomicAdd(out + 1, 64ull);
    }
}
__global__ void zero_words_kernel(unsigned long long *out, int n)
{
    if ((int)threadIdx.x < n) out[threadIdx.x] = 0ull;
}
}  // namespace

kb_status_t kb_check_draw_noise(int64_t *out_dev, void *hip_stream)
{
    if (!out_dev) return KB_ERR_NULL;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    unsigned long long *out = reinterpret_cast<unsigned long long *>(out_dev);
    hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, out, 2);
    hipLaunchKernelGGL(draw_noise_check_kernel, dim3((1u << 23) / 256), dim3(256), 0, s, out);
    return hipGetLastError() == hipSuccess ? KB_OK : KB_ERR_DEVICE;
}

kb_status_t kb_set_tuning(kb_t *kb, const char *name, int64_t value)
{
    if (!kb || !name) return KB_ERR_NULL;
    if (value < 0) return KB_ERR_INVALID_ARG;
    if (!strcmp(name, "sample_keys")) kb->tune_sample_keys = value;
    else if (!strcmp(name, "scan_config")) {
        ConfigInfo ci;
        if (value != 0 && (!scan_config_info(kb->dtype, (int)value, &ci) || is_whole_config((int)value))) return KB_ERR_INVALID_ARG;
        kb->tune_config = value;
    } else if (!strcmp(name, "small_path")) {
        if (value > 1) return KB_ERR_INVALID_ARG;
        kb->tune_no_small_path = value == 0;
    } else if (!strcmp(name, "profile_stride")) {       // of a profiling session, every value-th scan launch is timed, the middle one of each run of `value` (0 = every one)
        kb->prof_stride = value > 0 ? (int)value : 1;
    } else if (!strcmp(name, "wg_per_cu")) {
        if (value > 8) return KB_ERR_INVALID_ARG;
        kb->tune_wg_per_cu = value;
    } else
        return KB_ERR_INVALID_ARG;
    return KB_OK;
}

static void drop_events(kb_t *kb)
{
    if (kb->prof_events) {
        for (int i = 0; i < 2 * kb->prof_max; ++i)
            if (kb->prof_events[i]) (void)hipEventDestroy(kb->prof_events[i]);
        free(kb->prof_events);
    }
    kb->prof_events = nullptr;
    kb->prof_max = kb->prof_used = 0;
}

kb_status_t kb_profile_begin(kb_t *kb, int32_t max_calls)
{
    if (!kb) return KB_ERR_NULL;
    if (max_calls < 1 || max_calls > 4096) return KB_ERR_INVALID_ARG;
    drop_events(kb);
    kb->prof_events = static_cast<hipEvent_t *>(calloc(2 * (size_t)max_calls, sizeof(hipEvent_t)));
    if (!kb->prof_events) return KB_ERR_INVALID_ARG;
    kb->prof_max = max_calls;
    kb->prof_seen = 0;
    for (int i = 0; i < 2 * max_calls; ++i)
        if (hipEventCreate(&kb->prof_events[i]) != hipSuccess) {
            drop_events(kb);
            return KB_ERR_DEVICE;
        }
    return KB_OK;
}

kb_status_t kb_profile_end(kb_t *kb, void *hip_stream, double *scan_ms_total, int32_t *calls)
{
    if (!kb || !scan_ms_total || !calls) return KB_ERR_NULL;
    if (!kb->prof_events) return KB_ERR_INVALID_ARG;
    kb_status_t st = KB_OK;
    if (hipStreamSynchronize(static_cast<hipStream_t>(hip_stream)) != hipSuccess) st = KB_ERR_DEVICE;
    double total = 0.0;
    for (int i = 0; st == KB_OK && i < kb->prof_used; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, kb->prof_events[2 * i], kb->prof_events[2 * i + 1]) != hipSuccess) st = KB_ERR_DEVICE;
        total += ms;
    }
    *scan_ms_total = total;
    *calls = kb->prof_used;
    drop_events(kb);
    return st;
}

int64_t kb_size(const kb_t *kb) { return kb ? kb->n : -1; }

kb_status_t kb_destroy(kb_t *kb)
{
    if (!kb) return KB_ERR_NULL;
    drop_events(kb);
    delete kb;
    return KB_OK;
}

const char *kb_status_string(kb_status_t s)
{
    switch (s) {
    case KB_OK: return "ok";
    case KB_ERR_NULL: return "required pointer is NULL";
    case KB_ERR_INVALID_ARG: return "argument out of range";
    case KB_ERR_DTYPE: return "dtype not supported for this call";
    case KB_ERR_CAPACITY: return "capacity exceeded";
    case KB_ERR_NOT_NORMALIZED: return "appended rows have not been normalized";
    case KB_ERR_NO_TAGS: return "query mask given for an untagged knowledge base";
    case KB_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case KB_ERR_DEVICE: return "HIP call or kernel launch failed";
    }
    return "unknown status";
}

}  // extern "C"
