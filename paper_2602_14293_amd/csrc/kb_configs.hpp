// Tile configurations of the scan kernel: X(id, key dtype, TK, TQ, WM, WN, RBA, NSTAGE, WGPC)
//   TK x TQ      keys x queries per work item         WM x WN  wavefront grid inside the workgroup
//   RBA          bytes of each key row per d-chunk    NSTAGE   chunk buffers in LDS
//   WGPC         workgroups resident per compute unit (LDS and registers are budgeted for it)
// (12, 16: small tiles for knowledge bases of some ten thousand rows, where a query is bound by the latency of its
//  launches and more, shorter work items finish sooner; 23, 24: whole cache lines of fp8 rows of a multiple of 128 bytes;
//  26: f32, where the matrix units are the bound, up to 64 queries, and small stores, whose time is one dot product's chain of
//  matrix instructions times the blocks a wave holds: 150,000 x 256 rows, 40 queries 102 -> 65 us, 8000 x 768 rows, 100 queries 82 -> 46)
#pragma once
#define KB_SCAN_CONFIGS_BF16(X)                  \
    X(1, KB_BF16, 128, 32, 4, 1, 128, 3, 2)      \
    X(2, KB_BF16, 128, 128, 2, 2, 64, 4, 2)      \
    X(3, KB_BF16, 128, 256, 2, 2, 64, 3, 2)      \
    X(12, KB_BF16, 64, 64, 2, 2, 128, 4, 2)      \
    X(16, KB_BF16, 64, 128, 2, 2, 128, 3, 2)
#define KB_SCAN_CONFIGS_F32(X)                   \
    X(1, KB_F32, 128, 32, 4, 1, 128, 3, 2)       \
    X(2, KB_F32, 128, 128, 2, 2, 64, 4, 2)       \
    X(3, KB_F32, 128, 256, 2, 2, 64, 3, 2)       \
    X(26, KB_F32, 64, 64, 2, 2, 128, 4, 2)
// ... the same for rows that are scored as two f16 values an element
#define KB_SCAN_CONFIGS_F32_SPLIT(X)                  \
    X(2, KB_F32_SPLIT, 128, 128, 2, 2, 64, 4, 2)      \
    X(3, KB_F32_SPLIT, 128, 256, 2, 2, 64, 3, 2)      \
    X(26, KB_F32_SPLIT, 64, 64, 2, 2, 128, 4, 2)
#define KB_SCAN_CONFIGS_FP8(X)                   \
    X(1, KB_FP8_E4M3, 128, 32, 4, 1, 64, 3, 2)   \
    X(2, KB_FP8_E4M3, 128, 128, 2, 2, 64, 3, 2)  \
    X(3, KB_FP8_E4M3, 128, 256, 2, 2, 64, 3, 1)  \
    X(23, KB_FP8_E4M3, 128, 32, 4, 1, 128, 3, 2)
// ... with fp8 queries as well (key type KB_FP8_Q8 inside the kernels): every row length, every batch size
#define KB_SCAN_CONFIGS_FP8_Q8(X)                \
    X(6, KB_FP8_Q8, 128, 64, 2, 2, 64, 3, 2)     \
    X(7, KB_FP8_Q8, 128, 128, 2, 2, 64, 3, 2)    \
    X(8, KB_FP8_Q8, 128, 256, 2, 2, 64, 3, 1)    \
    X(24, KB_FP8_Q8, 128, 32, 4, 1, 128, 3, 2)

// ... of the whole-store plan only (it also takes those above with query blocks of up to 128, but for 2 of bf16).  13: the shortest scans, one wavefront
// per workgroup with eight chunks of 128 bytes of each of its 32 keys in flight at once (fp8: eleven of 64).  14: some ten thousand rows and
// up to 64 queries, one tile per resident workgroup (65,536 x 768 keys: 23.7 us, 25.1 with config 12).  21: up to 128
// queries, two tiles of 128 rows per compute unit and more (65,536 x 1024 keys, 128 queries: 39.6 us, 44.4 with config 16,
// whose 64 rows meet twice as many query bytes; 196,000 rows 110 against 120; 16,384 rows 15.8 against 14.1, and with rows
// of 512 bytes 30.6 against 28.1).
#define KB_SCAN_WHOLE_CONFIGS_BF16(X)            \
    X(13, KB_BF16, 32, 32, 1, 1, 128, 9, 2)      \
    X(14, KB_BF16, 128, 64, 4, 1, 128, 3, 2)     \
    X(21, KB_BF16, 128, 128, 4, 2, 128, 4, 1)
#define KB_SCAN_WHOLE_CONFIGS_FP8(X)             \
    X(13, KB_FP8_E4M3, 32, 32, 1, 1, 64, 12, 2)
// ... with fp8 queries (the dense plan only)
#define KB_SCAN_DENSE_CONFIGS_FP8_Q8(X)          \
    X(25, KB_FP8_Q8, 32, 32, 1, 1, 64, 15, 2)
// ... and of a kernel of its own, for f32 rows (kb_scan_f32.hip): tiles of 16 rows
constexpr int SMALL_F32_CONFIG = 15;

// Software-pipelined configurations (kb_scan_sp.hpp): XS(id, key dtype, TQ, NSA, NSB); 256-row tiles, 512 threads,
// NSA / NSB = ring depth of key / query chunks in LDS.
// bf16: the loads are issued between the MFMAs (IL mode).  Rows of 384 bytes (longer ones: the full-line kernel); call on 2^20 rows, 200
// queries, in us: 170, with a ring of five 175.  Rows of 256 bytes stay with the tiled kernel: 128 against 133 there, but slower on most
// stores (67,054 rows, 256 queries 50 against 43, 266,059 rows, 200 queries 64 against 59, 1,444,949 rows, 166 queries 194 against 190).
#define KB_SCAN_SP_CONFIGS_BF16_IL(XI) \
    XI(17, KB_BF16, 256, 4, 4)
// fp8 with bf16 queries: rows of 192 bytes, and those that are no multiple of 128 (192 bytes, 200 queries, per item: 8.0 us, tiled kernel 16.6)
#define KB_SCAN_SP_CONFIGS_FP8(XS)  \
    XS(4, KB_FP8_E4M3, 256, 3, 3)
// ... with fp8 queries as well (the fp8 matrix instruction): XQ(id, key dtype, TQ, NSA, NSB).  Rings of four take rows of 256 bytes and
// up, rings of three rows of 128 and 192.  Per item (256 rows x 256 queries) and compute unit, 2^20 rows, 200 queries, in us:
//   row bytes                 128    192    256    320    384    576    960
//   tiled kernel             12.4   14.2   16.9   19.6   22.3   29.5   44.1
//   rings of three            4.6    5.5    6.3    9.0    9.2   14.9   25.4
//   rings of four              -      -     5.9    7.2    8.2   11.5   19.1
//   five of keys, four of queries (before)  -  7.5    8.2   11.4   19.3
#define KB_SCAN_SP_CONFIGS_FP8_Q8(XQ) \
    XQ(5, KB_FP8_E4M3, 256, 4, 4) \
    XQ(27, KB_FP8_E4M3, 256, 3, 3)

// Full-line configurations (kb_scan_wide.hpp): XW(id, key dtype, TQ); 256-row tiles, 512 threads, 128-byte row pieces.
#define KB_SCAN_WIDE_CONFIGS_BF16(XW) \
    XW(18, KB_BF16, 256)              \
    XW(19, KB_BF16, 128)
// ... for fp8 keys with fp8 queries
#define KB_SCAN_WIDE_CONFIGS_FP8_Q8(XW) \
    XW(20, KB_FP8_E4M3, 256)
// ... for fp8 keys with bf16 queries: rows of a multiple of 128 elements, 256 at least
#define KB_SCAN_WIDE_CONFIGS_FP8(XW) \
    XW(22, KB_FP8_E4M3, 256)
