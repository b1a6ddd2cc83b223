// nw_kernels.h -- the per-length kernel instances, compiled in separate
// translation units (k_inst.hip) and collected into one table.
#pragma once

#include "nw_internal.h"

namespace nw {

// Row-length ranges compiled in separate translation units (build time).
#define NW_LA_SPLITS X(0, 14) X(15, 22) X(23, 29) X(30, 35) X(36, 40) X(41, 44) X(45, 48)

// Row-length classes of the width-8 persistent batched kernels.
#define NW_CLASS8 X(0, 7) X(8, 15) X(16, 23) X(24, 31) X(32, 39) X(40, 47) X(48, 48)
constexpr int kNumClass8 = 7;

// Ranges of row lengths of the query kernel, one translation unit each: kQuerySpan
// lengths, the last one more.
#define NW_QUERY X(0, 15) X(16, 31) X(32, 48)
constexpr int kQuerySpan = 16, kNumQuery = 3;

// Classes of four lengths of the bit-plane kernels, by translation unit.
#define NW_BITS_SPLITS X(0, 1) X(2, 2) X(3, 3) X(4, 4) X(5, 5) X(6, 6) X(7, 7) X(8, 8) X(9, 9) X(10, 10) X(11, 11)

// Bit-plane triangle and edge kernels: translation units (variant, range of lengths).
#define NW_TRI_BITS X(0, 0) X(0, 1) X(1, 0) X(1, 1) X(2, 0) X(2, 1) X(2, 2) X(2, 3) X(3, 0) X(3, 1) X(3, 2) X(3, 3) X(4, 0) X(4, 1) X(4, 2) X(4, 3) X(5, 0) X(5, 1) X(6, 0) X(6, 1) X(6, 2) X(6, 3)

struct KernelTables {
    const void *tri[kMaxLen + 1];
    const void *tri_code1[kMaxLen + 1];  // the same with score codes and dword stores, one row pair a step
    const void *tri_code2[kMaxLen + 1];  // two row pairs a step (rows 1 .. 16; else NULL)
    const void *probe_thr[kMaxLen + 1];  // threshold pre-pass by selection
    const void *topk[kMaxLen + 1];
    const void *topk_code[kMaxLen + 1];  // the same with the score-code epilogue
    const void *topk_bits[2][2][kMaxLen / 4];   // bit planes, classes of 4 lengths: [Bits2, Bits3][without, with histogram]
    // triangle: Bits2 int8, Bits2 int16, Bits3 int8, Bits3 int16, Bits3 int16 with 16-bit staging
    const void *tri_bits[5][4];                 // [variant][range of lengths]
    int tri_bits_threads[5][4];                 // and their threads per workgroup
    const void *edges_bits[2][4];               // threshold edges: Bits2, Bits3
    const void *edges[kMaxLen + 1];      // threshold edge emitter
    const void *persist1[kMaxLen + 1];   // persistent batched kernel, one per row length
    const void *persist8[kNumClass8];    // persistent batched kernel, one per class of 8 lengths
    const void *class8[kNumClass8];      // small-dictionary triangle kernel, one per class of 8 lengths
    const void *query[kNumQuery];        // queries, one per range of lengths
};

#define X(lo, hi) void nw_fill_##lo(KernelTables &t);
NW_LA_SPLITS
#undef X
#define X(v, r) void nw_fill_tri_bits_##v##_##r(KernelTables &t);
NW_TRI_BITS
#undef X
#define X(lo, hi) void nw_fill_bits_##lo(KernelTables &t);
NW_BITS_SPLITS
#undef X
#define X(lo, hi) void nw_fill_class_##lo(KernelTables &t);
NW_CLASS8
#undef X
#define X(lo, hi) void nw_fill_query_##lo(KernelTables &t);
NW_QUERY
#undef X

const KernelTables &kernel_tables();

}  // namespace nw
