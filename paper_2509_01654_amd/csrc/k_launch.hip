// k_launch.hip -- launchers of every kernel, and the naive triangle kernel.
//
// Naive kernel (k_tri_naive): the paper's GPU scheme (Section 4.2): one thread
// per pair index, a 1-D grid, idx -> (row, column) through the closed form of
// the row index, and one DP per thread with its scratch in shared memory (one
// row of the score matrix instead of the whole matrix).
#define NW_LAUNCH_TU 1
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "k_batch.h"
#include "k_diag.h"
#include "k_edges.h"
#include "k_edges_bits.h"
#include "k_probe.h"
#include "k_query.h"
#include "k_topk.h"
#include "k_topk_bits.h"
#include "k_topk_code.h"
#include "k_tri_bits.h"
#include "k_tri_code.h"
#include "k_tri_tiled.h"
#include "nw_fork.h"
#include "nw_kernels.h"

namespace nw {

// CAP: scratch row capacity (longest word + 1); NT: threads per block.  The
// score goes to out (OUT_I8 / OUT_I16) or, if it passes the slice, to E.
template <int CAP, int NT>
__global__ __launch_bounds__(NT) void k_tri_naive(DevVocab V, uint64_t idx_begin, uint64_t idx_end, void *out,
                                                  int out_kind, EdgeSink E)
{
    __shared__ int16_t rows[NT][CAP];
    int16_t *row = rows[threadIdx.x];   // this thread's scratch: one row of the score matrix
    const int64_t n = V.n;
    const int gap = V.gap;
    const double z = (double)n - 0.5;
    for (uint64_t idx = idx_begin + (uint64_t)blockIdx.x * NT + threadIdx.x; idx < idx_end;
         idx += (uint64_t)gridDim.x * NT) {
        // r = floor(z - sqrt(z^2 - 2 idx)), z = n - 1/2 (Section 4.2), then an
        // integer fix-up so rounding can never pick the wrong row
        int64_t r = (int64_t)floor(z - sqrt(z * z - 2.0 * (double)idx));
        if (r < 0) r = 0;
        if (r > n - 2) r = n - 2;
        while (r > 0 && row_start_idx(n, r) > idx) --r;
        while (r + 1 < n - 1 && row_start_idx(n, r + 1) <= idx) ++r;
        const int64_t c = r + 1 + (int64_t)(idx - row_start_idx(n, r));
        const int la = V.clen[r], lb = V.clen[c];
        const uint8_t *A = V.csym + r * V.WB;
        const uint8_t *B = V.csym + c * V.WB;
        for (int j = 0; j <= lb; ++j) row[j] = (int16_t)(gap * j);
        for (int i = 1; i <= la; ++i) {
            int diag = row[0];
            row[0] = (int16_t)(gap * i);
            const int a = A[i - 1];
            for (int j = 1; j <= lb; ++j) {
                const int bsym = B[j - 1];
                const int sim = V.has_submat ? (int)V.submat[a * V.alphabet + bsym] : (a == bsym ? V.match : V.mismatch);
                const int up = row[j];
                int v = diag + sim;
                v = max(v, up + gap);
                v = max(v, (int)row[j - 1] + gap);
                diag = up;
                row[j] = (int16_t)v;
            }
        }
        const int score = row[lb];
        if (out_kind == OUT_I8)
            static_cast<int8_t *>(out)[idx - idx_begin] = (int8_t)score;
        else if (out_kind == OUT_I16)
            static_cast<int16_t *>(out)[idx - idx_begin] = (int16_t)score;
        else if (edge_passes(E, score, la, lb))
            edge_direct(E, (int32_t)r, (int32_t)c, score);
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
const KernelTables &kernel_tables()
{
    static KernelTables t;
    static bool init = [] {
#define X(lo, hi) nw_fill_##lo(t);
        NW_LA_SPLITS
#undef X
#define X(v, r) nw_fill_tri_bits_##v##_##r(t);
        NW_TRI_BITS
#undef X
#define X(lo, hi) nw_fill_bits_##lo(t);
        NW_BITS_SPLITS
#undef X
#define X(lo, hi) nw_fill_class_##lo(t);
        NW_CLASS8
#undef X
#define X(lo, hi) nw_fill_query_##lo(t);
        NW_QUERY
#undef X
        return true;
    }();
    (void)init;
    return t;
}

// A launch through a fork (a stream, or a node of the graph being captured).
static hipError_t launch_dyn(const void *fn, dim3 grid, size_t lds, StreamFork &fork, void **args,
                             int threads = kThreads)
{
    if (lds > 65536) {
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return fork.launch(fn, grid, dim3(threads), lds, args);
}

// Row of pair index idx in the row-major triangle of n words: the largest u
// with S_{u-1} = (n-1)u - u(u-1)/2 <= idx (Section 4.2), by bisection.
static int64_t row_of_index(int64_t n, uint64_t idx)
{
    auto start = [n](int64_t u) { return (uint64_t)(n - 1) * (uint64_t)u - (uint64_t)u * (uint64_t)(u - 1) / 2u; };
    int64_t lo = 0, hi = n - 2;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) / 2;
        if (start(mid) <= idx) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Grid of a triangle launch over pair indices [idx_begin, idx_end): the whole
// column-major block-pair space, or a row-major window over the block rows
// the range touches when that is smaller.
struct TriGrid {
    uint32_t blocks, rb0, rbn;
};
static TriGrid tri_grid(const DevVocab &V, uint64_t idx_begin, uint64_t idx_end)
{
    const uint64_t all = (uint64_t)V.nb * (V.nb + 1) / 2;
    const uint32_t r0 = (uint32_t)(row_of_index(V.n, idx_begin) / V.CB);
    const uint32_t r1 = (uint32_t)(row_of_index(V.n, idx_end - 1) / V.CB);
    const uint64_t win = (uint64_t)(r1 - r0 + 1) * (uint64_t)V.nb;
    if (win < all) return {(uint32_t)win, r0, r1 - r0 + 1};
    return {(uint32_t)all, 0, 0};
}

// How many runs of row pairs a launch of `tiles` tiles cuts each tile of a
// row length into (at most maxrp row pairs per tile).  A launch with fewer
// tiles than workgroup slots (256 CUs x 6) splits its tiles into runs of at
// least kMinRowPairs row pairs, up to about four workgroups per slot; short
// runs cost more than they balance.
static uint32_t tile_chunks(uint64_t tiles, uint32_t maxrp)
{
    constexpr uint64_t kTargetWorkgroups = 256 * 6 * 4;
    constexpr uint64_t kSplitBelow = 2048;
    constexpr uint32_t kMinRowPairs = 16;
    if (tiles >= kSplitBelow) return 1;
    const uint32_t want = (uint32_t)((kTargetWorkgroups + tiles - 1) / tiles);
    return std::max<uint32_t>(1, std::min(want, maxrp / kMinRowPairs));
}

// NW_EPILOGUE=plain keeps the kernels with the plain integer epilogue where
// the score-code kernels would apply (both are exact; for comparisons).
static bool plain_epilogue_only()
{
    static const bool only = [] {
        const char *e = std::getenv("NW_EPILOGUE");
        return e && std::strcmp(e, "plain") == 0;
    }();
    return only;
}

// NW_DP=packed keeps the packed binary16 kernels where the bit-plane kernels
// would apply (both are exact; for comparisons).
static bool packed_dp_only()
{
    static const bool only = [] {
        const char *e = std::getenv("NW_DP");
        return e && std::strcmp(e, "packed") == 0;
    }();
    return only;
}

// The scalar parameters of a dictionary's bit-plane scheme.
static int bit_tab(const DevVocab &V) { return V.bits == 2 ? Bits2::kTab : Bits3::kTab; }
static int bit_wmax(const DevVocab &V) { return V.bits == 2 ? Bits2::kWmax : Bits3::kWmax; }

// Launches of the packed triangle kernels of dictionaries up to
// kClassLaunchMaxWords words: one per class of 8 row lengths present.
static uint32_t class_launches(const DevVocab &V, const uint32_t *h_maxrp)
{
    uint32_t launches = 0;
    for (int lo = 0; lo <= V.lmax; lo += 8) {
        uint32_t rows = 0;
        for (int LA = lo; LA <= std::min(lo + 7, (int)V.lmax); ++LA) rows += h_maxrp[LA];
        launches += rows > 0;
    }
    return launches;
}

// The launches of a bit-plane triangle or edge call over the lengths present in h_maxrp:
// ranges of row lengths (bits_span), the longest rows first.
struct LengthRange {
    int lo, hi, range;
};
static std::vector<LengthRange> bits_launches(const DevVocab &V, const uint32_t *h_maxrp)
{
    std::vector<LengthRange> out;
    const int span = V.bits == 2 ? bits_span<Bits2>() : bits_span<Bits3>();
    for (int r = (V.lmax - 1) / span; r >= 0; --r) {
        int lo = r == 0 ? 0 : r * span + 1, hi = std::min((r + 1) * span, (int)V.lmax);
        while (lo <= hi && h_maxrp[lo] == 0) ++lo;
        while (lo <= hi && h_maxrp[hi] == 0) --hi;
        if (lo <= hi) out.push_back({lo, hi, r});
    }
    return out;
}

// Whether planes are the faster for the scores of pair indices [idx_begin, idx_end)
// of a dictionary of up to kClassLaunchMaxWords words.  They score 32 rows at once,
// so the least time of a workgroup is 7 (two planes) or 22 (three) instructions for
// every cell of the longest words, against 1 for a packed pair of rows; they save
// launches (one per 24 or 12 row lengths against one per 8) and the rows of a block
// outside the range.  The lines are from 2,500 random calls timed on both sides
// (2 .. 16,384 words, 4 to 200 symbols, mixed, narrow and single lengths to 48, whole
// triangles and ranges); the choice costs 1.2 % (two planes) and 1.6 % (three) over
// the better side on average, planes wherever they apply 6 % and 18 %.
// - Two planes, and three up to 12 symbols: but for short calls that are one launch
//   on either side.  Words of one length, int16, packed / planes, us: two planes, 200
//   words of 24 / 48 symbols 30 / 40, 48 / 73, 700 words 34 / 40, 66 / 74, 1,500
//   words of 24 symbols 58 / 40; three, 700 / 1,500 / 2,300 words of 12 symbols 28 /
//   43, 48 / 49, 79 / 54.
// - Three planes past 12 symbols: packed up to 2,304 words (with 16-bit staging in
//   windows of a block, words to 48 symbols 197 / 277), then by estimates, us,
//   fitted to the calls above (log error 0.23 packed, 0.21 planes).  A million pairs
//   of 5,000 words of 30..48 symbols 131 / 234, of 16,384 words 475 / 257; 3,000 words
//   to 24 symbols 149 / 97.
static bool planes_faster(const DevVocab &V, const uint32_t *h_maxrp, uint64_t idx_begin, uint64_t idx_end)
{
    constexpr int kPlanesShortWords = 12;
    constexpr int64_t kOneLaunchWords = 4096, kPlanesAboveWords = 2304;
    const uint64_t pairs = idx_end - idx_begin;
    const uint32_t np = class_launches(V, h_maxrp), nb = (uint32_t)bits_launches(V, h_maxrp).size();
    if (V.bits == 2 || V.lmax <= kPlanesShortWords)
        return np > nb || V.n > kOneLaunchWords || pairs >= (V.bits == 2 ? 330000u : 900000u);
    if (V.n <= kPlanesAboveWords) return false;
    double block_pairs = 0, rows = 0, symbols = 0;   // pairs of the block rows the range touches
    const int64_t r0 = row_of_index(V.n, idx_begin) / V.CB, r1 = row_of_index(V.n, idx_end - 1) / V.CB;
    for (int64_t r = r0; r <= r1; ++r)
        block_pairs += (double)(std::min<int64_t>(V.n, (r + 1) * V.CB) - r * V.CB) * (double)(V.n - r * V.CB);
    for (int LA = 0; LA <= V.lmax; ++LA) {
        rows += h_maxrp[LA];
        symbols += (double)LA * h_maxrp[LA];
    }
    const double cells = symbols / rows * (symbols / rows) * 1e-9;   // of a pair of mean lengths, in 1e9
    const int steps = std::max(1, V.TW / (tri_bits_wide(V) ? 512 : 256));   // 64-column steps of a wavefront
    const double packed = 40 + 8.4 * np + 65 * block_pairs * cells;
    const double planes = 45 + 0.75 * V.lmax + 0.025 * steps * V.lmax * V.lmax + 26 * (double)pairs * cells;
    return planes < packed;
}

// Scores (not edges) of dictionaries the bit planes hold, where the staging
// and one group of the longest row words fit in LDS.  16-bit staging covers
// every score range of Bits3; Bits2 ranges fit a byte (at most 5 x 48 values).
// Above kClassLaunchMaxWords words planes are the faster in every form measured.
static bool triangle_bits_applies(const DevVocab &V, const uint32_t *h_maxrp, uint64_t idx_begin, uint64_t idx_end,
                                  int out_kind)
{
    if (V.bits == 0 || out_kind == OUT_EDGES || packed_dp_only()) return false;
    const bool w16 = tri_bits_wide(V);
    if (w16 && V.bits == 2) return false;
    if (tri_bits_lds_bytes(V.lmax, bit_tab(V), V, w16, 1) > kMaxLdsBytes) return false;
    return V.n > kClassLaunchMaxWords || planes_faster(V, h_maxrp, idx_begin, idx_end);
}

static hipError_t launch_triangle_bits(const DevVocab &V, const uint32_t *h_maxrp, uint64_t idx_begin, uint64_t idx_end,
                                       int out_kind, void *d_out, StreamFork &fork)
{
    const KernelTables &tab = kernel_tables();
    const bool w16 = tri_bits_wide(V);
    const int scheme = w16 ? 4 : 2 * (V.bits - 2) + (out_kind == OUT_I8 ? 0 : 1);
    const int64_t row0 = row_of_index(V.n, idx_begin), row1 = row_of_index(V.n, idx_end - 1);
    uint32_t rb0 = (uint32_t)(row0 / V.CB);
    const uint32_t nr = (uint32_t)(row1 / V.CB) - rb0 + 1;
    const std::vector<LengthRange> launches = bits_launches(V, h_maxrp);
    // Groups a workgroup takes at a time: one table build serves them, but they
    // run one after the other, so fewer where the call has less than kEnough
    // workgroups.  Four / one, words of one length, int16, us: 2,300 words of 24
    // symbols 90 / 48, 4,000 words of 24 symbols under a matrix 295 / 191.
    int most = kTriBitGroups;
    {
        constexpr uint64_t kEnough = 1024;
        const uint64_t tiles = std::max<uint64_t>(1, (uint64_t)nr * V.nwin / 2);
        const uint64_t groups = ((uint64_t)std::min<int64_t>(row1 - row0 + 1, V.CB) + kBitRows - 1) / kBitRows;
        uint64_t lengths = 0;
        for (int LA = 0; LA <= V.lmax; ++LA) lengths += h_maxrp[LA] != 0;
        while (most > 1 && tiles * std::max(std::min(lengths, groups), groups / most) < kEnough) most /= 2;
    }
    // A workgroup takes one chunk of row groups (blockIdx.z) against nw
    // windows, its tables serving all of them: as many as leave kWorkgroups
    // workgroups.
    auto parts = [&](const LengthRange &L) {
        const uint32_t lds = tri_bits_lds_bytes(L.hi, bit_tab(V), V, w16, most);
        uint32_t parts = 1;
        for (int LA = L.lo; LA <= L.hi; ++LA) {
            // rows of longest length LA: those of that length, and up to a
            // group's worth of shorter ones at either end
            const uint32_t groups = h_maxrp[LA] * 2 / kBitRows + 2;
            const uint32_t kg = (uint32_t)tri_bits_groups(LA, bit_tab(V), V.alphabet, V.TW, V.CB, w16, lds, most);
            if (h_maxrp[LA]) parts = std::max(parts, (groups + kg - 1) / kg);
        }
        return parts;
    };
    constexpr uint64_t kWorkgroups = 8192;
    uint64_t chunks = 0;
    for (const LengthRange &L : launches) chunks += (uint64_t)parts(L) * (uint64_t)(L.hi - L.lo + 1);
    int nw = (int)std::max<uint64_t>(1, std::min<uint64_t>(8, chunks * nr * V.nwin / 2 / kWorkgroups));
    uint32_t nset = ((uint32_t)V.nwin + nw - 1) / nw;
    for (const LengthRange &L : launches) {
        DevVocab Vc = V;
        uint64_t ib = idx_begin, ie = idx_end;
        void *po = d_out;
        uint32_t lds = tri_bits_lds_bytes(L.hi, bit_tab(V), V, w16, most);
        int hi = L.hi;
        void *args[] = {&Vc, &ib, &ie, &po, &rb0, &nset, &nw, &hi, &lds, &most};
        hipError_t e = launch_dyn(tab.tri_bits[scheme][L.range],
                                  dim3(nr * nset, (uint32_t)(L.hi - L.lo + 1), parts(L)), lds, fork, args,
                                  tab.tri_bits_threads[scheme][L.range]);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

uint32_t triangle_launches(const DevVocab &V, const uint32_t *h_maxrp, int out_kind)
{
    if (V.n < 2) return 0;
    if (triangle_bits_applies(V, h_maxrp, 0, (uint64_t)V.n * (uint64_t)(V.n - 1) / 2, out_kind))
        return (uint32_t)bits_launches(V, h_maxrp).size();
    if (V.n <= kClassLaunchMaxWords) return class_launches(V, h_maxrp);
    uint32_t launches = 0;
    for (int LA = 0; LA <= V.lmax; ++LA) launches += h_maxrp[LA] > 0;
    return launches;
}

hipError_t launch_triangle_tiled(const DevVocab &V, const uint32_t *h_maxrp, uint64_t idx_begin, uint64_t idx_end,
                                 int out_kind, void *d_out, hipStream_t stream, const EdgeSink *E, StreamFork *shared)
{
    if (idx_begin >= idx_end || V.n < 2) return hipSuccess;
    const TriGrid G = tri_grid(V, idx_begin, idx_end);
    const KernelTables &tab = kernel_tables();
    StreamFork own(stream);
    if (!shared) {
        hipError_t ef = own.begin();
        if (ef != hipSuccess) return ef;
    }
    StreamFork &fork = shared ? *shared : own;
    if (triangle_bits_applies(V, h_maxrp, idx_begin, idx_end, out_kind)) {
        const hipError_t e = launch_triangle_bits(V, h_maxrp, idx_begin, idx_end, out_kind, d_out, fork);
        if (e != hipSuccess) return e;
        return shared ? hipSuccess : own.end();
    }
    if (V.n <= kClassLaunchMaxWords) {
        // small dictionaries: one launch per class of 8 row lengths
        // (k_tri_class; the per-length launches would be bound by launch cost)
        for (int c = 0; c < kNumClass8 && 8 * c <= V.lmax; ++c) {
            const int lo = 8 * c, hi = std::min(8 * c + 7, (int)V.lmax);
            uint32_t rows = 0, maxrp = 0;
            size_t lds = 0;
            for (int LA = lo; LA <= hi; ++LA) {
                rows += h_maxrp[LA];
                maxrp = std::max(maxrp, h_maxrp[LA]);
                lds = std::max<size_t>(lds, tri_lds_bytes(LA, V.alphabet, V.CB));
            }
            if (rows == 0) continue;
            // runs of at least two row pairs, about 2048 workgroups per launch
            const uint64_t ny = (uint64_t)(hi - lo + 1);
            uint32_t chunks = (uint32_t)std::max<uint64_t>(
                1, std::min<uint64_t>((2048 + G.blocks * ny - 1) / (G.blocks * ny), (maxrp + 1) / 2));
            uint32_t rpc = (maxrp + chunks - 1) / chunks;
            DevVocab Vc = V;
            uint64_t ib = idx_begin, ie = idx_end;
            void *po = d_out;
            int ok = out_kind;
            EdgeSink es = E ? *E : EdgeSink{};
            uint32_t rb0 = G.rb0, rbn = G.rbn;
            void *args[] = {&Vc, &ib, &ie, &po, &ok, &es, &rb0, &rbn, &chunks, &rpc};
            hipError_t e = launch_dyn(tab.class8[c], dim3((uint32_t)((uint64_t)G.blocks * chunks), (uint32_t)ny), lds,
                                      fork, args);
            if (e != hipSuccess) return e;
        }
        return shared ? hipSuccess : own.end();
    }
    const bool code_ok = out_kind != OUT_EDGES && !plain_epilogue_only();
    for (int LA = 0; LA <= V.lmax; ++LA) {
        if (h_maxrp[LA] == 0) continue;   // no block has row pairs of this length
        uint32_t chunks = tile_chunks(G.blocks, h_maxrp[LA]);
        uint32_t rpc = (h_maxrp[LA] + chunks - 1) / chunks;
        int esz = out_kind == OUT_I8 ? 1 : 2;
        const int R = code_ok && tab.tri_code2[LA] && tri_code_applies(V, LA, esz, 2)   ? 2
                      : code_ok && tri_code_applies(V, LA, esz, 1) ? 1
                                                                   : 0;
        if (R) {
            // runs of whole steps
            rpc = (rpc + R - 1) / R * R;
            DevVocab Vc = V;
            uint64_t ib = idx_begin, ie = idx_end;
            void *po = d_out;
            uint32_t rb0 = G.rb0, rbn = G.rbn;
            void *args[] = {&Vc, &ib, &ie, &po, &esz, &rb0, &rbn, &chunks, &rpc};
            hipError_t e = launch_dyn(R == 2 ? tab.tri_code2[LA] : tab.tri_code1[LA],
                                      dim3((uint32_t)((uint64_t)G.blocks * chunks)),
                                      tri_code_lds_bytes(LA, V.alphabet, V.CB, esz, R), fork, args);
            if (e != hipSuccess) return e;
            continue;
        }
        DevVocab Vc = V;
        uint64_t ib = idx_begin, ie = idx_end;
        void *po = d_out;
        int ok = out_kind;
        EdgeSink es = E ? *E : EdgeSink{};
        uint32_t rb0 = G.rb0, rbn = G.rbn;
        void *args[] = {&Vc, &ib, &ie, &po, &ok, &es, &rb0, &rbn, &chunks, &rpc};
        hipError_t e = launch_dyn(tab.tri[LA], dim3((uint32_t)((uint64_t)G.blocks * chunks)),
                                  tri_lds_bytes(LA, V.alphabet, V.CB), fork, args);
        if (e != hipSuccess) return e;
    }
    return shared ? hipSuccess : own.end();
}

// Parts the 64-word column steps of a tile are dealt to: a launch of few tiles
// (each one workgroup per row length) halves them until it has 384, or four
// steps, one per wavefront, are left.  20k words (210 tiles): main pass
// 0.53 -> 0.35 ms; 30k words with a matrix (465 tiles, larger tables to
// build): 3.7 ms whole, 4.0 ms in three parts.
static int col_splits(uint64_t tiles, int CB)
{
    int s = 1;
    while (tiles * s < 384 && 2 * s <= CB / 256) s *= 2;
    return s;
}

// How many row groups a workgroup of the edge emitter takes at a time (most), and
// over how many workgroups a tile's groups of one length are dealt (parts).  With
// all of them in turn, a tile of a dictionary of few lengths is one long chain
// while the chip idles: below kEnough workgroups they are dealt, down to one group
// each.  Words of one length, packed / a workgroup a tile / dealt, us: 2,300 words
// of 24 symbols under a matrix 320 / 516 / 168, 700 words of 48 symbols 275 / 471
// / 107.
static void bits_parts(const DevVocab &V, const uint32_t *h_maxrp, const LengthRange &L, uint64_t tiles, int &most,
                       uint32_t &parts)
{
    constexpr uint64_t kEnough = 2048;
    uint32_t lengths = 0, groups = 1;
    for (int LA = L.lo; LA <= L.hi; ++LA) {
        lengths += h_maxrp[LA] != 0;
        // groups with their longest word of length LA: its words, and up to a
        // group's worth of shorter ones
        if (h_maxrp[LA]) groups = std::max(groups, h_maxrp[LA] * 2 / kBitRows + 1);
    }
    groups = std::min(groups, (uint32_t)V.CB / kBitRows);
    most = kBitMaxGroups;
    parts = 1;
    while (parts < groups && tiles * lengths * parts < kEnough) parts *= 2;
    if (parts > 1) {
        most = (int)std::min<uint32_t>(kBitMaxGroups, (groups + parts - 1) / parts);
        parts = (groups + most - 1) / most;
    }
}

// A few words make one workgroup, whose 32-row steps take longer than the packed
// rows.  Packed / planes, us: one length of 48 symbols, 6 words 91 / 106, 8 words
// 104 / 106 (two planes); 12 words 143 / 190, 16 words 173 / 191, lengths 1..48, 24
// words 174 / 213, 32 words 207 / 217 (three).
static int64_t edges_bits_min_words(const DevVocab &V) { return V.bits == 2 ? 8 : 32; }
static bool edges_bits_applies(const DevVocab &V)
{
    return V.bits != 0 && V.n >= edges_bits_min_words(V) && !packed_dp_only() && edges_bits_lds_bytes(V.lmax, bit_tab(V), bit_wmax(V), V, 1) <= kMaxLdsBytes;
}

hipError_t launch_edges_tiled(const DevVocab &V, const uint32_t *h_maxrp, uint64_t idx_begin, uint64_t idx_end,
                              const EdgeSink &E, hipStream_t stream)
{
    if (idx_begin >= idx_end || V.n < 2) return hipSuccess;
    const TriGrid G = tri_grid(V, idx_begin, idx_end);
    const KernelTables &tab = kernel_tables();
    StreamFork fork(stream);
    hipError_t ef = fork.begin();
    if (ef != hipSuccess) return ef;
    if (edges_bits_applies(V)) {
        for (const LengthRange &L : bits_launches(V, h_maxrp)) {
            DevVocab Vc = V;
            EdgeSink Ec = E;
            EdgeRange X;
            X.idx_begin = idx_begin;
            X.idx_end = idx_end;
            X.row0 = (int32_t)row_of_index(V.n, idx_begin);
            X.row1 = (int32_t)row_of_index(V.n, idx_end - 1);
            X.rb0 = G.rb0;
            X.rbn = G.rbn;
            X.splits = col_splits(G.blocks, V.CB);
            X.hi = L.hi;
            uint32_t parts;
            bits_parts(V, h_maxrp, L, (uint64_t)G.blocks * X.splits, X.most, parts);
            uint32_t lds = edges_bits_lds_bytes(L.hi, bit_tab(V), bit_wmax(V), V, X.most);
            void *args[] = {&Vc, &Ec, &X, &lds};
            hipError_t e = launch_dyn(tab.edges_bits[V.bits - 2][L.range],
                                      dim3((uint32_t)((uint64_t)G.blocks * X.splits), (uint32_t)(L.hi - L.lo + 1), parts),
                                      lds, fork, args);
            if (e != hipSuccess) return e;
        }
        return fork.end();
    }
    for (int LA = 0; LA <= V.lmax; ++LA) {
        if (h_maxrp[LA] == 0) continue;
        uint32_t chunks = tile_chunks(G.blocks, h_maxrp[LA]);
        uint32_t rpc = (h_maxrp[LA] + chunks - 1) / chunks;
        DevVocab Vc = V;
        EdgeSink Ec = E;
        uint64_t ib = idx_begin, ie = idx_end;
        uint32_t rb0 = G.rb0, rbn = G.rbn;
        void *args[] = {&Vc, &Ec, &ib, &ie, &rb0, &rbn, &chunks, &rpc};
        hipError_t e = launch_dyn(tab.edges[LA], dim3((uint32_t)((uint64_t)G.blocks * chunks)),
                                  edges_lds_bytes(LA, V.alphabet, V.CB), fork, args);
        if (e != hipSuccess) return e;
    }
    return fork.end();
}

hipError_t launch_triangle_naive(const DevVocab &V, uint64_t idx_begin, uint64_t idx_end, int out_kind, void *d_out,
                                 hipStream_t stream, const EdgeSink *E)
{
    if (idx_begin >= idx_end) return hipSuccess;
    const uint64_t count = idx_end - idx_begin;
    const bool lng = V.lmax > kMaxLen;
    const uint64_t nt = lng ? 64 : 256;
    const uint64_t blocks = (count + nt - 1) / nt;
    const uint32_t grid = (uint32_t)(blocks < (1u << 20) ? blocks : (1u << 20));
    const EdgeSink es = E ? *E : EdgeSink{};
    if (!lng)
        hipLaunchKernelGGL((k_tri_naive<kMaxLen + 1, 256>), dim3(grid), dim3(256), 0, stream, V, idx_begin, idx_end,
                           d_out, out_kind, es);
    else
        hipLaunchKernelGGL((k_tri_naive<kLongMaxLen + 1, 64>), dim3(grid), dim3(64), 0, stream, V, idx_begin, idx_end,
                           d_out, out_kind, es);
    return hipGetLastError();
}

bool diag_fits(const DevVocab &V)
{
    for (int c = 0; c < kDiagClasses; ++c)
        if (32 * c + 1 <= V.lmax && diag_lds_bytes(diag_rows_per_lane(c), V.alphabet, V.CB) > kMaxLdsBytes) return false;
    return true;
}

hipError_t launch_triangle_diag(const DevVocab &V, const uint32_t *h_maxrp, const uint32_t *h_maxdp,
                                uint64_t idx_begin, uint64_t idx_end, int out_kind, void *d_out, hipStream_t stream,
                                const EdgeSink *E)
{
    if (idx_begin >= idx_end || V.n < 2) return hipSuccess;
    // a class whose profile does not fit in LDS (large alphabets with long
    // words): the whole range goes through the one-thread-per-pair kernel
    if (!diag_fits(V)) return launch_triangle_naive(V, idx_begin, idx_end, out_kind, d_out, stream, E);
    const TriGrid G = tri_grid(V, idx_begin, idx_end);
    const KernelTables &tab = kernel_tables();
    StreamFork fork(stream);
    hipError_t ef = fork.begin();
    if (ef != hipSuccess) return ef;
    DevVocab Vc = V;
    uint64_t ib = idx_begin, ie = idx_end;
    void *po = d_out;
    int ok = out_kind;
    EdgeSink es = E ? *E : EdgeSink{};
    uint32_t rb0 = G.rb0, rbn = G.rbn;
    if (h_maxrp[0] != 0) {   // empty row words: score gap * lb, the register-row kernel of length 0
        uint32_t one = 1, all = 0xFFFFFFFFu;
        void *args[] = {&Vc, &ib, &ie, &po, &ok, &es, &rb0, &rbn, &one, &all};
        hipError_t e = launch_dyn(tab.tri[0], dim3(G.blocks), tri_lds_bytes(0, V.alphabet, V.CB), fork, args);
        if (e != hipSuccess) return e;
    }
    for (int c = 0; c < kDiagClasses; ++c) {
        const int R = diag_rows_per_lane(c);
        const uint32_t maxrp = h_maxdp[c];   // most row pairs of this class in one block
        if (maxrp == 0) continue;
        // runs of row pairs so that a launch has about kDiagWorkgroups workgroups
        constexpr uint64_t kDiagWorkgroups = 2048;
        uint32_t chunks = (uint32_t)std::min<uint64_t>(maxrp, std::max<uint64_t>(1, (kDiagWorkgroups + G.blocks - 1) / G.blocks));
        uint32_t rpc = (maxrp + chunks - 1) / chunks;
        static const void *const kDiag[kDiagClasses] = {
            reinterpret_cast<const void *>(&k_tri_diag<2>),  reinterpret_cast<const void *>(&k_tri_diag<4>),
            reinterpret_cast<const void *>(&k_tri_diag<6>),  reinterpret_cast<const void *>(&k_tri_diag<8>),
            reinterpret_cast<const void *>(&k_tri_diag<10>), reinterpret_cast<const void *>(&k_tri_diag<12>),
            reinterpret_cast<const void *>(&k_tri_diag<14>), reinterpret_cast<const void *>(&k_tri_diag<16>)};
        const void *fn = kDiag[c];
        void *args[] = {&Vc, &ib, &ie, &po, &ok, &es, &rb0, &rbn, &chunks, &rpc};
        const size_t lds = diag_lds_bytes(R, V.alphabet, V.CB);
        hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        e = fork.launch(fn, dim3((uint32_t)((uint64_t)G.blocks * chunks)), dim3(kDiagThreads), lds, args);
        if (e != hipSuccess) return e;
    }
    return fork.end();
}

hipError_t launch_query(const DevVocab &V, const RowSet &R, const uint32_t *h_off, const ColSet &C, int k,
                        int nsplit, uint64_t *partial, hipStream_t stream, bool fork_streams)
{
    const KernelTables &tab = kernel_tables();
    StreamFork fork(stream);
    if (fork_streams) {
        hipError_t ef = fork.begin();
        if (ef != hipSuccess) return ef;
    }
    int64_t per = (C.nslots + nsplit - 1) / nsplit;
    per = (per + kThreads - 1) / kThreads * kThreads;
    for (int c = 0; c < kNumQuery; ++c) {
        const int lo = kQuerySpan * c;
        int hi = c + 1 < kNumQuery ? lo + kQuerySpan - 1 : kMaxLen;
        const uint32_t np = h_off[hi + 1] - h_off[lo];
        if (np == 0) continue;
        while (h_off[hi + 1] == h_off[hi]) --hi;   // the longest present: its profile is the largest
        QueryArgs Q;
        Q.R = R;
        Q.C = C;
        Q.wtab = V.wtab;
        Q.alphabet = V.alphabet;
        Q.gap = V.gap;
        Q.lo = V.lo;
        Q.k = k;
        Q.per = per;
        Q.nsplit = nsplit;
        Q.partial = partial;
        void *args[] = {&Q};
        hipError_t e = launch_dyn(tab.query[c], dim3(np, nsplit), query_lds_bytes(hi, V.alphabet, k), fork, args);
        if (e != hipSuccess) return e;
    }
    return fork_streams ? fork.end() : hipSuccess;
}

// NW_PREPASS=lists keeps the list pre-pass (k_query_class + merge) where the
// selection would apply (both give the same keys; for comparisons).
static bool list_prepass_only()
{
    static const bool only = [] {
        const char *e = std::getenv("NW_PREPASS");
        return e && std::strcmp(e, "lists") == 0;
    }();
    return only;
}

bool probe_thr_applies(const DevVocab &V)
{
    return !list_prepass_only() && V.hi - V.lo <= kProbeMaxCode && V.pslots <= kProbeMaxSlots &&
           probe_lds_bytes(kMaxLen, V.alphabet, V.pslots) <= 65536u;
}

hipError_t launch_probe_thr(const DevVocab &V, const RowSet &R, const uint32_t *h_off, int m, uint64_t *thr,
                            hipStream_t stream)
{
    if (!probe_thr_applies(V)) return hipErrorNotSupported;
    const KernelTables &tab = kernel_tables();
    StreamFork fork(stream);
    hipError_t ef = fork.begin();
    if (ef != hipSuccess) return ef;
    const int rpw = 1;   // a workgroup per row pair: measured best of 1, 2, 4, 8 and 16
    for (int LA = 0; LA <= kMaxLen; ++LA) {
        const uint32_t np = h_off[LA + 1] - h_off[LA];
        if (np == 0) continue;
        ProbeArgs Q;
        Q.R = R;
        Q.C.sym = V.psym;
        Q.C.len = V.plen;
        Q.C.orig = V.porig;
        Q.C.nslots = V.pslots;
        Q.rank = V.prank;
        Q.wtab = V.wtab;
        Q.alphabet = V.alphabet;
        Q.gap = V.gap;
        Q.lo = V.lo;
        Q.m = m;
        Q.rpw = rpw;
        Q.n = V.n;
        Q.nprobe = V.nprobe;
        Q.thr = thr;
        void *args[] = {&Q};
        hipError_t e = launch_dyn(tab.probe_thr[LA], dim3((np + rpw - 1) / rpw), probe_lds_bytes(LA, V.alphabet, V.pslots),
                                  fork, args);
        if (e != hipSuccess) return e;
    }
    return fork.end();
}

hipError_t launch_merge(const uint64_t *partial, int P, int kin, int64_t rows, int kout, int lo, int16_t *score,
                        int32_t *index, uint64_t *thr, int rank, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    if ((int64_t)P * kin >= 1024) {   // many keys per row: a workgroup each
        hipLaunchKernelGGL(k_merge_lists_wg, dim3((uint32_t)rows), dim3(256), 0, stream, partial, P, kin, rows, kout, lo,
                           score, index, thr, rank);
        return hipGetLastError();
    }
    const uint32_t grid = (uint32_t)((rows + 3) / 4);
    hipLaunchKernelGGL(k_merge_lists, dim3(grid), dim3(256), 0, stream, partial, P, kin, rows, kout, lo, score, index,
                       thr, rank);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_column_layout(const uint8_t *csym, const uint8_t *len, const uint16_t *col,
                                                       int window, int WB, int64_t begin, int64_t end, uint32_t *ccol)
{
    const int64_t t = begin + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= end) return;
    const int lane = (int)(t & 63);
    const int64_t gq = t >> 6, g = gq / kColDwords;
    const int q = (int)(gq % kColDwords);
    const int64_t slot = g * 64 + lane;
    const int lb = len[slot], front = (int)len[g * 64 + 63] - lb;
    // padding slots have length 0 and read nothing
    const uint8_t *w = csym + (slot / window * window + (lb ? (int)col[slot] : 0)) * WB;
    uint32_t x = 0;
    for (int k = 0; k < 4; ++k) {
        const int i = 4 * q + k - front;
        if (i >= 0 && i < lb) x |= (uint32_t)w[i] << (8 * k);
    }
    ccol[t] = x;
}

hipError_t launch_column_layout(const DevVocab &V, const uint8_t *len, const uint16_t *col, int window, int64_t nslots,
                                uint32_t *ccol, hipStream_t stream)
{
    // a thread per dword, in launches of 2^30 threads (a grid holds fewer than 2^32)
    constexpr int64_t kSlice = (int64_t)1 << 30;
    const int64_t ndw = nslots * kColDwords;
    for (int64_t b = 0; b < ndw; b += kSlice) {
        const int64_t e = std::min(ndw, b + kSlice);
        hipLaunchKernelGGL(k_column_layout, dim3((uint32_t)((e - b + 255) / 256)), dim3(256), 0, stream, V.csym, len, col,
                           window, V.WB, b, e, ccol);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// The main pass takes the bit-plane kernels where the scoring fits them and
// the histogram copies fit beside one group of row words.
static bool topk_bits_applies(const DevVocab &V, const TopkArgs &T)
{
    if (V.bits == 0 || packed_dp_only()) return false;
    return (T.hist == nullptr || T.nbins <= kBitMaxBins) && T.lo <= V.lo &&
           topk_bits_lds_bytes(V.lmax, bit_tab(V), bit_wmax(V), V, T.nbins, T.hist != nullptr) <= kMaxLdsBytes;
}

hipError_t launch_topk_main(const DevVocab &V, const uint32_t *h_bitlens, const TopkArgs &T, hipStream_t stream)
{
    if (V.n < 2) return hipSuccess;
    const uint32_t nblk_pairs = (uint32_t)((uint64_t)V.nb * (V.nb + 1) / 2);
    const KernelTables &tab = kernel_tables();
    StreamFork fork(stream);
    hipError_t ef = fork.begin();
    if (ef != hipSuccess) return ef;
    const bool bits = topk_bits_applies(V, T);
    if (bits) {
        const int h = T.hist != nullptr;
        const uint64_t tiles = (uint64_t)nblk_pairs * (T.phase_hi - T.phase_lo + 1) / T.phase_mod;
        const bool rect = T.phase_lo == T.phase_hi;
        const uint32_t grid = rect ? (uint32_t)V.nb * ((uint32_t)(V.nb - T.phase_lo + T.phase_mod - 1) / (uint32_t)T.phase_mod)
                                   : nblk_pairs;
        if (rect && T.phase_lo >= V.nb) return fork.end();
        for (int c = 0; c < kBitClasses && bit_class_lo(c) <= V.lmax; ++c) {
            if (h_bitlens[c] == 0) continue;
            DevVocab Vc = V;
            TopkArgs Tc = T;
            Tc.bit_lds = topk_bits_lds_bytes(std::min(bit_class_hi(c), (int)V.lmax), bit_tab(V), bit_wmax(V), V, T.nbins, h);
            Tc.col_splits = col_splits(tiles, V.CB);
            Tc.phase_rect = rect;
            void *args[] = {&Vc, &Tc};
            hipError_t e = launch_dyn(tab.topk_bits[V.bits - 2][h][c], dim3(grid * (uint32_t)Tc.col_splits, h_bitlens[c]),
                                      Tc.bit_lds, fork, args);
            if (e != hipSuccess) return e;
        }
        return fork.end();
    }
    for (int LA = 0; LA <= V.lmax; ++LA) {
        DevVocab Vc = V;
        TopkArgs Tc = T;
        hipError_t e;
        if (!plain_epilogue_only() && topk_code_applies(V, T, LA)) {
            // score codes within [0, 1024), the histogram in LDS below 64 KiB
            Tc.hist_in_lds = T.hist != nullptr;
            Tc.wt_in_lds = topk_code_wt_in_lds(V, T, LA);
            void *args[] = {&Vc, &Tc};
            e = launch_dyn(tab.topk_code[LA], dim3(nblk_pairs),
                           topk_code_lds_bytes(LA, V.alphabet, T.nbins, Tc.hist_in_lds, V.CB, Tc.wt_in_lds), fork, args);
        } else {
            // the histogram copies go to LDS when they fit beside the profiles
            // (large alphabets with wide score ranges add to global bins instead)
            Tc.hist_in_lds = T.hist != nullptr && T.nbins <= kLdsHistMax &&
                             topk_lds_bytes(LA, V.alphabet, T.nbins, 1, V.CB) <= kMaxLdsBytes;
            void *args[] = {&Vc, &Tc};
            e = launch_dyn(tab.topk[LA], dim3(nblk_pairs), topk_lds_bytes(LA, V.alphabet, T.nbins, Tc.hist_in_lds, V.CB),
                           fork, args);
        }
        if (e != hipSuccess) return e;
    }
    return fork.end();
}

__global__ void k_scatter_lists(const int16_t *qs, const int32_t *qi, const int32_t *words, uint32_t B, int kq, int k,
                                int16_t *score, int32_t *index)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= B) return;
    const int32_t w = words[t];
    int o = 0;
    for (int c = 0; c < kq && o < k; ++c) {
        const int32_t j = qi[(size_t)t * kq + c];
        if (j == w) continue;   // no self-loops
        score[(size_t)w * k + o] = qs[(size_t)t * kq + c];
        index[(size_t)w * k + o] = j;
        ++o;
    }
    for (; o < k; ++o) {
        score[(size_t)w * k + o] = (int16_t)-32768;
        index[(size_t)w * k + o] = -1;
    }
}

hipError_t launch_scatter_lists(const int16_t *qs, const int32_t *qi, const int32_t *words, uint32_t B, int kq, int k,
                                int16_t *score, int32_t *index, hipStream_t stream)
{
    if (B == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter_lists, dim3((B + 255) / 256), dim3(256), 0, stream, qs, qi, words, B, kq, k, score,
                       index);
    return hipGetLastError();
}

namespace {
// Bytes carried by one upload launch (kernel arguments are at most 4 KiB).
constexpr uint32_t kUploadChunk = 3072;
struct UploadChunk {
    uint32_t off, n;
    uint8_t bytes[kUploadChunk];
};
// dst[c.off .. c.off + c.n) = c.bytes[0 .. c.n)
__global__ __launch_bounds__(256) void k_upload(uint8_t *dst, UploadChunk c)
{
    for (uint32_t i = threadIdx.x; i < c.n; i += blockDim.x) dst[c.off + i] = c.bytes[i];
}
}  // namespace

hipError_t launch_upload(void *dst, const void *src, uint64_t bytes, hipStream_t stream)
{
    for (uint64_t o = 0; o < bytes; o += kUploadChunk) {
        UploadChunk c;
        c.off = (uint32_t)o;
        c.n = (uint32_t)std::min<uint64_t>(kUploadChunk, bytes - o);
        std::memcpy(c.bytes, static_cast<const uint8_t *>(src) + o, c.n);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, stream, static_cast<uint8_t *>(dst), c);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_reset_counters(uint32_t *counters, int n, hipStream_t stream)
{
    hipLaunchKernelGGL(k_reset_counters, dim3((n + 63) / 64), dim3(64), 0, stream, counters, n);
    return hipGetLastError();
}

hipError_t launch_tighten(const uint32_t *cnt, const uint64_t *lists, uint32_t cap, int64_t n, int k, uint64_t *thr,
                          hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tighten, dim3((uint32_t)((n + 3) / 4)), dim3(256), 0, stream, cnt, lists, cap, n, k, thr);
    return hipGetLastError();
}

hipError_t launch_select(const uint32_t *cnt, const uint64_t *lists, uint32_t cap, int64_t n, int k, int lo,
                         int16_t *score, int32_t *index, uint32_t *ovf_count, int32_t *ovf_list, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const uint32_t grid = (uint32_t)((n + 3) / 4);
    hipLaunchKernelGGL(k_select, dim3(grid), dim3(256), 0, stream, cnt, lists, cap, n, k, lo, score, index, ovf_count,
                       ovf_list);
    return hipGetLastError();
}

}  // namespace nw
