// k_edges_bits.h -- the threshold edge emitter in bit planes (nw_bits.h): every
// pair of a tile is scored and tested against the weight slice 32 at a time.
//
// Layout and loop are those of k_topk_bits: a workgroup takes a block pair
// (r, b), the groups of 32 row words of one longest length LA and a share of
// the column block's 64-slot steps.  The slice is an interval of scores for
// each pair of lengths, so an interval of G for each (row word, column
// length): its ends are kept as planes in LDS per group and column length,
// and two comparisons (one function per plane each) test 32 pairs.  Passing
// pairs go to a queue of the wavefront's own; 192 of them are written at a
// time, one global atomic reserving their places.
//
// Bound: vector issue (the DP) where few pairs pass; where many do, the atomics
// on the one counter, about 12 ns each.  Hence the long queue (17,000 words of up
// to 16 symbols under a matrix, a fifth of the pairs pass: 9.7 ms packed, 5.9 ms
// with 64 at a time, 2.2 ms), and in a tile cut by the range the rows outside it
// are left out before the DP (333 rows of 600,000 words, 28 million edges: 18.1
// ms packed, 39.6 ms with the range tested at the queue, 6.7 ms).  Where hardly a
// pair passes, the longer drain and the mask cost 2 %: 100,000 words of up to 32
// symbols, the normalised slice [60, 100], 2.11 ms with 64 at a time, 2.16 here (with
// its graph and an ego network 13.7 ms packed, 2.5 ms).
#pragma once

#include "k_edges.h"
#include "k_topk_bits.h"

namespace nw {

constexpr uint32_t kEdgeBitsLds = 32u * 1024u;   // aim: five workgroups per CU
constexpr int kEdgeDrain = 192;                  // queue entries written at a time
constexpr int kEdgeQueue = kEdgeDrain + 64;      // entries of a wavefront's queue

__host__ __device__ constexpr uint32_t edges_bits_group_bytes(int LA, int tab, int wmax, int alphabet, int lmax)
{
    return bit_group_bytes(LA, tab, alphabet) + 2u * bit_thr_dwords(LA, wmax) * 4u * (uint32_t)(lmax + 1);
}
__host__ __device__ constexpr uint32_t edges_bits_fixed_bytes() { return (uint32_t)(kThreads / 64) * kEdgeQueue * 4u + 16u; }
__host__ __device__ inline int edges_bits_groups(int LA, int tab, int wmax, int alphabet, int lmax, uint32_t lds)
{
    const uint32_t per = edges_bits_group_bytes(LA, tab, wmax, alphabet, lmax), fixed = edges_bits_fixed_bytes();
    if (lds < fixed + per) return 0;
    const uint32_t kg = (lds - fixed) / per;
    return kg < (uint32_t)kBitMaxGroups ? (int)kg : kBitMaxGroups;
}
__host__ __device__ inline uint32_t edges_bits_lds_bytes(int LA, int tab, int wmax, const DevVocab &V, int most)
{
    const uint32_t per = edges_bits_group_bytes(LA, tab, wmax, V.alphabet, V.lmax), fixed = edges_bits_fixed_bytes();
    return bit_lds_bytes(fixed, per, kEdgeBitsLds, (uint32_t)most);
}

// The scores of the slice for a pair whose longer word has m (>= 1) symbols:
// smin .. smax (clamped to a range that keeps the later sums in 32 bits).
__device__ __forceinline__ void edge_scores(const EdgeSink &E, int m, int &smin, int &smax)
{
    int64_t a = E.lo, b = E.hi;
    if (E.normalised) {   // lo * m <= 100 s den <= hi * m
        const int64_t d = 100ll * E.den;
        const int64_t x = (int64_t)E.lo * m, y = (int64_t)E.hi * m;
        a = x >= 0 ? (x + d - 1) / d : -(-x / d);
        b = y >= 0 ? y / d : -((-y + d - 1) / d);
    }
    smin = (int)min(max(a, -(int64_t)100000), (int64_t)100000);
    smax = (int)min(max(b, -(int64_t)100000), (int64_t)100000);
}

// The pair indices of a call, the rows they lie in, and how its launches are cut.
struct EdgeRange {
    uint64_t idx_begin, idx_end;
    int32_t row0, row1;   // rows row0 .. row1 hold a pair of the range
    uint32_t rb0, rbn;    // tiles (tile_block_pair)
    int splits;           // parts the column steps of a tile are dealt to
    int hi;               // longest row length of the launch
    int most;             // row groups a workgroup takes at a time, at most
};

template <int LA, class S>
__device__ __forceinline__ void edges_bits_tile(const DevVocab &V, const EdgeSink &E, const EdgeRange &X, uint32_t r,
                                                uint32_t b, int part, uint32_t lds_bytes, uint8_t *lds)
{
    const uint64_t idx_begin = X.idx_begin, idx_end = X.idx_end;
    const int splits = X.splits;
    const uint32_t *rgo = V.rg_off + (size_t)r * (V.lmax + 1) + LA;
    const uint32_t gbeg = rgo[0], gend = rgo[1];
    if (gbeg >= gend) return;
    const int64_t n = V.n, CB = V.CB;
    const int64_t I0 = (int64_t)r * CB, I1 = min(I0 + CB, n);
    const int64_t J0 = (int64_t)b * CB, J1 = min(J0 + CB, n);
    // skip a tile outside [idx_begin, idx_end); test every passing pair only
    // when the tile straddles a bound (uniform)
    bool whole;
    {
        const int64_t jlo = (r == b) ? I0 + 1 : J0;
        if (jlo >= J1) return;
        const uint64_t first = row_start_idx(n, I0) + (uint64_t)(jlo - I0 - 1);
        const int64_t ilast = (r == b) ? J1 - 2 : I1 - 1;
        const uint64_t last = row_start_idx(n, ilast) + (uint64_t)(J1 - 1 - ilast - 1);
        if (last < idx_begin || first >= idx_end) return;
        whole = first >= idx_begin && last < idx_end;
    }

    constexpr int P = sum_planes<LA, S>();
    constexpr int PD = P > 0 ? P : 1;
    constexpr int PT = thr_planes<LA, S>();
    constexpr int TD = (int)bit_thr_dwords(LA, S::kWmax);
    constexpr int GMAX = S::kWmax * LA;
    const int A = V.alphabet, pabs = -V.gap, lmax = V.lmax;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kg = min(edges_bits_groups(LA, S::kTab, S::kWmax, A, lmax, lds_bytes), X.most);
    if (kg < 1) return;   // the launch's LDS holds a group (edges_bits_lds_bytes)
    const uint32_t gstride = edges_bits_group_bytes(LA, S::kTab, S::kWmax, A, lmax);
    const uint32_t thr_at = bit_group_bytes(LA, S::kTab, A);
    const uint32_t thr_b = (uint32_t)TD * 4u * (uint32_t)(lmax + 1);   // bytes of one end's planes
    const uint32_t lds0 = lds_addr_of(lds);
    uint32_t *queue = reinterpret_cast<uint32_t *>(lds + (uint32_t)kg * gstride) + wave * kEdgeQueue;
    uint32_t *counter = reinterpret_cast<uint32_t *>(lds + (uint32_t)kg * gstride + (kThreads / 64) * kEdgeQueue * 4u);
    const bool diag = r == b;
    const bool count_only = E.cap == 0 && whole;
    const int steps = ((int)CB / 64 - part + splits - 1) / splits;
    uint32_t counted = 0;   // this lane's pairs, when only counting

    // chunks of kg groups, every gridDim.z-th
    for (uint32_t gc = gbeg + blockIdx.z * (uint32_t)kg; gc < gend; gc += gridDim.z * (uint32_t)kg) {
        const int ng = (int)min((uint32_t)kg, gend - gc);
        build_groups<LA, S, kThreads>(V, I0, ng, lds, gstride,
                                      [&](int g, int q) { return ((int64_t)gc + g) * kBitRows + q; });
        // the ends of the slice as planes of G: lanes 0..31 the row words of
        // a group for one column length, lanes 32..63 for the next
        for (int x = wave; x < ng * ((lmax + 2) / 2); x += kThreads / 64) {
            const int ln = (int)in_vgpr((uint32_t)lane);   // (kept from hoisting the lane compares)
            const int g = x / ((lmax + 2) / 2);
            const int lb = 2 * (x % ((lmax + 2) / 2)) + (ln >> 5);
            const int64_t slot = ((int64_t)gc + g) * kBitRows + (ln & 31);
            int smin, smax;
            edge_scores(E, max(max((int)V.blen[slot], lb), 1), smin, smax);
            const int off = pabs * (LA + lb);
            const int t0 = min(max(smin + off, 0), GMAX + 1), t1 = min(max(smax + 1 + off, 0), GMAX + 1);
            uint32_t m0 = 0, m1 = 0;
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                const uint64_t b0 = __ballot((t0 >> q) & 1), b1 = __ballot((t1 >> q) & 1);
                if ((ln & 31) == q) {
                    m0 = ln & 32 ? (uint32_t)(b0 >> 32) : (uint32_t)b0;
                    m1 = ln & 32 ? (uint32_t)(b1 >> 32) : (uint32_t)b1;
                }
            }
            if ((ln & 31) < PT && lb <= lmax) {
                uint32_t *t = reinterpret_cast<uint32_t *>(lds + (uint32_t)g * gstride + thr_at) + lb * TD + (ln & 31);
                t[0] = m0;
                t[thr_b / 4] = m1;
            }
        }
        if (tid == 0) *counter = 0;
        __syncthreads();

        int qn = 0;   // entries in this wavefront's queue (wave-uniform)
        // entry x, and whether its pair lies in the range
        auto entry = [&](int x, int64_t &u, int64_t &j, int &s) {
            const uint32_t e = queue[x];
            const int64_t slot = J0 + (int64_t)(e & 0xFFFu);
            u = bit_group<LA, S>(lds + (uint32_t)(e >> 17 & 7u) * gstride, A).cu[e >> 12 & 31u];
            j = J0 + V.bcol[slot];
            s = (int)(e >> 20) - pabs * (LA + (int)V.blen[slot]);
            if (whole) return true;
            const uint64_t idx = row_start_idx(n, u) + (uint64_t)(j - u - 1);
            return idx >= idx_begin && idx < idx_end;
        };
        // write the first m entries (at most kEdgeDrain)
        auto drain = [&](int m) {
            int64_t u, j;
            int s;
            uint32_t total = (uint32_t)m;
            if (!whole) {
                total = 0;
#pragma unroll 1
                for (int x = 0; x < m; x += 64) total += (uint32_t)__popcll(__ballot(x + lane < m && entry(x + lane, u, j, s)));
            }
            if (total == 0) return;
            unsigned long long base = 0;
            if (lane == 0) base = atomicAdd(E.count, (unsigned long long)total);
            base = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base) |
                   (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)) << 32;
            if (base >= E.cap) return;   // past the capacity: counted only
#pragma unroll 1
            for (int x = 0; x < m; x += 64) {
                const bool keep = x + lane < m && entry(x + lane, u, j, s);
                const uint64_t k = __ballot(keep);
                const uint64_t q = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(k >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)k, 0u));
                if (keep && q < E.cap) {
                    E.ei[q] = (int32_t)u;
                    E.ej[q] = (int32_t)j;
                    E.es[q] = (int16_t)s;
                }
                base += (unsigned long long)__popcll(k);
            }
        };
        for (;;) {
            uint32_t taken = 0;
            if (lane == 0) taken = atomicAdd(counter, 1u);
            taken = (uint32_t)__builtin_amdgcn_readfirstlane((int)taken);
            if (taken >= (uint32_t)steps) break;
            const int st = part + (steps - 1 - (int)taken) * splits;   // longest words first
            const ColWords W = col_words(V.ccol, V.blen, J0 / 64 + st, lane);
            const uint32_t col = V.bcol[J0 + st * 64 + lane];
            const int64_t j = J0 + col;
            for (int g = 0; g < ng; ++g) {
                const uint32_t gb = (uint32_t)g * gstride;
                const BitGroup G = bit_group<LA, S>(lds + gb, A);
                // pairs that count: present words, rows of the range, and each
                // unordered pair once (in a diagonal block only j > u)
                uint32_t valid = col != 0xFFFFu ? ~0u : 0u;
                if (!whole) {
                    const int32_t u = G.cu[lane & (kBitRows - 1)];
                    const uint32_t rows = (uint32_t)__ballot(u >= X.row0 && u <= X.row1);
                    if (rows == 0) continue;
                    valid &= rows;
                }
                BitColumn<LA, S> C;
                C.run(W, lds0 + gb);
                if constexpr (LA > 0) {
                    if (__builtin_amdgcn_readfirstlane((int)G.rowmask[LA - 1]) != ~0) C.fill_short_rows(G.rowmask, pabs);
                }
                if (diag || LA == 0 || __builtin_amdgcn_readfirstlane(G.cu[0]) < 0) {
                    uint32_t absent = 0;
#pragma unroll 4
                    for (int q = 0; q < kBitRows; ++q) {
                        const int32_t u = G.cu[q];
                        absent = absent >> 1 | (u < 0 || (diag && j <= u) ? 0x80000000u : 0u);
                    }
                    valid &= ~absent;
                }
                uint32_t s[PD];
                if constexpr (P > 0) C.template sum<P>(s); else s[0] = 0;
                auto planes = [&](uint32_t at, uint32_t (&t)[PT]) {
#pragma unroll
                    for (int q = 0; q < TD / 4; ++q) {
                        const u32x4 x = *(const lds_u32x4 *)(uintptr_t)(at + 16u * (uint32_t)q);
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (4 * q + k < PT) t[4 * q + k < PT ? 4 * q + k : 0] = x[k];
                    }
                };
                uint32_t t0[PT], t1[PT];
                const uint32_t ta = lds0 + gb + thr_at + (uint32_t)W.lb * (TD * 4u);
                planes(ta, t0);
                planes(ta + thr_b, t1);
                uint32_t ev = at_least<PD, PT>(s, t0) & ~at_least<PD, PT>(s, t1) & valid;
                if (count_only) {
                    counted += (uint32_t)__builtin_popcount(ev);
                    continue;
                }
                uint64_t any = __ballot(ev != 0);
                while (any) {
                    if (ev) {
                        const uint32_t q = (uint32_t)__builtin_ctz(ev);
                        const uint32_t at = (uint32_t)qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u));
                        queue[at] = pair_sum<PD>(s, q) << 20 | (uint32_t)g << 17 | q << 12 | (uint32_t)(st * 64 + lane);
                        ev &= ev - 1u;
                    }
                    qn += (int)__popcll(any);
                    if (qn >= kEdgeDrain) {
                        drain(kEdgeDrain);
                        const uint32_t e = queue[kEdgeDrain + lane];
                        qn -= kEdgeDrain;
                        if (lane < qn) queue[lane] = e;
                    }
                    any = __ballot(ev != 0);
                }
            }
        }
        if (qn) drain(qn);
        __syncthreads();
    }
    if (count_only) {
#pragma unroll
        for (int d = 32; d; d >>= 1) counted += (uint32_t)__shfl_xor((int)counted, d);
        if (lane == 0 && counted) atomicAdd(E.count, (unsigned long long)counted);
    }
}

// Longest row lengths LO .. HI, one per blockIdx.y, the longest first;
// blockIdx.x = tile * splits + part, blockIdx.z = the part of the row groups.
template <int LO, int HI, class S>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(bits_min_waves<HI, S>())))
void k_edges_bits(DevVocab V, EdgeSink E, EdgeRange X, uint32_t lds_bytes)
{
    extern __shared__ __align__(16) uint8_t lds[];
    uint32_t r, b;
    if (!tile_block_pair(blockIdx.x / (uint32_t)X.splits, X.rb0, X.rbn, V.nb, r, b)) return;
    const int part = (int)(blockIdx.x % (uint32_t)X.splits);
    const int LA = X.hi - (int)blockIdx.y;
    if (LA < LO || LA > HI) return;
    bit_length_dispatch<LO, HI>(
        LA, [&](auto la) { edges_bits_tile<decltype(la)::value, S>(V, E, X, r, b, part, lds_bytes, lds); });
}

}  // namespace nw
