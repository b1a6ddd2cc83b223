// k_topk_bits.h -- main pass of the fused top-k in bit planes (nw_bits.h).
//
// The same computation as k_topk_code and k_topk_tiled: every unordered pair
// of the block pair scored once, offered to both endpoints' candidate lists
// when it reaches their thresholds, counted once in the histogram.
//
// A workgroup takes a block pair (r, b) and block r's groups of 32 row words
// whose longest word has LA symbols, kg groups at a time: their symbol tables
// and threshold planes are built in LDS, then the wavefronts take the column
// block's 64-slot steps one by one from an LDS counter (longest words first)
// and run each against every group of the chunk.  No barrier falls inside a
// chunk.  Everything after the DP stays in planes:
//
// * the sum of the last column's differences (about two functions per plane
//   bit, all 32 pairs at once) is G; score = G + p (LA + lb);
// * thresholds: a pair reaches its row word's threshold when G is at least
//   that threshold's score - p (LA + lb), a number per (row word, lb) kept as
//   planes in LDS, and its column word's likewise with one number per lane:
//   one comparison function per plane each;
// * the pairs that reach one (about one in a thousand) are packed as (G, row
//   word, column slot) into a queue of the wavefront's own; once it holds 64
//   they are tested exactly and appended to the global lists by 64 lanes at
//   once, so no DP step waits on a global atomic;
// * histogram: where G takes at most kBitHistRegs values, a lane counts each
//   value's pairs (one function and one population count per value and 32
//   pairs) in a register over all groups of the chunk, and adds the counters
//   to the LDS copies once per column step; otherwise the planes are turned
//   to bytes and every pair adds to its bin.
//
// Bound: vector issue.  The DP's functions are 0.22 lane-instructions per cell;
// counted over the 600,000-word main pass, with columns run past a lane's own
// word, short rows, sums, tests and histogram, 0.32, where the packed form
// takes 1.18: 409 -> 82 ms.
#pragma once

#include "k_topk.h"
#include "nw_bits.h"

namespace nw {

constexpr int kBitHistRegs = 52;     // most values of G counted in registers
constexpr int kBitQueue = 128;       // queue entries per wavefront (64 are drained at a time)
constexpr uint32_t kBitTopkLds = 40u * 1024u;   // aim: four workgroups per CU
constexpr int kBitMaxBins = 512;     // histogram bins that fit in LDS copies
constexpr int kBitMaxGroups = 8;     // groups per chunk (3 bits of a queue entry)

template <int LA, class S>
__host__ __device__ constexpr bool bit_hist_regs() { return S::kWmax * LA + 1 <= kBitHistRegs; }
__host__ __device__ constexpr uint32_t bit_thr_dwords(int LA, int wmax)
{
    return (uint32_t)((bit_width((uint32_t)(wmax * LA + 1)) + 3) / 4 * 4);
}
// LDS: kg groups with their threshold planes, the wavefronts' queues, the
// histogram copies and the step counter.
__host__ __device__ constexpr uint32_t topk_bits_group_bytes(int LA, int tab, int wmax, int alphabet, int lmax)
{
    return bit_group_bytes(LA, tab, alphabet) + bit_thr_dwords(LA, wmax) * 4u * (uint32_t)(lmax + 1);
}
__host__ __device__ constexpr uint32_t topk_bits_fixed_bytes(int nbins, int has_hist)
{
    return (uint32_t)(kThreads / 64) * kBitQueue * 4u + ((topk_hist_bytes(nbins, has_hist) + 15u) & ~15u) + 16u;
}
// Groups per chunk within lds bytes (0 when not even one fits).
__host__ __device__ inline int topk_bits_groups(int LA, int tab, int wmax, int alphabet, int lmax, int nbins, int has_hist,
                                               uint32_t lds)
{
    const uint32_t per = topk_bits_group_bytes(LA, tab, wmax, alphabet, lmax);
    const uint32_t fixed = topk_bits_fixed_bytes(nbins, has_hist);
    if (lds < fixed + per) return 0;
    const uint32_t kg = (lds - fixed) / per;
    return kg < (uint32_t)kBitMaxGroups ? (int)kg : kBitMaxGroups;
}
// LDS of a launch whose longest row words have LA symbols: what is aimed at,
// or what one group needs.
__host__ __device__ inline uint32_t topk_bits_lds_bytes(int LA, int tab, int wmax, const DevVocab &V, int nbins, int has_hist)
{
    const uint32_t fixed = topk_bits_fixed_bytes(nbins, has_hist);
    const uint32_t per = topk_bits_group_bytes(LA, tab, wmax, V.alphabet, V.lmax);
    return bit_lds_bytes(fixed, per, kBitTopkLds, (uint32_t)kBitMaxGroups);
}

// One block pair's groups of longest length LA against every splits-th column
// step of the block, from step `part`.
template <int LA, class S, bool HIST>
__device__ __forceinline__ void topk_bits_tile(const DevVocab &V, const TopkArgs &T, uint32_t r, uint32_t b, int part,
                                               uint8_t *lds)
{
    const uint32_t *rgo = V.rg_off + (size_t)r * (V.lmax + 1) + LA;
    const uint32_t gbeg = rgo[0], gend = rgo[1];
    if (gbeg >= gend) return;

    constexpr int P = sum_planes<LA, S>();
    constexpr int PD = P > 0 ? P : 1;
    constexpr int PT = thr_planes<LA, S>();
    constexpr int TD = (int)bit_thr_dwords(LA, S::kWmax);
    constexpr int GMAX = S::kWmax * LA;
    constexpr bool REGS = HIST && bit_hist_regs<LA, S>();
    const int64_t I0 = (int64_t)r * V.CB, J0 = (int64_t)b * V.CB;
    const int A = V.alphabet, pabs = -V.gap, lmax = V.lmax;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kg = topk_bits_groups(LA, S::kTab, S::kWmax, A, lmax, T.nbins, HIST, T.bit_lds);
    if (kg < 1) return;   // the launch's LDS holds a group (topk_bits_lds_bytes)
    const uint32_t gstride = topk_bits_group_bytes(LA, S::kTab, S::kWmax, A, lmax);
    const uint32_t thr_at = bit_group_bytes(LA, S::kTab, A);
    const uint32_t lds0 = lds_addr_of(lds);
    uint32_t *queue = reinterpret_cast<uint32_t *>(lds + (uint32_t)kg * gstride) + wave * kBitQueue;
    uint32_t *hist_all = reinterpret_cast<uint32_t *>(lds + (uint32_t)kg * gstride + (kThreads / 64) * kBitQueue * 4u);
    const uint32_t hs = hist_stride(T.nbins);
    uint32_t *counter = hist_all + ((topk_hist_bytes(T.nbins, HIST) + 15u) & ~15u) / 4u;
    uint32_t *hist = hist_all + (lane & (kHistCopies - 1)) * hs;   // this lane's copy
    if constexpr (HIST)
        for (int i = tid; i < kHistCopies * (int)hs; i += kThreads) hist_all[i] = 0;
    const bool diag = r == b;
    const int steps = (V.CB / 64 - part + T.col_splits - 1) / T.col_splits;

    for (uint32_t gc = gbeg; gc < gend; gc += (uint32_t)kg) {
        const int ng = (int)min((uint32_t)kg, gend - gc);
        build_groups<LA, S, kThreads>(V, I0, ng, lds, gstride,
                                      [&](int g, int q) { return ((int64_t)gc + g) * kBitRows + q; });
        // threshold planes: lanes 0..31 the row words of a group for one
        // length lb, lanes 32..63 for the next
        for (int x = wave; x < ng * ((lmax + 2) / 2); x += kThreads / 64) {
            const int ln = (int)in_vgpr((uint32_t)lane);   // (kept from hoisting the lane compares)
            const int g = x / ((lmax + 2) / 2);
            const int lb = 2 * (x % ((lmax + 2) / 2)) + (ln >> 5);
            const int64_t slot = ((int64_t)gc + g) * kBitRows + (ln & 31);
            const uint32_t col = V.bcol[slot];
            int t = GMAX + 1;
            if (col != 0xFFFFu) t = min(max(key_score(T.thr[I0 + col], T.lo) + pabs * (LA + lb), 0), GMAX + 1);
            uint32_t mine = 0;
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                const uint64_t bal = __ballot((t >> q) & 1);
                const uint32_t half = ln & 32 ? (uint32_t)(bal >> 32) : (uint32_t)bal;
                if ((ln & 31) == q) mine = half;
            }
            if ((ln & 31) < PT && lb <= lmax)
                reinterpret_cast<uint32_t *>(lds + (uint32_t)g * gstride + thr_at)[lb * TD + (ln & 31)] = mine;
        }
        if (tid == 0) *counter = 0;
        __syncthreads();

        int qn = 0;   // entries in this wavefront's queue (wave-uniform)
        // the exact tests of up to 64 entries, and the appends
        auto drain = [&](int m) {
            if (lane < m) {
                const uint32_t e = queue[lane];
                const int64_t slot = J0 + (int64_t)(e & 0xFFFu);
                const int g = (int)(e >> 17 & 7u);
                const int64_t u = bit_group<LA, S>(lds + (uint32_t)g * gstride, A).cu[e >> 12 & 31u];
                const int64_t j = J0 + V.bcol[slot];
                const int s = (int)(e >> 20) - pabs * (LA + (int)V.blen[slot]);
                const uint64_t ku = nb_key(s, T.lo, (uint32_t)j), kj = nb_key(s, T.lo, (uint32_t)u);
                if (ku >= T.thr[u]) emit_candidate(T, u, ku);
                if (kj >= T.thr[j]) emit_candidate(T, j, kj);
            }
        };
        for (;;) {
            uint32_t taken = 0;
            if (lane == 0) taken = atomicAdd(counter, 1u);
            taken = (uint32_t)__builtin_amdgcn_readfirstlane((int)taken);
            if (taken >= (uint32_t)steps) break;
            const int st = part + (steps - 1 - (int)taken) * T.col_splits;   // longest words first
            const ColWords W = col_words(V.ccol, V.blen, J0 / 64 + st, lane);
            const uint32_t col = V.bcol[J0 + st * 64 + lane];
            const int64_t j = J0 + col;
            // the lane's threshold as a mask per plane
            uint32_t cm[PT];
            {
                int t = GMAX + 1;
                if (col != 0xFFFFu) t = min(max(key_score(T.thr[j], T.lo) + pabs * (LA + W.lb), 0), GMAX + 1);
#pragma unroll
                for (int q = 0; q < PT; ++q) cm[q] = (uint32_t)__builtin_amdgcn_sbfe(t, q, 1);
            }
            uint32_t cnt[REGS ? GMAX + 1 : 1];
            if constexpr (REGS)
#pragma unroll
                for (int i = 0; i <= GMAX; ++i) cnt[i] = 0;
            // bin of G = 0 for this lane
            uint32_t *bin0 = hist + (-pabs * (LA + W.lb) - T.lo);

            for (int g = 0; g < ng; ++g) {
                const uint32_t gb = (uint32_t)g * gstride;
                BitColumn<LA, S> C;
                C.run(W, lds0 + gb);
                const BitGroup G = bit_group<LA, S>(lds + gb, A);
                // pairs that count: present words, and each unordered pair
                // once (in a diagonal block only j > u)
                uint32_t valid = col != 0xFFFFu ? ~0u : 0u;
                uint32_t absent = 0;
                if (LA > 0) {
                    // words of the group shorter than LA (the first is the shortest)
                    const uint32_t last = (uint32_t)__builtin_amdgcn_readfirstlane((int)G.rowmask[LA > 0 ? LA - 1 : 0]);
                    if (last != ~0u) C.fill_short_rows(G.rowmask, pabs);
                }
                if (diag || LA == 0 || __builtin_amdgcn_readfirstlane(G.cu[0]) < 0) {
#pragma unroll 4
                    for (int q = 0; q < kBitRows; ++q) {
                        const int32_t u = G.cu[q];
                        absent = absent >> 1 | (u < 0 || (diag && j <= u) ? 0x80000000u : 0u);
                    }
                }
                valid &= ~absent;
                uint32_t s[PD];
                if constexpr (P > 0) C.template sum<P>(s); else s[0] = 0;
                // thresholds
                uint32_t rt[TD];
                {
                    const uint32_t ta = lds0 + gb + thr_at + (uint32_t)W.lb * (TD * 4u);
#pragma unroll
                    for (int q = 0; q < TD / 4; ++q) {
                        const u32x4 x = *(const lds_u32x4 *)(uintptr_t)(ta + 16u * (uint32_t)q);
                        rt[4 * q] = x[0]; rt[4 * q + 1] = x[1]; rt[4 * q + 2] = x[2]; rt[4 * q + 3] = x[3];
                    }
                }
                uint32_t rr[PT];
#pragma unroll
                for (int q = 0; q < PT; ++q) rr[q] = rt[q];
                uint32_t ev = (at_least<PD, PT>(s, rr) | at_least<PD, PT>(s, cm)) & valid;
                uint64_t any = __ballot(ev != 0);
                while (any) {
                    if (ev) {
                        const uint32_t q = (uint32_t)__builtin_ctz(ev);
                        const uint32_t at = (uint32_t)qn + __builtin_amdgcn_mbcnt_hi((uint32_t)(any >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)any, 0u));
                        queue[at] = pair_sum<PD>(s, q) << 20 | (uint32_t)g << 17 | q << 12 | (uint32_t)(st * 64 + lane);
                        ev &= ev - 1u;
                    }
                    qn += (int)__popcll(any);
                    if (qn >= 64) {
                        drain(64);
                        // the rest of the queue moves to its front
                        const uint32_t e = queue[64 + lane];
                        qn -= 64;
                        if (lane < qn) queue[lane] = e;
                    }
                    any = __ballot(ev != 0);
                }
                if constexpr (REGS) {
                    count_values<GMAX>(s, valid, cnt);
                } else if constexpr (HIST) {
                    uint32_t by[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) by[q] = q < P ? s[q < P ? q : 0] : 0u;
                    planes_to_bytes(by);
#pragma unroll
                    for (int q = 0; q < 8; ++q)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            uint32_t x = by[q] >> (8 * k) & 0xFFu;
                            if constexpr (P > 8) x |= (s[P > 8 ? 8 : 0] >> (8 * k + q) & 1u) << 8;
                            if (valid >> (8 * k + q) & 1u) atomicAdd(bin0 + x, 1u);
                        }
                }
            }
            if constexpr (REGS) {
#pragma unroll
                for (int x = 0; x <= GMAX; ++x)
                    if (cnt[x]) atomicAdd(bin0 + x, cnt[x]);
            }
        }
        drain(qn);
        __syncthreads();
    }
    if constexpr (HIST) {
        for (int i = tid; i < T.nbins; i += kThreads) {
            uint32_t sum = 0;
            for (int c = 0; c < kHistCopies; ++c) sum += hist_all[c * hs + i];
            if (sum) atomicAdd(&T.hist[i], (unsigned long long)sum);
        }
    }
}

// Waves per SIMD asked of the compiler: what its registers hold without
// spilling inside the column loop.
template <int C, class S>
constexpr int topk_bits_min_waves()
{
    constexpr int LA = 4 * C + 4;
    return S::kPlanes == 2 ? (LA <= 16 ? 4 : LA <= 32 ? 3 : 1) : (LA <= 4 ? 4 : LA <= 20 ? 3 : 1);
}

// Longest lengths 4C+1 .. 4C+4 (and 0, for C = 0): blockIdx.y picks one of the
// lengths block r has groups of, blockIdx.x the block pair and column part.
// One launch per class of four lengths instead of one per length: small
// dictionaries are bound by the host's cost of a launch.  Workgroups without
// work are kept few (30k words under a matrix: main pass 3.06 -> 2.93 ms
// against one for every tile and length; 600k words the same).
template <int C, class S, bool HIST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(topk_bits_min_waves<C, S>())))
void k_topk_bits(DevVocab V, TopkArgs T)
{
    extern __shared__ __align__(16) uint8_t lds[];
    uint32_t r, b;
    const uint32_t tile = blockIdx.x / (uint32_t)T.col_splits;
    if (T.phase_rect) {
        r = tile % (uint32_t)V.nb;
        b = r + tile / (uint32_t)V.nb * (uint32_t)T.phase_mod + (uint32_t)T.phase_lo;
        if (b >= (uint32_t)V.nb) return;
    } else {
        decode_block_pair(tile, r, b);
        const int ph = (int)((b - r) % (uint32_t)T.phase_mod);
        if (ph < T.phase_lo || ph > T.phase_hi) return;
    }
    const int part = (int)(blockIdx.x % (uint32_t)T.col_splits);
    // the blockIdx.y-th length of the class, from the longest, that the block has
    const uint32_t *rgo = V.rg_off + (size_t)r * (V.lmax + 1);
    int LA = min(bit_class_hi(C), V.lmax), skip = (int)blockIdx.y;
    for (; LA >= bit_class_lo(C); --LA)
        if (rgo[LA + 1] > rgo[LA] && skip-- == 0) break;
    if (LA < bit_class_lo(C)) return;
    bit_length_dispatch<bit_class_lo(C), bit_class_hi(C)>(
        LA, [&](auto la) { topk_bits_tile<decltype(la)::value, S, HIST>(V, T, r, b, part, lds); });
}

}  // namespace nw
