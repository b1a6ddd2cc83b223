// k_probe_bits.h -- the threshold pre-pass of the all-pairs top-k in bit planes
// (nw_bits.h, Bits2): the keys of k_probe.h for a lane's word at a time.
//
// Every word needs its key of rank m against the M probes (k_probe.h).  Here a
// lane holds a word and the 32 bits of a plane are 32 probes, so everything
// after the DP is the lane's own:
//   0. k_probe_tables builds the symbol tables of the probes' groups once, in
//      scratch memory: set A in length order (the probe slots), set B in rank
//      order (probe i = word probe_word(i));
//   1. k_probe_bits runs set A: every probe's score adds to the lane's
//      histogram in LDS (16-bit counts, two to a dword, so the 64 lanes of an
//      add hit 64 banks);
//   2. each lane walks its histogram down to the code c that holds rank m and
//      the place r of the wanted key among the keys of code c;
//   3. k_probe_bits runs set B: keys of equal score rank by index, and the
//      groups come in index order, so the lane counts its pairs of code c (one
//      comparison function per plane) until the r-th.
// Two DP passes of 7 functions per cell and 32 pairs replace one of 32 packed
// instructions per cell and 32 pairs with two LDS adds and stores per pair.
// 600,000 words, 8,192 probes: 15.6 ms (k_probe_thr) -> 10.0 ms.  Below 131,073
// words the workgroups are too few for it (100k words: 3.0 ms against 2.1).
#pragma once

#include "nw_bits.h"

namespace nw {

constexpr uint32_t kProbeTabLds = 16u * 1024u;   // tables of a chunk of groups
constexpr int kProbeRegsLen = 10;                // rows whose values are counted in registers (31 of them)
constexpr int kProbeBitsMaxLen = 32;   // longest word: one kernel holds every length, and longer rows would cost all of them registers

struct ProbeBitsArgs {
    uint8_t *scratch;    // int32 longest length per group, then the groups, gstride apart
    uint32_t gstride;    // bit_group_bytes of the longest word
    uint32_t nA, nB;     // groups of the two sets
    uint32_t npad;       // leading padding slots of set A
    int m;               // rank of the wanted key
    uint64_t *thr;       // [n] the key of each word, by caller index
};
__host__ __device__ inline uint64_t probe_bits_lens_bytes(uint32_t groups) { return ((uint64_t)groups * 4u + 255u) & ~255ull; }

// Workgroup g builds group g (set A, then set B).
__global__ __launch_bounds__(kThreads) void k_probe_tables(DevVocab V, ProbeBitsArgs Q)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t g = blockIdx.x;
    const bool setb = g >= Q.nA;
    DevVocab Vp = V;
    Vp.bsym = setb ? V.csym : V.psym;
    Vp.blen = setb ? V.clen : V.plen;
    Vp.bcol = V.prank;   // caller indices are not used here: any array of the size
    const uint32_t g0 = setb ? g - Q.nA : g;
    auto slot_of = [&](int, int b) -> int64_t {
        const int64_t i = (int64_t)g0 * kBitRows + b;
        if (!setb) return i >= (int64_t)Q.npad ? i : -1;
        return i < V.nprobe ? (int64_t)probe_word((uint64_t)i, (uint64_t)V.n, (uint64_t)V.nprobe) : -1;
    };
    const int b = threadIdx.x & 31;
    const int64_t s = slot_of(0, b);
    int LA = s >= 0 ? (int)Vp.blen[s] : 0;
#pragma unroll
    for (int d = 16; d; d >>= 1) LA = max(LA, __shfl_xor(LA, d));
    LA = __builtin_amdgcn_readfirstlane(LA);   // the same in every wavefront
    bit_length_dispatch<0, kProbeBitsMaxLen>(LA, [&](auto la) __attribute__((always_inline)) {
        build_tables<decltype(la)::value, Bits2, kThreads>(Vp, 1, lds, 0u, slot_of);
    });
    __syncthreads();
    const uint32_t bytes = bit_group_bytes(LA, Bits2::kTab, V.alphabet);
    u32x4 *dst = reinterpret_cast<u32x4 *>(Q.scratch + probe_bits_lens_bytes(Q.nA + Q.nB) + (uint64_t)g * Q.gstride);
    const u32x4 *src = reinterpret_cast<const u32x4 *>(lds);
    for (uint32_t i = threadIdx.x; i < bytes / 16u; i += kThreads) dst[i] = src[i];
    if (threadIdx.x == 0) reinterpret_cast<int32_t *>(Q.scratch)[g] = LA;
}

// One group against the lane's word: planes of G - p-fill, as the other
// bit-plane kernels form it.
template <int LA, int P>
__device__ __forceinline__ void probe_group(const DevVocab &V, const ColWords &W, const uint8_t *lds, uint32_t at,
                                            uint32_t (&s)[P > 0 ? P : 1])
{
    BitColumn<LA, Bits2> C;
    C.run(W, lds_addr_of(lds) + at);
    if constexpr (LA > 0) {
        const uint32_t *rowmask = bit_group<LA, Bits2>(const_cast<uint8_t *>(lds) + at, V.alphabet).rowmask;
        if (__builtin_amdgcn_readfirstlane((int)rowmask[LA - 1]) != ~0) C.fill_short_rows(rowmask, -V.gap);
    }
    if constexpr (P > 0) C.template sum<P>(s); else s[0] = 0;
}

// A wavefront takes 64 slots.  LDS: the tables of a chunk, then a histogram of
// (bins + 1) / 2 x 64 dwords per wavefront.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_probe_bits(DevVocab V, ProbeBitsArgs Q)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t steps = (int64_t)V.nb * V.CB / 64;
    const int64_t st = (int64_t)blockIdx.x * (kThreads / 64) + wave;
    const bool active = st < steps;   // (CB is a multiple of 256: the last workgroup is whole)
    const ColWords W = col_words(V.ccol, V.blen, active ? st : 0, lane);
    const int32_t u = active ? V.borig[st * 64 + lane] : -1;
    const int pabs = -V.gap, nbins = V.hi - V.lo + 1;
    const uint32_t hdw = (uint32_t)(nbins + 1) / 2u * 64u;   // dwords of a histogram
    uint32_t *hist = reinterpret_cast<uint32_t *>(lds + kProbeTabLds) + (uint32_t)wave * hdw + (uint32_t)lane;
    const uint32_t hist_a = lds_addr_of(hist);
    for (uint32_t i = 0; i < hdw; i += 64) hist[i] = 0;
    const int32_t *lens = reinterpret_cast<const int32_t *>(Q.scratch);
    const uint8_t *tabs = Q.scratch + probe_bits_lens_bytes(Q.nA + Q.nB);

    // groups [g0, g1) of the scratch, `room` bytes of tables at a time:
    // body(first group, groups, their LA, their place in LDS) for each run of
    // one LA; more(): false ends the walk (evaluated by the whole workgroup)
    auto walk = [&](uint32_t g0, uint32_t g1, uint32_t room, auto &&body, auto &&more) __attribute__((always_inline)) {
        for (uint32_t g = g0; g < g1;) {
            __syncthreads();   // the LDS of the chunk before is done with
            uint32_t e = g, used = 0;
            while (e < g1) {
                const uint32_t by = bit_group_bytes(__builtin_amdgcn_readfirstlane(lens[e]), Bits2::kTab, V.alphabet);
                if (e > g && used + by > room) break;
                const u32x4 *src = reinterpret_cast<const u32x4 *>(tabs + (uint64_t)e * Q.gstride);
                u32x4 *dst = reinterpret_cast<u32x4 *>(lds + used);
                for (uint32_t i = tid; i < by / 16u; i += kThreads) dst[i] = src[i];
                used += by;
                ++e;
            }
            __syncthreads();
            uint32_t at = 0;
            while (g < e) {
                const int LA = __builtin_amdgcn_readfirstlane(lens[g]);
                uint32_t run = 1;
                while (g + run < e && __builtin_amdgcn_readfirstlane(lens[g + run]) == LA) ++run;
                body(g, run, LA, at);
                at += run * bit_group_bytes(LA, Bits2::kTab, V.alphabet);
                g += run;
            }
            if (!more()) break;
        }
    };

    // 1. the histogram over set A: of short rows, each value's pairs counted
    // in a register over a run of groups; of longer ones, a pair at a time
    auto add = [&](uint32_t bin, uint32_t cnt) __attribute__((always_inline)) {
        __atomic_fetch_add(lds_ptr(hist_a + (bin >> 1) * 256u), cnt << ((bin & 1u) * 16u), __ATOMIC_RELAXED);
    };
    walk(
        0, Q.nA, kProbeTabLds,
        [&](uint32_t g, uint32_t run, int LA, uint32_t at) __attribute__((always_inline)) {
            bit_length_dispatch<0, kProbeBitsMaxLen>(LA, [&](auto la) __attribute__((always_inline)) {
                constexpr int L = decltype(la)::value, P = sum_planes<L, Bits2>(), GMAX = Bits2::kWmax * L;
                constexpr bool REGS = L <= kProbeRegsLen;
                // (in_vgpr: kept from hoisting one value per length out of the walk)
                const int off = -pabs * (L + (int)in_vgpr((uint32_t)W.lb)) - V.lo;   // bin of G = 0
                uint32_t cnt[REGS ? GMAX + 1 : 1];
#pragma unroll
                for (int x = 0; x < (REGS ? GMAX + 1 : 1); ++x) cnt[x] = 0;
                for (uint32_t q = 0; q < run; ++q) {
                    const uint32_t base = (g + q) * kBitRows;
                    if (base + kBitRows <= Q.npad) continue;
                    const uint32_t valid = Q.npad <= base ? ~0u : ~0u << (Q.npad - base);
                    uint32_t s[P > 0 ? P : 1];
                    probe_group<L, P>(V, W, lds, at + q * bit_group_bytes(L, Bits2::kTab, V.alphabet), s);
                    if constexpr (REGS) {
                        count_values<GMAX>(s, valid, cnt);
                    } else {
                        uint32_t by[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i) by[i] = i < P ? s[i < P ? i : 0] : 0u;
                        planes_to_bytes(by);
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                if (valid >> (8 * k + i) & 1u) add((by[i] >> (8 * k) & 0xFFu) + (uint32_t)off, 1u);
                            __builtin_amdgcn_sched_barrier(0);   // four addresses at a time in registers
                        }
                    }
                }
                if constexpr (REGS) {
                    // (a value no pair has may lie outside the histogram)
#pragma unroll
                    for (int x = 0; x <= GMAX; ++x)
                        if (cnt[x]) add((uint32_t)(x + off), cnt[x]);
                }
            });
        },
        [] { return true; });

    // 2. the code c of rank m, and the place r (1-based) among its keys
    int c = 0;
    uint32_t need = 0;
    {
        uint32_t above = 0;
        for (int bin = nbins - 1; bin >= 0; --bin) {
            const uint32_t cnt = *lds_ptr(hist_a + (uint32_t)(bin >> 1) * 256u) >> ((bin & 1) * 16) & 0xFFFFu;
            if (need == 0 && above + cnt >= (uint32_t)Q.m) {
                c = bin;
                need = (uint32_t)Q.m - above;
            }
            above += cnt;
            if (__ballot(need == 0) == 0) break;
        }
    }
    const bool found_code = need != 0;
    if (u < 0) need = 0;   // padding slots look for nothing

    // 3. the need-th probe, in index order, of code c (the histograms' LDS
    // holds tables now)
    uint32_t rank = 0;
    walk(
        Q.nA, Q.nA + Q.nB, kProbeTabLds + 4u * hdw * (kThreads / 64),
        [&](uint32_t g, uint32_t run, int LA, uint32_t at) __attribute__((always_inline)) {
            bit_length_dispatch<0, kProbeBitsMaxLen>(LA, [&](auto la) __attribute__((always_inline)) {
                constexpr int L = decltype(la)::value, P = sum_planes<L, Bits2>();
                constexpr int GMAX = Bits2::kWmax * L;
                for (uint32_t q = 0; q < run; ++q) {
                    if (__ballot(need != 0) == 0) return;
                    const uint32_t base = (g + q - Q.nA) * kBitRows;
                    const uint32_t left = (uint32_t)V.nprobe - base;
                    const uint32_t valid = left >= kBitRows ? ~0u : (1u << left) - 1u;
                    uint32_t s[P > 0 ? P : 1];
                    probe_group<L, P>(V, W, lds, at + q * bit_group_bytes(L, Bits2::kTab, V.alphabet), s);
                    const int t = (int)in_vgpr((uint32_t)(c + pabs * W.lb)) + V.lo + pabs * L;   // G of code c
                    uint32_t eq = t >= 0 && t <= GMAX ? valid : 0u;
#pragma unroll
                    for (int p = 0; p < P; ++p)
                        eq = lut3<0x90>(eq, s[p], (uint32_t)__builtin_amdgcn_sbfe(t, p, 1));   // eq & ~(s ^ t)
                    const uint32_t cnt = (uint32_t)__builtin_popcount(eq);
                    if (need != 0) {
                        if (cnt >= need) {
                            while (--need) eq &= eq - 1u;
                            rank = base + (uint32_t)__builtin_ctz(eq);
                        } else {
                            need -= cnt;
                        }
                    }
                }
            });
        },
        [&] { return __syncthreads_or(need != 0) != 0; });

    if (u >= 0) {
        const uint64_t j = probe_word(rank, (uint64_t)V.n, (uint64_t)V.nprobe);
        Q.thr[u] = found_code ? ((uint64_t)(uint32_t)c << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)j) : 0;
    }
}

}  // namespace nw
