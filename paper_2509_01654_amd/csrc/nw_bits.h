// nw_bits.h -- the recurrence of nw_dp.h in bit planes: 32 row words at once.
//
// With G[i][j] = M[i][j] - p(i+j) (nw_dp.h) neighbouring cells differ by
//     v = G[i][j] - G[i-1][j]   and   h = G[i][j] - G[i][j-1],
// and both lie in [0, wmax], wmax the largest w = sim - 2p: G never falls
// along a row or a column, and dropping one symbol loses at most one match.
// A cell takes the differences above (h) and to the left (v) to those below
// and to the right:
//     t = max(w, h, v),   v' = t - h,   h' = t - v,
// and G[LA][lb] is the sum of the v of the last column.  A weight below 0
// gives the same t as 0, since h, v >= 0.
//
// A difference of B bits is held as B planes: bit b of a plane belongs to the
// pair (row word b, lane word), for 32 row words b of (nearly) equal length.
// A cell of 32 pairs is then a small network of three-input boolean functions
// (v_bitop3_b32), one vector instruction per function and 32 pairs:
//     Bits2  (match weight 3, every mismatch weight 1: +1 / -1 / gap -1 and
//            whatever shifts to it): 2 planes, 7 functions per cell;
//     Bits3  (any similarity with w <= 7): 3 planes, 22 functions per cell.
// The packed binary16 form of nw_dp.h issues 32 lane-instructions for the
// same 32 cells, at about two thirds of the rate: on MI355X v_bitop3_b32 was
// measured at 56e12 lane-instructions/s, v_pk_maximum3_f16 at 37e12.
//
// The column symbol enters through a table in LDS: row c holds, per row
// position, which of the 32 row words have symbol c there (Bits2, one dword)
// or the planes of their weights against c (Bits3, three dwords): 4 or 12
// bytes of LDS reads per 32 cells, against 64 in the packed form.
//
// Row words: 32 consecutive slots of a length-sorted block.  The kernel is
// compiled for the longest, LA; the rows past a shorter word are replaced,
// after the last column, by v = -p, so that G - |p|(LA + lb) is every pair's
// score whatever the row word's own length (needs |p| <= wmax).
// Column words: 64 consecutive slots, one per lane, front-padded to the
// longest of them; after each column a lane that has not begun yet resets its
// differences to the boundary's 0.
#pragma once

#include "nw_tile_common.h"
#include "nw_topk.h"

namespace nw {

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

constexpr int kBitRows = 32;                     // row words of a group
constexpr int kColDwords = kWordBytes / 4;       // symbol dwords of a column word

template <int IMM>
__device__ __forceinline__ uint32_t lut3(uint32_t a, uint32_t b, uint32_t c)
{
    // bit of IMM: (a << 2 | b << 1 | c)
    return __builtin_amdgcn_bitop3_b32(a, b, c, IMM);
}
constexpr int kXor3 = 0x96, kMaj = 0xE8, kMux = 0xCA;   // a^b^c; majority; a ? b : c
constexpr int kGt = 0xB2;    // a > b, or a == b and c: one bit of a comparison
constexpr int kBorrow = 0x8E;   // a < b, or a == b and c: the borrow of a - b - c

struct Bits2 {
    static constexpr int kPlanes = 2, kTab = 1, kWmax = 3;
    // v, h in and out; w[0] = the pairs whose symbols match
    template <bool FIRST, bool TOP>
    static __device__ __forceinline__ void cell(const uint32_t (&w)[1], uint32_t (&v)[2], uint32_t (&h)[2])
    {
        const uint32_t M = w[0];
        if constexpr (FIRST && TOP) {          // h = v = 0
            v[0] = h[0] = ~0u;
            v[1] = h[1] = M;
        } else if constexpr (FIRST) {          // v = 0
            const uint32_t h0 = h[0], h1 = h[1];
            v[0] = lut3<0x31>(M, h0, h1);      // M ? ~h0 : ~(h0 | h1)
            v[1] = M & ~h1;
            h[0] = lut3<0xFD>(M, h0, h1);      // M | h0 | ~h1
            h[1] = M | h1;
        } else if constexpr (TOP) {            // h = 0
            const uint32_t v0 = v[0], v1 = v[1];
            h[0] = lut3<0x31>(M, v0, v1);
            h[1] = M & ~v1;
            v[0] = lut3<0xFD>(M, v0, v1);
            v[1] = M | v1;
        } else {
            const uint32_t h0 = h[0], h1 = h[1], v0 = v[0], v1 = v[1];
            const uint32_t x0 = lut3<0x32>(M, h1, v1);
            const uint32_t x1 = lut3<0xF8>(M, h1, h0);
            const uint32_t x2 = lut3<0x98>(h1, v1, x1);
            h[0] = lut3<0x29>(v1, v0, x2);
            h[1] = lut3<0x46>(v0, x1, x2);
            v[0] = lut3<0x16>(h0, v0, h[0]);
            v[1] = lut3<0x4C>(h0, x0, v[0]);
        }
    }
};

struct Bits3 {
    static constexpr int kPlanes = 3, kTab = 3, kWmax = 7;
    static __device__ __forceinline__ void max2(const uint32_t (&a)[3], const uint32_t (&b)[3], uint32_t (&t)[3])
    {
        const uint32_t g = lut3<kGt>(a[2], b[2], lut3<kGt>(a[1], b[1], a[0] & ~b[0]));
#pragma unroll
        for (int q = 0; q < 3; ++q) t[q] = lut3<kMux>(g, a[q], b[q]);
    }
    static __device__ __forceinline__ void sub(const uint32_t (&a)[3], const uint32_t (&b)[3], uint32_t (&d)[3])
    {
        const uint32_t br0 = ~a[0] & b[0], br1 = lut3<kBorrow>(a[1], b[1], br0);
        d[2] = lut3<kXor3>(a[2], b[2], br1);
        d[1] = lut3<kXor3>(a[1], b[1], br0);
        d[0] = a[0] ^ b[0];
    }
    template <bool FIRST, bool TOP>
    static __device__ __forceinline__ void cell(const uint32_t (&w)[3], uint32_t (&v)[3], uint32_t (&h)[3])
    {
        uint32_t t[3], o[3];
        if constexpr (FIRST && TOP) {
#pragma unroll
            for (int q = 0; q < 3; ++q) v[q] = h[q] = w[q];
        } else if constexpr (FIRST) {          // v = 0: t = max(w, h)
            max2(w, h, t);
            sub(t, h, v);
#pragma unroll
            for (int q = 0; q < 3; ++q) h[q] = t[q];
        } else if constexpr (TOP) {
            max2(w, v, t);
            sub(t, v, h);
#pragma unroll
            for (int q = 0; q < 3; ++q) v[q] = t[q];
        } else {
            uint32_t m[3];
            max2(h, v, m);
            max2(w, m, t);
            sub(t, v, o);
            sub(t, h, v);
#pragma unroll
            for (int q = 0; q < 3; ++q) h[q] = o[q];
        }
    }
};

// Planes of a sum of LA differences.
__host__ __device__ constexpr int bit_width(uint32_t x) { return x == 0 ? 0 : 1 + bit_width(x >> 1); }
template <int LA, class S>
__host__ __device__ constexpr int sum_planes() { return bit_width((uint32_t)(S::kWmax * LA)); }
// Planes that also hold the value one past the largest sum (a threshold no pair reaches).
template <int LA, class S>
__host__ __device__ constexpr int thr_planes() { return bit_width((uint32_t)(S::kWmax * LA + 1)); }

// Bytes of a table row: LA positions, an odd number of 16-byte units, so the
// rows of different symbols spread over the LDS bank groups.
__host__ __device__ constexpr uint32_t bit_row_units(int LA, int tab) { return (uint32_t)((LA * tab + 3) / 4) | 1u; }
__host__ __device__ constexpr uint32_t bit_row_bytes(int LA, int tab) { return LA == 0 ? 0u : 16u * bit_row_units(LA, tab); }
__host__ __device__ constexpr uint32_t bit_tab_bytes(int LA, int tab, int alphabet)
{
    return bit_row_bytes(LA, tab) * (uint32_t)alphabet;
}

// Column words of the 64 slots of a group, as the lanes read them: dword q of
// lane l at ccol[(group * kColDwords + q) * 64 + l]; the symbols start
// (longest - own length) bytes in, the bytes before and after are symbol 0.
struct ColWords {
    const uint32_t *p;   // lane 0's dword 0 (wave-uniform)
    uint32_t dw0;        // this lane's dword 0
    int ncols;           // longest word of the 64 (wave-uniform)
    int npad;            // ncols - shortest (wave-uniform)
    int lb;              // this lane's length
};

// 16-byte units of a table row held in registers: enough to cover the LDS
// latency, few enough that long rows leave room for waves.
constexpr int kRowWindow = 4;

template <int LA, class S>
struct BitColumn {
    static constexpr int N = LA > 0 ? LA : 1;
    static constexpr int NQ = (LA * S::kTab + 3) / 4;
    uint32_t v[N][S::kPlanes];

    // The table row passes through a window of NW 16-byte units, unit u in
    // row[u % NW].
    static constexpr int NW = NQ < 1 ? 1 : NQ < kRowWindow ? NQ : kRowWindow;

    // One column, its table row at LDS address cur; the window holds the first
    // NW units.  A unit is replaced as soon as the cells that read it are done:
    // by the unit NW further on, or, past the end of the row, by the next
    // column's (at next) for the same place, so reads are in flight a window
    // ahead of their use.  The scheduling barriers keep them there.
    template <bool FIRST>
    __device__ __forceinline__ void column(u32x4 (&row)[NW], uint32_t cur, uint32_t next)
    {
        uint32_t h[S::kPlanes];
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            uint32_t w[S::kTab];
#pragma unroll
            for (int q = 0; q < S::kTab; ++q) w[q] = row[((i * S::kTab + q) >> 2) % NW][(i * S::kTab + q) & 3];
            if (i == 0)
                S::template cell<FIRST, true>(w, v[i], h);
            else
                S::template cell<FIRST, false>(w, v[i], h);
            // the units whose last dword was this cell's
            const int done = i + 1 == LA ? NQ : (i + 1) * S::kTab / 4, before = i * S::kTab / 4;
            if (done > before) {
#pragma unroll
                for (int u = before; u < done; ++u) {
                    const uint32_t at = u + NW < NQ ? cur + 16u * (uint32_t)(u + NW) : next + 16u * (uint32_t)(u % NW);
                    row[u % NW] = *(const lds_u32x4 *)(uintptr_t)at;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    __device__ __forceinline__ void reset_unless(bool begun)
    {
        uint32_t m = begun ? ~0u : 0u;
        asm volatile("" : "+v"(m));   // stays behind its (uniform) branch: most steps have one length
#pragma unroll
        for (int i = 0; i < LA; ++i)
#pragma unroll
            for (int q = 0; q < S::kPlanes; ++q) v[i][q] &= m;
    }

    // Run the columns of the lane's word against the table at LDS address tab.
    __device__ __forceinline__ void run(const ColWords &W, uint32_t tab)
    {
        const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
        for (int i = 0; i < LA; ++i)
#pragma unroll
            for (int q = 0; q < S::kPlanes; ++q) v[i][q] = 0u;
        if constexpr (LA > 0) {
            constexpr uint32_t RB = bit_row_bytes(LA, S::kTab);
            const uint32_t tv = in_vgpr(tab);
            const int nc = W.ncols;
            if (nc == 0) return;
            const int first = nc - W.lb;   // the lane's first real column
            // one column a trip (a longer loop body costs instruction cache:
            // a launch runs many lengths); the symbol after the last is one
            // of the word's or 0, in either case a row of the table
            const int lastq = (nc - 1) >> 2;
            uint32_t dw = W.dw0, dn = W.p[(uint32_t)(64 * min(1, lastq)) + lane];
            u32x4 row[NW];
            uint32_t cur = tv + (dw & 0xFFu) * RB;
            load_row<NW>(row, cur);
            dw >>= 8;
            uint32_t next = tv + (dw & 0xFFu) * RB;
            column<true>(row, cur, next);
            if (0 < W.npad) reset_unless(first <= 0);
            for (int c = 1; c < nc; ++c) {
                if ((c & 3) == 3) {
                    dw = dn;
                    dn = W.p[(uint32_t)(64 * min((c >> 2) + 2, lastq)) + lane];
                } else {
                    dw >>= 8;
                }
                cur = next;
                next = tv + (dw & 0xFFu) * RB;
                column<false>(row, cur, next);
                if (c < W.npad) reset_unless(c >= first);
            }
        }
    }

    // Rows past a row word's own length take v = pabs: rowmask[i] (LDS) has
    // the row words longer than i.
    __device__ __forceinline__ void fill_short_rows(const uint32_t *rowmask, int pabs)
    {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            const uint32_t m = rowmask[i];
#pragma unroll
            for (int q = 0; q < S::kPlanes; ++q) v[i][q] = lut3<kMux>(m, v[i][q], (uint32_t)-(pabs >> q & 1));
        }
    }

    // Planes of the sum of the differences: full adders (two functions for
    // three bits of one weight) down to one bit per weight.
    template <int P>
    __device__ __forceinline__ void sum(uint32_t (&g)[P])
    {
        constexpr int CAP = S::kPlanes * N + 8;
        uint32_t cur[CAP], nxt[CAP];
        add_level<0, 0, P>(cur, nxt, g);
    }

  private:
    // Weight W: NC carries from the weight below in cur, plus the planes W of v.
    template <int W, int NC, int P, int CAP>
    __device__ __forceinline__ void add_level(uint32_t (&cur)[CAP], uint32_t (&nxt)[CAP], uint32_t (&g)[P])
    {
        if constexpr (W < P) {
            constexpr int NV = W < S::kPlanes ? LA : 0;
            constexpr int T = NC + NV;
            if constexpr (W < S::kPlanes) {
#pragma unroll
                for (int i = 0; i < LA; ++i) cur[NC + i] = v[i][W];
            }
            if constexpr (T == 0) {
                g[W] = 0u;
                add_level<W + 1, 0, P>(nxt, cur, g);
            } else {
                // fold three at a time into the running bit
                constexpr int FA = (T - 1) / 2;          // full adders
                constexpr bool HA = ((T - 1) & 1) != 0;  // one half adder
                uint32_t s = cur[0];
#pragma unroll
                for (int k = 0; k < FA; ++k) {
                    const uint32_t a = cur[1 + 2 * k], b = cur[2 + 2 * k];
                    nxt[k] = lut3<kMaj>(s, a, b);
                    s = lut3<kXor3>(s, a, b);
                }
                if constexpr (HA) {
                    nxt[FA] = s & cur[T - 1];
                    s = s ^ cur[T - 1];
                }
                g[W] = s;
                add_level<W + 1, FA + (HA ? 1 : 0), P>(nxt, cur, g);
            }
        }
    }
};

// Pairs whose sum (planes g) is at least the threshold (planes r).
template <int P, int PT>
__device__ __forceinline__ uint32_t at_least(const uint32_t (&g)[P], const uint32_t (&r)[PT])
{
    uint32_t c = ~0u;
#pragma unroll
    for (int q = 0; q < PT; ++q) c = q < P ? lut3<kGt>(g[q < P ? q : 0], r[q], c) : (c & ~r[q]);
    return c;
}

// The sum of pair b (0 .. 31) from its planes.
template <int P>
__device__ __forceinline__ uint32_t pair_sum(const uint32_t (&g)[P], uint32_t b)
{
    uint32_t x = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) x |= ((g[q] >> b) & 1u) << q;
    return x;
}

// cnt[x] += the pairs of `valid` whose sum is x, x = 0 .. GMAX: the low three
// planes select one of eight masks, the others one function per value.
template <int GMAX, int P>
__device__ __forceinline__ void count_values(const uint32_t (&s)[P], uint32_t valid, uint32_t (&cnt)[GMAX + 1])
{
    uint32_t low[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        uint32_t m = valid;
        if (GMAX > 0) m &= (x & 1) ? s[0] : ~s[0];
        if (P > 1) m &= (x & 2) ? s[P > 1 ? 1 : 0] : ~s[P > 1 ? 1 : 0];
        if (P > 2) m &= (x & 4) ? s[P > 2 ? 2 : 0] : ~s[P > 2 ? 2 : 0];
        low[x] = m;
    }
#pragma unroll
    for (int x = 0; x <= GMAX; ++x) {
        uint32_t m = low[x & 7];
#pragma unroll
        for (int q = 3; q < P; ++q) m &= (x >> q & 1) ? s[q] : ~s[q];
        cnt[x] += (uint32_t)__builtin_popcount(m);
    }
}

// Eight planes to bytes: byte k of o[j] is the value of pair 8k + j (three
// rounds of exchanges, each swapping half of the bits of two planes).
__device__ __forceinline__ void planes_to_bytes(uint32_t (&p)[8])
{
    auto swap = [](uint32_t &a, uint32_t &b, int s, uint32_t m) {
        const uint32_t na = (a & m) | ((b << s) & ~m);
        const uint32_t nb = ((a >> s) & m) | (b & ~m);
        a = na;
        b = nb;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) swap(p[i], p[i + 4], 4, 0x0F0F0F0Fu);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (!(i & 2)) swap(p[i], p[i + 2], 2, 0x33333333u);
#pragma unroll
    for (int i = 0; i < 8; i += 2) swap(p[i], p[i + 1], 1, 0x55555555u);
}

// 32 x 32 bit transposition: bit b of m[c] becomes what bit c of m[b] was.
template <int W, uint32_t MASK>
__device__ __forceinline__ void transpose_round(uint32_t (&m)[32])
{
#pragma unroll
    for (int k = 0; k < 32; ++k)
        if (!(k & W)) {
            const uint32_t a = m[k], b = m[k + W];
            m[k] = (a & MASK) | ((b << W) & ~MASK);
            m[k + W] = ((a >> W) & MASK) | (b & ~MASK);
        }
}
__device__ __forceinline__ void transpose32(uint32_t (&m)[32])
{
    transpose_round<16, 0x0000FFFFu>(m);
    transpose_round<8, 0x00FF00FFu>(m);
    transpose_round<4, 0x0F0F0F0Fu>(m);
    transpose_round<2, 0x33333333u>(m);
    transpose_round<1, 0x55555555u>(m);
}

// ---------------------------------------------------------------- LDS tables
// LDS of a launch: `fixed` bytes and as many groups of `per` bytes as fit
// `aim`, at least one and at most `most`; no more is asked for, so that short
// rows get more workgroups per CU.
__host__ __device__ constexpr uint32_t bit_lds_bytes(uint32_t fixed, uint32_t per, uint32_t aim, uint32_t most)
{
    const uint32_t fit = aim > fixed ? (aim - fixed) / per : 0u;
    return fixed + per * (fit < 1u ? 1u : fit < most ? fit : most);
}
// One group of row words in LDS: its table, the row masks and caller indices.
__host__ __device__ constexpr uint32_t bit_group_bytes(int LA, int tab, int alphabet)
{
    return bit_tab_bytes(LA, tab, alphabet) + (((uint32_t)LA * 4u + 15u) & ~15u) + kBitRows * 4u;
}

struct BitGroup {
    uint32_t *tab;      // [alphabet][bit_row_bytes / 4]
    uint32_t *rowmask;  // [LA] row words longer than i
    int32_t *cu;        // [32] caller index of the row word, -1 when absent
};
template <int LA, class S>
__device__ __forceinline__ BitGroup bit_group(uint8_t *base, int alphabet)
{
    BitGroup G;
    G.tab = reinterpret_cast<uint32_t *>(base);
    G.rowmask = reinterpret_cast<uint32_t *>(base + bit_tab_bytes(LA, S::kTab, alphabet));
    G.cu = reinterpret_cast<int32_t *>(base + bit_group_bytes(LA, S::kTab, alphabet) - kBitRows * 4u);
    return G;
}

// Build n groups into lds, `stride` bytes apart.  slot_of(g, b) is the slot
// of row word b of group g (block origin I0), -1 for none.  All threads of
// the workgroup call it; the caller's barrier after it completes the build.
// It clears the tables first, so no thread may still read the old groups
// when it is entered.
// (build_tables: all but the caller indices.)
template <int LA, class S, int NT, typename SlotOf>
__device__ __forceinline__ void build_tables(const DevVocab &V, int n, uint8_t *lds, uint32_t stride, SlotOf slot_of)
{
    // kept from hoisting the addresses of the build over the caller's loop
    const int tid = (int)in_vgpr(threadIdx.x);
    const int A = V.alphabet;
    constexpr uint32_t RD = bit_row_bytes(LA, S::kTab) / 4;
    const uint32_t tdw = bit_tab_bytes(LA, S::kTab, A) / 4;
    if constexpr (LA > 0 && S::kTab == 1) {
        for (int g = 0; g < n; ++g) {
            u32x4 *t = reinterpret_cast<u32x4 *>(lds + (uint32_t)g * stride);
            for (uint32_t i = tid; i < tdw / 4; i += NT) t[i] = u32x4{0u, 0u, 0u, 0u};
        }
        __syncthreads();
        // thread (row word b of group g, position i): one bit of one row
        for (int x = tid; x < n * LA * kBitRows; x += NT) {
            const int b = x & (kBitRows - 1), gi = x >> 5;
            const int i = gi % LA, g = gi / LA;
            const int64_t slot = slot_of(g, b);
            if (slot >= 0 && i < (int)V.blen[slot]) {
                const uint32_t c = V.bsym[slot * V.WB + i];
                uint32_t *t = reinterpret_cast<uint32_t *>(lds + (uint32_t)g * stride);
                atomicOr(&t[c * RD + (uint32_t)i], 1u << b);
            }
        }
    }
    if constexpr (LA > 0 && S::kTab == 3) {
        // task (group, position i, 32 symbols c0 ..): the weight planes of the
        // 32 row words against those symbols, one 32 x 32 bit transposition
        // per plane (wplanes[x][plane][c / 32] has the planes of w(x, c))
        const int nh = (A + 31) / 32;
        const int tasks = n * LA * nh * 3;
        for (int x = tid; x < tasks; x += NT) {
            const int q = x % 3, y = x / 3;
            const int hf = y % nh, z = y / nh;
            const int i = z % LA, g = z / LA;
            uint32_t m[32];
#pragma unroll
            for (int b = 0; b < 32; ++b) {
                const int64_t slot = slot_of(g, b);
                m[b] = 0u;
                if (slot >= 0 && i < (int)V.blen[slot])
                    m[b] = V.wplanes[((uint32_t)V.bsym[slot * V.WB + i] * 3u + (uint32_t)q) * 8u + (uint32_t)hf];
            }
            transpose32(m);
            uint32_t *t = reinterpret_cast<uint32_t *>(lds + (uint32_t)g * stride);
#pragma unroll
            for (int c = 0; c < 32; ++c)
                if (hf * 32 + c < A) t[(uint32_t)(hf * 32 + c) * RD + (uint32_t)(i * 3 + q)] = m[c];
        }
    }
    if constexpr (LA > 0) {
        // a wavefront takes two groups, a lane one row word of one of them
        const int lane = tid & 63;
        const int half = lane >> 5, b = lane & 31;
        for (int x = tid >> 6; x < (n + 1) / 2; x += NT / 64) {
            const int g = 2 * x + half;
            const int64_t slot = g < n ? slot_of(g, b) : -1;
            const int len = slot >= 0 ? (int)V.blen[slot] : 0;
            uint32_t m0 = 0, m1 = 0;
#pragma unroll
            for (int i = 0; i < LA; ++i) {
                const uint64_t bal = __ballot(len > i);
                const uint32_t mine = half ? (uint32_t)(bal >> 32) : (uint32_t)bal;
                if (b == (i & 31)) (i < 32 ? m0 : m1) = mine;
            }
            if (g < n) {
                uint32_t *rm = bit_group<LA, S>(lds + (uint32_t)g * stride, A).rowmask;
                if (b < LA) rm[b] = m0;
                if (b + 32 < LA) rm[b + 32] = m1;
            }
        }
    }
}

template <int LA, class S, int NT, typename SlotOf>
__device__ __forceinline__ void build_groups(const DevVocab &V, int64_t I0, int n, uint8_t *lds, uint32_t stride,
                                             SlotOf slot_of)
{
    build_tables<LA, S, NT>(V, n, lds, stride, slot_of);
    const int tid = (int)in_vgpr(threadIdx.x);
    const int A = V.alphabet;
    for (int x = tid; x < n * kBitRows; x += NT) {
        const int g = x >> 5, b = x & (kBitRows - 1);
        const int64_t slot = slot_of(g, b);
        const uint32_t col = slot >= 0 ? (uint32_t)V.bcol[slot] : 0xFFFFu;
        BitGroup G = bit_group<LA, S>(lds + (uint32_t)g * stride, A);
        G.cu[b] = col == 0xFFFFu ? -1 : (int32_t)(I0 + col);
    }
}

// The column words of 64 slots (group cg of the column array ccol, lengths
// clen) for this lane: the loads, and then the wave-uniform lengths.
__device__ __forceinline__ ColWords col_words_load(const uint32_t *ccol, const uint8_t *clen, int64_t cg, int lane)
{
    ColWords W;
    W.p = ccol + cg * (kColDwords * 64);
    W.dw0 = W.p[(uint32_t)lane];
    W.lb = (clen + cg * 64)[(uint32_t)lane];
    W.ncols = W.npad = 0;
    return W;
}
__device__ __forceinline__ void col_words_lengths(ColWords &W)
{
    W.ncols = __builtin_amdgcn_readlane(W.lb, 63);
    W.npad = W.ncols - __builtin_amdgcn_readfirstlane(W.lb);
}
__device__ __forceinline__ ColWords col_words(const uint32_t *ccol, const uint8_t *clen, int64_t cg, int lane)
{
    ColWords W = col_words_load(ccol, clen, cg, lane);
    col_words_lengths(W);
    return W;
}

// Launch classes of four longest lengths: class C has 4C+1 .. 4C+4, and class
// 0 also length 0.
constexpr int kBitClasses = kMaxLen / 4;
__host__ __device__ constexpr int bit_class_lo(int C) { return C == 0 ? 0 : 4 * C + 1; }
__host__ __device__ constexpr int bit_class_hi(int C) { return 4 * C + 4; }
// f(integral_constant<int, LA>) for the (wave-uniform) LA in [LO, HI].
template <int LO, int HI, typename F>
__device__ __forceinline__ void bit_length_dispatch(int LA, F &&f)
{
    if constexpr (LO == HI) {
        f(std::integral_constant<int, LO>{});
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (LA <= MID)
            bit_length_dispatch<LO, MID>(LA, f);
        else
            bit_length_dispatch<MID + 1, HI>(LA, f);
    }
}

// Row lengths of one launch of the triangle and edge kernels, all in one
// kernel: a launch ends with the
// workgroups of its last lengths alone on the chip, so few and full launches
// win (50k words of up to 20 symbols: one launch of 0 .. 24 against five of
// four lengths each), as far as the registers of the longest rows leave the
// short ones the waves that LDS admits.
template <class S>
constexpr int bits_span() { return S::kPlanes == 2 ? 24 : 12; }
template <class S>
constexpr int bits_ranges() { return kMaxLen / bits_span<S>(); }

// Waves per SIMD asked of the compiler: what its registers hold without
// spilling inside the column loop.
template <int HI, class S>
constexpr int bits_min_waves()
{
    return S::kPlanes == 2 ? (HI <= 24 ? 4 : 1) : (HI <= 12 ? 4 : HI <= 24 ? 3 : 1);
}

}  // namespace nw
