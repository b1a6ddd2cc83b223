// k_tri_bits.h -- the triangle kernel (int8 / int16 scores of the row-major
// upper triangle, Section 4.1 of the paper) in bit planes (nw_bits.h).
//
// A workgroup takes a block r of row words, a window of TW consecutive
// caller-order column words and one longest row length LA.  For every group of
// 32 row words of that length its wavefronts run the window's 64-word steps
// (length-sorted, dealt so that each wavefront gets long and short ones), turn
// the planes of G to one byte per pair (three rounds of bit exchanges), add
// the lane's p (LA + lb) to four pairs at a time, and stage the 32 bytes of a
// column word at its caller-order place: LDS dword S[j][column] holds the rows
// j, j+8, j+16, j+24.  Then the workgroup writes the 32 row segments: a thread
// reads eight columns, exchanges bytes to rows and stores 8 bytes (16 for
// int16) per row, at whatever alignment the row segment has.  (Shifting the
// bytes to dword boundaries first took 130 lane-instructions per 16 scores,
// a third of the kernel; this takes about 25.)
//
// Bytes hold score + bias, 0 .. 255 (bias 128 for int8, -lo for int16).
// Dictionaries of more than 256 score values (int16, W16) stage 16-bit scores,
// two rows per dword.
//
// Rows without a pair in the range [idx_begin, idx_end) right of the diagonal
// are left out: a tile that holds such rows first lists the others (in slot
// order, so still sorted by length) and groups those.
//
// Bound: vector issue; at 7 symbols about 11 lane-instructions of DP and 7 of
// sums, byte exchange, staging and stores per pair.  50,000 words, int8:
// 2.79 ms with the packed DP (k_tri_code), 0.69 ms (1.8 TB/s of scores)
// here; 20,000 words of 1..25 symbols under a matrix, int16: 2.26 -> 0.82 ms.
#pragma once

#include "nw_bits.h"

namespace nw {

constexpr int kTriBitGroups = 4;    // groups whose tables are built at a time, at most
constexpr uint32_t kTriBitsLds = 40u * 1024u;   // aim: four workgroups per CU

struct alignas(16) TriRow {
    uint64_t addr;   // output address of column 0 of the window (may lie outside the buffer)
    int32_t cs, cl;  // columns [cs, cl) of the window are stored
};

__host__ __device__ constexpr uint32_t tri_stage_stride(int TW) { return (uint32_t)(TW + 4) * 4u; }   // bytes of S[j]
__host__ __device__ constexpr uint32_t tri_bits_group_bytes(int LA, int tab, int alphabet)
{
    return bit_group_bytes(LA, tab, alphabet) + kBitRows * (uint32_t)sizeof(TriRow);
}
// LDS: the staging rows (before them, in the same place, the row list), the
// list's counts and the groups.
__host__ __device__ constexpr uint32_t tri_bits_fixed_bytes(int TW, int CB, bool w16)
{
    const uint32_t stage = tri_stage_stride(TW) * (w16 ? 16u : 8u), list = (uint32_t)CB * 2u;
    return ((stage > list ? stage : list) + 15u & ~15u) + 64u;
}
__host__ __device__ inline int tri_bits_groups(int LA, int tab, int alphabet, int TW, int CB, bool w16, uint32_t lds, int most)
{
    const uint32_t per = tri_bits_group_bytes(LA, tab, alphabet), fixed = tri_bits_fixed_bytes(TW, CB, w16);
    if (lds < fixed + per) return 0;
    const uint32_t kg = (lds - fixed) / per;
    return kg < (uint32_t)most ? (int)kg : most;
}
// LDS of a launch whose longest row words have LA symbols, for at most `most`
// (1 .. kTriBitGroups) groups at a time.
__host__ __device__ inline uint32_t tri_bits_lds_bytes(int LA, int tab, const DevVocab &V, bool w16, int most)
{
    const uint32_t fixed = tri_bits_fixed_bytes(V.TW, V.CB, w16), per = tri_bits_group_bytes(LA, tab, V.alphabet);
    return bit_lds_bytes(fixed, per, kTriBitsLds, (uint32_t)most);
}
// More than 256 score values: 16-bit staging.
__host__ __device__ inline bool tri_bits_wide(const DevVocab &V) { return V.hi - V.lo > 255; }

// Four dwords of four row bytes each (x[c] = column c) to four dwords of four
// columns each (d[k] = row byte k).
__device__ __forceinline__ void bytes_to_rows(const u32x4 &x, uint32_t (&d)[4])
{
    const uint32_t t0 = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), t1 = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
    const uint32_t u0 = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u), u1 = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    d[0] = __builtin_amdgcn_perm(u0, t0, 0x05040100u);
    d[1] = __builtin_amdgcn_perm(u0, t0, 0x07060302u);
    d[2] = __builtin_amdgcn_perm(u1, t1, 0x05040100u);
    d[3] = __builtin_amdgcn_perm(u1, t1, 0x07060302u);
}

#define NW_GLOBAL __attribute__((address_space(1)))
// Row segments start at any byte: stores of 8 or 16 bytes at any alignment
// (the hardware splits one that crosses a cache line).
typedef uint32_t u32x2_a1 __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint16_t u16_a1 __attribute__((aligned(1)));

// A row's info as the whole wavefront reads it, in scalar registers.
__device__ __forceinline__ TriRow uniform_row(const TriRow &R)
{
    TriRow u;
    u.addr = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)R.addr) |
             (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(R.addr >> 32)) << 32;
    u.cs = __builtin_amdgcn_readfirstlane(R.cs);
    u.cl = __builtin_amdgcn_readfirstlane(R.cl);
    return u;
}

// Store the eight elements of row R at window columns f .. f+7, e their output
// bytes (2 dwords int8, 4 dwords int16): one store where all lie in [cs, cl),
// else element by element.
template <int ES>
__device__ __forceinline__ void store_eight(const TriRow &R, int f, const uint32_t (&e)[2 * ES])
{
    NW_GLOBAL uint8_t *const g = (NW_GLOBAL uint8_t *)R.addr + (uint32_t)(f * ES);
    if (f >= R.cs && f + 8 <= R.cl) {
        if constexpr (ES == 1)
            *(NW_GLOBAL u32x2_a1 *)g = u32x2_a1{e[0], e[1]};
        else
            *(NW_GLOBAL u32x4_a1 *)g = u32x4_a1{e[0], e[1], e[2], e[3]};
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (f + i >= R.cs && f + i < R.cl) {
                if constexpr (ES == 1)
                    g[i] = (uint8_t)(e[i / 4] >> (8 * (i & 3)));
                else
                    ((NW_GLOBAL u16_a1 *)g)[i] = (uint16_t)(e[i / 2] >> (16 * (i & 1)));
            }
    }
}

template <int LA, class S, int ES, bool W16, int NT>
__device__ __forceinline__ void tri_bits_tile(const DevVocab &V, uint32_t r, uint32_t w0, int nw, uint32_t part, uint64_t idx_begin,
                                              uint64_t idx_end, void *out, uint32_t lds_bytes, int most, uint8_t *lds)
{
    constexpr int P = sum_planes<LA, S>();
    constexpr int PD = P > 0 ? P : 1;
    const int64_t n = V.n;
    const int TW = V.TW, A = V.alphabet, pabs = -V.gap;
    const int64_t I0 = (int64_t)r * V.CB, I1 = min(I0 + V.CB, n);
    // the windows w0 .. w0 + nw - 1, less those left of the block's diagonal
    if ((int64_t)w0 * TW < I0) {
        const int skip = (int)((I0 - (int64_t)w0 * TW) / TW);
        if (skip >= nw) return;
        w0 += (uint32_t)skip;
        nw -= skip;
    }
    nw = min(nw, (int)((uint32_t)V.nwin - w0));
    const int64_t Jbeg = (int64_t)w0 * TW, Jend = min(Jbeg + (int64_t)nw * TW, n);
    if (Jend <= I0 + 1) return;   // no column right of the block's first row
    // rows [u0, u1) of the block have a pair of these windows in the range
    int64_t u0 = I0, u1 = min(I1, Jend - 1);
    {
        auto first = [&](int64_t u) { return row_start_idx(n, u) + (uint64_t)(max(Jbeg, u + 1) - u - 1); };
        auto last = [&](int64_t u) { return row_start_idx(n, u) + (uint64_t)(Jend - 1 - u - 1); };
        if (last(u1 - 1) < idx_begin || first(u0) >= idx_end) return;
        // both ends grow with u: bisect
        if (last(u0) < idx_begin) {
            int64_t lo = u0, hi = u1 - 1;   // last(lo) < idx_begin <= last(hi)
            while (hi - lo > 1) {
                const int64_t m = (lo + hi) / 2;
                if (last(m) < idx_begin) lo = m; else hi = m;
            }
            u0 = hi;
        }
        if (first(u1 - 1) >= idx_end) {
            int64_t lo = u0, hi = u1 - 1;   // first(hi) >= idx_end
            while (hi > lo) {
                const int64_t m = (lo + hi) / 2;
                if (first(m) >= idx_end) hi = m; else lo = m + 1;
            }
            u1 = hi;
            if (u1 <= u0) return;
        }
    }
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    constexpr int NWAVE = NT / 64;
    const uint32_t lds0 = lds_addr_of(lds);
    const uint32_t SS = tri_stage_stride(TW);
    constexpr uint32_t SJ = W16 ? 16u : 8u;
    uint16_t *rows = reinterpret_cast<uint16_t *>(lds);
    uint32_t *counts = reinterpret_cast<uint32_t *>(lds + tri_bits_fixed_bytes(TW, V.CB, W16) - 64u);
    uint8_t *groups = lds + tri_bits_fixed_bytes(TW, V.CB, W16);
    const uint32_t gstride = tri_bits_group_bytes(LA, S::kTab, A);
    const int kg = tri_bits_groups(LA, S::kTab, A, TW, V.CB, W16, lds_bytes, most);
    if (kg < 1) return;   // the launch's LDS holds a group (tri_bits_lds_bytes)

    // the groups of this length: the block's own, or groups of the listed rows
    const bool listed = u0 > I0 || u1 < I1;
    uint32_t gbeg, gend, nlist = 0;
    if (!listed) {
        const uint32_t *rgo = V.rg_off + (size_t)r * (V.lmax + 1) + LA;
        gbeg = rgo[0];
        gend = rgo[1];
        if (gbeg >= gend) return;
    } else {
        auto keep = [&](int s) {
            const uint32_t col = V.bcol[I0 + s];
            return col != 0xFFFFu && I0 + col >= u0 && I0 + col < u1;
        };
        // the wavefronts' shares: a multiple of 64 slots (CB / 64 is at least
        // 4 and, from 8 on, a multiple of NWAVE)
        const int share = V.CB / min(NWAVE, V.CB / 64);
        const int s0 = min(wave * share, V.CB), s1 = min(s0 + share, V.CB);
        uint32_t c = 0;
        for (int s = s0; s < s1; s += 64) c += (uint32_t)__popcll(__ballot(keep(s + lane)));
        if (lane == 0) counts[wave] = c;
        if (tid < 2) counts[NWAVE + tid] = 0;
        __syncthreads();
        uint32_t at = 0;
        for (int q = 0; q < NWAVE; ++q) {
            if (q < wave) at += counts[q];
            nlist += counts[q];
        }
        for (int s = s0; s < s1; s += 64) {
            const bool k = keep(s + lane);
            const uint64_t m = __ballot(k);
            if (k)
                rows[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    (uint16_t)(s + lane);
            at += (uint32_t)__popcll(m);
        }
        __syncthreads();
        // groups of the list with a shorter, and with at most this, longest length
        const uint32_t ng = (nlist + kBitRows - 1) / kBitRows;
        for (uint32_t g = tid; g < ng; g += NT) {
            const int len = V.blen[I0 + rows[min(g * kBitRows + kBitRows, nlist) - 1]];
            if (len < LA) atomicAdd(&counts[NWAVE], 1u);
            if (len <= LA) atomicAdd(&counts[NWAVE + 1], 1u);
        }
        __syncthreads();
        gbeg = counts[NWAVE];
        gend = counts[NWAVE + 1];
        if (gbeg >= gend) return;
    }

    const int steps = TW / 64;
    const uint32_t nparts = gridDim.z;
    const int bias = W16 ? 0 : ES == 1 ? 128 : -V.lo;
    // chunks of kg groups, every nparts-th.  The row list lies where the rows
    // are staged: a listed tile's parts take one chunk each (the launch has
    // enough parts)
    for (uint32_t gc = gbeg + part * (uint32_t)kg; gc < gend; gc += nparts * (uint32_t)kg) {
        const int ng = (int)min((uint32_t)kg, gend - gc);
        auto slot_of = [&](int g, int b) -> int64_t {
            const uint32_t q = (gc + (uint32_t)g) * kBitRows + (uint32_t)b;
            if (!listed) return (int64_t)q;
            return q < nlist ? I0 + rows[q] : -1;
        };
        build_groups<LA, S, NT>(V, I0, ng, groups, gstride, slot_of);
        __syncthreads();
        for (int wi = 0; wi < nw; ++wi) {
        const uint32_t w = w0 + (uint32_t)wi;
        const int64_t J0 = (int64_t)w * TW, J1 = min(J0 + TW, n);
        for (int x = tid; x < ng * kBitRows; x += NT) {
            const int64_t u = bit_group<LA, S>(groups + (uint32_t)(x >> 5) * gstride, A).cu[x & 31];
            TriRow R{0, 0, 0};
            if (u >= 0) {
                const int64_t base = (int64_t)row_start_idx(n, u) + (J0 - u - 1);   // pair index of column 0
                R.addr = (uint64_t)(uintptr_t)out + (uint64_t)((base - (int64_t)idx_begin) * ES);
                R.cs = (int32_t)min(max(max((int64_t)0, u + 1 - J0), (int64_t)idx_begin - base), (int64_t)TW);
                R.cl = (int32_t)max(min(J1 - J0, (int64_t)idx_end - base), (int64_t)0);
            }
            reinterpret_cast<TriRow *>(groups + (uint32_t)(x >> 5) * gstride + bit_group_bytes(LA, S::kTab, A))[x & 31] = R;
        }
        __syncthreads();
        // this wavefront's steps, taken from either end in turn; the next
        // step's words are loaded while one runs
        const int nq = wave < steps ? (steps - 1 - wave) / NWAVE + 1 : 0;
        auto step_of = [&](int q) { return q * NWAVE + ((q & 1) && (q + 1) * NWAVE <= steps ? NWAVE - 1 - wave : wave); };
        auto load = [&](int q, ColWords &W, uint32_t &col) {
            const int st = step_of(q);
            W = col_words_load(V.tccol, V.tlen, (int64_t)w * steps + st, lane);
            col = V.tcol[(int64_t)w * TW + st * 64 + lane];
        };
        ColWords Wn;
        uint32_t coln = 0;
        if (nq > 0) load(0, Wn, coln);
        for (int g = 0; g < ng; ++g) {
            const uint32_t gb = (uint32_t)(groups - lds) + (uint32_t)g * gstride;
            const BitGroup G = bit_group<LA, S>(lds + gb, A);
            bool mixed = false;
            if constexpr (LA > 0) mixed = __builtin_amdgcn_readfirstlane((int)G.rowmask[LA - 1]) != ~0;
            for (int q = 0; q < nq; ++q) {
                ColWords W = Wn;
                const uint32_t at = lds0 + 4u * (coln == 0xFFFFu ? (uint32_t)TW : coln);   // padding: the spare column
                col_words_lengths(W);
                load(q + 1 < nq ? q + 1 : 0, Wn, coln);
                BitColumn<LA, S> C;
                C.run(W, lds0 + gb);
                if (mixed) C.fill_short_rows(G.rowmask, pabs);
                uint32_t s[PD];
                if constexpr (P > 0) C.template sum<P>(s); else s[0] = 0;
                uint32_t by[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) by[i] = i < P ? s[i < P ? i : 0] : 0u;
                planes_to_bytes(by);
                const int off = bias - pabs * (LA + W.lb);
                if constexpr (!W16) {
                    const uint32_t o4 = (uint32_t)off * 0x01010101u;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        // every byte plus off lies in [0, 255]: the packed add
                        // carries between bytes only where a ninth plane was cut off
                        uint32_t x = by[i] + o4;
                        if constexpr (P > 8) {
                            const uint32_t ob = ((uint32_t)off & 0xFFu) * 0x01010101u;
                            x = ((by[i] & 0x7F7F7F7Fu) + (ob & 0x7F7F7F7Fu)) ^ ((by[i] ^ ob) & 0x80808080u);
                        }
                        *lds_ptr(at + (uint32_t)i * SS) = x;
                    }
                } else {
                    const uint32_t o2 = ((uint32_t)off & 0xFFFFu) * 0x00010001u;
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        // rows i, i+16 and rows i+8, i+24 as 16-bit sums, plus off modulo 2^16
                        uint32_t a = by[i] & 0x00FF00FFu, c = (by[i] >> 8) & 0x00FF00FFu;
                        if constexpr (P > 8) {
                            a |= ((s[P > 8 ? 8 : 0] >> i) & 0x00010001u) << 8;
                            c |= ((s[P > 8 ? 8 : 0] >> (8 + i)) & 0x00010001u) << 8;
                        }
                        a = ((a & 0x7FFF7FFFu) + (o2 & 0x7FFF7FFFu)) ^ ((a ^ o2) & 0x80008000u);
                        c = ((c & 0x7FFF7FFFu) + (o2 & 0x7FFF7FFFu)) ^ ((c ^ o2) & 0x80008000u);
                        *lds_ptr(at + (uint32_t)(2 * i) * SS) = a;
                        *lds_ptr(at + (uint32_t)(2 * i + 1) * SS) = c;
                    }
                }
            }
            __syncthreads();
            // the row segments: a wavefront takes every NWAVE-th staging row, a
            // lane eight columns of it at a time
            const TriRow *info = reinterpret_cast<const TriRow *>(lds + gb + bit_group_bytes(LA, S::kTab, A));
            for (int j = wave; j < (int)SJ; j += NWAVE) {
                constexpr int NR = W16 ? 2 : 4;   // rows of a staging dword
                TriRow R[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) R[k] = uniform_row(info[W16 ? (j >> 1) + 8 * (j & 1) + 16 * k : j + 8 * k]);
                for (int c = 8 * lane; c < TW; c += 512) {
                    const uint32_t at = lds0 + (uint32_t)j * SS + 4u * (uint32_t)c;
                    const u32x4 x0 = *(const lds_u32x4 *)(uintptr_t)at, x1 = *(const lds_u32x4 *)(uintptr_t)(at + 16u);
                    uint32_t e[NR][2 * ES];
                    if constexpr (!W16) {
                        uint32_t d0[4], d1[4];
                        bytes_to_rows(x0, d0);
                        bytes_to_rows(x1, d1);
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            if constexpr (ES == 1) {
                                e[k][0] = d0[k] ^ 0x80808080u;
                                e[k][1] = d1[k] ^ 0x80808080u;
                            } else {
                                const u16x2 lo2 = u16x2{(uint16_t)V.lo, (uint16_t)V.lo};
                                auto widen = [&](uint32_t y, uint32_t sel) {
                                    return __builtin_bit_cast(
                                        uint32_t, __builtin_bit_cast(u16x2, __builtin_amdgcn_perm(0u, y, sel)) + lo2);
                                };
                                e[k][0] = widen(d0[k], 0x0C010C00u);
                                e[k][1] = widen(d0[k], 0x0C030C02u);
                                e[k][2 * ES - 2] = widen(d1[k], 0x0C010C00u);
                                e[k][2 * ES - 1] = widen(d1[k], 0x0C030C02u);
                            }
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < NR; ++k) {
                            const uint32_t sel = k ? 0x07060302u : 0x05040100u;
                            e[k][0] = __builtin_amdgcn_perm(x0[1], x0[0], sel);
                            e[k][1] = __builtin_amdgcn_perm(x0[3], x0[2], sel);
                            e[k][2 * ES - 2] = __builtin_amdgcn_perm(x1[1], x1[0], sel);
                            e[k][2 * ES - 1] = __builtin_amdgcn_perm(x1[3], x1[2], sel);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NR; ++k) store_eight<ES>(R[k], c, e[k]);
                }
            }
            __syncthreads();
        }
        }
    }
}

// Threads of a workgroup: eight wavefronts where the 64 KB of 16-bit staging
// and the tables leave one workgroup per CU; four elsewhere (with eight for
// every Bits3 row past 12 symbols, 20,000 words under a matrix took 1.15 ms
// against 0.88: the registers then fit one workgroup instead of three).
template <int HI, bool W16>
constexpr int tri_bits_threads() { return W16 && HI > 12 ? 512 : 256; }

// Longest row lengths LO .. HI, one per blockIdx.y, the longest first;
// blockIdx.x = (row block - rb0) * nset + set, set s being the windows s * nw
// .. s * nw + nw - 1; blockIdx.z = the part of the groups.
template <int LO, int HI, class S, int ES, bool W16>
__global__ __launch_bounds__((tri_bits_threads<HI, W16>())) __attribute__((amdgpu_waves_per_eu(bits_min_waves<HI, S>())))
void k_tri_bits(DevVocab V, uint64_t idx_begin, uint64_t idx_end, void *out, uint32_t rb0, uint32_t nset, int nw,
                int hi, uint32_t lds_bytes, int most)
{
    extern __shared__ __align__(16) uint8_t lds[];
    const uint32_t r = rb0 + blockIdx.x / nset, w0 = blockIdx.x % nset * (uint32_t)nw;
    const int LA = hi - (int)blockIdx.y;
    if (LA < LO || LA > HI) return;
    bit_length_dispatch<LO, HI>(LA, [&](auto la) {
        tri_bits_tile<decltype(la)::value, S, ES, W16, tri_bits_threads<HI, W16>()>(V, r, w0, nw, blockIdx.z, idx_begin, idx_end, out, lds_bytes,
                                                                                  most, lds);
    });
}

}  // namespace nw
