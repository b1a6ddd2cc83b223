// k_query.h -- per-row top-k of a set of row words against a column set.
//
// Used for served queries (rows = query words, columns = the dictionary) and
// for the threshold pre-pass of the all-pairs top-k (rows = every dictionary
// word, columns = the probe subset).  A neighbour list is the first k of
// {(score(q, d), d)} sorted by (score descending, index ascending); there is
// no self-exclusion here (the all-pairs path accounts for it).
//
// k_query_class<LO, HI>: a workgroup takes one row pair of a length in LO .. HI
// (the two words of a pair have one length and fill the two binary16 halves of
// the DP) and one split of the column slots.  It builds the pair's LDS profile,
// then each wavefront walks its share of the split (64 length-sorted column
// words per step) and keeps a sorted wave list of the best k keys for each of
// the two rows.  With several splits the four wave lists of a row are merged in
// LDS (wavefront 0 for the first row, 1 for the second) into the split's list,
// written to `partial`, row-major [row][split][k]; with one split (many rows,
// nothing to spread) the four wave lists go out as they are, [row][wave][k].
// Either way a row has query_lists(nsplit) lists of k keys.
//
// A launch per range of 16 lengths, not per length: a batch of mixed lengths is
// at most three launches on the caller's stream, its row pairs side by side, with
// no need of other streams.  8 / 256 / 1,000 queries of mixed lengths against
// 200,000 words to 20 symbols, us: 141 / 719 / 1,681 with a launch per length
// spread over the library's streams, 111 / 448 / 1,218 here.  (Ranges of 8: one
// launch more for most batches, 4 queries of 600,000 words to 40 symbols 324
// against 271; longer ranges cost the short rows the registers of the long.)
//
// k_merge_lists: one wavefront per row merges its P partial lists into the
// final top-k (and optionally reports the key of a given rank);
// k_merge_lists_wg does the same with a workgroup per row, for rows with many
// partial keys (a few queries spread over many splits).
#pragma once

#include "nw_tile_common.h"
#include "nw_topk.h"

namespace nw {

struct QueryArgs {
    RowSet R;
    ColSet C;
    const uint16_t *wtab;
    int alphabet;
    int gap;
    int lo;                 // lower score bound (key origin)
    int k;                  // list length, 1..64
    int64_t per;            // column slots per split (multiple of 256)
    int nsplit;
    uint64_t *partial;      // [rows][nsplit][k]
};

// LDS: the profile, then the wave lists of both rows of the pair (2 x 4 x k keys).
__host__ __device__ constexpr uint32_t query_lds_bytes(int LA, int alphabet, int k)
{
    return profile_bytes(LA, alphabet) + 2u * 4u * 8u * (uint32_t)k;
}

// Row pair p of length LA.
template <int LA>
__device__ __forceinline__ void query_tile(const QueryArgs &Q, uint32_t p, uint8_t *lds)
{
    const int split = blockIdx.y;
    const int64_t c0 = (int64_t)split * Q.per;
    const int64_t c1 = min(c0 + Q.per, Q.C.nslots);

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int32_t a0 = Q.R.pairs[2 * p], a1 = Q.R.pairs[2 * p + 1];
    build_profile<LA>(Q.wtab, Q.alphabet, reinterpret_cast<uint32_t *>(lds), Q.R.sym + (int64_t)a0 * kWordBytes,
                      Q.R.sym + (int64_t)(a1 >= 0 ? a1 : a0) * kWordBytes, profile_role(tid, Q.alphabet));
    __syncthreads();
    uint64_t list0 = 0, list1 = 0, thr0 = 0, thr1 = 0;
    // the next step's column word is loaded while this step's DP and
    // list offers run (a split is a few steps, so load latency would
    // otherwise dominate a lightly loaded GPU)
    int64_t base = c0 + wave * 64;
    int lb_n = 0;
    int32_t d_n = -1;
    uint32_t bw_n[kWordBytes / 4];
    if (base < c1) {
        lb_n = Q.C.len[base + lane];
        d_n = Q.C.orig[base + lane];
        load_word(bw_n, Q.C.sym + (base + lane) * kWordBytes);
    }
    for (; base < c1; base += kThreads) {
        const int lb = lb_n;
        const int32_t d = d_n;
        uint32_t bw[kWordBytes / 4];
#pragma unroll
        for (int q = 0; q < kWordBytes / 4; ++q) bw[q] = bw_n[q];
        const int64_t nx = base + kThreads + lane;
        if (base + kThreads < c1) {
            lb_n = Q.C.len[nx];
            d_n = Q.C.orig[nx];
            load_word(bw_n, Q.C.sym + nx * kWordBytes);
        }
        const int lbmax_w = __builtin_amdgcn_readlane(lb, 63);
        int s0, s1;
        pair_scores_regs<LA>(bw, lb, lbmax_w, lds, Q.gap, s0, s1);
        const uint64_t key0 = d >= 0 ? nb_key(s0, Q.lo, (uint32_t)d) : 0;
        const uint64_t key1 = d >= 0 ? nb_key(s1, Q.lo, (uint32_t)d) : 0;
        wl_offer(list0, thr0, key0, Q.k, lane);
        if (a1 >= 0) wl_offer(list1, thr1, key1, Q.k, lane);
    }
    if (Q.nsplit == 1) {   // uniform: the wave lists are the row's partial lists
        if (lane < Q.k) {
            Q.partial[((int64_t)Q.R.orig[a0] * 4 + wave) * Q.k + lane] = list0;
            if (a1 >= 0) Q.partial[((int64_t)Q.R.orig[a1] * 4 + wave) * Q.k + lane] = list1;
        }
        return;
    }
    uint64_t *wl = reinterpret_cast<uint64_t *>(lds + profile_bytes(LA, Q.alphabet));   // [2 rows][4 waves][k]
    if (lane < Q.k) {
        wl[(0 * 4 + wave) * Q.k + lane] = list0;
        wl[(1 * 4 + wave) * Q.k + lane] = list1;
    }
    __syncthreads();
    // wavefront h merges the four wave lists of row h of the pair
    if (wave < 2 && (wave == 0 || a1 >= 0)) {
        const uint64_t *src = wl + wave * 4 * Q.k;
        uint64_t list = 0, t = 0;
        for (int base2 = 0; base2 < 4 * Q.k; base2 += 64) {
            const int i = base2 + lane;
            wl_offer(list, t, i < 4 * Q.k ? src[i] : 0, Q.k, lane);
        }
        const int32_t row = Q.R.orig[wave == 0 ? a0 : a1];
        if (lane < Q.k) Q.partial[((int64_t)row * Q.nsplit + split) * Q.k + lane] = list;
    }
}

template <int LA, int HI>
__device__ __forceinline__ void query_dispatch(const QueryArgs &Q, int la, uint32_t p, uint8_t *lds)
{
    if constexpr (LA <= HI) {
        if (la == LA)
            query_tile<LA>(Q, p, lds);
        else
            query_dispatch<LA + 1, HI>(Q, la, p, lds);
    }
}

// blockIdx.x = the row pair among those of lengths LO .. HI, blockIdx.y = the split.
template <int LO, int HI>
__global__ __launch_bounds__(kThreads) void k_query_class(QueryArgs Q)
{
    extern __shared__ __align__(16) uint8_t lds[];
    // the offsets are loaded together: testing one after the other chains their loads
    uint32_t off[HI - LO + 2];
#pragma unroll
    for (int l = 0; l <= HI - LO + 1; ++l) off[l] = Q.R.off[LO + l];
    const uint32_t p = off[0] + blockIdx.x;
    int la = LO;
#pragma unroll
    for (int l = 1; l <= HI - LO + 1; ++l) la += p >= off[l] ? 1 : 0;
    query_dispatch<LO, HI>(Q, la, p, lds);
}

#ifdef NW_LAUNCH_TU   // non-template kernels: compiled in the launcher unit only
// One wavefront per row: merge P sorted lists of kin keys into the top kout.
// Writes scores/indices (padding INT16_MIN / -1) when score != NULL and the
// key of rank `rank` (0 when the list is shorter) to thr when thr != NULL.
__global__ __launch_bounds__(256) void k_merge_lists(const uint64_t *partial, int P, int kin, int64_t rows, int kout,
                                                     int lo, int16_t *score, int32_t *index, uint64_t *thr, int rank)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const uint64_t *src = partial + row * (int64_t)P * kin;
    const int total = P * kin;
    uint64_t list = 0, t = 0;
    offer_range(list, t, src, 0, total, kout, lane);
    if (score != nullptr && lane < kout) {
        score[row * kout + lane] = list ? (int16_t)key_score(list, lo) : (int16_t)-32768;
        index[row * kout + lane] = list ? key_index(list) : -1;
    }
    if (thr != nullptr) {
        const uint64_t v = readlane64(list, rank - 1);
        if (lane == 0) thr[row] = v;
    }
}

// The same with one workgroup per row: wavefront w merges the w-th quarter of
// the row's P * kin keys, then wavefront 0 merges the four lists (LDS).
__global__ __launch_bounds__(256) void k_merge_lists_wg(const uint64_t *partial, int P, int kin, int64_t rows, int kout,
                                                        int lo, int16_t *score, int32_t *index, uint64_t *thr, int rank)
{
    __shared__ uint64_t quarter[4 * 64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row = blockIdx.x;
    if (row >= rows) return;   // uniform over the workgroup
    const uint64_t *src = partial + row * (int64_t)P * kin;
    const int total = P * kin;
    const int per = (total + 3) / 4;
    const int b0 = min(total, wave * per), b1 = min(total, b0 + per);
    uint64_t list = 0, t = 0;
    offer_range(list, t, src, b0, b1, kout, lane);
    if (lane < kout) quarter[wave * kout + lane] = list;
    __syncthreads();
    if (wave != 0) return;
    uint64_t fin = 0, tf = 0;
    for (int base = 0; base < 4 * kout; base += 64) {
        const int i = base + lane;
        wl_offer(fin, tf, i < 4 * kout ? quarter[i] : 0, kout, lane);
    }
    if (score != nullptr && lane < kout) {
        score[row * kout + lane] = fin ? (int16_t)key_score(fin, lo) : (int16_t)-32768;
        index[row * kout + lane] = fin ? key_index(fin) : -1;
    }
    if (thr != nullptr) {
        const uint64_t v = readlane64(fin, rank - 1);
        if (lane == 0) thr[row] = v;
    }
}

#endif

}  // namespace nw
