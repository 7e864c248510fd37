// The k smallest of n keys by one workgroup, without a sort: a search for the cut.
//
// Keys are rank_key values (segments.hpp), the order is (key, index).  The cut is built from the
// most significant bits down, two bits per step: the workgroup counts the keys below the three
// candidate cuts (ballots of keys held in registers; nothing but 16 LDS adds and one barrier a
// step) and keeps the largest candidate that has fewer than k keys below it.  A candidate with
// exactly k keys below it ends the search: for values that differ that is after about 20 of the
// 32 bits.  Only if entries equal to the cut have to be told apart by index (repeated values) a
// prefix count over the workgroup follows.
//
// Bound by latency: 10-16 steps of a ballot count, a barrier and an LDS read.  Measured, whole
// kernels: 11.1 us at 4 sequences of 2880 tokens (a count of the entries that come before each
// entry, which reads n keys per entry: 64 us); kept tokens and slots of 8 sets of 1024 7.9 us and of a
// set of 2304 9.3 us (24 + 5 and 52 + 6 us).
#pragma once

#include "common.hpp"

namespace skipffn {

constexpr int TOPK_THREADS = 1024;
constexpr int TOPK_WAVES = TOPK_THREADS / 64;
constexpr uint32_t TOPK_NONE = 0xFFFFFFFFu;     // key of an absent entry: below no candidate

struct TopkShared {
    int below[3][4];                             // counts of three steps in rotation (one barrier a step)
    int scan[16 * TOPK_WAVES];
    int total;
};
// entries with key < cut are among the k smallest, and the first `ties` (in index order) of those with key == cut
struct TopkCut { uint32_t cut; int ties; };

// Entry i * TOPK_THREADS + threadIdx.x is key(i), i < nv = ceil(n / TOPK_THREADS); MAXV > 0: nv <= MAXV and the
// loops over i are unrolled (keys in registers), MAXV == 0: any nv.  0 < k < n, uniform.
template <int MAXV, class Key>
__device__ __forceinline__ TopkCut topk_cut(Key&& key, int nv, int k, TopkShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 4) sh.below[0][tid] = 0;
    __syncthreads();
    uint32_t p = 0;
    int less = 0;                                // keys below p
    int cur = 0;
    for (int shift = 30; shift >= 0; shift -= 2) {
        const uint32_t c1 = p | (1u << shift), c2 = p | (2u << shift), c3 = p | (3u << shift);
        int n1 = 0, n2 = 0, n3 = 0;
        auto count = [&](uint32_t v) {
            n1 += __popcll(__ballot(v < c1));
            n2 += __popcll(__ballot(v < c2));
            n3 += __popcll(__ballot(v < c3));
        };
        if constexpr (MAXV > 0) {
#pragma unroll
            for (int i = 0; i < MAXV; ++i)
                if (i < nv) count(key(i));
        } else {
            for (int i = 0; i < nv; ++i) count(key(i));
        }
        const int nxt = cur == 2 ? 0 : cur + 1;
        if (lane < 3) atomicAdd(&sh.below[cur][lane], lane == 0 ? n1 : (lane == 1 ? n2 : n3));
        if (tid < 4) sh.below[nxt][tid] = 0;     // last read two steps ago
        __syncthreads();
        const int b1 = sh.below[cur][0], b2 = sh.below[cur][1], b3 = sh.below[cur][2];
        cur = nxt;
        if (b1 == k) return TopkCut{c1, 0};
        if (b2 == k) return TopkCut{c2, 0};
        if (b3 == k) return TopkCut{c3, 0};
        if (b3 < k)      { p = c3; less = b3; }
        else if (b2 < k) { p = c2; less = b2; }
        else if (b1 < k) { p = c1; less = b1; }
    }
    return TopkCut{p, k - less};
}

// before[i] = number of entries flagged by flag(i) that precede entry i * TOPK_THREADS + threadIdx.x;
// returns how many are flagged in all
template <int MAXV, class Flag>
__device__ __forceinline__ int topk_prefix(Flag&& flag, int nv, TopkShared& sh, int (&before)[MAXV]) {
    static_assert(MAXV <= 16, "size of TopkShared::scan");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();                             // scan[] of an earlier call has been read
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (i < nv) {
            const uint64_t m = __ballot(flag(i));
            before[i] = lanes_below(m);
            if (lane == 0) sh.scan[i * TOPK_WAVES + wave] = __popcll(m);
        }
    __syncthreads();
    if (wave == 0) {
        int carry = 0;
        for (int q = 0; q < nv * TOPK_WAVES; q += 64) {
            const bool in = q + lane < nv * TOPK_WAVES;
            const int v = in ? sh.scan[q + lane] : 0;
            const int inc = wave_inclusive_sum(v);
            if (in) sh.scan[q + lane] = carry + inc - v;
            carry += __builtin_amdgcn_readlane(inc, 63);
        }
        if (lane == 0) sh.total = carry;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (i < nv) before[i] += sh.scan[i * TOPK_WAVES + wave];
    return sh.total;
}

// For short lists (4 n <= TOPK_THREADS): how many of the n keys in LDS come before entry threadIdx.x / 4 in the order
// (key, index); four lanes share an entry.  All lanes of a wavefront call it (entries from n on count something).
__device__ __forceinline__ int rank_in_lds(const uint32_t* keys, int n) {
    const int t = threadIdx.x >> 2;
    const uint64_t mine = ((uint64_t)keys[t < n ? t : 0] << 32) | (uint32_t)t;
    int before = 0;
#pragma unroll 4
    for (int u = threadIdx.x & 3; u < n; u += 4) before += (((uint64_t)keys[u] << 32) | (uint32_t)u) < mine ? 1 : 0;
    before += __shfl_xor(before, 1);
    return before + __shfl_xor(before, 2);
}

}  // namespace skipffn
