// The k smallest of n keys by one workgroup, without a sort: a search for the cut.
//
// Keys are rank_key values (segments.hpp), the order is (key, index).  The range of the keys is cut into 2048 equal parts, the
// keys are counted per part in LDS, and a prefix sum finds the part in which the k-th lies; that part is cut again, three times at
// most (32 bits in steps of 11), as a rule twice: a part of the second cut that ends at the k-th key ends the search.  Only if
// entries equal to the cut have to be told apart by index (repeated values) a prefix count over the workgroup follows.
//
// Bound by latency: four barriers and an LDS round trip between each two for every cut.  Measured, whole
// kernels, us: 7.0 at 4 sequences of 2880 tokens (two bits a step, counted with ballots, 10-16 steps of a barrier each: 11.6; a rank for every
// entry by counting, 64 entries to a workgroup: 9.2); kept tokens and slots of 8 sets of 1024 5.5 (8.1) and of a set of 2304
// 6.1 (10.2).
#pragma once

#include "common.hpp"

namespace skipffn {

constexpr int TOPK_THREADS = 1024;
constexpr int TOPK_WAVES = TOPK_THREADS / 64;
constexpr uint32_t TOPK_NONE = 0xFFFFFFFFu;     // key of an absent entry: below no candidate

constexpr int TOPK_BINS = 2048;
struct TopkShared {
    int hist[2][TOPK_BINS];                      // of a cut, and cleared for the next one
    uint32_t lo[TOPK_WAVES], hi[TOPK_WAVES];
    int count[TOPK_WAVES];
    int part, before, inside;                    // the part with the k-th key, keys before and in it
    int scan[16 * TOPK_WAVES];
    int total;
};
// entries with key < cut are among the k smallest, and the first `ties` (in index order) of those with key == cut
struct TopkCut { uint32_t cut; int ties; };

// Entry i * TOPK_THREADS + threadIdx.x is key(i), i < nv = ceil(n / TOPK_THREADS); MAXV > 0: nv <= MAXV and the
// loops over i are unrolled (keys in registers), MAXV == 0: any nv.  0 < k < n, uniform.
template <int MAXV, class Key>
__device__ __forceinline__ TopkCut topk_cut(Key&& key, int nv, int k, TopkShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto for_keys = [&](auto&& f) {
        if constexpr (MAXV > 0) {
#pragma unroll
            for (int i = 0; i < MAXV; ++i)
                if (i < nv) f(key(i));
        } else {
            for (int i = 0; i < nv; ++i) f(key(i));
        }
    };
    constexpr int PER = TOPK_BINS / TOPK_THREADS;
    static_assert(PER == 2, "two bins a thread");
    // the range of the keys that are numbers, and how many they are
    uint32_t lo = TOPK_NONE, hi = 0;
    int m = 0;
    for_keys([&](uint32_t v) {
        if (v != TOPK_NONE) {
            lo = v < lo ? v : lo;
            hi = v > hi ? v : hi;
            ++m;
        }
    });
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t l = __shfl_xor(lo, off), h = __shfl_xor(hi, off);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
        m += __shfl_xor(m, off);
    }
    if (lane == 0) { sh.lo[wave] = lo; sh.hi[wave] = hi; sh.count[wave] = m; }
#pragma unroll
    for (int q = 0; q < PER; ++q) sh.hist[0][tid + q * TOPK_THREADS] = 0;
    __syncthreads();
    m = 0;
#pragma unroll
    for (int w = 0; w < TOPK_WAVES; ++w) {
        lo = sh.lo[w] < lo ? sh.lo[w] : lo;
        hi = sh.hi[w] > hi ? sh.hi[w] : hi;
        m += sh.count[w];
    }
    if (m <= k) return TopkCut{TOPK_NONE, k - m};        // all numbers, and the first of the others
    for (int cur = 0;; cur ^= 1) {
        // lo <= hi, and the k-th key is the k-th smallest of those in [lo, hi], of which there are more than k
        const int width = 32 - __builtin_clz((hi - lo) | 1u), shift = width > 11 ? width - 11 : 0;
        for_keys([&](uint32_t v) {
            if (v >= lo && v <= hi) atomicAdd(&sh.hist[cur][(v - lo) >> shift], 1);
        });
        __syncthreads();
        const int h0 = sh.hist[cur][2 * tid], h1 = sh.hist[cur][2 * tid + 1];
        const int incl = wave_inclusive_sum(h0 + h1);
        if (lane == 63) sh.count[wave] = incl;
#pragma unroll
        for (int q = 0; q < PER; ++q) sh.hist[cur ^ 1][tid + q * TOPK_THREADS] = 0;
        __syncthreads();
        int before = incl - h0 - h1;
#pragma unroll
        for (int w = 0; w < TOPK_WAVES - 1; ++w) before += w < wave ? sh.count[w] : 0;
        if (before < k && k <= before + h0 + h1) {       // one thread
            const bool second = k > before + h0;
            sh.part = 2 * tid + (second ? 1 : 0);
            sh.before = second ? before + h0 : before;
            sh.inside = second ? h1 : h0;
        }
        __syncthreads();
        const uint32_t from = lo + ((uint32_t)sh.part << shift);
        const int b = sh.before, in = sh.inside;
        if (k == b + in) return TopkCut{from + (1u << shift), 0};       // more keys follow up to hi: no wrap
        if (shift == 0) return TopkCut{from, k - b};
        k -= b;
        const uint32_t to = from + ((1u << shift) - 1);
        lo = from;
        hi = to < hi ? to : hi;
    }
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
