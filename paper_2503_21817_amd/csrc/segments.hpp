// Token sets described by a device-side offset table: set i is positions [seg[i], seg[i+1]) of
// a token list of n_tok entries.  Sets are cut into chunks of CH positions, one workgroup per
// chunk; a launch covers the upper bound ceil(n_tok / CH) + S chunks and workgroups past the
// real count exit.  Bounds are clamped so that a malformed table cannot send a read outside
// the list.
#pragma once

#include "common.hpp"

namespace skipffn {

__device__ __forceinline__ void seg_bounds(const int32_t* __restrict__ seg, int i, int n_tok, int& b, int& e) {
    e = seg[i + 1];
    e = e < 0 ? 0 : (e > n_tok ? n_tok : e);
    b = seg[i];
    b = b < 0 ? 0 : (b > e ? e : b);
}
// chunk q -> (set s, first position t0, count nt); false past the last chunk.  Called by whole
// wavefronts: a lane takes a set, a prefix sum over the lanes finds the chunk's set.  (A scalar walk over the
// sets costs a load's latency per few sets before a workgroup knows its rows: the reducing kernels of the
// summary layer 13.4 -> 11.7 and 7.3 -> 5.9 us at 32 sets.)  FEW_SETS (S <= 2): the scalar loads are the faster way:
// forward + backward of the summary layer 26.9 / 27.5 us at one set of 16 tokens, C = 4096.
constexpr int SEG_FEW_SETS = 2;
template <int CH, bool FEW_SETS>
__device__ __forceinline__ bool locate_chunk(const int32_t* __restrict__ seg, int S, int n_tok, int q,
                                             int& s, int& t0, int& nt) {
    if constexpr (FEW_SETS) {
        int b0, e0, b1, e1;
        seg_bounds(seg, 0, n_tok, b0, e0);
        seg_bounds(seg, S - 1, n_tok, b1, e1);
        const int nc0 = (e0 - b0 + CH - 1) / CH, nc1 = S == 2 ? (e1 - b1 + CH - 1) / CH : 0;
        if (q >= nc0 + nc1) return false;
        s = q < nc0 ? 0 : 1;
        const int e = s == 0 ? e0 : e1;
        t0 = s == 0 ? b0 + q * CH : b1 + (q - nc0) * CH;
        nt = e - t0 < CH ? e - t0 : CH;
        return true;
    }
    const int lane = threadIdx.x & 63;
    int cc = 0;
    for (int i0 = 0; i0 < S; i0 += 64) {
        int b = 0, e = 0;
        if (i0 + lane < S) seg_bounds(seg, i0 + lane, n_tok, b, e);
        const int nc = (e - b + CH - 1) / CH;
        const int incl = wave_inclusive_sum(nc);
        const uint64_t past = __ballot(q < cc + incl);
        if (past != 0) {
            const int l = __builtin_ctzll(past);
            b = __builtin_amdgcn_readlane(b, l);
            e = __builtin_amdgcn_readlane(e, l);
            s = i0 + l;
            t0 = b + (q - cc - __builtin_amdgcn_readlane(incl - nc, l)) * CH;
            nt = e - t0 < CH ? e - t0 : CH;
            return true;
        }
        cc += __builtin_amdgcn_readlane(incl, 63);
    }
    return false;
}
// chunks [q0, q1) of set s, clamped to the nq_max chunks the launch covers (called by whole wavefronts)
template <int CH, bool FEW_SETS>
__device__ __forceinline__ void chunk_range(const int32_t* __restrict__ seg, int s, int n_tok, int nq_max,
                                            int& q0, int& q1) {
    int cc = 0;
    if constexpr (FEW_SETS) {
        int b, e;
        seg_bounds(seg, 0, n_tok, b, e);
        cc = s == 0 ? 0 : (e - b + CH - 1) / CH;
    } else {
        const int lane = threadIdx.x & 63;
        for (int i0 = 0; i0 < s; i0 += 64) {
            int b = 0, e = 0;
            if (i0 + lane < s) seg_bounds(seg, i0 + lane, n_tok, b, e);
            cc += __builtin_amdgcn_readlane(wave_inclusive_sum((e - b + CH - 1) / CH), 63);
        }
    }
    int b, e;
    seg_bounds(seg, s, n_tok, b, e);
    q0 = cc < nq_max ? cc : nq_max;
    q1 = cc + (e - b + CH - 1) / CH;
    q1 = q1 < nq_max ? q1 : nq_max;
}

__device__ __forceinline__ void unpack8s(const u32x4& v, float* f) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = bf16lo_to_f32(v[j]);
        f[2 * j + 1] = bf16hi_to_f32(v[j]);
    }
}

// The order of the selections: "DESCENDING ? larger first : smaller first", equal values (+0 and
// -0 are equal) ordered by index.  The order is total: a NaN comes after every number (NaNs among
// themselves by index), so exactly min(k, n) entries have rank < k whatever the values are.
// rank_key maps a value to an unsigned key that increases along that order (equal values share a key).
template <bool DESCENDING>
__device__ __forceinline__ uint32_t rank_key(float v) {
    if (v != v) return 0xFFFFFFFFu;
    uint32_t b = __float_as_uint(v);
    if (b == 0x80000000u) b = 0u;                               // -0 == +0
    // increasing with v; numbers (infinities included) map into [0x007FFFFF, 0xFF800000], and so does the
    // complement of that range, so 0xFFFFFFFF is left to the NaNs in both orders
    const uint32_t asc = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    return DESCENDING ? ~asc : asc;
}

__device__ __forceinline__ float block_sum256(float v, float* red) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

}  // namespace skipffn
