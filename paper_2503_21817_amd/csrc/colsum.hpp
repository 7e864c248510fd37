// Column sums of fp32 partial rows: out[c] (+)= sum_q part[q][c], for the gradients that leave a kernel as one row per
// workgroup.  32 columns (a 128-byte line per row) per workgroup, the rows dealt to 32 lanes, four loads in flight each;
// every lane sums its rows in order and the lanes are added in order, so the result does not vary.
//
// Bound by latency: C / 32 workgroups.  With 8 lanes and two loads in flight 11.5 us at 608 rows of 4096 and 21 us at
// 1200 rows; here 4.8 and 6.2 us.
#pragma once

#include "common.hpp"

namespace skipffn {

constexpr int COLSUM_LANES = 32;
constexpr int COLSUM_THREADS = 32 * COLSUM_LANES;

__device__ __forceinline__ void column_sum(const float* __restrict__ part, int rows, int C, float* __restrict__ out,
                                           int accumulate) {
    __shared__ float lanes[COLSUM_LANES][33];
    const int cx = threadIdx.x & 31, sy = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + cx;
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (c < C) {
        int q = sy;
        for (; q + 3 * COLSUM_LANES < rows; q += 4 * COLSUM_LANES)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] += part[(int64_t)(q + k * COLSUM_LANES) * C + c];
        for (; q < rows; q += COLSUM_LANES) a[0] += part[(int64_t)q * C + c];
    }
    lanes[sy][cx] = (a[0] + a[1]) + (a[2] + a[3]);
    __syncthreads();
    if (sy == 0 && c < C) {
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < COLSUM_LANES; ++k) v += lanes[k][cx];
        out[c] = accumulate ? out[c] + v : v;
    }
}

}  // namespace skipffn
