// Column sums of fp32 partial rows: out[c] (+)= sum_q part[q][c], for the gradients that leave a kernel as one row per
// workgroup.  32 columns (a 128-byte line per row) per workgroup, the rows dealt to LANES lanes, four loads in flight
// each; every lane sums its rows in order and the lanes are added in order, so the result does not vary.
//
// Bound by latency: C / 32 workgroups.  With 8 lanes and two loads in flight 11.5 us at 608 rows of 4096 and 21 us at
// 1200 rows; with 32 lanes 4.8 and 6.2 us.  Up to 32 rows 8 lanes have one round of loads as well, and the workgroup is
// a quarter of the size: 0.3 us less at 9 rows of 4096 (0.6 us more at 60 rows).
#pragma once

#include "common.hpp"

namespace skipffn {

constexpr int COLSUM_LANES = 32, COLSUM_LANES_FEW = 8;
constexpr int COLSUM_FEW_ROWS = 32;           // up to here COLSUM_LANES_FEW

template <int LANES>
__device__ __forceinline__ void column_sum(const float* __restrict__ part, int rows, int C, float* __restrict__ out,
                                           int accumulate) {
    __shared__ float lanes[LANES][33];
    const int cx = threadIdx.x & 31, sy = threadIdx.x >> 5;
    const int c = blockIdx.x * 32 + cx;
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (c < C) {
        int q = sy;
        for (; q + 3 * LANES < rows; q += 4 * LANES)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] += part[(int64_t)(q + k * LANES) * C + c];
        for (; q < rows; q += LANES) a[0] += part[(int64_t)q * C + c];
    }
    lanes[sy][cx] = (a[0] + a[1]) + (a[2] + a[3]);
    __syncthreads();
    if (sy == 0 && c < C) {
        float v = 0.0f;
#pragma unroll
        for (int k = 0; k < LANES; ++k) v += lanes[k][cx];
        out[c] = accumulate ? out[c] + v : v;
    }
}

}  // namespace skipffn
