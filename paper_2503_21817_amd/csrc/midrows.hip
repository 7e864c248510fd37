// Kernels and launchers of the tiles of all rows (midrows.hpp).
#include "midrows.hpp"

namespace skipffn {

template <int MT, bool GATE_UP, bool NORM>
__global__ __launch_bounds__(SLAB_THREADS) void mid_rows_kernel(MidRowsArgs P) {
    mid_rows_tile<MT, GATE_UP, NORM, GATE_UP && !NORM && MT == 4>(P, (int)blockIdx.x);
}

// H = silu(sum_z gate) * sum_z up over the slabs of a split gate/up GEMM; one thread per 8 columns of a row, the
// slabs added in order, two of them in flight.
constexpr int SWIGLU_THREADS = 256;
__global__ __launch_bounds__(SWIGLU_THREADS) void swiglu_reduce_kernel(MidRowsArgs P) {
    const int R = effective_rows(P.rows, P.r_dev), chunks = P.N >> 3;
    const int64_t gid = (int64_t)blockIdx.x * SWIGLU_THREADS + threadIdx.x;
    const int r = (int)(gid / chunks), c = (int)(gid - (int64_t)r * chunks);
    if (r >= R) return;
    const float* p = P.partial + (int64_t)r * 2 * P.N + c * 8;
    const int64_t zstride = (int64_t)P.rows * 2 * P.N;
    float g[8], u[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) g[j] = u[j] = 0.0f;
    auto load = [&](int z, f32x4 (&v)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = *reinterpret_cast<const f32x4*>(p + z * zstride + (q >> 1) * P.N + (q & 1) * 4);
    };
    auto add = [&](const f32x4 (&v)[4]) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            g[j] += v[0][j]; g[4 + j] += v[1][j];
            u[j] += v[2][j]; u[4 + j] += v[3][j];
        }
    };
    int z = 0;
    for (; z + 2 <= P.splits; z += 2) {
        f32x4 a[4], b[4];
        load(z, a);
        load(z + 1, b);
        add(a);
        add(b);
    }
    if (z < P.splits) {
        f32x4 a[4];
        load(z, a);
        add(a);
    }
    u32x4 h, gb, ub;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float g0 = g[2 * k], g1 = g[2 * k + 1], u0 = u[2 * k], u1 = u[2 * k + 1];
        h[k] = pack_bf16x2(g0 * sigmoid_f(g0) * u0, g1 * sigmoid_f(g1) * u1);
        gb[k] = pack_bf16x2(g0, g1);
        ub[k] = pack_bf16x2(u0, u1);
    }
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(P.H) + (uint32_t)r * P.h_row + (uint32_t)c * P.h_chunk) = h;
    if (P.G != nullptr) {
        const int64_t o = (int64_t)r * P.N + c * 8;
        *reinterpret_cast<u32x4*>(P.G + o) = gb;
        *reinterpret_cast<u32x4*>(P.U + o) = ub;
    }
}

template <int MT, bool GATE_UP, bool NORM = false>
static hipError_t launch_mid(const MidRowsArgs& a, hipStream_t s) {
    const int tiles_m = (a.rows + 16 * MT - 1) / (16 * MT), cols = GATE_UP ? a.cols : SLAB_B_ROWS;
    const int tiles_n = (a.N + cols - 1) / cols;
    hipLaunchKernelGGL((mid_rows_kernel<MT, GATE_UP, NORM>), dim3((unsigned)(tiles_m * tiles_n * a.splits)), dim3(SLAB_THREADS),
                       kSlabLds<16 * MT>, s, a);
    return hipGetLastError();
}
template <bool GATE_UP>
static hipError_t launch_mid_rows(const MidRowsArgs& a, hipStream_t s) {
    if (a.rows <= 0 || a.N <= 0) return hipSuccess;
    // as few row tiles as 256 rows allow, and those no taller than they have to be
    const int tiles_m = mid_row_tiles(a.rows), per = (a.rows + tiles_m - 1) / tiles_m;
    if (per <= 64) return launch_mid<4, GATE_UP>(a, s);
    if (per <= 128) return launch_mid<8, GATE_UP>(a, s);
    if (per <= 192) return launch_mid<12, GATE_UP>(a, s);
    return launch_mid<16, GATE_UP>(a, s);
}

template <int MT, bool GATE_UP, bool NORM = false>
static hipError_t mid_lds_limit() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&mid_rows_kernel<MT, GATE_UP, NORM>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSlabLds<16 * MT>);
}
hipError_t mid_rows_init() {
    hipError_t e;
    if ((e = mid_lds_limit<4, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<4, true, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<4, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<8, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<8, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<12, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<12, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<16, true>()) != hipSuccess) return e;
    return mid_lds_limit<16, false>();
}

MidRowsArgs mid_rows_gate_up_args(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                  const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major_h, int cols) {
    MidRowsArgs a{};
    a.rows = rows; a.r_dev = r_dev; a.N = I; a.K = C;
    a.A = xn; a.a_bytes = (uint32_t)((int64_t)rows * C * 2);
    a.B0 = w_gate; a.B1 = w_up; a.b_bytes = (uint32_t)((int64_t)I * C * 2);
    a.splits = 1; a.cols = cols; a.H = H; a.G = G; a.U = U;
    a.h_row = chunk_major_h ? 16u : (uint32_t)I * 2; a.h_chunk = chunk_major_h ? (uint32_t)rows * 16 : 16u;
    return a;
}
MidRowsArgs mid_rows_down_args(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down, int splits,
                               float* partial) {
    MidRowsArgs a{};
    a.rows = rows; a.r_dev = r_dev; a.N = C; a.K = I;
    a.A = H; a.a_bytes = (uint32_t)((int64_t)rows * I * 2);
    a.B0 = w_down; a.b_bytes = (uint32_t)((int64_t)C * I * 2);
    a.splits = splits; a.partial = partial;
    return a;
}

hipError_t launch_mid_rows_gate_up(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                   const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major_h, int splits,
                                   int cols, float* partial, const RowNorm* norm, const float* rstd, hipStream_t s) {
    MidRowsArgs a = mid_rows_gate_up_args(xn, rows, r_dev, C, I, w_gate, w_up, H, G, U, chunk_major_h, cols);
    a.splits = splits; a.partial = partial; a.rstd = rstd;
    if (rstd != nullptr && (rows > kNormInMidRows || splits > 1)) return hipErrorInvalidValue;
    if (norm != nullptr) {                    // one row tile; a part of K would not know a row's norm
        if (rows > kNormInMidRows || splits > 1 || norm->gain != nullptr) return hipErrorInvalidValue;
        a.A = norm->hidden; a.a_bytes = (uint32_t)(norm->T * C * 2);
        a.idx = norm->idx; a.eps = norm->eps;
        return rows <= 0 || I <= 0 ? hipSuccess : launch_mid<4, true, true>(a, s);
    }
    const hipError_t e = launch_mid_rows<true>(a, s);
    if (e != hipSuccess || splits <= 1 || rows <= 0) return e;
    const int64_t threads = (int64_t)rows * (I >> 3);
    hipLaunchKernelGGL(swiglu_reduce_kernel, dim3((unsigned)((threads + SWIGLU_THREADS - 1) / SWIGLU_THREADS)),
                       dim3(SWIGLU_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_mid_rows_down(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down,
                                int splits, float* partial, hipStream_t s) {
    return launch_mid_rows<false>(mid_rows_down_args(H, rows, r_dev, C, I, w_down, splits, partial), s);
}

}  // namespace skipffn
