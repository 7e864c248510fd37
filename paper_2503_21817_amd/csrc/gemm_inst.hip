// Instantiations and launcher of the bf16 MFMA GEMM core.
#include <algorithm>

#include "kernels.hpp"
#include "stream.hpp"

namespace skipffn {

// dH with the SwiGLU backward in its epilogue and dW_down, which depend on each other in nothing, in one grid: workgroups
// [0, n0) run a tile of dH each (the longer ones, dispatched first), the rest lists of tiles of dW_down, so the last round
// of one fills with work of the other.  n0 is a multiple of 8 (workgroups past the tiles leave at once): both problems see the
// round-robin XCD assignment from its start.  dW_down as a stream, sums stored from registers, us a launch before / after:
// 368 rows 126 / 122, 640 rows 177 / 172, 2944 rows 604 / 590, 4096 rows 811 / 805.
__global__ __launch_bounds__(GEMM_THREADS) void gemm_dh_dw_down_kernel(GemmArgs P0, GemmArgs P1, int n0) {
    const int b = (int)blockIdx.x;
    if (b < n0)
        gemm_block<true, false, EPI_SWIGLU_BWD>(P0, b);
    else
        stream_tall<EPI_STORE>(P1, b - n0, (int)gridDim.x - n0);
}

template <bool A_KC, bool B_KC, int EPI>
static hipError_t set_lds_limit() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_kernel<A_KC, B_KC, EPI>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS_BYTES);
}

static hipError_t set_stream_lds(void (*kernel)(GemmArgs)) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kStreamLds);
}

hipError_t gemm_init() {
    hipError_t e;
    if ((e = set_stream_lds(&stream_gemm_kernel<EPI_STORE>)) != hipSuccess) return e;
    if ((e = set_stream_lds(&stream_gemm_rows_kernel<EPI_SWIGLU>)) != hipSuccess) return e;
    if ((e = set_stream_lds(&stream_gemm_kernel<EPI_PARTIAL>)) != hipSuccess) return e;
    if ((e = set_stream_lds(&stream_gemm_kernel<EPI_RESID_SCATTER>)) != hipSuccess) return e;
    if ((e = set_stream_lds(&stream_gemm_balanced_kernel)) != hipSuccess) return e;
    if ((e = set_lds_limit<true, false, EPI_PARTIAL>()) != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_bf16_streamk_kernel<true, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS_BYTES);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_dh_dw_down_kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS_BYTES);
    if (e != hipSuccess) return e;
    return hipSuccess;
}

static void finish_args(int epi, GemmArgs& a) {
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = epi == EPI_SWIGLU ? (a.N + BN / 2 - 1) / (BN / 2) : (a.N + BN - 1) / BN;
    if (a.splits < 1) a.splits = 1;
    if (a.batch < 1) a.batch = 1;
    // a last tile row of at most 128 rows runs on 128-row tiles (one workgroup per tile: the gate/up GEMM);
    // the kernel looks at the effective row count
    a.tail_narrow = (epi == EPI_SWIGLU && a.splits == 1 && a.batch == 1) ? 1 : 0;
}
// workgroups of a one-tile-per-workgroup launch
static unsigned grid_blocks(const GemmArgs& a) { return (unsigned)(a.tiles_m * a.tiles_n * a.splits * a.batch); }

template <bool A_KC, bool B_KC, int EPI>
static hipError_t launch_one(const GemmArgs& a, hipStream_t s) {
    const unsigned blocks = grid_blocks(a);
    hipLaunchKernelGGL((gemm_bf16_kernel<A_KC, B_KC, EPI>), dim3(blocks), dim3(GEMM_THREADS),
                       GEMM_LDS_BYTES, s, a);
    return hipGetLastError();
}

// One workgroup per CU, a multiple of the 8 XCDs; fewer where the tiles, counted at their smallest height, are fewer
template <int EPI>
static hipError_t launch_stream(void (*kernel)(GemmArgs), const GemmArgs& a, hipStream_t s) {
    const int height = EPI == EPI_SWIGLU ? 128 : 256;
    const unsigned cus = (unsigned)(a.ncu >= 8 ? a.ncu / 8 * 8 : 8);
    const unsigned tiles = ((unsigned)((a.M + height - 1) / height * a.tiles_n * a.splits * a.batch) + 7) / 8 * 8;
    hipLaunchKernelGGL(kernel, dim3(tiles < cus ? tiles : cus), dim3(GEMM_THREADS), kStreamLds, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm_dual(int which, GemmArgs& a0, GemmArgs& a1, hipStream_t s) {
    if (which != DUAL_DH_DWDOWN) return hipErrorInvalidValue;
    finish_args(EPI_SWIGLU_BWD, a0);
    finish_args(EPI_STORE, a1);
    const int real0 = (int)grid_blocks(a0), n0 = (real0 + 7) / 8 * 8, tiles1 = (int)grid_blocks(a1);
    if (real0 <= 0 || tiles1 <= 0) return hipErrorInvalidValue;
    // lists of about 16 slabs (of short tiles several, whose ends overlap; no longer: they also even out the end of the
    // grid), and no fewer lists than compute units
    const int slabs = std::max((a1.K + BK - 1) / BK, 1), per = std::max(std::min(16 / slabs, tiles1 / std::max(a1.ncu, 1)), 1);
    const int n1 = ((tiles1 + per - 1) / per + 7) / 8 * 8;
    hipLaunchKernelGGL(gemm_dh_dw_down_kernel, dim3((unsigned)(n0 + n1)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a0, a1, n0);
    return hipGetLastError();
}

hipError_t launch_gemm_streamk(bool a_kc, bool b_kc, GemmArgs& a, int nbg, hipStream_t s) {
    finish_args(EPI_PARTIAL, a);
    if (a.tiles_m <= 0 || a.tiles_n <= 0) return hipSuccess;
    if (nbg < 1 || !a_kc || a.batch != 1) return hipErrorInvalidValue;
    a.splits = nbg;
    const unsigned blocks = (unsigned)(a.tiles_n * nbg);
    if (b_kc)
        hipLaunchKernelGGL(stream_gemm_balanced_kernel, dim3(blocks), dim3(GEMM_THREADS), kStreamLds, s, a);
    else
        hipLaunchKernelGGL((gemm_bf16_streamk_kernel<true, false>), dim3(blocks), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm(bool a_kc, bool b_kc, int epi, GemmArgs& a, hipStream_t s) {
    finish_args(epi, a);
    if (grid_blocks(a) == 0 || a.tiles_n <= 0) return hipSuccess;
    if (a_kc && b_kc && epi == EPI_SWIGLU) return launch_stream<EPI_SWIGLU>(&stream_gemm_rows_kernel<EPI_SWIGLU>, a, s);
    if (a_kc && b_kc && epi == EPI_PARTIAL) return launch_stream<EPI_PARTIAL>(&stream_gemm_kernel<EPI_PARTIAL>, a, s);
    if (a_kc && b_kc && epi == EPI_RESID_SCATTER) return launch_stream<EPI_RESID_SCATTER>(&stream_gemm_kernel<EPI_RESID_SCATTER>, a, s);
    if (a_kc && b_kc && epi == EPI_STORE) return launch_stream<EPI_STORE>(&stream_gemm_kernel<EPI_STORE>, a, s);
    if (a_kc && !b_kc && epi == EPI_PARTIAL) return launch_one<true, false, EPI_PARTIAL>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace skipffn
