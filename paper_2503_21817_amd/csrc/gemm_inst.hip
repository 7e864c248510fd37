// Kernels and launchers of the bf16 MFMA GEMM core.
#include <algorithm>

#include "kernels.hpp"
#include "stream.hpp"

namespace skipffn {

__global__ __launch_bounds__(GEMM_THREADS) void gemm_bf16_kernel(GemmArgs P) {
    gemm_block<EPI_PARTIAL>(P, (int)blockIdx.x);
}

// the balanced split with two K-contiguous operands: grid = tiles_n * nbg workgroups (P.splits carries nbg)
__global__ __launch_bounds__(GEMM_THREADS) void stream_gemm_balanced_kernel(GemmArgs P) {
    stream_balanced(P, (int)blockIdx.x, (int)gridDim.x / P.splits, P.splits);
}

// ---- balanced split-K for GEMMs that leave through fp32 partial slabs (see streamk.hpp) ------
// grid = tiles_n * nbg workgroups (P.splits carries nbg); EPI_PARTIAL only
__global__ __launch_bounds__(GEMM_THREADS) void gemm_bf16_streamk_kernel(GemmArgs P) {
    const int nbg = P.splits, tiles_n = (int)gridDim.x / nbg;
    const int Meff = effective_rows(P.M, P.m_dev);
    const int Keff = effective_rows(P.K, P.k_dev);
    const int g = (Meff + BM - 1) / BM;
    const int kt = ((Keff + BK - 1) / BK) * P.pairs;
    if (g == 0 || kt == 0) return;
    const StreamKPlan p = streamk_plan(g, kt, nbg);
    int tn, j;
    balanced_share(p, tiles_n, (int)blockIdx.x, tn, j);
    StreamKIter it = streamk_begin(p, j);
    StreamKSeg sg;
    bool first = true;
    while (streamk_next(p, it, sg)) {      // uniform over the workgroup
        if (!first) lds_barrier();          // the staging buffers of the previous epilogue are free again
        first = false;
        gemm_tile<EPI_PARTIAL>(P, sg.i, tn, sg.slot, sg.kb, sg.ke, Meff, Keff);
    }
}

// dH with the SwiGLU backward in its epilogue and dW_down, which depend on each other in nothing, in one grid: workgroups
// [0, n0) run a tile of dH each (the longer ones, dispatched first), the rest lists of tiles of dW_down, so the last round
// of one fills with work of the other.  n0 is a multiple of 8 (workgroups past the tiles leave at once): both problems see the
// round-robin XCD assignment from its start.  dW_down as a stream, sums stored from registers, us a launch before / after:
// 368 rows 120 / 120, 640 rows 165 / 160, 2944 rows 609 / 598, 4096 rows 792 / 791.
__global__ __launch_bounds__(GEMM_THREADS) void gemm_dh_dw_down_kernel(GemmArgs P0, GemmArgs P1, int n0) {
    const int b = (int)blockIdx.x;
    if (b < n0)
        gemm_block<EPI_SWIGLU_BWD>(P0, b);
    else
        stream_tall<EPI_STORE>(P1, b - n0, (int)gridDim.x - n0);
}

// A GEMM into fp32 slabs (dXn, dH; K cut evenly) and weight gradients in one grid: workgroups [0, n0) run the first, the others
// lists of tiles of the second.
__global__ __launch_bounds__(GEMM_THREADS) void gemm_partial_dw_kernel(GemmArgs P0, GemmArgs P1, int n0) {
    const int b = (int)blockIdx.x;
    if (b < n0)
        gemm_block<EPI_PARTIAL>(P0, b);
    else
        stream_tall<EPI_STORE>(P1, b - n0, (int)gridDim.x - n0);
}

template <class... Args>
static hipError_t set_lds(void (*kernel)(Args...)) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS_BYTES);
}

hipError_t gemm_init() {
    hipError_t e;
    if ((e = set_lds(&stream_gemm_kernel<EPI_STORE>)) != hipSuccess) return e;
    if ((e = set_lds(&stream_gemm_rows_kernel<EPI_SWIGLU>)) != hipSuccess) return e;
    if ((e = set_lds(&stream_gemm_rows_kernel<EPI_PARTIAL>)) != hipSuccess) return e;
    if ((e = set_lds(&stream_gemm_rows_kernel<EPI_RESID_SCATTER>)) != hipSuccess) return e;
    if ((e = set_lds(&stream_gemm_balanced_kernel)) != hipSuccess) return e;
    if ((e = set_lds(&gemm_bf16_kernel)) != hipSuccess) return e;
    if ((e = set_lds(&gemm_bf16_streamk_kernel)) != hipSuccess) return e;
    if ((e = set_lds(&gemm_partial_dw_kernel)) != hipSuccess) return e;
    return set_lds(&gemm_dh_dw_down_kernel);
}

static void finish_args(int epi, GemmArgs& a) {
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = epi == EPI_SWIGLU ? (a.N + BN / 2 - 1) / (BN / 2) : (a.N + BN - 1) / BN;
    if (a.splits < 1) a.splits = 1;
    if (a.batch < 1) a.batch = 1;
}
// workgroups of a one-tile-per-workgroup launch
static unsigned grid_blocks(const GemmArgs& a) { return (unsigned)(a.tiles_m * a.tiles_n * a.splits * a.batch); }

// One workgroup per CU, a multiple of the 8 XCDs; fewer where the tiles, counted at their smallest height, are fewer
template <int EPI>
static unsigned stream_workgroups(const GemmArgs& a) {
    const int height = EPI == EPI_STORE ? 256 : 128;
    const unsigned cus = (unsigned)(a.ncu >= 8 ? a.ncu / 8 * 8 : 8);
    const unsigned tiles = ((unsigned)((a.M + height - 1) / height * a.tiles_n * a.splits * a.batch) + 7) / 8 * 8;
    return tiles < cus ? tiles : cus;
}
// Tiles by the row count, planned here where the host knows it: some twenty divisions, 2-3 us at the start of every workgroup.
// Layer forward, us, planned on the device / here:  C = 1024, I = 3584: 1200 rows 53.8 / 51.1;  C = 2048, I = 7168: 640 rows 73.6 /
// 70.7, 1472 rows 137.0 / 134.4;  C = 4096, I = 14336: 300 rows 132.8 / 129.9, 1472 rows 406.3 / 405.6.  (A kernel for each height
// was no faster than that.)
template <int EPI>
static hipError_t launch_stream_rows(const GemmArgs& a, hipStream_t s) {
    const unsigned workgroups = stream_workgroups<EPI>(a);
    StreamRows plan{0, 0};
    if (a.m_dev == nullptr && a.k_dev == nullptr) {
        const int slabs = ((a.K + BK - 1) / BK + a.splits - 1) / a.splits;
        plan = stream_rows_plan(a.M, a.tiles_n * a.splits, slabs, (int)workgroups, a.outT0 != nullptr, EPI == EPI_SWIGLU);
    }
    hipLaunchKernelGGL(stream_gemm_rows_kernel<EPI>, dim3(workgroups), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a, plan);
    return hipGetLastError();
}

// workgroups of dW_down beside dH: lists of about 16 slabs (of short tiles several, whose ends overlap; no longer: they also even
// out the end of the grid), and no fewer lists than compute units
static int dw_down_lists(const GemmArgs& a) {
    const int tiles = (int)grid_blocks(a), slabs = std::max((a.K + BK - 1) / BK, 1);
    const int per = std::max(std::min(16 / slabs, tiles / std::max(a.ncu, 1)), 1);
    return ((tiles + per - 1) / per + 7) / 8 * 8;
}
hipError_t launch_gemm_dh_dw_down(GemmArgs& a0, GemmArgs& a1, hipStream_t s) {
    finish_args(EPI_SWIGLU_BWD, a0);
    finish_args(EPI_STORE, a1);
    const int real0 = (int)grid_blocks(a0), n0 = (real0 + 7) / 8 * 8, tiles1 = (int)grid_blocks(a1);
    if (real0 <= 0 || tiles1 <= 0) return hipErrorInvalidValue;
    const int n1 = dw_down_lists(a1);
    hipLaunchKernelGGL(gemm_dh_dw_down_kernel, dim3((unsigned)(n0 + n1)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a0, a1, n0);
    return hipGetLastError();
}

hipError_t launch_gemm_partial_dw(GemmArgs& a0, GemmArgs& a1, int n0, int n1, hipStream_t s) {
    finish_args(EPI_PARTIAL, a0);
    finish_args(EPI_STORE, a1);
    if (grid_blocks(a0) == 0 || grid_blocks(a1) == 0) return hipErrorInvalidValue;
    if (n0 % 8 != 0 || (unsigned)n0 < grid_blocks(a0) || n1 < 8 || n1 % 8 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_partial_dw_kernel, dim3((unsigned)(n0 + n1)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a0, a1, n0);
    return hipGetLastError();
}

hipError_t launch_gemm_dh_partial_dw_down(GemmArgs& a0, GemmArgs& a1, hipStream_t s) {
    finish_args(EPI_PARTIAL, a0);
    finish_args(EPI_STORE, a1);
    return launch_gemm_partial_dw(a0, a1, (int)((grid_blocks(a0) + 7) / 8 * 8), dw_down_lists(a1), s);
}

hipError_t launch_gemm_streamk(bool b_kc, GemmArgs& a, int nbg, hipStream_t s) {
    finish_args(EPI_PARTIAL, a);
    if (a.tiles_m <= 0 || a.tiles_n <= 0) return hipSuccess;
    if (nbg < 1 || a.batch != 1 || (b_kc && a.pairs != 1)) return hipErrorInvalidValue;
    a.splits = nbg;
    const unsigned blocks = (unsigned)(a.tiles_n * nbg);
    if (b_kc)
        hipLaunchKernelGGL(stream_gemm_balanced_kernel, dim3(blocks), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a);
    else
        hipLaunchKernelGGL(gemm_bf16_streamk_kernel, dim3(blocks), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a);
    return hipGetLastError();
}

hipError_t launch_gemm(bool b_kc, int epi, GemmArgs& a, hipStream_t s) {
    finish_args(epi, a);
    if (grid_blocks(a) == 0 || a.tiles_n <= 0) return hipSuccess;
    if (b_kc && a.pairs != 1) return hipErrorInvalidValue;
    const int kt = std::max((a.K + BK - 1) / BK, 1);         // a part of K without slabs would end a list of tiles
    if (b_kc && (a.splits - 1) * ((kt + a.splits - 1) / a.splits) >= kt) return hipErrorInvalidValue;
    if (b_kc && epi == EPI_SWIGLU) return launch_stream_rows<EPI_SWIGLU>(a, s);
    if (b_kc && epi == EPI_PARTIAL) return launch_stream_rows<EPI_PARTIAL>(a, s);
    if (b_kc && epi == EPI_RESID_SCATTER) return launch_stream_rows<EPI_RESID_SCATTER>(a, s);
    if (b_kc && epi == EPI_STORE) {
        hipLaunchKernelGGL(stream_gemm_kernel<EPI_STORE>, dim3(stream_workgroups<EPI_STORE>(a)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a);
        return hipGetLastError();
    }
    if (b_kc || epi != EPI_PARTIAL || a.batch != 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_bf16_kernel, dim3(grid_blocks(a)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a);
    return hipGetLastError();
}

}  // namespace skipffn
