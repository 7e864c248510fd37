// The forward GEMMs of a layer whose row count is on the device, far below its bound as a rule (the bound is the number of
// tokens, the count that of the retained ones).  The host can plan for the bound only: these kernels hold the paths of all counts
// and take the one that the count wants: tiles of all rows up to 256 (also of a handful, which a call with the count on the host
// would run on registers), lists of tiles or the balanced split beyond.  Everything about a path stands where it is
// (midrows.hpp, stream.hpp); the reducing kernel reads the same plans (rowops.hip).
//
// Gate/up of more than 16384 columns or so is more tiles of all rows than the chip holds at once, and from 129 rows their second round costs more
// than tiles of 128 rows that read the weights twice.  Layer forward, us, tiles of all rows / lists:  C = 5120, I = 20480: 154 rows 200 / 183,
// 250 rows 247 / 220;  C = 4096, I = 17408: 154 rows 137 / 130, 250 rows 169 / 152;  C = 1024, I = 24576, 200 rows 77 / 71;
// up to 128 rows (100, C = 5120, I = 20480) the tiles of all rows take 165, the bound's plan 179.
//
// One kernel for all paths, although the longer ones set its registers (the arguments of all paths are loaded at the start and
// some spill, outside the loops): a kernel for each, of which all but one leave at once, cost 4.5 us an idle launch.  The
// arguments are read only: a field assigned here moves the whole structure to vector registers (640 rows 20 % slower).
//
// C = 4096, I = 14336, us a layer's gate/up, down and reduction, plan of the bound / of the count:  bound 2944 rows, 640
// retained 133 + 83 + 13 / 133 + 70 + 12;  bound 616, 184 retained 67 + 50 + 5 / 57 + 38 + 7;  bound 3080, 1600 retained 289
// + 207 / 291 + 152 + 16.
#include <algorithm>

#include "midrows.hpp"
#include "stream.hpp"

namespace skipffn {

// up to 256 rows
template <bool GATE_UP>
__device__ __forceinline__ void mid_rows_of_count(const MidRowsArgs& M, const int rows, const int block) {
    if (rows <= 64) mid_rows_tile<4, GATE_UP>(M, block);
    else if (rows <= 128) mid_rows_tile<8, GATE_UP>(M, block);
    else if (rows <= 192) mid_rows_tile<12, GATE_UP>(M, block);
    else mid_rows_tile<16, GATE_UP>(M, block);
}

// lists: workgroups that run lists of tiles; mid: workgroups of the tiles of all rows, which take up to MID_MAX rows (a constant: as an
// argument, or by a comparison of these two, 1 to 2 % on every count, in scalar registers that spill)
template <int MID_MAX>
__global__ __launch_bounds__(GEMM_THREADS) void gate_up_count_kernel(GemmArgs P, MidRowsArgs M, int lists, int mid) {
    const int rows = uniform(effective_rows(P.M, P.m_dev)), block = (int)blockIdx.x;
    if (rows <= MID_MAX) {
        if (block < mid) mid_rows_of_count<true>(M, rows, block);
    } else if (block < lists) {
        stream_rows<EPI_SWIGLU>(P, stream_plan_of_count<EPI_SWIGLU>(P, 1, lists), 1, block, lists);
    }
}
__global__ __launch_bounds__(GEMM_THREADS) void down_count_kernel(GemmArgs P, MidRowsArgs M, RowPlans plans, int lists, int mid) {
    const int rows = uniform(effective_rows(P.M, P.m_dev)), block = (int)blockIdx.x;
    if (rows <= 256) {
        if (block < mid) mid_rows_of_count<false>(M, rows, block);
        return;
    }
    const KPartition k = row_plan(plans, (rows + BM - 1) / BM);
    const int nbg = uniform(k.sk_nbg), splits = uniform(k.splits);
    if (nbg > 0) {
        if (block < P.tiles_n * nbg) stream_balanced(P, block, P.tiles_n, nbg);
    } else if (block < lists) {
        if (splits > 1) stream_rows<EPI_PARTIAL>(P, stream_plan_of_count<EPI_PARTIAL>(P, splits, lists), splits, block, lists);
        else stream_rows<EPI_RESID_SCATTER>(P, stream_plan_of_count<EPI_RESID_SCATTER>(P, 1, lists), 1, block, lists);
    }
}

hipError_t count_rows_init() {
    const void* kernels[] = {reinterpret_cast<const void*>(&gate_up_count_kernel<256>), reinterpret_cast<const void*>(&gate_up_count_kernel<128>),
                             reinterpret_cast<const void*>(&down_count_kernel)};
    for (const void* k : kernels) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS_BYTES);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
static_assert(kSlabLds<64> <= GEMM_LDS_BYTES && kSlabLds<128> <= GEMM_LDS_BYTES && kSlabLds<192> <= GEMM_LDS_BYTES &&
              kSlabLds<256> <= GEMM_LDS_BYTES, "the rings of all paths fit");

static int list_workgroups(const GemmArgs& a) { return a.ncu >= 8 ? a.ncu / 8 * 8 : 8; }

hipError_t launch_gate_up_count(GemmArgs& a, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if (a.m_dev == nullptr || a.out1 != nullptr) return hipErrorInvalidValue;
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN / 2 - 1) / (BN / 2);
    a.splits = a.batch = 1;
    const MidRowsArgs m = mid_rows_gate_up_args(a.A0, a.M, a.m_dev, a.K, a.N, a.B0, a.B1, static_cast<bf16_t*>(a.out0), nullptr,
                                                nullptr, false, gate_up_cols(256, a.N, a.ncu));
    const int lists = list_workgroups(a), mid = (a.N + m.cols - 1) / m.cols;
    const auto kernel = mid <= a.ncu ? &gate_up_count_kernel<256> : &gate_up_count_kernel<128>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)std::max(lists, mid)), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a, m, lists, mid);
    return hipGetLastError();
}

hipError_t launch_down_count(GemmArgs& a, const RowPlans& plans, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if (a.m_dev == nullptr || plans.mid_splits < 1) return hipErrorInvalidValue;
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN - 1) / BN;
    a.batch = 1;
    const MidRowsArgs m = mid_rows_down_args(a.A0, 256, a.m_dev, a.N, a.K, a.B0, plans.mid_splits, a.partial);
    const int lists = list_workgroups(a), mid = (a.N + SLAB_B_ROWS - 1) / SLAB_B_ROWS * plans.mid_splits;
    int blocks = std::max(lists, mid);
    const int kt = std::max((a.K + BK - 1) / BK, 1);
    for (int t = 2; t <= a.tiles_m; ++t) {
        const KPartition k = row_plan(plans, t);
        blocks = std::max(blocks, a.tiles_n * k.sk_nbg);
        // a part of K without slabs would end a list of tiles
        if (k.sk_nbg == 0 && (k.splits < 1 || (k.splits - 1) * ((kt + k.splits - 1) / k.splits) >= kt)) return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(down_count_kernel, dim3((unsigned)blocks), dim3(GEMM_THREADS), GEMM_LDS_BYTES, s, a, m, plans, lists, mid);
    return hipGetLastError();
}

}  // namespace skipffn
