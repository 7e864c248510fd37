// The two forward GEMMs for a handful of retained rows (decode steps, very short prompts): all rows against
// every weight of the layer, so the time is that of streaming the weights from HBM once.
//
// One workgroup owns 16 output columns (16 rows of W_gate and the same 16 of W_up, or 16 rows of W_down)
// and ALL of K, cut over its wavefronts; the wavefronts' sums meet in LDS, so the epilogue sees complete sums and
// nothing goes through fp32 slabs in memory.  Weights go from HBM straight to the MFMA operand registers (a
// K-contiguous fragment is 16 bytes per lane): no LDS stage and no barrier in the loop, only loads.  The source asks for FR_UNROLL
// k-steps in flight per wavefront; with the norm inside, the compiler keeps them (98 to 212 registers), without it gate/up's
// loads sink to their uses (34 to 48 registers), so what the two forms differ by is in part this.
//
// The activations are the same for every workgroup and come from L2, which is what grows with the rows: they
// lie chunk-major ([K / 8][rows][8]) where no caller reads them, so that a load is one contiguous piece (row-major,
// 16 rows x 64 bytes at a stride of K: 89 against 81 us a layer at 8 rows, 102 against 87 at 16); lanes of absent
// rows are out of range and cost nothing.  More columns per workgroup (32, 64) would read them less
// often, but leave fewer workgroups: no faster below 32 rows, up to 60 % slower at C = 2048.
//
// Measured at C = 4096, I = 14336, 8 rows: down 24.6 us (4.8 TB/s of weights; the loads alone, without activations and
// epilogue, 21), where tiles with split K take 25.8 + 5.5 for the reduction; gate/up 48.6, slower than the tiles of
// midrows.hip (42), which read the activations once per 64 columns.  Which layers and row counts come here, each GEMM for
// itself: layout.hpp.
#include "kernels.hpp"

namespace skipffn {

constexpr int FR_COLS = 16;                   // output columns per workgroup
constexpr int FR_UNROLL = 8;                  // k-steps of 32 loaded together
// RMSNorm of the rows beside their product: no, x * rstd, x * gain * rstd
enum FewNorm : int { NORM_NONE = 0, NORM_PLAIN = 1, NORM_GAIN = 2 };
constexpr int FR_WAVES_GU = 4, FR_WAVES_DOWN = 8;      // wavefronts that share K

struct FewRowsArgs {
    int rows; const int32_t* r_dev;           // row bound, optional device count
    int N, K;                                 // output columns, contraction length (multiples of 8)
    // activations: 16-byte chunk c (8 k) of row r at byte r * a_row + c * a_chunk
    const bf16_t* A; uint32_t a_bytes, a_row, a_chunk;
    const bf16_t* B0; const bf16_t* B1; uint32_t b_bytes;   // [N][K]; B1 = W_up
    // gate/up: H as A with strides h_row, h_chunk; G, U [rows][N], optional
    bf16_t* H; uint32_t h_row, h_chunk; bf16_t* G; bf16_t* U;
    const int32_t* idx; const bf16_t* res; bf16_t* out; int no_residual;   // down: res, out [T][N]
    const bf16_t* gain; float eps;            // gate/up that normalises its rows itself: A = hidden [T][K], rows idx
    const float* rstd;                        // gate/up, optional: A holds rows that are yet to be multiplied by this, 1 / rms of each
};

template <int MT, int WAVES, bool GATE_UP, int NORM>
__global__ __launch_bounds__(WAVES * 64) void few_rows_kernel(FewRowsArgs P) {
    constexpr int NW = GATE_UP ? 2 : 1;       // weight matrices
    static_assert(MT <= WAVES, "a wavefront of the epilogue per 16 rows");
    __shared__ f32x4 red[WAVES][NW * MT][64];
    __shared__ float red_ss[NORM != NORM_NONE ? WAVES : 1][MT][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int R = effective_rows(P.rows, P.r_dev);
    if (R <= 0) return;                       // uniform
    const int n0 = blockIdx.x * FR_COLS;
    const int r16 = lane & 15, kq = lane >> 4;           // row of the fragment, the lane's chunk of 8 k

    // results of the epilogue threads: row em, columns en .. en + 3
    const int em = wave * 16 + r16, en = n0 + 4 * kq;
    const bool mine = wave < MT && em < R && en < P.N;
    const int irow = !GATE_UP && mine ? P.idx[em] : 0;
    float rstd = 1.0f;
    if (GATE_UP && NORM == NORM_NONE && P.rstd != nullptr && mine) rstd = P.rstd[em];

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(P.A, P.a_bytes), rb0 = make_rsrc(P.B0, P.b_bytes),
                                 rb1 = make_rsrc(GATE_UP ? P.B1 : P.B0, P.b_bytes);
    const uint32_t b_off = n0 + r16 < P.N ? (uint32_t)(((int64_t)(n0 + r16) * P.K + kq * 8) * 2) : kOobOffset;
    uint32_t a_off[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = m * 16 + r16;
        a_off[m] = row < R ? (uint32_t)(NORM != NORM_NONE ? P.idx[row] : row) * P.a_row + (uint32_t)kq * P.a_chunk : kOobOffset;
    }
    const uint32_t a_step = 4 * P.a_chunk;

    f32x4 acc[NW][MT];
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[w][m] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float ss[MT];                             // squares of the lane's k of its rows
#pragma unroll
    for (int m = 0; m < MT; ++m) ss[m] = 0.0f;
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(P.gain, NORM == NORM_GAIN ? (uint32_t)P.K * 2 : 0u);
    auto normalise = [&](int m, u32x4& av, const u32x4& gv) {
        bf16x8 x = __builtin_bit_cast(bf16x8, av);
        ss[m] = add_squares(x, ss[m]);
        if (NORM == NORM_GAIN) {
            float g[8];
            unpack_bf16x8(__builtin_bit_cast(bf16x8, gv), g);
            av = __builtin_bit_cast(u32x4, scale_bf16x8(x, g));
        }
    };
    auto mfma = [&](int w, int m, const u32x4& bv, const u32x4& av) {
        // weights first: a lane's four results are four consecutive columns of one row
        acc[w][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bv), __builtin_bit_cast(bf16x8, av),
                                                            acc[w][m], 0, 0, 0);
    };

    // k-steps [s, s_end) of this wavefront; those below s_full lie inside K
    const int steps = (P.K + 31) / 32, per = (steps + WAVES - 1) / WAVES;
    int s = wave * per;
    const int s_end = s + per < steps ? s + per : steps;
    const int s_full = s_end < P.K / 32 ? s_end : P.K / 32;
    u32x4 b[NW][FR_UNROLL], a[MT][FR_UNROLL], g[NORM == NORM_GAIN ? FR_UNROLL : 1];
    auto load_batch = [&]() {
#pragma unroll
        for (int u = 0; u < FR_UNROLL; ++u) {
            b[0][u] = __builtin_amdgcn_raw_buffer_load_b128(rb0, (int)b_off, (s + u) * 64, 0);
            if (NW == 2) b[NW - 1][u] = __builtin_amdgcn_raw_buffer_load_b128(rb1, (int)b_off, (s + u) * 64, 0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                a[m][u] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_off[m], (int)((uint32_t)(s + u) * a_step), 0);
            if (NORM == NORM_GAIN) g[u] = __builtin_amdgcn_raw_buffer_load_b128(rg, kq * 16, (s + u) * 64, 0);
        }
    };
    auto mfma_batch = [&]() {
#pragma unroll
        for (int u = 0; u < FR_UNROLL; ++u)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (NORM != NORM_NONE) normalise(m, a[m][u], g[NORM == NORM_GAIN ? u : 0]);
#pragma unroll
                for (int w = 0; w < NW; ++w) mfma(w, m, b[w][u], a[m][u]);
            }
    };
    const bool any_batch = s + FR_UNROLL <= s_full;
    if (any_batch) load_batch();
    // the epilogue's residual: two dependent loads, behind the first weights
    int64_t orow = 0;
    u32x2 resid = {0u, 0u};
    if (!GATE_UP && mine) {
        orow = (int64_t)irow * P.N + en;
        if (!P.no_residual) resid = *reinterpret_cast<const u32x2*>(P.res + orow);
    }
    if (any_batch) {
        mfma_batch();
        for (s += FR_UNROLL; s + FR_UNROLL <= s_full; s += FR_UNROLL) {
            load_batch();
            mfma_batch();
        }
    }
    for (; s < s_end; ++s) {                  // fewer than a batch; the last step of a ragged K is masked
        const bool in = s * 32 + kq * 8 < P.K;
        const uint32_t bo = in && b_off != kOobOffset ? b_off + (uint32_t)s * 64u : kOobOffset;
        u32x4 bt[NW];
        bt[0] = buf_load16(rb0, bo);
        if (NW == 2) bt[NW - 1] = buf_load16(rb1, bo);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            u32x4 at = buf_load16(ra, in && a_off[m] != kOobOffset ? a_off[m] + (uint32_t)s * a_step : kOobOffset);
            if (NORM != NORM_NONE)
                normalise(m, at, NORM == NORM_GAIN ? buf_load16(rg, in ? (uint32_t)(s * 64 + kq * 16) : kOobOffset) : u32x4{0u, 0u, 0u, 0u});
#pragma unroll
            for (int w = 0; w < NW; ++w) mfma(w, m, bt[w], at);
        }
    }

#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
        for (int m = 0; m < MT; ++m) red[wave][w * MT + m][lane] = acc[w][m];
    if (NORM != NORM_NONE) {
#pragma unroll
        for (int m = 0; m < MT; ++m) red_ss[wave][m][lane] = ss[m];
    }
    __syncthreads();
    if (NORM != NORM_NONE && wave < MT) {
        float sq = red_ss[0][wave][lane];
#pragma unroll
        for (int q = 1; q < WAVES; ++q) sq += red_ss[q][wave][lane];
        rstd = rstd_of_lanes(sq, P.K, P.eps);
    }
    if (!mine) return;
    f32x4 v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        v[w] = red[0][w * MT + wave][lane];
#pragma unroll
        for (int q = 1; q < WAVES; ++q) v[w] += red[q][w * MT + wave][lane];
    }
    if (GATE_UP) {
        f32x4 g = v[0], u = v[NW - 1];
        g *= rstd;
        u *= rstd;
        float h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = g[j] * sigmoid_f(g[j]) * u[j];
        *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(P.H) + (uint32_t)em * P.h_row + (uint32_t)(en >> 3) * P.h_chunk +
                                  (en & 4) * 2) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
        if (P.G != nullptr) {
            const int64_t o = (int64_t)em * P.N + en;
            *reinterpret_cast<u32x2*>(P.G + o) = u32x2{pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3])};
            *reinterpret_cast<u32x2*>(P.U + o) = u32x2{pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3])};
        }
    } else {
        f32x4 y = v[0];
        if (!P.no_residual) {
            y[0] += bf16lo_to_f32(resid[0]); y[1] += bf16hi_to_f32(resid[0]);
            y[2] += bf16lo_to_f32(resid[1]); y[3] += bf16hi_to_f32(resid[1]);
        }
        *reinterpret_cast<u32x2*>(P.out + orow) = u32x2{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    }
}

template <int WAVES, bool GATE_UP, int NORM = NORM_NONE>
static hipError_t launch_few_rows(const FewRowsArgs& a, hipStream_t s) {
    if (a.rows <= 0 || a.N <= 0) return hipSuccess;
    const dim3 grid((unsigned)((a.N + FR_COLS - 1) / FR_COLS)), block(WAVES * 64);
    if (a.rows <= 16)
        hipLaunchKernelGGL((few_rows_kernel<1, WAVES, GATE_UP, NORM>), grid, block, 0, s, a);
    else if (a.rows <= 32)
        hipLaunchKernelGGL((few_rows_kernel<2, WAVES, GATE_UP, NORM>), grid, block, 0, s, a);
    else if (a.rows <= kFewRowsMax)
        hipLaunchKernelGGL((few_rows_kernel<4, WAVES, GATE_UP, NORM>), grid, block, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_few_rows_gate_up(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                   const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major, bool chunk_major_h,
                                   const RowNorm* norm, const float* rstd, hipStream_t s) {
    FewRowsArgs a{};
    a.rstd = rstd;
    a.rows = rows; a.r_dev = r_dev; a.N = I; a.K = C;
    a.A = xn; a.a_bytes = (uint32_t)((int64_t)rows * C * 2);
    a.a_row = chunk_major ? 16u : (uint32_t)C * 2; a.a_chunk = chunk_major ? (uint32_t)rows * 16 : 16u;
    a.B0 = w_gate; a.B1 = w_up; a.b_bytes = (uint32_t)((int64_t)I * C * 2);
    a.H = H; a.h_row = chunk_major_h ? 16u : (uint32_t)I * 2; a.h_chunk = chunk_major_h ? (uint32_t)rows * 16 : 16u;
    a.G = G; a.U = U;
    if (norm != nullptr) {
        a.A = norm->hidden; a.a_bytes = (uint32_t)(norm->T * C * 2); a.a_row = (uint32_t)C * 2; a.a_chunk = 16u;
        a.idx = norm->idx; a.gain = norm->gain; a.eps = norm->eps;
        return norm->gain != nullptr ? launch_few_rows<FR_WAVES_GU, true, NORM_GAIN>(a, s)
                                     : launch_few_rows<FR_WAVES_GU, true, NORM_PLAIN>(a, s);
    }
    return launch_few_rows<FR_WAVES_GU, true>(a, s);
}

hipError_t launch_few_rows_down(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down,
                                const int32_t* idx, const bf16_t* res, bf16_t* out, int no_residual, bool chunk_major,
                                hipStream_t s) {
    FewRowsArgs a{};
    a.rows = rows; a.r_dev = r_dev; a.N = C; a.K = I;
    a.A = H; a.a_bytes = (uint32_t)((int64_t)rows * I * 2);
    a.a_row = chunk_major ? 16u : (uint32_t)I * 2; a.a_chunk = chunk_major ? (uint32_t)rows * 16 : 16u;
    a.B0 = w_down; a.b_bytes = (uint32_t)((int64_t)C * I * 2);
    a.idx = idx; a.res = res; a.out = out; a.no_residual = no_residual;
    return launch_few_rows<FR_WAVES_DOWN, false>(a, s);
}

}  // namespace skipffn
