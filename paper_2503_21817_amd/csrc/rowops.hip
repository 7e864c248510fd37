// Memory-bound row kernels of the Skip-FFN block: 16-byte accesses, fp32 arithmetic.
// Rows are addressed through the retained index list, so only the R retained rows are
// touched (Section 4.2: skipped tokens keep their residual and see no FFN work).
// Kernels that reduce over a row give the row to one 256-thread workgroup (R is a few
// thousand at most, so a wavefront per row would leave most of the chip without work in
// flight); purely elementwise ones run one thread per 16-byte chunk.
#include <type_traits>

#include "colsum.hpp"
#include "gemm.hpp"
#include "kernels.hpp"

namespace skipffn {

constexpr int ROW_THREADS = 256;
constexpr int RMS_MAXV = 4;                   // register-resident row up to C = 256*8*4 = 8192

__device__ __forceinline__ void unpack8(const u32x4& v, float* f) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = bf16lo_to_f32(v[j]);
        f[2 * j + 1] = bf16hi_to_f32(v[j]);
    }
}
__device__ __forceinline__ u32x4 pack8(const float* f) {
    u32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = pack_bf16x2(f[2 * j], f[2 * j + 1]);
    return v;
}
// sum over the 256 threads of a workgroup (one call per kernel: `red` is not reused)
__device__ __forceinline__ float block_sum(float v, float* red) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// ---- bit copy of skipped rows (out-of-place calls) ---------------------------------------
// A wavefront takes a row t and copies it unless t is in the ascending list idx.  The search probes 64 positions at a
// time: two dependent loads up to 4096 entries, where halving takes 12 before the copy can begin; the row is then
// copied with eight loads in flight per lane (a row of 4096 at once).  616 rows 7.8 -> 5.2 us, 1232 rows 9.8 ->
// 6.1, 4928 rows 16.4 -> 14.0.  It depends on nothing but the hidden states (the gradient), so it shares a launch with the first
// kernel of the call that reads them too.
constexpr int ROWS_PER_BLOCK = ROW_THREADS / 64;   // copy kernels: one wavefront per row
static unsigned skipped_blocks(const SkippedRows& sk) {
    return sk.dst == nullptr ? 0u : (unsigned)((sk.T + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK);
}
__device__ __forceinline__ void copy_skipped_rows(const SkippedRows& sk, const int block, const int R) {
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)block * ROWS_PER_BLOCK + (threadIdx.x >> 6);
    const int32_t* idx = sk.idx;
    if (t >= sk.T) return;
    int lo = 0, hi = R;              // the first position with idx[pos] >= t lies in [lo, hi]
    while (hi - lo > 63) {
        const int step = (hi - lo + 63) >> 6;
        const int p = lo + lane * step;
        const int below = __popcll(__ballot(p < hi && idx[p < hi ? p : lo] < t));    // ascending: a prefix of the lanes
        const int end = lo + below * step;
        if (below == 0) hi = lo;
        else { lo = end - step + 1; hi = end < hi ? end : hi; }
    }
    const int p = lo + lane;
    if (__ballot(p <= hi && p < R && idx[p < R ? p : 0] == t) != 0) return;   // retained: written by the scatter epilogue
    const u32x4* s = static_cast<const u32x4*>(sk.src) + t * sk.row_chunks;
    u32x4* d = static_cast<u32x4*>(sk.dst) + t * sk.row_chunks;
    int64_t c = lane;
    for (; c + 7 * 64 < sk.row_chunks; c += 8 * 64) {
        u32x4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = s[c + k * 64];
#pragma unroll
        for (int k = 0; k < 8; ++k) d[c + k * 64] = v[k];
    }
    for (; c < sk.row_chunks; c += 64) d[c] = s[c];
}

// ---- gather + RMSNorm -------------------------------------------------------------
// n(x) = x * rsqrt(mean(x^2) + eps) * gain for the rows idx[r]; x is read once
// (held in registers), the un-normalised row is optionally copied for backward.
template <bool IN_REGS>
__global__ __launch_bounds__(ROW_THREADS) void gather_rmsnorm_kernel(
    const bf16_t* __restrict__ hidden, const int32_t* __restrict__ idx, int Rbound,
    const int32_t* __restrict__ r_dev, int C, float eps, const bf16_t* __restrict__ gain,
    bf16_t* __restrict__ xrows, bf16_t* __restrict__ xn, int64_t xn_row, int xn_chunk, int scaled, float* __restrict__ rstd_out,
    SkippedRows sk) {
    __shared__ float red[4];
    const int R = effective_rows(Rbound, r_dev);
    const int tid = threadIdx.x;
    const int r = blockIdx.x;
    if (r >= Rbound) return copy_skipped_rows(sk, r - Rbound, R);
    if (r >= R) return;                       // the whole workgroup leaves together
    const int chunks = C >> 3;
    const u32x4* src = reinterpret_cast<const u32x4*>(hidden + (int64_t)idx[r] * C);
    const u32x4* gsrc = reinterpret_cast<const u32x4*>(gain);
    u32x4* dxn = reinterpret_cast<u32x4*>(xn) + r * xn_row;      // strides in 16-byte chunks
    u32x4* dxr = xrows ? reinterpret_cast<u32x4*>(xrows + (int64_t)r * C) : nullptr;

    u32x4 held[IN_REGS ? RMS_MAXV : 1];
    float ss = 0.0f;
    if (IN_REGS) {
#pragma unroll
        for (int v = 0; v < RMS_MAXV; ++v) {
            int c = tid + ROW_THREADS * v;
            if (c < chunks) {
                held[v] = src[c];
                float f[8];
                unpack8(held[v], f);
#pragma unroll
                for (int j = 0; j < 8; ++j) ss += f[j] * f[j];
            }
        }
    } else {
        for (int c = tid; c < chunks; c += ROW_THREADS) {
            float f[8];
            unpack8(src[c], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) ss += f[j] * f[j];
        }
    }
    ss = block_sum(ss, red);
    const float rstd = 1.0f / sqrtf(ss / (float)C + eps);
    if (tid == 0) rstd_out[r] = rstd;

    auto emit = [&](int c, const u32x4& raw) {
        float f[8];
        unpack8(raw, f);
        if (gain != nullptr) {
            float g[8];
            unpack8(gsrc[c], g);
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = f[j] * rstd * g[j];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = f[j] * rstd;
        }
        dxn[(int64_t)c * xn_chunk] = scaled ? pack8(f) : raw;
        if (dxr) dxr[c] = raw;
    };
    if (IN_REGS) {
#pragma unroll
        for (int v = 0; v < RMS_MAXV; ++v) {
            int c = tid + ROW_THREADS * v;
            if (c < chunks) emit(c, held[v]);
        }
    } else {
        for (int c = tid; c < chunks; c += ROW_THREADS) emit(c, src[c]);
    }
}

hipError_t launch_gather_rmsnorm(const bf16_t* hidden, const int32_t* idx, int R,
                                 const int32_t* r_dev, int C, float eps, const bf16_t* gain,
                                 bf16_t* xrows, bf16_t* xn, float* rstd, bool chunk_major, bool scaled, const SkippedRows& sk,
                                 hipStream_t s) {
    if (R <= 0) return hipSuccess;
    const int64_t xn_row = chunk_major ? 1 : C >> 3;
    const int xn_chunk = chunk_major ? R : 1;
    dim3 grid((unsigned)R + skipped_blocks(sk)), block(ROW_THREADS);
    profile_mark_begin(KC_GATHER_RMSNORM, s);
    if (C <= ROW_THREADS * 8 * RMS_MAXV)
        hipLaunchKernelGGL(gather_rmsnorm_kernel<true>, grid, block, 0, s, hidden, idx, R, r_dev, C,
                           eps, gain, xrows, xn, xn_row, xn_chunk, scaled ? 1 : 0, rstd, sk);
    else
        hipLaunchKernelGGL(gather_rmsnorm_kernel<false>, grid, block, 0, s, hidden, idx, R, r_dev, C,
                           eps, gain, xrows, xn, xn_row, xn_chunk, scaled ? 1 : 0, rstd, sk);
    profile_mark_end(KC_GATHER_RMSNORM, s);
    return hipGetLastError();
}

// ---- split-K reduce + residual + scatter ----------------------------------------------
// out[idx[r]][c] = bf16( res[idx[r]][c] + sum_z partial[z][r][c] ), summed in z order.
// One thread per 16-byte chunk of the output.
// number of partial slabs to add for row r, column col
__device__ __forceinline__ int partial_count(const PartialLayout& pl, int R, int r, int col) {
    if (pl.sk_nbg == 0) return pl.splits;
    const StreamKPlan p = streamk_plan((R + BM - 1) / BM, pl.sk_kt, pl.sk_nbg);
    (void)col;                       // the count depends on the m-tile only
    return streamk_count(p, r / BM);
}

// zrows: rows of a slab
__device__ __forceinline__ void resid_scatter_chunk(const float* __restrict__ partial, const PartialLayout& pl, const int zrows,
                                                    const int R, const int C, const int r, const int c, const int row,
                                                    const bf16_t* res, bf16_t* out, const int no_residual) {
    const int64_t orow = (int64_t)row * C;
    const int64_t zstride = (int64_t)zrows * C;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
    const float* p = partial + (int64_t)r * C + c * 8;
    const int splits = partial_count(pl, R, r, c * 8);
    const u32x4 xraw = no_residual ? u32x4{0u, 0u, 0u, 0u} : *reinterpret_cast<const u32x4*>(res + orow + c * 8);
    // four slabs in flight, then two (few rows: a load after the other is all the time there is)
    int z = 0;
    auto add = [&](auto count) {
        constexpr int N = decltype(count)::value;
        f32x4 a[N], b[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            a[k] = *reinterpret_cast<const f32x4*>(p + (z + k) * zstride);
            b[k] = *reinterpret_cast<const f32x4*>(p + (z + k) * zstride + 4);
        }
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[j] += a[k][j];
                acc[4 + j] += b[k][j];
            }
        z += N;
    };
    while (z + 4 <= splits) add(std::integral_constant<int, 4>{});
    if (z + 2 <= splits) add(std::integral_constant<int, 2>{});
    if (z < splits) add(std::integral_constant<int, 1>{});
    if (!no_residual) {
        float x[8];
        unpack8(xraw, x);
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += x[j];
    }
    *reinterpret_cast<u32x4*>(out + orow + c * 8) = pack8(acc);
}
__global__ __launch_bounds__(ROW_THREADS) void resid_scatter_kernel(
    const float* __restrict__ partial, PartialLayout pl, int Rbound, const int32_t* __restrict__ r_dev,
    int C, const int32_t* __restrict__ idx, const bf16_t* res, bf16_t* out, int no_residual) {
    const int R = effective_rows(Rbound, r_dev), chunks = C >> 3;
    const int64_t g = (int64_t)blockIdx.x * ROW_THREADS + threadIdx.x;
    const int r = (int)(g / chunks), c = (int)(g - (int64_t)r * chunks);
    if (r < R) resid_scatter_chunk(partial, pl, Rbound, R, C, r, c, idx[r], res, out, no_residual);
}
// Bound by its chain of loads: count, its plan, row, slabs.  Row and plan at once, the plan by a scalar load, two slabs in flight:  1871 rows of 3072
// columns, two slabs, 21.7 -> 18.7 us;  644 of 8192 17.8 -> 15.8;  100 of 4096, eight slabs, 5.6 -> 5.2 (with the plan in the arguments 16.0, 14.0).
__global__ __launch_bounds__(ROW_THREADS) void resid_scatter_count_kernel(
    const float* __restrict__ partial, RowPlans plans, int ktiles, int Rbound, const int32_t* __restrict__ r_dev,
    int C, const int32_t* __restrict__ idx, const bf16_t* res, bf16_t* out, int no_residual) {
    const int chunks = C >> 3;
    const int64_t g = (int64_t)blockIdx.x * ROW_THREADS + threadIdx.x;
    const int r = (int)(g / chunks), c = (int)(g - (int64_t)r * chunks);
    // the row's index on the way while the count and its plan come in, one after the other (idx holds the bound)
    int row = idx[r < Rbound ? r : 0];
    const int R = effective_rows(Rbound, r_dev);
    if (R <= 0) return;
    const bool all_rows = R <= 256;
    const KPartition k = all_rows ? KPartition{plans.mid_splits, 0} : row_plan(plans, (R + BM - 1) / BM);
    asm volatile("" : "+v"(row));                                       // (not moved past the branch)
    if (r >= R || (!all_rows && k.splits == 1 && k.sk_nbg == 0)) return;                // ..: the GEMM has written the rows itself
    resid_scatter_chunk(partial, PartialLayout{k.splits, k.sk_nbg, ktiles}, all_rows ? 256 : Rbound, R, C, r, c, row, res, out, no_residual);
}

hipError_t launch_resid_scatter_count(const float* partial, const RowPlans& plans, int ktiles, int R, int sum_rows, const int32_t* r_dev, int C,
                                      const int32_t* idx, const bf16_t* res, bf16_t* out, int no_residual, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    const int64_t total = (int64_t)sum_rows * (C >> 3);
    profile_mark_begin(KC_RESID_SCATTER, s);
    hipLaunchKernelGGL(resid_scatter_count_kernel, dim3((unsigned)((total + ROW_THREADS - 1) / ROW_THREADS)), dim3(ROW_THREADS), 0, s,
                       partial, plans, ktiles, R, r_dev, C, idx, res, out, no_residual);
    profile_mark_end(KC_RESID_SCATTER, s);
    return hipGetLastError();
}

hipError_t launch_resid_scatter(const float* partial, PartialLayout pl, int R, const int32_t* r_dev,
                                int C, const int32_t* idx, const bf16_t* res, bf16_t* out,
                                int no_residual, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    const int64_t total = (int64_t)R * (C >> 3);
    dim3 grid((unsigned)((total + ROW_THREADS - 1) / ROW_THREADS)), block(ROW_THREADS);
    profile_mark_begin(KC_RESID_SCATTER, s);
    hipLaunchKernelGGL(resid_scatter_kernel, grid, block, 0, s, partial, pl, R, r_dev, C, idx,
                       res, out, no_residual);
    profile_mark_end(KC_RESID_SCATTER, s);
    return hipGetLastError();
}

// ---- row gather (upstream gradient rows; skip KV-cache of Section 4.3) -----------------
__global__ __launch_bounds__(ROW_THREADS) void gather_rows_kernel(
    const u32x4* __restrict__ src, u32x4* __restrict__ dst, int64_t row_chunks,
    const int32_t* __restrict__ idx, int Rbound, const int32_t* __restrict__ r_dev) {
    const int R = effective_rows(Rbound, r_dev);
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * ROWS_PER_BLOCK + (threadIdx.x >> 6);
    if (r >= R) return;
    const u32x4* s = src + (int64_t)idx[r] * row_chunks;
    u32x4* d = dst + (int64_t)r * row_chunks;
    for (int64_t c = lane; c < row_chunks; c += 64) d[c] = s[c];
}

hipError_t launch_gather_rows(const void* src, void* dst, int64_t row_bytes, const int32_t* idx,
                              int R, const int32_t* r_dev, hipStream_t s) {
    if (R <= 0 || row_bytes <= 0) return hipSuccess;
    dim3 grid((R + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK), block(ROW_THREADS);
    profile_mark_begin(KC_GATHER_ROWS, s);
    hipLaunchKernelGGL(gather_rows_kernel, grid, block, 0, s, static_cast<const u32x4*>(src),
                       static_cast<u32x4*>(dst), row_bytes / 16, idx, R, r_dev);
    profile_mark_end(KC_GATHER_ROWS, s);
    return hipGetLastError();
}

// ---- skip KV-cache over a whole cache (Section 4.3) --------------------------------------------
// One thread per 16-byte chunk of the compacted cache; blockIdx.y walks the slabs.  Cache rows
// are short (one head of one token: 256 bytes for d = 128), so a wavefront per row would
// leave three quarters of its lanes idle.
__global__ __launch_bounds__(ROW_THREADS) void kv_compact_kernel(
    const char* __restrict__ src, char* __restrict__ dst, int64_t n_slabs, int row_chunks,
    int64_t src_slab_bytes, int64_t dst_slab_bytes, const int32_t* __restrict__ idx, int Rbound,
    const int32_t* __restrict__ r_dev) {
    const int R = effective_rows(Rbound, r_dev);
    const int64_t g = (int64_t)blockIdx.x * ROW_THREADS + threadIdx.x;
    const int r = (int)(g / row_chunks), c = (int)(g - (int64_t)r * row_chunks);
    if (r >= R) return;
    const int64_t so = (int64_t)idx[r] * row_chunks + c, d_o = (int64_t)r * row_chunks + c;
    for (int64_t sl = blockIdx.y; sl < n_slabs; sl += gridDim.y) {
        const u32x4* s = reinterpret_cast<const u32x4*>(src + sl * src_slab_bytes);
        u32x4* d = reinterpret_cast<u32x4*>(dst + sl * dst_slab_bytes);
        d[d_o] = s[so];
    }
}

hipError_t launch_kv_compact(const void* src, void* dst, int64_t n_slabs, int64_t row_bytes,
                             int64_t src_slab_bytes, int64_t dst_slab_bytes, const int32_t* idx,
                             int R, const int32_t* r_dev, hipStream_t s) {
    if (R <= 0 || row_bytes <= 0 || n_slabs <= 0) return hipSuccess;
    const int row_chunks = (int)(row_bytes / 16);
    const int64_t per_slab = (int64_t)R * row_chunks;
    dim3 grid((unsigned)((per_slab + ROW_THREADS - 1) / ROW_THREADS),
              (unsigned)(n_slabs < 65535 ? n_slabs : 65535)), block(ROW_THREADS);
    profile_mark_begin(KC_KV_COMPACT, s);
    hipLaunchKernelGGL(kv_compact_kernel, grid, block, 0, s, static_cast<const char*>(src),
                       static_cast<char*>(dst), n_slabs, row_chunks, src_slab_bytes, dst_slab_bytes,
                       idx, R, r_dev);
    profile_mark_end(KC_KV_COMPACT, s);
    return hipGetLastError();
}

// ---- row gather with a transposed copy ------------------------------------------------------
// dst[r][:] = src[row(r)][:] (optional) and dstT[c][r] = src[row(r)][c], where row(r) = idx[r]
// (or r when idx is null).  dstT has leading dimension ldT (a multiple of 8 >= the row
// bound); columns r >= R of dstT are written as zeros so that K-slabs reading past R see
// zeros.  The weight-gradient GEMMs contract over R: a copy with R contiguous lets them read
// this operand with plain 16-byte LDS reads instead of transposing ones.
// A launch takes up to two such copies of the same rows, and the skipped rows: each is a few us of latency at small sizes.
constexpr int TR_TILE = 64;
struct TransposeArgs {
    TransposeJob job[2];
    int blocks[2], tiles_r;                              // workgroups of a job, tiles of TR_TILE rows
    int Rbound; const int32_t* r_dev; int ldT;
    SkippedRows sk;
};
__global__ __launch_bounds__(256) void gather_transpose_kernel(TransposeArgs P) {
    __shared__ bf16_t tile[TR_TILE][TR_TILE + 2];
    const int R = effective_rows(P.Rbound, P.r_dev);
    int b = (int)blockIdx.x;
    if (b >= P.blocks[0] + P.blocks[1]) return copy_skipped_rows(P.sk, b - P.blocks[0] - P.blocks[1], R);
    const bool second = b >= P.blocks[0];                // uniform
    if (second) b -= P.blocks[0];
    const bf16_t* src = second ? P.job[1].src : P.job[0].src;
    const int32_t* idx = second ? P.job[1].idx : P.job[0].idx;
    bf16_t* dst = second ? P.job[1].dst : P.job[0].dst;
    bf16_t* dstT = second ? P.job[1].dstT : P.job[0].dstT;
    const int C = second ? P.job[1].C : P.job[0].C, ldT = P.ldT;
    const int r0 = b % P.tiles_r * TR_TILE, c0 = b / P.tiles_r * TR_TILE;
    const int t = threadIdx.x;
    // phase 1: 64 rows x 64 columns, 16 bytes per access
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = t + 256 * i;
        const int rr = q >> 3, ch = q & 7;
        const int r = r0 + rr, c = c0 + ch * 8;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (r < R && c < C) {
            const int64_t srow = idx ? (int64_t)idx[r] : (int64_t)r;
            v = *reinterpret_cast<const u32x4*>(src + srow * C + c);
            if (dst) *reinterpret_cast<u32x4*>(dst + (int64_t)r * C + c) = v;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            tile[rr][ch * 8 + 2 * k] = (bf16_t)(v[k] & 0xffffu);
            tile[rr][ch * 8 + 2 * k + 1] = (bf16_t)(v[k] >> 16);
        }
    }
    __syncthreads();
    // phase 2: 64 output rows (columns of src) x 64 r values = 8 chunks of 16 bytes each
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = t + 256 * i;
        const int cc = q >> 3, ch = q & 7;
        const int c = c0 + cc, r = r0 + ch * 8;
        if (c < C && r < ldT) {
            u32x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = (uint32_t)tile[ch * 8 + 2 * k][cc] | ((uint32_t)tile[ch * 8 + 2 * k + 1][cc] << 16);
            *reinterpret_cast<u32x4*>(dstT + (int64_t)c * ldT + r) = v;
        }
    }
}

hipError_t launch_gather_transpose(const TransposeJob* jobs, int count, int R, const int32_t* r_dev, int ldT, const SkippedRows& sk,
                                   hipStream_t s) {
    if (R <= 0 || count <= 0) return hipSuccess;
    if (count > 2) return hipErrorInvalidValue;
    TransposeArgs a{};
    a.tiles_r = (ldT + TR_TILE - 1) / TR_TILE;
    for (int j = 0; j < count; ++j) {
        a.job[j] = jobs[j];
        a.blocks[j] = a.tiles_r * ((jobs[j].C + TR_TILE - 1) / TR_TILE);
    }
    a.Rbound = R; a.r_dev = r_dev; a.ldT = ldT; a.sk = sk;
    profile_mark_begin(KC_GATHER_ROWS, s);
    hipLaunchKernelGGL(gather_transpose_kernel, dim3((unsigned)(a.blocks[0] + a.blocks[1]) + skipped_blocks(sk)), dim3(256), 0, s, a);
    profile_mark_end(KC_GATHER_ROWS, s);
    return hipGetLastError();
}

// ---- SwiGLU backward of a dH that comes as fp32 slabs -----------------------------------------
// dG, dU [R][I] and their transposed copies [I][ldT] (zeros past the last row), a tile of 64 x 64 a workgroup as above: S + 1 reads and
// two writes of R * I values beside the copies.  When it pays: dh_splits.
template <int S>
__global__ __launch_bounds__(256) void swiglu_bwd_reduce_kernel(SwigluBwdArgs P) {
    __shared__ bf16_t tile[2][TR_TILE][TR_TILE + 2];
    const int R = effective_rows(P.R, P.r_dev);
    const int r0 = (int)blockIdx.x * TR_TILE, c0 = (int)blockIdx.y * TR_TILE, t = threadIdx.x;
    const int64_t zstride = (int64_t)P.R * P.I;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = t + 256 * i, rr = q >> 3, ch = q & 7, r = r0 + rr, c = c0 + ch * 8;
        u32x4 dg = {0u, 0u, 0u, 0u}, du = {0u, 0u, 0u, 0u};
        if (r < R && c < P.I) {
            const int64_t o = (int64_t)r * P.I + c;
            f32x4 v[S][2];
#pragma unroll
            for (int z = 0; z < S; ++z)
#pragma unroll
                for (int h = 0; h < 2; ++h) v[z][h] = *reinterpret_cast<const f32x4*>(P.partial + z * zstride + o + 4 * h);
            float g[8], u[8];
            unpack8(*reinterpret_cast<const u32x4*>(P.G + o), g);
            unpack8(*reinterpret_cast<const u32x4*>(P.U + o), u);
            float a[8], b[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float dh = v[0][j >> 2][j & 3];
#pragma unroll
                for (int z = 1; z < S; ++z) dh += v[z][j >> 2][j & 3];
                const float sg = sigmoid_f(g[j]);
                a[j] = dh * u[j] * sg * (1.0f + g[j] * (1.0f - sg));
                b[j] = dh * g[j] * sg;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                dg[k] = pack_bf16x2(a[2 * k], a[2 * k + 1]);
                du[k] = pack_bf16x2(b[2 * k], b[2 * k + 1]);
            }
            *reinterpret_cast<u32x4*>(P.dG + o) = dg;
            *reinterpret_cast<u32x4*>(P.dU + o) = du;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            tile[0][rr][ch * 8 + 2 * k] = (bf16_t)(dg[k] & 0xffffu);
            tile[0][rr][ch * 8 + 2 * k + 1] = (bf16_t)(dg[k] >> 16);
            tile[1][rr][ch * 8 + 2 * k] = (bf16_t)(du[k] & 0xffffu);
            tile[1][rr][ch * 8 + 2 * k + 1] = (bf16_t)(du[k] >> 16);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = (t + 256 * i) & 511, m = i >> 1, cc = q >> 3, ch = q & 7, c = c0 + cc, r = r0 + ch * 8;
        if (c < P.I && r < P.ldT) {
            u32x4 v;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = (uint32_t)tile[m][ch * 8 + 2 * k][cc] | ((uint32_t)tile[m][ch * 8 + 2 * k + 1][cc] << 16);
            *reinterpret_cast<u32x4*>((m == 0 ? P.dGT : P.dUT) + (int64_t)c * P.ldT + r) = v;
        }
    }
}

hipError_t launch_swiglu_bwd_reduce(const SwigluBwdArgs& a, hipStream_t s) {
    if (a.R <= 0 || a.I <= 0) return hipSuccess;
    const dim3 grid((unsigned)((a.ldT + TR_TILE - 1) / TR_TILE), (unsigned)((a.I + TR_TILE - 1) / TR_TILE)), block(256);
    if (grid.y > 65535) return hipErrorInvalidValue;
    switch (a.splits) {
        case 2: hipLaunchKernelGGL(swiglu_bwd_reduce_kernel<2>, grid, block, 0, s, a); break;
        case 3: hipLaunchKernelGGL(swiglu_bwd_reduce_kernel<3>, grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL(swiglu_bwd_reduce_kernel<4>, grid, block, 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__global__ __launch_bounds__(ROW_THREADS) void passthrough_kernel(SkippedRows sk, int Rbound, const int32_t* __restrict__ r_dev) {
    copy_skipped_rows(sk, (int)blockIdx.x, effective_rows(Rbound, r_dev));
}

hipError_t launch_passthrough(const SkippedRows& sk, int R, const int32_t* r_dev, hipStream_t s) {
    if (sk.dst == nullptr || sk.T <= 0 || sk.row_chunks <= 0) return hipSuccess;
    profile_mark_begin(KC_PASSTHROUGH, s);
    hipLaunchKernelGGL(passthrough_kernel, dim3(skipped_blocks(sk)), dim3(ROW_THREADS), 0, s, sk, R < 0 ? 0 : R, r_dev);
    profile_mark_end(KC_PASSTHROUGH, s);
    return hipGetLastError();
}

// ---- RMSNorm backward + residual gradient + scatter ----------------------------------------
// With xh = x * rstd and dxh = dxn * gain:
//   dx = rstd * (dxh - xh * mean_c(dxh * xh));  dX[idx[r]] = bf16(dY[r] + dx)
// dxn arrives as `splits` fp32 partial sums [z][r][c] (the split-K slabs of the
// dG*W_gate + dU*W_up GEMM), added here in z order.
// With GAIN_GRAD a workgroup walks a strip of GAIN_STRIP rows and also accumulates the
// gradient of the gain, dgain[c] = sum_r dxn[r][c] * x[r][c] * rstd[r], over its strip into
// gpart[strip][c]; gain_grad_reduce_kernel adds the strips in order (deterministic).
template <bool IN_REGS, bool GAIN_GRAD>
__global__ __launch_bounds__(ROW_THREADS) void rmsnorm_bwd_scatter_kernel(
    const float* __restrict__ part, PartialLayout pl, int Rbound, const int32_t* __restrict__ r_dev,
    int C, const bf16_t* __restrict__ xrows, const float* __restrict__ rstd_in,
    const bf16_t* __restrict__ gain, const bf16_t* __restrict__ dY,
    const int32_t* __restrict__ idx, bf16_t* dX, float* __restrict__ gpart) {
    __shared__ float red[4];
    const int R = effective_rows(Rbound, r_dev);
    const int tid = threadIdx.x;
    constexpr int STRIP = GAIN_GRAD ? GAIN_STRIP : 1;
    const int r_begin = blockIdx.x * STRIP;
    if (r_begin >= R) return;                 // the whole workgroup leaves together
    const int r_end = r_begin + STRIP < R ? r_begin + STRIP : R;
    const int chunks = C >> 3;
    const int64_t zstride = (int64_t)Rbound * C;
    const u32x4* gs = reinterpret_cast<const u32x4*>(gain);
    constexpr int MAXV = 2;                   // register-resident row: C <= 256 * 8 * 2 = 4096
    float gacc[IN_REGS ? MAXV : 1][8];
    if (IN_REGS && GAIN_GRAD) {
#pragma unroll
        for (int v = 0; v < MAXV; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) gacc[v][j] = 0.0f;
    }
    float* gp = GAIN_GRAD ? gpart + (int64_t)blockIdx.x * C : nullptr;

    for (int r = r_begin; r < r_end; ++r) {
        const float rstd = rstd_in[r];
        const float* p = part + (int64_t)r * C;
        const u32x4* xs = reinterpret_cast<const u32x4*>(xrows + (int64_t)r * C);
        const int splits = partial_count(pl, R, r, 0);
        // d = dxn (sum of the split-K slabs)
        auto load_dxn = [&](int c, float* d) {
#pragma unroll
            for (int j = 0; j < 8; ++j) d[j] = 0.0f;
            for (int z = 0; z < splits; ++z) {
                f32x4 a = *reinterpret_cast<const f32x4*>(p + z * zstride + c * 8);
                f32x4 b = *reinterpret_cast<const f32x4*>(p + z * zstride + c * 8 + 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d[j] += a[j];
                    d[4 + j] += b[j];
                }
            }
        };
        auto apply_gain = [&](int c, float* d) {
            if (gain != nullptr) {
                float g[8];
                unpack8(gs[c], g);
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] *= g[j];
            }
        };
        const u32x4* dys = reinterpret_cast<const u32x4*>(dY + (int64_t)r * C);
        u32x4* out = reinterpret_cast<u32x4*>(dX + (int64_t)idx[r] * C);
        auto emit = [&](int c, const float* d, const float* x, const u32x4& dyraw, float dot) {
            float gy[8], o[8];
            unpack8(dyraw, gy);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = gy[j] + rstd * (d[j] - (x[j] * rstd) * dot);
            out[c] = pack8(o);
        };

        if (IN_REGS) {
            // the row (sum of the split-K slabs, x and dY) is read once and kept in registers
            float d[MAXV][8], x[MAXV][8];
            u32x4 dyraw[MAXV];
            float dot = 0.0f;
#pragma unroll
            for (int v = 0; v < MAXV; ++v) {
                int c = tid + ROW_THREADS * v;
                if (c < chunks) {
                    load_dxn(c, d[v]);
                    unpack8(xs[c], x[v]);
                    dyraw[v] = dys[c];
                    if (GAIN_GRAD) {
#pragma unroll
                        for (int j = 0; j < 8; ++j) gacc[v][j] += d[v][j] * (x[v][j] * rstd);
                    }
                    apply_gain(c, d[v]);
#pragma unroll
                    for (int j = 0; j < 8; ++j) dot += d[v][j] * (x[v][j] * rstd);
                }
            }
            dot = block_sum(dot, red) / (float)C;
#pragma unroll
            for (int v = 0; v < MAXV; ++v) {
                int c = tid + ROW_THREADS * v;
                if (c < chunks) emit(c, d[v], x[v], dyraw[v], dot);
            }
        } else {
            float dot = 0.0f;
            for (int c = tid; c < chunks; c += ROW_THREADS) {
                float d[8], x[8];
                load_dxn(c, d);
                unpack8(xs[c], x);
                if (GAIN_GRAD) {
                    // the strip's partial lives in global memory: each thread owns its chunks
                    f32x4* g0 = reinterpret_cast<f32x4*>(gp + c * 8);
                    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
                    if (r > r_begin) { lo = g0[0]; hi = g0[1]; }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        lo[j] += d[j] * (x[j] * rstd);
                        hi[j] += d[4 + j] * (x[4 + j] * rstd);
                    }
                    g0[0] = lo; g0[1] = hi;
                }
                apply_gain(c, d);
#pragma unroll
                for (int j = 0; j < 8; ++j) dot += d[j] * (x[j] * rstd);
            }
            dot = block_sum(dot, red) / (float)C;
            for (int c = tid; c < chunks; c += ROW_THREADS) {
                float d[8], x[8];
                load_dxn(c, d);
                apply_gain(c, d);
                unpack8(xs[c], x);
                emit(c, d, x, dys[c], dot);
            }
        }
        if (STRIP > 1) __syncthreads();       // `red` is reused by the next row
    }
    if (IN_REGS && GAIN_GRAD) {
#pragma unroll
        for (int v = 0; v < MAXV; ++v) {
            int c = tid + ROW_THREADS * v;
            if (c < chunks) {
                f32x4* g0 = reinterpret_cast<f32x4*>(gp + c * 8);
                f32x4 lo = {gacc[v][0], gacc[v][1], gacc[v][2], gacc[v][3]};
                f32x4 hi = {gacc[v][4], gacc[v][5], gacc[v][6], gacc[v][7]};
                g0[0] = lo; g0[1] = hi;
            }
        }
    }
}

// dgain[c] (+)= sum over strips of gpart[strip][c]
template <int LANES>
__global__ __launch_bounds__(32 * LANES) void gain_grad_reduce_kernel(
    const float* __restrict__ gpart, int Rbound, const int32_t* __restrict__ r_dev, int C,
    float* __restrict__ dgain, int accumulate) {
    const int R = effective_rows(Rbound, r_dev);
    column_sum<LANES>(gpart, (R + GAIN_STRIP - 1) / GAIN_STRIP, C, dgain, accumulate);
}

hipError_t launch_rmsnorm_bwd_scatter(const float* dxn_partial, PartialLayout pl, int R,
                                      const int32_t* r_dev, int C, const bf16_t* xrows,
                                      const float* rstd, const bf16_t* gain, const bf16_t* dY,
                                      const int32_t* idx, bf16_t* dX, float* gain_partial,
                                      float* dgain, int accumulate, hipStream_t s) {
    if (R <= 0) return hipSuccess;
    const bool gg = dgain != nullptr;
    dim3 grid(gg ? (R + GAIN_STRIP - 1) / GAIN_STRIP : R), block(ROW_THREADS);
    profile_mark_begin(KC_RMSNORM_BWD, s);
    if (C <= 4096) {
        if (gg)
            hipLaunchKernelGGL((rmsnorm_bwd_scatter_kernel<true, true>), grid, block, 0, s, dxn_partial,
                               pl, R, r_dev, C, xrows, rstd, gain, dY, idx, dX, gain_partial);
        else
            hipLaunchKernelGGL((rmsnorm_bwd_scatter_kernel<true, false>), grid, block, 0, s, dxn_partial,
                               pl, R, r_dev, C, xrows, rstd, gain, dY, idx, dX, gain_partial);
    } else {
        if (gg)
            hipLaunchKernelGGL((rmsnorm_bwd_scatter_kernel<false, true>), grid, block, 0, s, dxn_partial,
                               pl, R, r_dev, C, xrows, rstd, gain, dY, idx, dX, gain_partial);
        else
            hipLaunchKernelGGL((rmsnorm_bwd_scatter_kernel<false, false>), grid, block, 0, s, dxn_partial,
                               pl, R, r_dev, C, xrows, rstd, gain, dY, idx, dX, gain_partial);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && gg) {
        const dim3 cols((C + 31) / 32);
        if ((R + GAIN_STRIP - 1) / GAIN_STRIP <= COLSUM_FEW_ROWS)
            hipLaunchKernelGGL(gain_grad_reduce_kernel<COLSUM_LANES_FEW>, cols, dim3(32 * COLSUM_LANES_FEW), 0, s,
                               gain_partial, R, r_dev, C, dgain, accumulate);
        else
            hipLaunchKernelGGL(gain_grad_reduce_kernel<COLSUM_LANES>, cols, dim3(32 * COLSUM_LANES), 0, s, gain_partial, R,
                               r_dev, C, dgain, accumulate);
        e = hipGetLastError();
    }
    profile_mark_end(KC_RMSNORM_BWD, s);
    return e;
}

// ---- zero fill (a kernel, so that it can be captured in a HIP graph) -----------------------
__global__ __launch_bounds__(256) void fill_zero_kernel(u32x4* p, size_t chunks) {
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t stride = (size_t)gridDim.x * 256;
    u32x4 z = {0u, 0u, 0u, 0u};
    for (; i < chunks; i += stride) p[i] = z;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    size_t chunks = bytes / 16;     // callers pass multiples of 16
    size_t blocks = (chunks + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    profile_mark_begin(KC_FILL, s);
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                       static_cast<u32x4*>(p), chunks);
    profile_mark_end(KC_FILL, s);
    return hipGetLastError();
}

}  // namespace skipffn
