// Adaptive summary layer (Section 4.2, the summary-token equation):
//     x^s = softmax(X w^T)^T X        X = a set of visual tokens [n, C], w [C]
// one summary row per token set, forward and backward.  Memory-bound: X is read once from
// HBM per pass (a second read of the same rows inside a workgroup hits L2).
//
// A token set s is the rows tok[seg[s] .. seg[s+1]) of the hidden states; tok and seg live
// on the device, so set sizes need not be known on the host.  Every set is cut into chunks
// of SUM_CH tokens, one workgroup per chunk ("flash" style): a chunk produces its own
// maximum m, denominator d = sum exp(s_t - m) and unnormalised weighted row sum; a second
// small kernel merges the chunks of a set.  The launch covers the upper bound
// ceil(n_tok / SUM_CH) + S chunks; workgroups past the real count exit.
#include "colsum.hpp"
#include "kernels.hpp"
#include "segments.hpp"

namespace skipffn {

constexpr int SUM_THREADS = 256;
static_assert(SUM_CH == 16, "four wavefronts of four tokens");
constexpr float kNoScore = -3.0e38f;      // score of an out-of-range token index: weight 0

// dots of four rows of `hidden` (row index < 0: skipped, result 0) with the row `b`, by one
// wavefront.  Loads are issued for two column steps of all four rows before any arithmetic, so
// that ten 16-byte loads per lane are in flight (a skipped row reads row 0: always in bounds).
__device__ __forceinline__ void wave_dot4(const bf16_t* __restrict__ hidden, int C, const int* rows,
                                          const bf16_t* __restrict__ b, int chunks, int lane, float* out) {
    const u32x4* pb = reinterpret_cast<const u32x4*>(b);
    const u32x4* pr[4];
    float scale[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        pr[k] = reinterpret_cast<const u32x4*>(hidden + (int64_t)(rows[k] >= 0 ? rows[k] : 0) * C);
        scale[k] = rows[k] >= 0 ? 1.0f : 0.0f;
    }
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    int c = lane;
    for (; c + 64 < chunks; c += 128) {
        u32x4 x0[4], x1[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) { x0[k] = pr[k][c]; x1[k] = pr[k][c + 64]; }
        const u32x4 w0 = pb[c], w1 = pb[c + 64];
        float y0[8], y1[8];
        unpack8s(w0, y0);
        unpack8s(w1, y1);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float a[8], d[8];
            unpack8s(x0[k], a);
            unpack8s(x1[k], d);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[k] += a[j] * y0[j] + d[j] * y1[j];
        }
    }
    if (c < chunks) {
        u32x4 x0[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x0[k] = pr[k][c];
        float y0[8];
        unpack8s(pb[c], y0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float a[8];
            unpack8s(x0[k], a);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[k] += a[j] * y0[j];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) out[k] = wave_sum(acc[k]) * scale[k];
}

// ---- forward, per chunk ---------------------------------------------------------------------
template <bool FEW_SETS>
__global__ __launch_bounds__(SUM_THREADS) void summary_chunk_fwd_kernel(
    const bf16_t* __restrict__ hidden, int64_t T, int C, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ seg, int S, int n_tok, const bf16_t* __restrict__ w,
    float* __restrict__ scores, float* __restrict__ part_acc, float* __restrict__ part_md) {
    __shared__ float sc[SUM_CH];
    __shared__ int rowid[SUM_CH];
    int s, t0, nt;
    if (!locate_chunk<SUM_CH, FEW_SETS>(seg, S, n_tok, (int)blockIdx.x, s, t0, nt)) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int chunks = C >> 3;
    // phase A: scores s_t = X_t . w, four tokens per wavefront (SUM_CH = 16 = 4 waves x 4)
    {
        int rows[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = wv * 4 + k;
            int row = -1;
            if (i < nt) {
                row = tok[t0 + i];
                if ((uint32_t)row >= (uint32_t)T) row = -1;
            }
            rows[k] = row;
        }
        float v[4];
        wave_dot4(hidden, C, rows, w, chunks, lane, v);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = wv * 4 + k;
                if (i < nt) {
                    const float sv = rows[k] >= 0 ? v[k] : kNoScore;
                    sc[i] = sv;
                    rowid[i] = rows[k];
                    if (scores != nullptr) scores[t0 + i] = sv;
                }
            }
        }
    }
    __syncthreads();
    float m = kNoScore;
    for (int i = 0; i < nt; ++i) m = fmaxf(m, sc[i]);
    float e[SUM_CH];
    float d = 0.0f;
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i) {
        e[i] = (i < nt && rowid[i] >= 0) ? __expf(sc[i] - m) : 0.0f;
        d += e[i];
    }
    // phase B: every thread owns 16-byte column chunks: sum_t e_t X_t.  The sixteen row loads of
    // a chunk are unconditional and issued together; an absent token reads zeros, no row: its weight 0 times
    // an infinity or a NaN would not be 0.
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(hidden, (uint32_t)(T * C * 2));
    uint32_t ro[SUM_CH];
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i)
        ro[i] = i < nt && rowid[i] >= 0 ? (uint32_t)rowid[i] * (uint32_t)C * 2u : kOobOffset;
    float* pa = part_acc + (int64_t)blockIdx.x * C;
    for (int c = tid; c < chunks; c += SUM_THREADS) {
        u32x4 xr[SUM_CH];
#pragma unroll
        for (int i = 0; i < SUM_CH; ++i) xr[i] = buf_load16(rx, ro[i] + (uint32_t)c * 16u);
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
        for (int i = 0; i < SUM_CH; ++i) {
            float x[8];
            unpack8s(xr[i], x);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += e[i] * x[j];
        }
        f32x4 lo = {acc[0], acc[1], acc[2], acc[3]}, hi = {acc[4], acc[5], acc[6], acc[7]};
        *reinterpret_cast<f32x4*>(pa + c * 8) = lo;
        *reinterpret_cast<f32x4*>(pa + c * 8 + 4) = hi;
    }
    if (tid == 0) {
        part_md[2 * blockIdx.x] = m;
        part_md[2 * blockIdx.x + 1] = d;
    }
}

// The same with the rows of the chunk in registers, V <= 2 pieces of 8 columns a thread (C <= 4096): they are read once, all at the
// same time, and up to 768 chunks run at once.  Sixteen products are summed over the lanes together, half of them given away at
// every step.  C = 4096, held / read again from L2, us: 9216 tokens 18.0 / 26.5, 33600 tokens 66.8 / 96.0, 576 tokens 7.3 / 8.7.
// Three workgroups a CU leave a wavefront 168 registers; past 2048 columns four more are spilled (20 bytes a lane of scratch).
template <bool FEW_SETS, int V, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 3) void summary_held_fwd_kernel(
    const bf16_t* __restrict__ hidden, int64_t T, int C, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ seg, int S, int n_tok, const bf16_t* __restrict__ w,
    float* __restrict__ scores, float* __restrict__ part_acc, float* __restrict__ part_md) {
    constexpr int THREADS = WAVES * 64;
    __shared__ float dots[WAVES][SUM_CH];
    int s, t0, nt;
    if (!locate_chunk<SUM_CH, FEW_SETS>(seg, S, n_tok, (int)blockIdx.x, s, t0, nt)) return;   // uniform over the workgroup
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int chunks = C >> 3;
    t0 = __builtin_amdgcn_readfirstlane(t0);
    nt = __builtin_amdgcn_readfirstlane(nt);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(hidden, (uint32_t)(T * C * 2)), rw = make_rsrc(w, (uint32_t)C * 2);
    uint32_t col[V];
#pragma unroll
    for (int v = 0; v < V; ++v) col[v] = tid + v * THREADS < chunks ? (uint32_t)(tid + v * THREADS) * 16u : kOobOffset;
    int row[SUM_CH];                                     // -1: absent, reads row 0
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i) {
        const int r = i < nt ? tok[t0 + i] : -1;
        row[i] = __builtin_amdgcn_readfirstlane((uint32_t)r < (uint32_t)T ? r : -1);
    }
    u32x4 x[SUM_CH][V], wr[V];
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v)
            x[i][v] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)col[v], (int)((uint32_t)(row[i] >= 0 ? row[i] : 0) * (uint32_t)C * 2u), 0);
#pragma unroll
    for (int v = 0; v < V; ++v) wr[v] = buf_load16(rw, col[v]);
    float p[SUM_CH];
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i) p[i] = 0.0f;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        float y[8];
        unpack8s(wr[v], y);
#pragma unroll
        for (int i = 0; i < SUM_CH; ++i) {
            float f[8];
            unpack8s(x[i][v], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) p[i] += f[j] * y[j];
        }
    }
    // lane l ends with the sum over the lanes of token (l / 4) with its bits in the order the halves were given away
#pragma unroll
    for (int half = SUM_CH / 2, off = 32; half >= 1; half >>= 1, off >>= 1) {
        const bool upper = (lane & off) != 0;
#pragma unroll
        for (int i = 0; i < SUM_CH / 2; ++i)
            if (i < half) {
                const float give = upper ? p[i] : p[i + half], keep = upper ? p[i + half] : p[i];
                p[i] = keep + __shfl_xor(give, off, 64);
            }
    }
    p[0] += __shfl_xor(p[0], 2, 64);
    p[0] += __shfl_xor(p[0], 1, 64);
    if ((lane & 3) == 0) dots[wv][lane >> 2] = p[0];
    // the rows stay packed: their values unpacked for the products are not to be kept for the sums
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) asm volatile("" : "+v"(x[i][v]));
    __syncthreads();
    float e[SUM_CH];
    float m = kNoScore;
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i) {
        float dot = 0.0f;
#pragma unroll
        for (int q = 0; q < WAVES; ++q) dot += dots[q][i];
        e[i] = row[i] >= 0 ? dot : kNoScore;
        m = i < nt ? fmaxf(m, e[i]) : m;
    }
    if (scores != nullptr && tid < nt) {
        float own = kNoScore;
#pragma unroll
        for (int i = 0; i < SUM_CH; ++i) own = tid == i ? e[i] : own;
        scores[t0 + tid] = own;
    }
    float d = 0.0f;
#pragma unroll
    for (int i = 0; i < SUM_CH; ++i) {
        e[i] = row[i] >= 0 ? __expf(e[i] - m) : 0.0f;
        d += e[i];
    }
    float* pa = part_acc + (int64_t)blockIdx.x * C;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int c = tid + v * THREADS;
        if (c >= chunks) continue;
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
#pragma unroll
        for (int i = 0; i < SUM_CH; ++i) {
            if (row[i] < 0) continue;                    // uniform; weight 0 times an infinity or a NaN of row 0 is not 0
            float f[8];
            unpack8s(x[i][v], f);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += e[i] * f[j];
        }
        *reinterpret_cast<f32x4*>(pa + c * 8) = f32x4{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<f32x4*>(pa + c * 8 + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
    }
    if (tid == 0) {
        part_md[2 * blockIdx.x] = m;
        part_md[2 * blockIdx.x + 1] = d;
    }
}

// ---- forward, merge the chunks of a set -------------------------------------------------------
// grid (S, ceil(C / 8 / 64)): 64 column chunks x 4 interleaved chunk lanes per workgroup.
// out bf16 [S, C]; xs_f32 [S, C] and lse [S] for the backward.
// Bound by latency: the longest set's chunks, a quarter of them in a chain of loads.  Forward, us, one chunk / four of a lane in
// flight:  sets of 2 and 5000 tokens, C = 512 32 / 17, C = 4096 36.6 / 23.4, C = 8192 51.5 / 39.1;  16 of 576, C = 4096 25.2 / 23.3;
// 500 sets of 20 tokens even (eight in flight take 78 registers there: 22.1 / 23.6 at C = 2048).
constexpr int MERGE_Q = 256;              // chunk scales staged in LDS per pass
template <bool FEW_SETS>
__global__ __launch_bounds__(SUM_THREADS) void summary_merge_fwd_kernel(
    int C, const int32_t* __restrict__ seg, int n_tok, int nq_max, const float* __restrict__ part_acc,
    const float* __restrict__ part_md, bf16_t* __restrict__ out, float* __restrict__ xs_f32,
    float* __restrict__ lse) {
    __shared__ float scale[MERGE_Q];
    __shared__ float red[4];
    __shared__ float part4[4][64][8];
    const int s = blockIdx.x;
    const int tid = threadIdx.x;
    int q0, q1;
    chunk_range<SUM_CH, FEW_SETS>(seg, s, n_tok, nq_max, q0, q1);
    // global maximum and denominator of the set
    float M = kNoScore;
    for (int q = q0 + tid; q < q1; q += SUM_THREADS) M = fmaxf(M, part_md[2 * q]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    if ((tid & 63) == 0) red[tid >> 6] = M;
    __syncthreads();
    M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float dpart = 0.0f;
    for (int q = q0 + tid; q < q1; q += SUM_THREADS) dpart += part_md[2 * q + 1] * __expf(part_md[2 * q] - M);
    const float D = block_sum256(dpart, red);
    const float inv = D > 0.0f ? 1.0f / D : 0.0f;     // empty set: zero row
    const int cx = tid & 63, sy = tid >> 6;
    const int c = blockIdx.y * 64 + cx;
    const bool cok = c < (C >> 3);
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
    for (int qb = q0; qb < q1; qb += MERGE_Q) {
        const int nqb = q1 - qb < MERGE_Q ? q1 - qb : MERGE_Q;
        __syncthreads();
        if (tid < nqb) scale[tid] = __expf(part_md[2 * (qb + tid)] - M);
        __syncthreads();
        if (cok) {
            const float* pa = part_acc + (int64_t)qb * C + c * 8;
            auto add = [&](float sc, const f32x4& lo, const f32x4& hi) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[j] += sc * lo[j];
                    acc[4 + j] += sc * hi[j];
                }
            };
            int k = sy;
            for (; k + 12 < nqb; k += 16) {               // four chunks in flight, added in order
                f32x4 lo[4], hi[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    lo[u] = *reinterpret_cast<const f32x4*>(pa + (int64_t)(k + 4 * u) * C);
                    hi[u] = *reinterpret_cast<const f32x4*>(pa + (int64_t)(k + 4 * u) * C + 4);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) add(scale[k + 4 * u], lo[u], hi[u]);
            }
            for (; k < nqb; k += 4)
                add(scale[k], *reinterpret_cast<const f32x4*>(pa + (int64_t)k * C), *reinterpret_cast<const f32x4*>(pa + (int64_t)k * C + 4));
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) part4[sy][cx][j] = acc[j];
    __syncthreads();
    if (sy == 0 && cok) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            acc[j] = ((part4[0][cx][j] + part4[1][cx][j]) + (part4[2][cx][j] + part4[3][cx][j])) * inv;
        u32x4 pk;
#pragma unroll
        for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(acc[2 * j], acc[2 * j + 1]);
        *reinterpret_cast<u32x4*>(out + (int64_t)s * C + c * 8) = pk;
        if (xs_f32 != nullptr) {
            f32x4 lo = {acc[0], acc[1], acc[2], acc[3]}, hi = {acc[4], acc[5], acc[6], acc[7]};
            *reinterpret_cast<f32x4*>(xs_f32 + (int64_t)s * C + c * 8) = lo;
            *reinterpret_cast<f32x4*>(xs_f32 + (int64_t)s * C + c * 8 + 4) = hi;
        }
    }
    if (lse != nullptr && blockIdx.y == 0 && tid == 0) lse[s] = D > 0.0f ? M + __logf(D) : kNoScore;
}

// ---- backward, per chunk ------------------------------------------------------------------------
// With p_t = exp(s_t - lse), dp_t = g . X_t and delta = g . x^s (= sum_u p_u dp_u):
//   ds_t = p_t (dp_t - delta);  dX_t = p_t g + ds_t w  (added to grad_hidden row t);
//   dw = sum_t ds_t X_t  (per chunk into part_dw, summed by summary_dw_reduce_kernel)
template <bool FEW_SETS>
__global__ __launch_bounds__(SUM_THREADS) void summary_chunk_bwd_kernel(
    const bf16_t* __restrict__ hidden, int64_t T, int C, const int32_t* __restrict__ tok,
    const int32_t* __restrict__ seg, int S, int n_tok, const bf16_t* __restrict__ w,
    const float* __restrict__ xs_f32, const float* __restrict__ scores, const float* __restrict__ lse,
    const bf16_t* __restrict__ gout, bf16_t* grad_hidden, float* __restrict__ part_dw) {
    __shared__ float pp[SUM_CH], dss[SUM_CH];
    __shared__ int rowid[SUM_CH];
    __shared__ float red[4];
    int s, t0, nt;
    if (!locate_chunk<SUM_CH, FEW_SETS>(seg, S, n_tok, (int)blockIdx.x, s, t0, nt)) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int chunks = C >> 3;
    const bf16_t* g = gout + (int64_t)s * C;
    // delta = g . x^s
    float dl = 0.0f;
    for (int c = tid; c < chunks; c += SUM_THREADS) {
        float gg[8];
        unpack8s(*reinterpret_cast<const u32x4*>(g + c * 8), gg);
        const float* xp = xs_f32 + (int64_t)s * C + c * 8;
        f32x4 lo = *reinterpret_cast<const f32x4*>(xp), hi = *reinterpret_cast<const f32x4*>(xp + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) dl += gg[j] * lo[j] + gg[4 + j] * hi[j];
    }
    const float delta = block_sum256(dl, red);
    const float L = lse[s];
    {
        int rows[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = wv * 4 + k;
            int row = -1;
            if (i < nt) {
                row = tok[t0 + i];
                if ((uint32_t)row >= (uint32_t)T) row = -1;
            }
            rows[k] = row;
        }
        float dp[4];
        wave_dot4(hidden, C, rows, g, chunks, lane, dp);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = wv * 4 + k;
                if (i < nt) {
                    const float p = rows[k] >= 0 ? __expf(scores[t0 + i] - L) : 0.0f;
                    pp[i] = p;
                    dss[i] = p * (dp[k] - delta);
                    rowid[i] = rows[k];
                }
            }
        }
    }
    __syncthreads();
    float* pd = part_dw + (int64_t)blockIdx.x * C;
    for (int c = tid; c < chunks; c += SUM_THREADS) {
        float gg[8], ww[8], dw[8];
        unpack8s(*reinterpret_cast<const u32x4*>(g + c * 8), gg);
        unpack8s(*reinterpret_cast<const u32x4*>(w + c * 8), ww);
#pragma unroll
        for (int j = 0; j < 8; ++j) dw[j] = 0.0f;
        // eight tokens at a time: all loads first (the rows are distinct, which the compiler
        // cannot know, so a plain read-modify-write loop would serialise on memory latency)
#pragma unroll
        for (int i0 = 0; i0 < SUM_CH; i0 += 8) {
            u32x4 xr[8], gr[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int i = i0 + k;
                if (i < nt && rowid[i] >= 0) {
                    const int64_t o = (int64_t)rowid[i] * C + c * 8;
                    xr[k] = *reinterpret_cast<const u32x4*>(hidden + o);
                    gr[k] = *reinterpret_cast<const u32x4*>(grad_hidden + o);
                }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int i = i0 + k;
                if (i < nt && rowid[i] >= 0) {
                    float x[8], gh[8];
                    unpack8s(xr[k], x);
                    unpack8s(gr[k], gh);
                    const float p = pp[i], ds = dss[i];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        gh[j] += p * gg[j] + ds * ww[j];
                        dw[j] += ds * x[j];
                    }
                    u32x4 pk;
#pragma unroll
                    for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(gh[2 * j], gh[2 * j + 1]);
                    *reinterpret_cast<u32x4*>(grad_hidden + (int64_t)rowid[i] * C + c * 8) = pk;
                }
            }
        }
        f32x4 lo = {dw[0], dw[1], dw[2], dw[3]}, hi = {dw[4], dw[5], dw[6], dw[7]};
        *reinterpret_cast<f32x4*>(pd + c * 8) = lo;
        *reinterpret_cast<f32x4*>(pd + c * 8 + 4) = hi;
    }
}

// dw[c] (+)= sum over all chunks of part_dw[q][c]
template <int LANES, bool FEW_SETS>
__global__ __launch_bounds__(32 * LANES) void summary_dw_reduce_kernel(
    const float* __restrict__ part_dw, const int32_t* __restrict__ seg, int S, int n_tok, int nq_max,
    int C, float* __restrict__ dw, int accumulate) {
    int q0, q1;
    chunk_range<SUM_CH, FEW_SETS>(seg, S - 1, n_tok, nq_max, q0, q1);           // q1 = total number of chunks
    column_sum<LANES>(part_dw, q1, C, dw, accumulate);
}

// ---- launchers -----------------------------------------------------------------------------------
int64_t summary_max_chunks(int64_t n_tok, int64_t S) { return (n_tok + SUM_CH - 1) / SUM_CH + S; }

template <bool FEW_SETS>
static hipError_t summary_forward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok, const int32_t* seg, int64_t n_tok,
                                  int S, const bf16_t* w, bf16_t* out, float* scores, float* lse, float* xs_f32,
                                  float* part_acc, float* part_md, hipStream_t s) {
    const unsigned nq = (unsigned)summary_max_chunks(n_tok, S);
    if (C <= 1024)
        hipLaunchKernelGGL((summary_held_fwd_kernel<FEW_SETS, 1, 2>), dim3(nq), dim3(128), 0, s, hidden, T, C, tok, seg, S, (int)n_tok,
                           w, scores, part_acc, part_md);
    else if (C <= 2048)
        hipLaunchKernelGGL((summary_held_fwd_kernel<FEW_SETS, 1, 4>), dim3(nq), dim3(256), 0, s, hidden, T, C, tok, seg, S, (int)n_tok,
                           w, scores, part_acc, part_md);
    else if (C <= 4096)
        hipLaunchKernelGGL((summary_held_fwd_kernel<FEW_SETS, 2, 4>), dim3(nq), dim3(256), 0, s, hidden, T, C, tok, seg, S, (int)n_tok,
                           w, scores, part_acc, part_md);
    else
        hipLaunchKernelGGL(summary_chunk_fwd_kernel<FEW_SETS>, dim3(nq), dim3(SUM_THREADS), 0, s, hidden, T, C, tok, seg,
                           S, (int)n_tok, w, scores, part_acc, part_md);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 grid((unsigned)S, (unsigned)(((C >> 3) + 63) / 64));
    hipLaunchKernelGGL(summary_merge_fwd_kernel<FEW_SETS>, grid, dim3(SUM_THREADS), 0, s, C, seg, (int)n_tok, (int)nq,
                       part_acc, part_md, out, xs_f32, lse);
    return hipGetLastError();
}

hipError_t launch_summary_forward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok,
                                  const int32_t* seg, int64_t n_tok, int S, const bf16_t* w,
                                  bf16_t* out, float* scores, float* lse, float* xs_f32,
                                  float* part_acc, float* part_md, hipStream_t s) {
    if (S <= 0) return hipSuccess;
    profile_mark_begin(KC_SUMMARY_FWD, s);
    const hipError_t e = S <= SEG_FEW_SETS
        ? summary_forward<true>(hidden, T, C, tok, seg, n_tok, S, w, out, scores, lse, xs_f32, part_acc, part_md, s)
        : summary_forward<false>(hidden, T, C, tok, seg, n_tok, S, w, out, scores, lse, xs_f32, part_acc, part_md, s);
    profile_mark_end(KC_SUMMARY_FWD, s);
    return e;
}

template <bool FEW_SETS>
static hipError_t summary_backward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok, const int32_t* seg, int64_t n_tok,
                                   int S, const bf16_t* w, const float* xs_f32, const float* scores, const float* lse,
                                   const bf16_t* gout, bf16_t* grad_hidden, float* part_dw, float* dw, int accumulate,
                                   hipStream_t s) {
    const unsigned nq = (unsigned)summary_max_chunks(n_tok, S);
    hipLaunchKernelGGL(summary_chunk_bwd_kernel<FEW_SETS>, dim3(nq), dim3(SUM_THREADS), 0, s, hidden, T, C, tok, seg,
                       S, (int)n_tok, w, xs_f32, scores, lse, gout, grad_hidden, part_dw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 cols((unsigned)((C + 31) / 32));
    if (nq <= COLSUM_FEW_ROWS)
        hipLaunchKernelGGL((summary_dw_reduce_kernel<COLSUM_LANES_FEW, FEW_SETS>), cols, dim3(32 * COLSUM_LANES_FEW), 0, s,
                           part_dw, seg, S, (int)n_tok, (int)nq, C, dw, accumulate);
    else
        hipLaunchKernelGGL((summary_dw_reduce_kernel<COLSUM_LANES, FEW_SETS>), cols, dim3(32 * COLSUM_LANES), 0, s, part_dw,
                           seg, S, (int)n_tok, (int)nq, C, dw, accumulate);
    return hipGetLastError();
}

hipError_t launch_summary_backward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok,
                                   const int32_t* seg, int64_t n_tok, int S, const bf16_t* w,
                                   const float* xs_f32, const float* scores, const float* lse,
                                   const bf16_t* gout, bf16_t* grad_hidden, float* part_dw, float* dw,
                                   int accumulate, hipStream_t s) {
    if (S <= 0) return hipSuccess;
    profile_mark_begin(KC_SUMMARY_BWD, s);
    const hipError_t e = S <= SEG_FEW_SETS
        ? summary_backward<true>(hidden, T, C, tok, seg, n_tok, S, w, xs_f32, scores, lse, gout, grad_hidden, part_dw, dw, accumulate, s)
        : summary_backward<false>(hidden, T, C, tok, seg, n_tok, S, w, xs_f32, scores, lse, gout, grad_hidden, part_dw, dw, accumulate, s);
    profile_mark_end(KC_SUMMARY_BWD, s);
    return e;
}

}  // namespace skipffn
