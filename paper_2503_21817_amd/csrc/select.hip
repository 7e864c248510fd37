// Retained-token selection for a backbone without global / local views (Section 4.1): per
// sequence, the n visual tokens whose features are most similar (cosine) to the CLS token
// are retained (mask 0), the rest are skipped (mask 1).  Two kernels: similarities (features read
// once), then per sequence a search for the cut between the retained and the skipped ones (a token is
// retained iff fewer than n tokens beat it; equal similarities: the lower index wins; a NaN
// similarity loses to every number), which gives the unique answer for the similarities computed; in a short
// sequence every token's rank is counted instead.
#include "kernels.hpp"
#include "segments.hpp"
#include "topk.hpp"

namespace skipffn {

constexpr int SEL_THREADS = 256;

// ---- cosine similarity to the sequence's CLS row, four tokens per wavefront ----------------
// Bound by latency (a few MB in all): the rows of all four tokens and the CLS row, two column steps of
// each, are loaded together; |cls|^2 comes from the CLS row that every wavefront reads anyway.
__global__ __launch_bounds__(SEL_THREADS) void cls_sim_kernel(
    const bf16_t* __restrict__ feat, const bf16_t* __restrict__ cls, const int32_t* __restrict__ seq_off,
    int B, int n_feat, int Cv, float* __restrict__ sim) {
    int b, t0, nt;
    if (!locate_chunk<SEL_CH, false>(seq_off, B, n_feat, (int)blockIdx.x, b, t0, nt)) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int chunks = Cv >> 3;
    const u32x4* pc = reinterpret_cast<const u32x4*>(cls + (int64_t)b * Cv);
    // tokens 4 wv .. 4 wv + 3 of the chunk (an absent one reads the chunk's first row)
    const u32x4* rows[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = wv * 4 + k;
        rows[k] = reinterpret_cast<const u32x4*>(feat + (int64_t)(t0 + (i < nt ? i : 0)) * Cv);
    }
    float dot[4] = {0.f, 0.f, 0.f, 0.f}, sq[4] = {0.f, 0.f, 0.f, 0.f}, cc = 0.0f;
    auto add = [&](const u32x4& yr, const u32x4 (&xr)[4]) {
        float y[8];
        unpack8s(yr, y);
#pragma unroll
        for (int j = 0; j < 8; ++j) cc += y[j] * y[j];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float x[8];
            unpack8s(xr[k], x);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                dot[k] += x[j] * y[j];
                sq[k] += x[j] * x[j];
            }
        }
    };
    int c = lane;
    for (; c + 64 < chunks; c += 128) {
        u32x4 x0[4], x1[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) { x0[k] = rows[k][c]; x1[k] = rows[k][c + 64]; }
        const u32x4 y0 = pc[c], y1 = pc[c + 64];
        add(y0, x0);
        add(y1, x1);
    }
    if (c < chunks) {
        u32x4 x0[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x0[k] = rows[k][c];
        add(pc[c], x0);
    }
    const float cls_norm = sqrtf(wave_sum(cc));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float d = wave_sum(dot[k]), q = wave_sum(sq[k]);
        if (lane == 0 && wv * 4 + k < nt) {
            const float den = sqrtf(q) * cls_norm;
            sim[t0 + wv * 4 + k] = den > 0.0f ? d / den : 0.0f;
        }
    }
}

// ---- mask: one workgroup per sequence searches the cut (topk.hpp) ----------------------------------
// Up to SEL_MAXV * 1024 tokens the keys stay in registers; a longer sequence reads its similarities
// again for every cut of the search (from L2).  Up to 256 tokens, four threads to each, counting the tokens that beat it
// takes less than the search's barriers.
constexpr int SEL_MAXV = 16;
constexpr int SEL_RANK_MAX = TOPK_THREADS / 4;

__global__ __launch_bounds__(TOPK_THREADS) void select_topn_kernel(
    const float* __restrict__ sim, const int32_t* __restrict__ seq_off, int n_feat, int n_keep,
    const int32_t* __restrict__ n_keep_dev, uint8_t* __restrict__ mask,
    const int32_t* __restrict__ token_pos, uint8_t* __restrict__ skip_mask, int64_t T) {
    __shared__ TopkShared sh;
    __shared__ uint32_t keys[SEL_RANK_MAX];
    const int b = blockIdx.x, tid = threadIdx.x;
    int lo, hi;
    seg_bounds(seq_off, b, n_feat, lo, hi);
    const int n = hi - lo;
    if (n <= 0) return;
    const int keep = n_keep_dev != nullptr ? n_keep_dev[b] : n_keep;
    const int nv = (n + TOPK_THREADS - 1) / TOPK_THREADS;
    const bool scatter = skip_mask != nullptr && token_pos != nullptr;
    auto put = [&](int t, bool in, int pos) {
        const uint8_t m = in ? 0 : 1;
        mask[lo + t] = m;
        if (scatter && (int64_t)pos >= 0 && (int64_t)pos < T) skip_mask[pos] = m;
    };
    if (n <= SEL_RANK_MAX) {                                   // uniform
        if (tid < n) keys[tid] = rank_key<true>(sim[lo + tid]);
        const int t = tid >> 2;
        const int pos = scatter && t < n ? token_pos[lo + t] : -1;
        __syncthreads();
        const bool in = rank_in_lds(keys, n) < keep;
        if (t < n && (tid & 3) == 0) put(t, in, pos);
        return;
    }
    const bool all_or_none = keep <= 0 || keep >= n;          // uniform
    if (nv <= SEL_MAXV && !all_or_none) {
        uint32_t key[SEL_MAXV];
        int pos[SEL_MAXV], before[SEL_MAXV];
#pragma unroll
        for (int i = 0; i < SEL_MAXV; ++i)
            if (i < nv) {
                const int t = i * TOPK_THREADS + tid;
                key[i] = t < n ? rank_key<true>(sim[lo + t]) : TOPK_NONE;
                pos[i] = scatter && t < n ? token_pos[lo + t] : -1;
                before[i] = 0;
            }
        const TopkCut cut = topk_cut<SEL_MAXV>([&](int i) { return key[i]; }, nv, keep, sh);
        if (cut.ties > 0)
            topk_prefix<SEL_MAXV>([&](int i) { return key[i] == cut.cut && i * TOPK_THREADS + tid < n; }, nv, sh, before);
#pragma unroll
        for (int i = 0; i < SEL_MAXV; ++i)
            if (i < nv) {
                const int t = i * TOPK_THREADS + tid;
                if (t < n) put(t, key[i] < cut.cut || (key[i] == cut.cut && before[i] < cut.ties), pos[i]);
            }
        return;
    }
    auto key_of = [&](int t) { return t < n ? rank_key<true>(sim[lo + t]) : TOPK_NONE; };
    TopkCut cut{keep > 0 ? TOPK_NONE : 0u, keep > 0 ? n : 0};  // everything (every key <= NONE), or nothing
    if (!all_or_none) cut = topk_cut<0>([&](int i) { return key_of(i * TOPK_THREADS + tid); }, nv, keep, sh);
    int ties_before = 0;                                       // entries equal to the cut in earlier chunks
    for (int i = 0; i < nv; ++i) {
        const int t = i * TOPK_THREADS + tid;
        const uint32_t key = key_of(t);
        int before[1] = {0};
        if (cut.ties > 0 && !all_or_none) {
            const int here = topk_prefix<1>([&](int) { return key == cut.cut && t < n; }, 1, sh, before);
            before[0] += ties_before;
            ties_before += here;
        }
        if (t < n) put(t, key < cut.cut || (key == cut.cut && before[0] < cut.ties), scatter ? token_pos[lo + t] : -1);
    }
}

hipError_t launch_select_retained(const bf16_t* feat, const bf16_t* cls, const int32_t* seq_off,
                                  int64_t n_feat, int B, int Cv, int n_keep, const int32_t* n_keep_dev,
                                  uint8_t* mask, float* sim, const int32_t* token_pos,
                                  uint8_t* skip_mask, int64_t T, hipStream_t s) {
    if (B <= 0 || n_feat <= 0) return hipSuccess;
    const unsigned nq = (unsigned)((n_feat + SEL_CH - 1) / SEL_CH + B);
    profile_mark_begin(KC_SELECT, s);
    hipLaunchKernelGGL(cls_sim_kernel, dim3(nq), dim3(SEL_THREADS), 0, s, feat, cls, seq_off, B,
                       (int)n_feat, Cv, sim);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(select_topn_kernel, dim3((unsigned)B), dim3(TOPK_THREADS), 0, s, sim, seq_off,
                           (int)n_feat, n_keep, n_keep_dev, mask, token_pos, skip_mask, T);
        e = hipGetLastError();
    }
    profile_mark_end(KC_SELECT, s);
    return e;
}

}  // namespace skipffn
