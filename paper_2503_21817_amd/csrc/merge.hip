// Token merge of the skipped (local) visual tokens (Section 4.1, the three bullet points):
//   1. cosine similarity between every pair of tokens of a set, averaged per token;
//   2. the k tokens of lowest average similarity are kept;
//   3. every other token is merged into the kept token it is most similar to (plain mean).
// The similarity matrices are dense contractions and run on the matrix cores (normalised rows
// times their transpose, fp32 out, all sets of a group in one grid); everything else is
// small and memory-bound and also runs for a whole group of sets per launch (blockIdx.y = set;
// the sets' row offsets travel in the kernel arguments, so nothing is copied to the device).
// Decisions that depend on floating point (which tokens are kept, where a token goes) are
// taken on the float32 averages / similarities computed here, with ties to the lower index,
// so they are unique for those values.  A token with a non-finite feature has NaN similarities:
// its average ranks after every number, so exactly min(k, n) tokens are kept whatever the input;
// a token whose similarities are all NaN goes to no slot (assign = -1) and gets a zero gradient.
#include "kernels.hpp"
#include "segments.hpp"
#include "slabloop.hpp"
#include "topk.hpp"

namespace skipffn {

constexpr int MG_THREADS = 256;

// ---- Xn = X / |X| (a zero row stays zero), one workgroup per row ------------------------------
__global__ __launch_bounds__(MG_THREADS) void row_normalize_kernel(const bf16_t* __restrict__ x, int C,
                                                                   bf16_t* __restrict__ xn) {
    __shared__ float red[4];
    const int64_t r = blockIdx.x;
    const int tid = threadIdx.x, chunks = C >> 3;
    const u32x4* src = reinterpret_cast<const u32x4*>(x + r * C);
    u32x4* dst = reinterpret_cast<u32x4*>(xn + r * C);
    float ss = 0.0f;
    for (int c = tid; c < chunks; c += MG_THREADS) {
        float f[8];
        unpack8s(src[c], f);
#pragma unroll
        for (int j = 0; j < 8; ++j) ss += f[j] * f[j];
    }
    ss = block_sum256(ss, red);
    const float inv = ss > 0.0f ? 1.0f / sqrtf(ss) : 0.0f;
    for (int c = tid; c < chunks; c += MG_THREADS) {
        float f[8];
        unpack8s(src[c], f);
        u32x4 pk;
#pragma unroll
        for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(f[2 * j] * inv, f[2 * j + 1] * inv);
        dst[c] = pk;
    }
}

// In the kernels below: set = blockIdx.y, rows [lo, lo + n) of the token list; S_set is its
// similarity matrix [n][ld] inside the group's buffer (stride sim_stride floats per set).

// ---- S_set = Xn Xn^T, fp32 ----------------------------------------------------------------------
// S is symmetric: only the 128 x 128 tiles on and above the diagonal are computed, the others are their mirror
// images (products commute and K is summed in one order, so the values are those of the full product).  Bound by
// the loop's phases and, for one set, by how many CUs have a tile: 36 tiles per set of 1024, 171 of 2304.  On 256 x 256
// tiles of the whole square (16 and 81): 82 us at one set of 2304 x 4096, here 37; 8 sets of 1024 x 1024 33 and
// 27 us.
__global__ __launch_bounds__(SLAB_THREADS) void selfsim_kernel(const bf16_t* __restrict__ xn, SegTable st, int pairs, int C,
                                                               int ld, int64_t sim_stride, float* __restrict__ sim) {
    constexpr int TILE = 128, NL = kSlabPieces<TILE>;
    static_assert(TILE == SLAB_B_ROWS && kSlabPiecesA<TILE> == 2, "square tiles");
    // workgroups are dealt round-robin to the 8 XCDs: each gets a contiguous range of the tiles, so that few sets (or
    // few rows of a set) share its L2
    const int nb = (int)gridDim.x, xcd = (int)blockIdx.x & 7, q8 = nb >> 3, rem8 = nb & 7;
    const int b = xcd * q8 + (xcd < rem8 ? xcd : rem8) + ((int)blockIdx.x >> 3);
    const int set = b / pairs;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    // pair p = tn (tn + 1) / 2 + tm, tm <= tn
    const int p = b - set * pairs;
    int tn = (int)((sqrtf(8.0f * (float)p + 1.0f) - 1.0f) * 0.5f);
    while (tn * (tn + 1) / 2 > p) --tn;
    while ((tn + 1) * (tn + 2) / 2 <= p) ++tn;
    const int tm = p - tn * (tn + 1) / 2;
    if (tn * TILE >= n) return;                          // whole workgroup leaves together
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(xn + (int64_t)lo * C, (uint32_t)((int64_t)n * C * 2));
    uint32_t goff[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int row = 8 * (wave * 2 + (l & 1)) + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        const int gr = (l < 2 ? tm : tn) * TILE + row;
        goff[l] = gr < n ? (uint32_t)(((int64_t)gr * C + c * 8) * 2) : kOobOffset;
    }
    f32x4 acc[TILE / 32][2];
    float ss[TILE / 32];
    slab_loop<TILE, 16>(rx, rx, goff, (wave & 3) * 32, 0, (C + BK - 1) / BK, 0, C, acc, ss);
    float* S = sim + set * sim_stride;
#pragma unroll
    for (int m = 0; m < TILE / 32; ++m)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const int i = tm * TILE + (wave >> 2) * 64 + m * 16 + (lane & 15);
            const int j = tn * TILE + (wave & 3) * 32 + f * 16 + 4 * (lane >> 4);
            if (i >= n || j >= n) continue;
            // ld is a multiple of 8 >= n: a quad that begins inside the row ends inside it
            *reinterpret_cast<f32x4*>(S + (int64_t)i * ld + j) = acc[m][f];
            if (tm != tn) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j + r < n) S[(int64_t)(j + r) * ld + i] = acc[m][f][r];
            }
        }
}

hipError_t merge_init() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&selfsim_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSlabLds<128>);
}

hipError_t launch_selfsim(const bf16_t* xn, int C, const SegTable& st, int n_max, float* sim, int ld,
                          int64_t sim_stride, hipStream_t s) {
    if (st.count <= 0 || n_max <= 0) return hipSuccess;
    const int t = (n_max + 127) / 128, pairs = t * (t + 1) / 2;
    hipLaunchKernelGGL(selfsim_kernel, dim3((unsigned)(pairs * st.count)), dim3(SLAB_THREADS), kSlabLds<128>, s,
                       xn, st, pairs, C, ld, sim_stride, sim);
    return hipGetLastError();
}

// ---- avg_i = (sum_j S_ij - S_ii) / (n - 1), one wavefront per row ------------------------------
// Bound by reading S (from L2 and the memory-side cache); 16 bytes per lane and load.  Rows of S start on 32 bytes.
__global__ __launch_bounds__(MG_THREADS) void sim_rowmean_kernel(const float* __restrict__ sim, SegTable st,
                                                                 int ld, int64_t sim_stride,
                                                                 float* __restrict__ avg) {
    const int set = blockIdx.y;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const float* row = sim + set * sim_stride + (int64_t)i * ld;
    float acc = 0.0f;
    int j = lane * 4;
    for (; j + 3 < n; j += 256) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += j + e == i ? 0.0f : v[e];
    }
    for (int e = j; e < n && e < j + 4; ++e) acc += e == i ? 0.0f : row[e];      // the lane of a ragged end
    acc = wave_sum(acc);
    if (lane == 0) avg[lo + i] = n > 1 ? acc / (float)(n - 1) : 0.0f;
}

// ---- which tokens are kept, and their slots ------------------------------------------------------
// One workgroup per set: the k tokens of lowest average (topk.hpp), then the position of every kept
// token among the kept ones, in index order.  slot_of[t] = slot or -1; kept_idx[set][slot] = lo + t, -1
// padding.
constexpr int MG_MAXV = MERGE_MAX_N / TOPK_THREADS;
__global__ __launch_bounds__(TOPK_THREADS) void merge_select_kernel(const float* __restrict__ avg, SegTable st,
                                                                    int k, int set_base,
                                                                    int32_t* __restrict__ slot_of,
                                                                    int32_t* __restrict__ kept_idx) {
    __shared__ TopkShared sh;
    const int set = blockIdx.x, tid = threadIdx.x;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    int32_t* kout = kept_idx + (int64_t)(set_base + set) * k;
    for (int s = (k < n ? k : n) + tid; s < k; s += TOPK_THREADS) kout[s] = -1;
    if (n <= 0) return;
    const int nv = (n + TOPK_THREADS - 1) / TOPK_THREADS;
    uint32_t key[MG_MAXV];
    int before[MG_MAXV];
    bool in[MG_MAXV];
#pragma unroll
    for (int i = 0; i < MG_MAXV; ++i) {
        const int t = i * TOPK_THREADS + tid;
        key[i] = t < n ? rank_key<false>(avg[lo + t]) : TOPK_NONE;
        before[i] = 0;
        in[i] = k >= n && t < n;
    }
    if (k > 0 && k < n) {                        // uniform
        const TopkCut cut = topk_cut<MG_MAXV>([&](int i) { return key[i]; }, nv, k, sh);
        if (cut.ties > 0)
            topk_prefix<MG_MAXV>([&](int i) { return key[i] == cut.cut && i * TOPK_THREADS + tid < n; }, nv, sh, before);
#pragma unroll
        for (int i = 0; i < MG_MAXV; ++i)
            in[i] = i * TOPK_THREADS + tid < n && (key[i] < cut.cut || (key[i] == cut.cut && before[i] < cut.ties));
    }
    topk_prefix<MG_MAXV>([&](int i) { return in[i]; }, nv, sh, before);
#pragma unroll
    for (int i = 0; i < MG_MAXV; ++i) {
        const int t = i * TOPK_THREADS + tid;
        if (t >= n) continue;
        // exactly min(k, n) tokens are in, so a slot is below k
        slot_of[lo + t] = in[i] ? before[i] : -1;
        if (in[i]) kout[before[i]] = lo + t;
    }
}

// ---- destination of every token: own slot if kept, else the most similar kept token ----------
__global__ __launch_bounds__(MG_THREADS) void merge_assign_kernel(const float* __restrict__ sim, SegTable st,
                                                                  int ld, int64_t sim_stride,
                                                                  const int32_t* __restrict__ slot_of,
                                                                  int32_t* __restrict__ assign) {
    const int set = blockIdx.y;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    const int lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int own = slot_of[lo + i];
    if (own >= 0) {
        if (lane == 0) assign[lo + i] = own;
        return;
    }
    const float* row = sim + set * sim_stride + (int64_t)i * ld;
    float best = -3.0e38f;
    int bj = 0x7fffffff;
    // four entries of S and four slots per lane and step, two steps' loads in flight; j ascending per lane, so a tie
    // keeps the lower index
    for (int j0 = lane * 4; j0 < n; j0 += 512) {
        float v[2][4];
        int sl[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int j = j0 + h * 256;
            if (j + 3 < n) {
                const f32x4 q = *reinterpret_cast<const f32x4*>(row + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[h][e] = q[e];
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                sl[h][e] = j + e < n ? slot_of[lo + j + e] : -1;
                if (j + 3 >= n) v[h][e] = j + e < n ? row[j + e] : 0.0f;
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (sl[h][e] >= 0 && v[h][e] > best) { best = v[h][e]; bj = j0 + h * 256 + e; }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float ov = __shfl_xor(best, off, 64);
        const int oj = __shfl_xor(bj, off, 64);
        if (ov > best || (ov == best && oj < bj)) { best = ov; bj = oj; }
    }
    if (lane == 0) assign[lo + i] = bj != 0x7fffffff ? slot_of[lo + bj] : -1;
}

// ---- out[set][slot] = mean of the rows assigned to the slot, added in index order --------------
__global__ __launch_bounds__(MG_THREADS) void merge_mean_kernel(const bf16_t* __restrict__ x, SegTable st, int C,
                                                                int k, int set_base,
                                                                const int32_t* __restrict__ assign,
                                                                bf16_t* __restrict__ out) {
    constexpr int WAVES = MG_THREADS / 64, SHARE = MERGE_MAX_N / WAVES;
    __shared__ int members[WAVES][SHARE];
    __shared__ int nmem[WAVES];
    const int set = blockIdx.y, slot = blockIdx.x;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    const int kk = k < n ? k : n;
    const int tid = threadIdx.x, chunks = C >> 3;
    u32x4* dst = reinterpret_cast<u32x4*>(out + ((int64_t)(set_base + set) * k + slot) * C);
    // a workgroup takes MG_THREADS chunks of the row: the largest slot of a set ends the kernel, and its row is split
    const int c = (int)blockIdx.z * MG_THREADS + tid;
    if (slot >= kk) {                       // fewer tokens than slots: zero rows
        if (c < chunks) dst[c] = u32x4{0u, 0u, 0u, 0u};
        return;
    }
    // the slot's members, in index order: every wavefront compacts a quarter of the set with ballots, eight loads in
    // flight (one wavefront over the whole set, a load at a time: 13 of this kernel's 33 us at 2304 tokens)
    {
        const int lane = tid & 63, wave = tid >> 6;
        const int share = ((n + WAVES - 1) / WAVES + 63) / 64 * 64;          // <= SHARE
        const int i1 = (wave + 1) * share < n ? (wave + 1) * share : n;
        int count = 0;
        for (int base = wave * share; base < i1; base += 512) {
            int a[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int i = base + q * 64 + lane;
                a[q] = i < i1 ? assign[lo + i] : -1;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint64_t m = __ballot(a[q] == slot);
                if (a[q] == slot) members[wave][count + lanes_below(m)] = base + q * 64 + lane;
                count += __popcll(m);
            }
        }
        if (lane == 0) nmem[wave] = count;
    }
    __syncthreads();
    int m = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m += nmem[w];
    const float inv = 1.0f / (float)(m > 0 ? m : 1);
    if (c < chunks) {
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.0f;
        auto add = [&](const u32x4& raw) {
            float f[8];
            unpack8s(raw, f);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += f[j];
        };
        for (int w = 0; w < WAVES; ++w) {
            const int cnt = nmem[w];
            auto row = [&](int q) { return *reinterpret_cast<const u32x4*>(x + (int64_t)(lo + members[w][q]) * C + c * 8); };
            int q = 0;
            for (; q + 8 <= cnt; q += 8) {                // eight rows in flight, added in order
                u32x4 r[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e] = row(q + e);
#pragma unroll
                for (int e = 0; e < 8; ++e) add(r[e]);
            }
            for (; q < cnt; ++q) add(row(q));
        }
        u32x4 pk;
#pragma unroll
        for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(acc[2 * j] * inv, acc[2 * j + 1] * inv);
        dst[c] = pk;
    }
}

// ---- gradient of the mean: dx[t] = dout[set][assign[t]] / (members of that slot) ---------------
// The kept set and the assignment are piecewise constant in x and carry no gradient.  Every
// workgroup recounts the members per slot of its set in LDS (integer adds: order-free), then
// its wavefronts write MB_ROWS rows.
constexpr int MB_ROWS = 4;            // one per wavefront: enough workgroups to fill the chip from 1024 tokens on

__global__ __launch_bounds__(MG_THREADS) void merge_bwd_kernel(const bf16_t* __restrict__ dout, SegTable st,
                                                               int C, int k, int set_base,
                                                               const int32_t* __restrict__ assign,
                                                               bf16_t* __restrict__ dx) {
    __shared__ int cnt[MERGE_MAX_N];
    const int set = blockIdx.y;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    const int r0 = blockIdx.x * MB_ROWS;
    if (r0 >= n) return;
    const int kk = k < n ? k : n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, chunks = C >> 3;
    for (int j = tid; j < kk; j += MG_THREADS) cnt[j] = 0;
    __syncthreads();
    for (int i0 = tid; i0 < n; i0 += 8 * MG_THREADS) {           // eight loads in flight
        int a[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) a[q] = i0 + q * MG_THREADS < n ? assign[lo + i0 + q * MG_THREADS] : -1;
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (a[q] >= 0 && a[q] < kk) atomicAdd(&cnt[a[q]], 1);
    }
    __syncthreads();
    for (int r = r0 + wave; r < r0 + MB_ROWS && r < n; r += 4) {
        const int a = assign[lo + r];
        u32x4* dst = reinterpret_cast<u32x4*>(dx + (int64_t)(lo + r) * C);
        if (a < 0 || a >= kk) {
            const u32x4 z = {0u, 0u, 0u, 0u};
            for (int c = lane; c < chunks; c += 64) dst[c] = z;
            continue;
        }
        const float m = (float)cnt[a];
        const u32x4* src = reinterpret_cast<const u32x4*>(dout + ((int64_t)(set_base + set) * k + a) * C);
        for (int c = lane; c < chunks; c += 64) {
            float f[8];
            unpack8s(src[c], f);
            u32x4 pk;
#pragma unroll
            for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(f[2 * j] / m, f[2 * j + 1] / m);
            dst[c] = pk;
        }
    }
}

// ---- launchers ---------------------------------------------------------------------------------------
hipError_t launch_merge_bwd_group(const bf16_t* dout, const SegTable& st, int n_max, int C, int k, int set_base,
                                  const int32_t* assign, bf16_t* dx, hipStream_t s) {
    if (st.count == 0 || n_max <= 0) return hipSuccess;
    hipLaunchKernelGGL(merge_bwd_kernel, dim3((unsigned)((n_max + MB_ROWS - 1) / MB_ROWS), (unsigned)st.count),
                       dim3(MG_THREADS), 0, s, dout, st, C, k, set_base, assign, dx);
    return hipGetLastError();
}

hipError_t launch_row_normalize(const bf16_t* x, int64_t rows, int C, bf16_t* xn, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(row_normalize_kernel, dim3((unsigned)rows), dim3(MG_THREADS), 0, s, x, C, xn);
    return hipGetLastError();
}

// steps after the similarity GEMMs for the sets of one table (set_base = index of its first set)
hipError_t launch_merge_group(const bf16_t* x, const SegTable& st, int n_max, int C, int k, int set_base,
                              const float* sim, int ld, int64_t sim_stride, float* avg,
                              int32_t* slot_of, int32_t* kept_idx, int32_t* assign, bf16_t* out,
                              hipStream_t s) {
    hipError_t e = hipSuccess;
    const unsigned sets = (unsigned)st.count;
    if (sets == 0) return e;
    if (n_max > 0) {
        hipLaunchKernelGGL(sim_rowmean_kernel, dim3((unsigned)((n_max + 3) / 4), sets), dim3(MG_THREADS), 0, s,
                           sim, st, ld, sim_stride, avg);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(merge_select_kernel, dim3(sets), dim3(TOPK_THREADS), 0, s, avg, st, k, set_base, slot_of,
                       kept_idx);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (n_max > 0) {
        hipLaunchKernelGGL(merge_assign_kernel, dim3((unsigned)((n_max + 3) / 4), sets), dim3(MG_THREADS), 0, s,
                           sim, st, ld, sim_stride, slot_of, assign);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (k > 0) {
        hipLaunchKernelGGL(merge_mean_kernel, dim3((unsigned)k, sets, (unsigned)(((C >> 3) + MG_THREADS - 1) / MG_THREADS)), dim3(MG_THREADS), 0, s, x, st, C, k,
                           set_base, assign, out);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace skipffn
