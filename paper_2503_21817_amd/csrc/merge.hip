// Token merge of the skipped (local) visual tokens (Section 4.1, the three bullet points):
//   1. cosine similarity between every pair of tokens of a set, averaged per token;
//   2. the k tokens of lowest average similarity are kept;
//   3. every other token is merged into the kept token it is most similar to (plain mean).
// The averages need no pair: with s the sum of a set's normalised rows, the sum of token i's similarities to the others is
// xn_i . (s - xn_i).  Only similarities of dropped tokens to kept ones are formed, on the matrix cores, and of those only each
// row's largest leaves the kernel.  (All similarities of a set, averaged and searched from memory: 43 of 78 us at 8 sets of
// 1024, k = 256.)  Every kernel runs for a whole group of sets per launch; the sets' row offsets travel in the kernel
// arguments, so nothing is copied to the device.
// Decisions that depend on floating point (which tokens are kept, where a token goes) are
// taken on the float32 averages / similarities computed here, with ties to the lower index,
// so they are unique for those values.  A token with a non-finite feature has NaN similarities, to
// every other, so all averages of its set are NaN (a set of one apart).  NaN ranks after every number and ties go to the lower index: the
// set's first min(k, n) tokens are kept.  A token whose similarities are all NaN goes to no slot (assign = -1)
// and gets a zero gradient.
#include <algorithm>
#include <type_traits>

#include "colsum.hpp"
#include "kernels.hpp"
#include "segments.hpp"
#include "slabloop.hpp"
#include "topk.hpp"

namespace skipffn {

constexpr int MG_THREADS = 256;

// In the kernels below: set = blockIdx.y, rows [lo, lo + n) of the token list.

// ---- Xn = X / |X| (a zero row stays zero), and the sum of the MERGE_CHUNK rows of a workgroup of Xn ----
// Bound by latency and HBM: a wavefront holds its two rows in registers, V chunks of each a lane, all loads in flight at once; its
// sum of them meets those of the other three in LDS, past 4096 columns 2048 of them at a time.  V = 0: rows of more than 8192
// columns, read again for the second step, 4096 columns at a time: 64 KB of LDS whatever the width.
// 9.3 us at 8192 rows of 1024 columns, 11.5 at 2304 of 4096 (16 rows a workgroup, read twice: 14.2 and 20.4).  4608 rows of
// 8192 columns: 30.5 us, of 4104 in 64 sets: 14.7 (read again, two loads in flight: 48 and 19; eight: 40 and 18.4).
__device__ __forceinline__ int64_t merge_part_row(const SegTable& st, int set, int chunk) {
    return (st.off[set] - st.off[0]) / MERGE_CHUNK + set + chunk;           // the sets' rows of `part` do not overlap
}
static_assert(MERGE_CHUNK == MG_THREADS / 64 * 2, "two rows a wavefront");
constexpr int MG_WIDE = 4096, MG_PIECE = 2048;
template <int V>
__global__ __launch_bounds__(MG_THREADS) void merge_normalize_kernel(const bf16_t* __restrict__ x, SegTable st, int C,
                                                                     bf16_t* __restrict__ xn, float* __restrict__ part) {
    extern __shared__ __align__(16) float sums[];        // [4][C], at most MG_WIDE columns
    const int set = blockIdx.y, n = st.off[set + 1] - st.off[set];
    if ((int)blockIdx.x * MERGE_CHUNK >= n) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, chunks = C >> 3;
    const int r = (int)blockIdx.x * MERGE_CHUNK + wave * 2;
    const bool has[2] = {r < n, r + 1 < n};              // uniform over a wavefront
    const int64_t row0 = st.off[set] + (has[0] ? r : 0), row1 = has[1] ? row0 + 1 : row0;
    const u32x4* src[2] = {reinterpret_cast<const u32x4*>(x + row0 * C), reinterpret_cast<const u32x4*>(x + row1 * C)};
    u32x4* dst[2] = {reinterpret_cast<u32x4*>(xn + row0 * C), reinterpret_cast<u32x4*>(xn + row1 * C)};
    constexpr int HELD = V > 0 ? V : 1;
    u32x4 held[2][HELD];
    float ss[2] = {0.0f, 0.0f};
    auto add = [](const u32x4& raw, float& s) {
        float f[8];
        unpack8s(raw, f);
#pragma unroll
        for (int j = 0; j < 8; ++j) s += f[j] * f[j];
    };
    // f(c, chunk c of the two rows) for c = first, first + 64, ...: eight loads in flight
    auto in_fours = [&](int c, const int end, auto&& f) {
        for (; c + 192 < end; c += 256) {
            u32x4 a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = src[0][c + 64 * u];
                b[u] = src[1][c + 64 * u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) f(c + 64 * u, a[u], b[u]);
        }
        for (; c < end; c += 64) f(c, src[0][c], src[1][c]);
    };
    if constexpr (V > 0) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int c = lane + 64 * v < chunks ? lane + 64 * v : 0;
            held[0][v] = src[0][c];
            held[1][v] = src[1][c];
        }
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (lane + 64 * v < chunks) {
                add(held[0][v], ss[0]);
                add(held[1][v], ss[1]);
            }
    } else {
        in_fours(lane, chunks, [&](int, const u32x4& a, const u32x4& b) {
            add(a, ss[0]);
            add(b, ss[1]);
        });
    }
    float inv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float v = wave_sum(ss[q]);
        inv[q] = v > 0.0f ? 1.0f / sqrtf(v) : 0.0f;
    }
    const int width = V > 0 && V <= 8 ? C : V > 8 ? MG_PIECE : C < MG_WIDE ? C : MG_WIDE;
    auto emit = [&](int c, int c0, const u32x4& a, const u32x4& b) {
        float sum[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) sum[j] = 0.0f;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (!has[q]) continue;                       // uniform
            float f[8];
            unpack8s(q == 0 ? a : b, f);
            u32x4 pk;
#pragma unroll
            for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(f[2 * j] * inv[q], f[2 * j + 1] * inv[q]);
            dst[q][c] = pk;
            unpack8s(pk, f);                             // the sum of what the similarities are formed of
#pragma unroll
            for (int j = 0; j < 8; ++j) sum[j] += f[j];
        }
        f32x4* to = reinterpret_cast<f32x4*>(sums + wave * width + (c - c0) * 8);
        to[0] = f32x4{sum[0], sum[1], sum[2], sum[3]};
        to[1] = f32x4{sum[4], sum[5], sum[6], sum[7]};
    };
    f32x4* out = reinterpret_cast<f32x4*>(part + merge_part_row(st, set, (int)blockIdx.x) * C);
    const f32x4* in = reinterpret_cast<const f32x4*>(sums);
    const int quads = width >> 2;
    auto write_sum = [&](int first, int count) {         // quads of columns
        for (int c = tid; c < count; c += MG_THREADS)
            out[first + c] = (in[c] + in[c + quads]) + (in[c + 2 * quads] + in[c + 3 * quads]);
    };
    if constexpr (V > 8) {
        constexpr int PIECE = MG_PIECE / 8;              // chunks
#pragma unroll
        for (int p = 0; p < V * 64 / PIECE; ++p) {
            const int c0 = p * PIECE;
            if (c0 >= chunks) break;                     // uniform
            if (p > 0) __syncthreads();                  // the piece before has been added
#pragma unroll
            for (int v = c0 / 64; v < (c0 + PIECE) / 64; ++v)
                if (lane + 64 * v < chunks) emit(lane + 64 * v, c0, held[0][v], held[1][v]);
            __syncthreads();
            write_sum(c0 * 2, (c0 + PIECE < chunks ? PIECE : chunks - c0) * 2);
        }
    } else if constexpr (V > 0) {
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (lane + 64 * v < chunks) emit(lane + 64 * v, 0, held[0][v], held[1][v]);
        __syncthreads();
        write_sum(0, quads);
    } else {
        for (int c0 = 0; c0 < chunks; c0 += MG_WIDE / 8) {
            const int c1 = c0 + MG_WIDE / 8 < chunks ? c0 + MG_WIDE / 8 : chunks;
            if (c0 > 0) __syncthreads();                 // the piece before has been added
            in_fours(c0 + lane, c1, [&](int c, const u32x4& a, const u32x4& b) { emit(c, c0, a, b); });
            __syncthreads();
            write_sum(c0 * 2, (c1 - c0) * 2);
        }
    }
}

// ---- s_set = the sum of the set's partial rows ------------------------------------------------------
template <int LANES>
__global__ __launch_bounds__(32 * LANES) void merge_sum_kernel(const float* __restrict__ part, SegTable st, int C, float* __restrict__ s) {
    const int set = blockIdx.y, n = st.off[set + 1] - st.off[set];
    if (n <= 0) return;
    column_sum<LANES>(part + merge_part_row(st, set, 0) * C, (n + MERGE_CHUNK - 1) / MERGE_CHUNK, C, s + (int64_t)set * C, 0);
}

// The same sums (lane by lane, added in the same order) where there are sets and columns enough for a workgroup of a quarter of the
// threads and four times the columns, up to 4 * LANES partial rows: all of them in flight at once.  36 sets of 377 x 4096: 14.1 -> 6.6 us,
// 29 of 310 x 2048 9 -> 4.0.
template <int LANES>
__global__ __launch_bounds__(256) void merge_sum_wide_kernel(const float* __restrict__ part, SegTable st, int C, float* __restrict__ s) {
    const int set = blockIdx.y, n = st.off[set + 1] - st.off[set];
    if (n <= 0) return;
    constexpr int V = LANES / 8;
    __shared__ f32x4 lanes[LANES][32];
    const int rows = (n + MERGE_CHUNK - 1) / MERGE_CHUNK, cx = threadIdx.x & 31, sy = threadIdx.x >> 5;
    const int q = (int)blockIdx.x * 32 + cx;             // columns 4 q .. 4 q + 3
    const f32x4* p = reinterpret_cast<const f32x4*>(part + merge_part_row(st, set, 0) * C) + q;
    const f32x4 zero{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 x[V][4];
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = sy + 8 * v + k * LANES;
            x[v][k] = q < C >> 2 && row < rows ? p[(int64_t)row * (C >> 2)] : zero;
        }
#pragma unroll
    for (int v = 0; v < V; ++v)
        lanes[sy + 8 * v][cx] = sy + 8 * v + 3 * LANES < rows ? (x[v][0] + x[v][1]) + (x[v][2] + x[v][3]) : (x[v][0] + x[v][1]) + x[v][2];
    __syncthreads();
    if (sy == 0 && q < C >> 2) {
        f32x4 v = zero;
#pragma unroll
        for (int k = 0; k < LANES; ++k) v += lanes[k][cx];
        reinterpret_cast<f32x4*>(s + (int64_t)set * C)[q] = v;
    }
}

// ---- avg_i = xn_i . (s - xn_i) / (n - 1), two rows per wavefront ------------------------------------
// SMALL: s is added here, from the partial rows (`s` points at them), at most MG_FEW_PARTS: sets of few tokens are bound by their
// launches.  200 sets of 16 tokens of 256 columns, four groups of launches: 94 -> 84 us a call, of 8192 columns 302 -> 278.  The partial
// rows are loaded together: 17 sets of 31 x 5912 17.4 -> 11.4 us.
constexpr int MG_FEW_PARTS = 4;
template <bool SMALL>
__global__ __launch_bounds__(MG_THREADS) void merge_average_kernel(const bf16_t* __restrict__ xn, SegTable st, int C,
                                                                   const float* __restrict__ s, float* __restrict__ avg) {
    constexpr int ROWS = 2;
    const int set = blockIdx.y, lo = st.off[set], n = st.off[set + 1] - lo;
    const int lane = threadIdx.x & 63, i = ((int)blockIdx.x * 4 + (threadIdx.x >> 6)) * ROWS;
    if (i >= n) return;
    const int chunks = C >> 3;
    const u32x4* row[ROWS];
    float d[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        row[r] = reinterpret_cast<const u32x4*>(xn + (int64_t)(lo + i + (i + r < n ? r : 0)) * C);
        d[r] = 0.0f;
    }
    const f32x4* ps = reinterpret_cast<const f32x4*>(s + (SMALL ? merge_part_row(st, set, 0) : (int64_t)set) * C);
    const int parts = SMALL ? (n + MERGE_CHUNK - 1) / MERGE_CHUNK : 1;
    auto sum_at = [&](int q) {                           // columns 4 q .. 4 q + 3
        f32x4 v = ps[q];
        if (SMALL) {
            f32x4 more[MG_FEW_PARTS];                    // in flight together; past the parts the first one again, not added
#pragma unroll
            for (int p = 1; p < MG_FEW_PARTS; ++p) more[p] = ps[(int64_t)(p < parts ? p : 0) * (C >> 2) + q];
#pragma unroll
            for (int p = 1; p < MG_FEW_PARTS; ++p)
                if (p < parts) v += more[p];
        }
        return v;
    };
    auto add = [&](float& dr, const u32x4& raw, const f32x4& lo4, const f32x4& hi4) {
        float x[8];
        unpack8s(raw, x);
#pragma unroll
        for (int j = 0; j < 8; ++j) dr += x[j] * ((j < 4 ? lo4[j & 3] : hi4[j & 3]) - x[j]);
    };
    int c = lane;
    for (; c + 64 < chunks; c += 128) {
        u32x4 a[2][ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            a[0][r] = row[r][c];
            a[1][r] = row[r][c + 64];
        }
        const f32x4 l0 = sum_at(2 * c), h0 = sum_at(2 * c + 1), l1 = sum_at(2 * c + 128), h1 = sum_at(2 * c + 129);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            add(d[r], a[0][r], l0, h0);
            add(d[r], a[1][r], l1, h1);
        }
    }
    if (c < chunks) {
        const f32x4 l0 = sum_at(2 * c), h0 = sum_at(2 * c + 1);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) add(d[r], row[r][c], l0, h0);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const float v = wave_sum(d[r]);
        if (lane == 0 && i + r < n) avg[lo + i + r] = n > 1 ? v / (float)(n - 1) : 0.0f;
    }
}

// ---- which tokens are kept, and their slots ------------------------------------------------------
// One workgroup per set: the k tokens of lowest average (topk.hpp), then the position of every kept
// token among the kept ones, in index order, and of every other among the others.  kept_idx[set][slot] = lo + t, -1
// padding; dropped[lo + position] = t.  goal[lo + t] = where token t goes: a key that grows with the similarity and, for equal
// ones, falls with the slot; a kept token's own slot, before every similarity, 0 for the others (no slot yet).
typedef unsigned long long goal_t;
__device__ __forceinline__ goal_t merge_goal(uint32_t key, int slot) { return (goal_t)key << 32 | (uint32_t)~slot; }
__device__ __forceinline__ int slot_of_goal(uint32_t lower) { return (int)~lower; }      // of goal 0: -1
constexpr uint32_t GOAL_KEPT = 0xFFFFFFFFu;   // rank_key of no number

constexpr int MG_MAXV = MERGE_MAX_N / TOPK_THREADS;
__global__ __launch_bounds__(TOPK_THREADS) void merge_select_kernel(const float* __restrict__ avg, SegTable st,
                                                                    int k, int set_base, goal_t* __restrict__ goal,
                                                                    int32_t* __restrict__ dropped, int32_t* __restrict__ kept_idx,
                                                                    int32_t* __restrict__ assign) {
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
        goal[lo + t] = in[i] ? merge_goal(GOAL_KEPT, before[i]) : 0;
        if (in[i]) kout[before[i]] = lo + t;
        else dropped[lo + t - before[i]] = t;
        if (k <= 0) assign[lo + t] = -1;         // no slot to go to
    }
}

// ---- the kept token that every dropped one is most similar to -------------------------------------
// Xn Xn^T of dropped rows and kept rows, gathered by their lists as they are loaded; a tile keeps the largest entry of each of its
// rows (ties: the lower slot) and adds it to the token's goal by an atomic maximum, whose order does not matter.  Bound by
// the loop's phases and by how many CUs have a tile; the launcher picks the tile.  8 sets of 1024 x 1024, k = 256: 12.0 us, a
// set of 2304 x 4096, k = 576: 22.2, 6 of 2880 x 1024, k = 1200: 49.7; all similarities on and above the diagonal, 128 x 128, and the search for the
// largest one in memory: 25.1 + 11.1, 34.5 + 10.1, 95 + 44.
template <int A_ROWS, int B_ROWS>
__global__ __launch_bounds__(SLAB_THREADS) void merge_target_kernel(const bf16_t* __restrict__ xn, SegTable st, int C, int k, int set_base,
                                                                    int tiles_m, int tiles_n, const int32_t* __restrict__ dropped,
                                                                    const int32_t* __restrict__ kept_idx, goal_t* __restrict__ goal) {
    constexpr int MI = A_ROWS / 32, NF = B_ROWS / 64;
    constexpr int NLA = kSlabPiecesA<A_ROWS>, NL = kSlabPieces<A_ROWS, B_ROWS>;
    // workgroups are dealt round-robin to the 8 XCDs: each gets a contiguous range of the tiles, so that few sets (or
    // few rows of a set) share its L2
    const int nb = (int)gridDim.x, xcd = (int)blockIdx.x & 7, q8 = nb >> 3, rem8 = nb & 7;
    const int b = xcd * q8 + (xcd < rem8 ? xcd : rem8) + ((int)blockIdx.x >> 3);
    const int set = b / (tiles_m * tiles_n), t = b - set * tiles_m * tiles_n, tm = t / tiles_n, tn = t - tm * tiles_n;
    const int lo = st.off[set], n = st.off[set + 1] - lo, kk = k < n ? k : n, nd = n - kk;
    if (tm * A_ROWS >= nd || tn * B_ROWS >= kk) return;  // whole workgroup leaves together
    const int32_t* rows_a = dropped + lo;                // relative to the set
    const int32_t* rows_b = kept_idx + (int64_t)(set_base + set) * k;        // absolute
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(xn + (int64_t)lo * C, (uint32_t)((int64_t)n * C * 2));
    uint32_t goff[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int row = 8 * (l < NLA ? wave * NLA + l : wave * NF + (l - NLA)) + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        const int i = (l < NLA ? tm * A_ROWS : tn * B_ROWS) + row;
        const bool in = i < (l < NLA ? nd : kk);
        const int gr = !in ? 0 : l < NLA ? rows_a[i] : rows_b[i] - lo;
        goff[l] = in ? (uint32_t)(((int64_t)gr * C + c * 8) * 2) : kOobOffset;
    }
    extern __shared__ __align__(16) char smem[];
    goal_t (*best)[A_ROWS] = reinterpret_cast<goal_t (*)[A_ROWS]>(smem);     // [4][A_ROWS], once the slabs have been read
    const int wm = wave >> 2, wn = wave & 3;
    f32x4 acc[MI][NF];
    float ss[MI];
    slab_loop<A_ROWS, 16, false, B_ROWS>(rx, rx, goff, wn * 16 * NF, 0, (C + BK - 1) / BK, 0, C, acc, ss);
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        goal_t g = 0;
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = tn * B_ROWS + wn * 16 * NF + f * 16 + 4 * (lane >> 4) + r;
                const float v = acc[m][f][r];
                if (j < kk && v == v) {
                    const goal_t o = merge_goal(rank_key<false>(v), j);
                    g = o > g ? o : g;
                }
            }
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const goal_t o = __shfl_xor(g, off, 64);
            g = o > g ? o : g;
        }
        if (lane < 16) best[wn][wm * (A_ROWS / 2) + m * 16 + lane] = g;
    }
    __syncthreads();
    const int i = tm * A_ROWS + (int)threadIdx.x;
    if ((int)threadIdx.x < A_ROWS && i < nd) {
        goal_t g = best[0][threadIdx.x];
#pragma unroll
        for (int w = 1; w < 4; ++w) g = best[w][threadIdx.x] > g ? best[w][threadIdx.x] : g;
        if (g != 0) atomicMax(&goal[lo + rows_a[i]], g);
    }
}

template <int A_ROWS, int B_ROWS>
constexpr int kTargetLds = kSlabLds<A_ROWS, B_ROWS>;
template <int A_ROWS, int B_ROWS>
static hipError_t target_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&merge_target_kernel<A_ROWS, B_ROWS>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kTargetLds<A_ROWS, B_ROWS>);
}
hipError_t merge_init() {
    hipError_t e;
    if ((e = target_lds<64, 64>()) != hipSuccess) return e;
    if ((e = target_lds<64, 128>()) != hipSuccess) return e;
    return target_lds<128, 128>();
}

template <int A_ROWS, int B_ROWS>
static void launch_target(const bf16_t* xn, const SegTable& st, int nd, int kk, int C, int k, int set_base, const int32_t* dropped,
                          const int32_t* kept_idx, goal_t* goal, hipStream_t s) {
    const int tiles_m = (nd + A_ROWS - 1) / A_ROWS, tiles_n = (kk + B_ROWS - 1) / B_ROWS;
    hipLaunchKernelGGL((merge_target_kernel<A_ROWS, B_ROWS>), dim3((unsigned)(tiles_m * tiles_n * st.count)), dim3(SLAB_THREADS),
                       (kTargetLds<A_ROWS, B_ROWS>), s, xn, st, C, k, set_base, tiles_m, tiles_n, dropped, kept_idx, goal);
}

// ---- out[set][slot] = mean of the rows that go to the slot; assign ----------------------------------
// A workgroup takes four slots, two wavefronts each, COLS pieces of 64 chunks of the row a wavefront at a time.  The slots of the
// set's tokens are staged in LDS once; of the two wavefronts of a slot one searches them, eight a lane at a time, and a prefix sum over
// the lanes gives every member its place in the list.  Then the members are added in index order, sixteen loads in flight: sixteen
// rows, or fewer rows of more pieces.  The staging and the search are most of the time of a short list, so a workgroup walks along
// the row where the groups of slots fill the chip by themselves (four of them a CU) and takes a part of it where they do not.
// us, a part of the row a workgroup whatever their number and the places read one by one / this:  64 sets of 576 x 4096, k = 518 207 /
// 107;  8 of 576 x 8192, k = 518 42 / 26;  64 of 64 x 4104, k = 57 23.4 / 15.2;  one slot of 144 rows of 256 16.8 / 10.1;
// 8 of 1024 x 1024, k = 256 6.4 / 6.6.  (A workgroup a slot, which reads the slots of all tokens for itself: 117, 23.8, 15.7, 10.4, 7.5.)
constexpr int MEAN_THREADS = 512, MEAN_SLOTS = 4, MEAN_COLS = 128;
__host__ __device__ constexpr int mean_lds_tokens(int n) { return (n + 511) / 512 * 512; }      // a wavefront searches 512 at a time
template <int COLS>
__global__ __launch_bounds__(MEAN_THREADS) void merge_mean_kernel(const bf16_t* __restrict__ x, SegTable st, int n_max, int C, int k,
                                                                  int set_base, const goal_t* __restrict__ goal,
                                                                  int32_t* __restrict__ assign, bf16_t* __restrict__ out) {
    extern __shared__ __align__(16) uint16_t lds16[];    // slots of the tokens, then the members of each slot
    __shared__ int members[MEAN_SLOTS];
    constexpr int ROWS = 16 / COLS;                      // in flight
    const int set = blockIdx.y;
    const int lo = st.off[set], n = st.off[set + 1] - lo;
    const int kk = k < n ? k : n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), chunks = C >> 3;
    const uint32_t* goal_slots = reinterpret_cast<const uint32_t*>(goal + lo);       // the lower halves
    const int padded = mean_lds_tokens(n);
    for (int i0 = tid; i0 < padded; i0 += 4 * MEAN_THREADS) {                        // four loads in flight
        int to[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + e * MEAN_THREADS;
            to[e] = i < n ? slot_of_goal(goal_slots[2 * i]) : -1;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = i0 + e * MEAN_THREADS;
            if (i < padded) lds16[i] = (uint16_t)to[e];                              // -1: no slot of 4096
            if (i < n && blockIdx.z == 0 && (i >> 6) % (int)gridDim.x == (int)blockIdx.x) assign[lo + i] = to[e];
        }
    }
    __syncthreads();
    const int mine = wave >> 1, slot = (int)blockIdx.x * MEAN_SLOTS + mine;
    uint16_t* list = lds16 + mean_lds_tokens(n_max) * (1 + mine);
    if ((wave & 1) == 0) {
        int m = 0;
        if (slot < kk)
            for (int i0 = 0; i0 < n; i0 += 512) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(lds16 + i0 + lane * 8);
                uint32_t hit = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    hit |= ((v[e] & 0xffffu) == (uint32_t)slot ? 1u << (2 * e) : 0u) | (v[e] >> 16 == (uint32_t)slot ? 2u << (2 * e) : 0u);
                const int here = __popc(hit), incl = wave_inclusive_sum(here);
                int at = m + incl - here;
                while (hit != 0) {
                    list[at++] = (uint16_t)(i0 + lane * 8 + __builtin_ctz(hit));
                    hit &= hit - 1;
                }
                m += __builtin_amdgcn_readlane(incl, 63);
            }
        if (lane == 0) members[mine] = m;
    }
    __syncthreads();
    const int m = __builtin_amdgcn_readfirstlane(members[mine]);
    if (slot >= k) return;
    const bf16_t* rows = x + (int64_t)lo * C;
    const float inv = 1.0f / (float)(m > 0 ? m : 1);     // a slot past the set's tokens: a row of zeros
    u32x4* dst = reinterpret_cast<u32x4*>(out + ((int64_t)(set_base + set) * k + slot) * C);
    for (int c0 = (int)blockIdx.z * MEAN_COLS * COLS + (wave & 1) * 64 + lane; c0 < chunks; c0 += (int)gridDim.z * MEAN_COLS * COLS) {
        int col[COLS];                                   // past the row: its last chunk in reach again, not stored
#pragma unroll
        for (int v = 0; v < COLS; ++v) col[v] = c0 + v * MEAN_COLS < chunks ? c0 + v * MEAN_COLS : c0;
        float acc[COLS][8];
#pragma unroll
        for (int v = 0; v < COLS; ++v)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[v][j] = 0.0f;
        // N rows of the list from q on, the first `count` of them added in order; their places are read together (a read of LDS
        // before each row's load was most of the kernel), the rows past the count are the first one again, as zeros
        auto add_rows = [&](auto batch, const int q, const int count) {
            constexpr int N = decltype(batch)::value;
            u32x4 r[N][COLS];
            uint32_t place[(N + 1) / 2];
#pragma unroll
            for (int h = 0; h < (N + 1) / 2; ++h)
                place[h] = (uint32_t)__builtin_amdgcn_readfirstlane((int)reinterpret_cast<const uint32_t*>(list + q)[h]);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const uint32_t row = e < count ? (e & 1 ? place[e >> 1] >> 16 : place[e >> 1] & 0xffffu) : place[0] & 0xffffu;
                const u32x4* p = reinterpret_cast<const u32x4*>(rows + (int64_t)row * C);
#pragma unroll
                for (int v = 0; v < COLS; ++v) r[e][v] = p[col[v]];
            }
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const uint32_t keep = e < count ? 0xffffffffu : 0u;
#pragma unroll
                for (int v = 0; v < COLS; ++v) {
                    float f[8];
                    unpack8s(r[e][v] & u32x4{keep, keep, keep, keep}, f);
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[v][j] += f[j];
                }
            }
        };
        int q = 0;
        for (; q + ROWS <= m; q += ROWS) add_rows(std::integral_constant<int, ROWS>{}, q, ROWS);
        const int rest = m - q;                          // uniform, below ROWS
        if (ROWS > 8 && rest > 8) add_rows(std::integral_constant<int, 16>{}, q, rest);
        else if (ROWS > 4 && rest > 4) add_rows(std::integral_constant<int, 8>{}, q, rest);
        else if (rest > 2) add_rows(std::integral_constant<int, 4>{}, q, rest);
        else if (rest == 2) add_rows(std::integral_constant<int, 2>{}, q, 2);
        else if (rest == 1) add_rows(std::integral_constant<int, 1>{}, q, 1);
#pragma unroll
        for (int v = 0; v < COLS; ++v) {
            u32x4 pk;
#pragma unroll
            for (int j = 0; j < 4; ++j) pk[j] = pack_bf16x2(acc[v][2 * j] * inv, acc[v][2 * j + 1] * inv);
            if (c0 + v * MEAN_COLS < chunks) dst[c0 + v * MEAN_COLS] = pk;
        }
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

// the sets of one table (set_base = index of its first set), n_max rows in the largest
hipError_t launch_merge_group(const bf16_t* x, const SegTable& st, int n_max, int C, int k, int set_base, const MergeScratch& ws,
                              float* avg, int32_t* kept_idx, int32_t* assign, bf16_t* out, int ncu, hipStream_t s) {
    const unsigned sets = (unsigned)st.count;
    if (sets == 0) return hipSuccess;
    goal_t* goal = static_cast<goal_t*>(ws.goal);
    hipError_t e;
    if (n_max > 0) {
        const int chunks = C >> 3, parts = (n_max + MERGE_CHUNK - 1) / MERGE_CHUNK;
        const dim3 rows((unsigned)parts, sets), threads(MG_THREADS);
        const size_t lds = (size_t)std::min(C, MG_WIDE) * 16;
        if (chunks <= 64) hipLaunchKernelGGL(merge_normalize_kernel<1>, rows, threads, lds, s, x, st, C, ws.xn, ws.part);
        else if (chunks <= 128) hipLaunchKernelGGL(merge_normalize_kernel<2>, rows, threads, lds, s, x, st, C, ws.xn, ws.part);
        else if (chunks <= 256) hipLaunchKernelGGL(merge_normalize_kernel<4>, rows, threads, lds, s, x, st, C, ws.xn, ws.part);
        else if (chunks <= 512) hipLaunchKernelGGL(merge_normalize_kernel<8>, rows, threads, lds, s, x, st, C, ws.xn, ws.part);
        else if (chunks <= 1024) hipLaunchKernelGGL(merge_normalize_kernel<16>, rows, threads, MG_PIECE * 16, s, x, st, C, ws.xn, ws.part);
        else hipLaunchKernelGGL(merge_normalize_kernel<0>, rows, threads, lds, s, x, st, C, ws.xn, ws.part);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (parts <= MG_FEW_PARTS) {
            hipLaunchKernelGGL(merge_average_kernel<true>, rows, threads, 0, s, ws.xn, st, C, ws.part, avg);
        } else {
            const dim3 cols((unsigned)((C + 31) / 32), sets), wide((unsigned)((C + 127) / 128), sets);
            const bool few = parts <= COLSUM_FEW_ROWS;
            if (parts <= 4 * COLSUM_LANES && (int64_t)wide.x * sets >= ncu) {
                if (few) hipLaunchKernelGGL(merge_sum_wide_kernel<COLSUM_LANES_FEW>, wide, threads, 0, s, ws.part, st, C, ws.sum);
                else hipLaunchKernelGGL(merge_sum_wide_kernel<COLSUM_LANES>, wide, threads, 0, s, ws.part, st, C, ws.sum);
            } else if (few) {
                hipLaunchKernelGGL(merge_sum_kernel<COLSUM_LANES_FEW>, cols, dim3(32 * COLSUM_LANES_FEW), 0, s, ws.part, st, C, ws.sum);
            } else {
                hipLaunchKernelGGL(merge_sum_kernel<COLSUM_LANES>, cols, dim3(32 * COLSUM_LANES), 0, s, ws.part, st, C, ws.sum);
            }
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(merge_average_kernel<false>, rows, threads, 0, s, ws.xn, st, C, ws.sum, avg);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(merge_select_kernel, dim3(sets), dim3(TOPK_THREADS), 0, s, avg, st, k, set_base, goal, ws.dropped, kept_idx, assign);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (k <= 0) return hipSuccess;
    if (n_max > k) {
        const int nd = n_max - k, best = merge_target_tile(nd, k, st.count, ncu);
        if (best == 0) launch_target<128, 128>(ws.xn, st, nd, k, C, k, set_base, ws.dropped, kept_idx, goal, s);
        else if (best == 1) launch_target<64, 128>(ws.xn, st, nd, k, C, k, set_base, ws.dropped, kept_idx, goal, s);
        else launch_target<64, 64>(ws.xn, st, nd, k, C, k, set_base, ws.dropped, kept_idx, goal, s);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int groups = (k + MEAN_SLOTS - 1) / MEAN_SLOTS, pieces = ((C >> 3) + MEAN_COLS - 1) / MEAN_COLS;
    const int64_t slot_groups = (int64_t)groups * st.count, room = (4 * (int64_t)ncu + slot_groups - 1) / slot_groups;
    const int cols = pieces >= 4 * room ? 4 : pieces >= 2 * room ? 2 : 1, row_parts = (pieces + cols - 1) / cols;
    const dim3 mean_grid((unsigned)groups, sets, (unsigned)std::min<int64_t>(row_parts, room));
    const size_t mean_lds = (size_t)mean_lds_tokens(n_max) * 2 * (1 + MEAN_SLOTS);
    auto mean = [&](auto kernel) { hipLaunchKernelGGL(kernel, mean_grid, dim3(MEAN_THREADS), mean_lds, s, x, st, n_max, C, k, set_base, goal, assign, out); };
    if (cols == 4) mean(merge_mean_kernel<4>);
    else if (cols == 2) mean(merge_mean_kernel<2>);
    else mean(merge_mean_kernel<1>);
    return hipGetLastError();
}

}  // namespace skipffn
