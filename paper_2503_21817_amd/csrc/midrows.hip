// The two forward GEMMs for up to 256 retained rows (decode batches, prefill of an image, small training batches).
//
// Bound by streaming the weights from HBM.  A tile is ALL rows (16 * MT of them) times 128 weight rows, so that every
// weight byte goes to one CU only and the tiles are many (I / 64 for gate/up; C / 128 with K split for down, whose
// fp32 slabs a reducing kernel adds).  What limits a CU is the bytes its address unit takes, weights and activations
// together: about 9 TB/s over the chip here.  Hence both operands go to LDS by direct loads of whole 128-byte lines
// (weights straight to registers, 16 rows x 64 bytes a load: 65 instead of 57 us at 184 rows), and the rows are not
// padded further than to 64.
//
// Two row groups of four wavefronts run one phase apart: one reads the fragments of its next slab of 64 k and issues
// loads, the other runs its MFMAs; two barriers a slab (the 256-row core has four, and twice the MFMAs between them).
// The LDS ring holds as many slabs as fit (6 to 3 for 64 to 256 rows).  Where rows are a multiple of 8 KB apart,
// workgroups of an XCD start at different slabs and wrap around: walking K in step they would all read the same few
// L2 and HBM channels (gate/up at 64 rows 52 -> 44 us).  At strides of 6, 4 and 28 KB it makes no difference, and K
// is summed in order.
//
// Measured at C = 4096, I = 14336 (the loads of the weights alone: 41 + 21 us): gate/up 42 / 49 / 57 / 64 us and down
// 26 / 32 / 35 / 42 us at 64 / 128 / 184 / 256 rows; 128-row tiles with the weights shared through L2: 73 and 41 at 184.
#include "kernels.hpp"

namespace skipffn {

constexpr int MID_THREADS = 512;
constexpr int MID_CHANNEL_K = 4096;           // rows this many k apart share their L2 channels
constexpr int MID_WROWS = 128;                // weight rows per tile: 64 of W_gate and 64 of W_up, or 128 of W_down

struct MidRowsArgs {
    int rows; const int32_t* r_dev;           // row bound (<= 16 * MT), optional device count
    int N, K;                                 // output columns, contraction length (multiples of 8)
    const bf16_t* A; uint32_t a_bytes;        // [rows][K]
    const bf16_t* B0; const bf16_t* B1; uint32_t b_bytes;   // [N][K]; gate/up: W_gate, W_up
    int splits;                               // gate/up: 1
    bf16_t* H; bf16_t* G; bf16_t* U;          // gate/up: [rows][N]; G, U optional
    float* partial;                           // down: [splits][rows][N]
};

// LDS ring of slabs of 64 k: 16 * MT rows of activations and 128 of weights, 128 bytes each
template <int MT>
constexpr int kMidStage = MT * 2048 + MID_WROWS * 128;
template <int MT>
constexpr int kMidStages = (160 * 1024) / kMidStage<MT>;
template <int MT>
constexpr int kMidLds = kMidStages<MT> * kMidStage<MT>;

template <int MT, bool GATE_UP>
__global__ __launch_bounds__(MID_THREADS) void mid_rows_kernel(MidRowsArgs P) {
    static_assert(MT % 4 == 0 && MT <= 16, "two row groups, whole 1 KB pieces per wavefront");
    constexpr int NST = kMidStages<MT>, STAGE = kMidStage<MT>, B_BASE = MT * 2048;
    constexpr int MI = MT / 2;                // row fragments of a wavefront
    constexpr int NLA = MT / 4, NL = NLA + 2; // 1 KB pieces of a slab each wavefront loads: activations, and all
    static_assert(NST >= 3, "two slabs in flight beside the one that is read");
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;  // row group, column quarter
    const int R = effective_rows(P.rows, P.r_dev);
    if (R <= 0) return;                       // uniform
    const int z = (int)blockIdx.x % P.splits;
    const int n0 = ((int)blockIdx.x / P.splits) * (GATE_UP ? MID_WROWS / 2 : MID_WROWS);
    const int r16 = lane & 15, kq = lane >> 4;

    const int ktiles = (P.K + BK - 1) / BK, per = (ktiles + P.splits - 1) / P.splits;
    const int kt0 = z * per, kt1 = kt0 + per < ktiles ? kt0 + per : ktiles;
    const int nk = kt1 > kt0 ? kt1 - kt0 : 0;
    // where in its K range the workgroup starts (blocks b, b + 8, ... share an XCD); see the note above
    const int rot = nk > 0 && P.K % MID_CHANNEL_K == 0 ? (int)(((blockIdx.x >> 3) * 2) % (unsigned)nk) : 0;

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(P.A, P.a_bytes),
                                 rb = make_rsrc(GATE_UP && wave >= 4 ? P.B1 : P.B0, P.b_bytes);
    // piece q of an operand slab = its rows 8 q .. 8 q + 7: lane -> row 8 q + lane / 8, the chunk whose swizzled
    // home is slot lane % 8
    uint32_t goff[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int q = l < NLA ? wave * NLA + l : wave * 2 + (l - NLA);
        const int row = 8 * q + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        const int gr = l < NLA ? row : n0 + (GATE_UP ? row & 63 : row);
        const bool in = l < NLA ? gr < R : gr < P.N;
        goff[l] = in ? (uint32_t)(((int64_t)gr * P.K + c * 8) * 2) : kOobOffset;
    }
    typedef __attribute__((address_space(3))) void* lds_void_ptr;
    auto lds_piece = [&](int stage, int l) {
        return smem + stage * STAGE + (l < NLA ? (wave * NLA + l) * 1024 : B_BASE + (wave * 2 + (l - NLA)) * 1024);
    };
    auto slab_of = [&](int j) { const int jr = j + rot; return kt0 + (jr < nk ? jr : jr - nk); };
    // a slab that may reach past K: k past the end are zeros
    auto load_masked = [&](int j) {
        const int slab = slab_of(j);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int q = l < NLA ? wave * NLA + l : wave * 2 + (l - NLA);
            const int row = 8 * q + (lane >> 3), kk = slab * BK + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
            const uint32_t off = goff[l] != kOobOffset && kk < P.K ? goff[l] + (uint32_t)slab * (BK * 2) : kOobOffset;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(l < NLA ? ra : rb, (lds_void_ptr)lds_piece(j % NST, l), 16, (int)off, 0, 0, 0);
        }
    };

    f32x4 acc[MI][2];
#pragma unroll
    for (int m = 0; m < MI; ++m)
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[m][f] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    uint32_t a_rd[2], b_rd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        a_rd[ks] = lds_addr_of(smem) + kc_off(wm * MI * 16 + r16, 4 * ks + kq);
        b_rd[ks] = lds_addr_of(smem) + B_BASE + kc_off(wn * (GATE_UP ? 16 : 32) + r16, 4 * ks + kq);
    }
    constexpr int B_NEXT = GATE_UP ? 8192 : 2048;      // the up columns, or the next 16
    auto phase_barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    bf16x8 af[2][MI], bfr[2][2];
    int st_rd = 0, st_ld = NST - 1;                     // stages slab j is read from and slab j + NST - 1 loaded to
    // the memory phase of slab j: the loads of slab j + NST - 1 spread between the fragment reads
    auto memory_phase = [&](int j, auto steady) {
        constexpr bool STEADY = decltype(steady)::value;
        if (!STEADY && j + NST - 1 < nk) load_masked(j + NST - 1);
        const int step = STEADY ? slab_of(j + NST - 1) * (BK * 2) : 0;
        const uint32_t so = (uint32_t)(st_rd * STAGE);
        const uint32_t aa[2] = {a_rd[0] + so, a_rd[1] + so}, ba[2] = {b_rd[0] + so, b_rd[1] + so};
        constexpr int NR = 2 * (MI + 2);
        static_for<NR>([&](auto r) {
            if constexpr (STEADY)
                static_for<NL>([&](auto l) {
                    if constexpr (l * NR / NL == r)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(l < NLA ? ra : rb, (lds_void_ptr)lds_piece(st_ld, l), 16, (int)goff[l], step, 0, 0);
                });
            constexpr int ks = r / (MI + 2), i = r % (MI + 2);
            if constexpr (i < 2) bfr[ks][i] = ds_read_b128_imm<i * B_NEXT>(ba[ks]);
            else af[ks][i - 2] = ds_read_b128_imm<(i - 2) * 2048>(aa[ks]);
        });
    };
    // slab j + 1 has landed; the slabs issued after it may still fly
    auto wait_next_slab = [&](auto steady) {
        if (decltype(steady)::value) SKIPFFN_WAIT_VMCNT((NST - 2) * NL); else SKIPFFN_WAIT_VMCNT(0);
    };
    auto iteration = [&](int j, auto steady) {
        memory_phase(j, steady);
        if (wm == 1) wait_next_slab(steady);
        SKIPFFN_WAIT_LGKMCNT0();
        phase_barrier();
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int m = 0; m < MI; ++m)
#pragma unroll
                for (int fj = 0; fj < 2; ++fj) {
                    const int f = (m & 1) ? 1 - fj : fj;
                    acc[m][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ks][f], af[ks][m], acc[m][f], 0, 0, 0);
                }
        __builtin_amdgcn_sched_barrier(0);
        if (wm == 0) wait_next_slab(steady);
        st_rd = st_rd + 1 == NST ? 0 : st_rd + 1;
        st_ld = st_ld + 1 == NST ? 0 : st_ld + 1;
        phase_barrier();
    };

    if (nk > 0) {
        const int ahead = nk < NST - 1 ? nk : NST - 1;
        for (int j = 0; j < ahead; ++j) load_masked(j);
        if (ahead == NST - 1) SKIPFFN_WAIT_VMCNT((NST - 2) * NL); else SKIPFFN_WAIT_VMCNT(0);
        phase_barrier();
        if (wm == 1) phase_barrier();                   // row group 1 runs one phase later
        int j = 0;
        const int full = kt1 * BK <= P.K ? nk : nk - 1;  // slabs inside K (rot == 0 if the last one is not)
        for (; j + NST - 1 < full; ++j) iteration(j, std::true_type{});
        for (; j < nk; ++j) iteration(j, std::false_type{});
        if (wm == 0) phase_barrier();
    }

#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int row = (wm * MI + m) * 16 + r16;
        if (row >= R) continue;
        if (GATE_UP) {
            const int n = n0 + wn * 16 + 4 * kq;
            if (n >= P.N) continue;
            const f32x4 g = acc[m][0], u = acc[m][1];
            float h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = g[j] * sigmoid_f(g[j]) * u[j];
            const int64_t o = (int64_t)row * P.N + n;
            *reinterpret_cast<u32x2*>(P.H + o) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
            if (P.G != nullptr) {
                *reinterpret_cast<u32x2*>(P.G + o) = u32x2{pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3])};
                *reinterpret_cast<u32x2*>(P.U + o) = u32x2{pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3])};
            }
        } else {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int n = n0 + wn * 32 + f * 16 + 4 * kq;
                if (n < P.N) *reinterpret_cast<f32x4*>(P.partial + ((int64_t)z * P.rows + row) * P.N + n) = acc[m][f];
            }
        }
    }
}

template <int MT, bool GATE_UP>
static hipError_t launch_mid(const MidRowsArgs& a, hipStream_t s) {
    const unsigned tiles = (unsigned)((a.N + (GATE_UP ? 63 : 127)) / (GATE_UP ? 64 : 128));
    hipLaunchKernelGGL((mid_rows_kernel<MT, GATE_UP>), dim3(tiles * (unsigned)a.splits), dim3(MID_THREADS), kMidLds<MT>, s, a);
    return hipGetLastError();
}
template <bool GATE_UP>
static hipError_t launch_mid_rows(const MidRowsArgs& a, hipStream_t s) {
    if (a.rows <= 0 || a.N <= 0) return hipSuccess;
    if (a.rows <= 64) return launch_mid<4, GATE_UP>(a, s);
    if (a.rows <= 128) return launch_mid<8, GATE_UP>(a, s);
    if (a.rows <= 192) return launch_mid<12, GATE_UP>(a, s);
    if (a.rows <= 256) return launch_mid<16, GATE_UP>(a, s);
    return hipErrorInvalidValue;
}

template <int MT, bool GATE_UP>
static hipError_t mid_lds_limit() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&mid_rows_kernel<MT, GATE_UP>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kMidLds<MT>);
}
hipError_t mid_rows_init() {
    hipError_t e;
    if ((e = mid_lds_limit<4, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<4, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<8, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<8, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<12, true>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<12, false>()) != hipSuccess) return e;
    if ((e = mid_lds_limit<16, true>()) != hipSuccess) return e;
    return mid_lds_limit<16, false>();
}

hipError_t launch_mid_rows_gate_up(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                   const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, hipStream_t s) {
    MidRowsArgs a{};
    a.rows = rows; a.r_dev = r_dev; a.N = I; a.K = C;
    a.A = xn; a.a_bytes = (uint32_t)((int64_t)rows * C * 2);
    a.B0 = w_gate; a.B1 = w_up; a.b_bytes = (uint32_t)((int64_t)I * C * 2);
    a.splits = 1; a.H = H; a.G = G; a.U = U;
    return launch_mid_rows<true>(a, s);
}

hipError_t launch_mid_rows_down(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down,
                                int splits, float* partial, hipStream_t s) {
    MidRowsArgs a{};
    a.rows = rows; a.r_dev = r_dev; a.N = C; a.K = I;
    a.A = H; a.a_bytes = (uint32_t)((int64_t)rows * I * 2);
    a.B0 = w_down; a.b_bytes = (uint32_t)((int64_t)C * I * 2);
    a.splits = splits; a.partial = partial;
    return launch_mid_rows<false>(a, s);
}

}  // namespace skipffn
