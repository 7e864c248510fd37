// Main loop of a workgroup tile of A_ROWS x 128 over slabs of 64 k, both operands K-contiguous ([rows][K] bf16), for
// GEMMs whose tiles are many and short of MFMA work: 8 wavefronts, 2 (A rows) x 4 (B rows), v_mfma_f32_16x16x32_bf16.
//
// Both operands come by 16-byte direct-to-LDS loads (a wave-wide load fills 1 KB: 8 rows of 128 bytes, swizzled on the
// global side) into a ring of as many slabs as fit 160 KB: 6 at 64 A rows, 5 at 128, 4 at 192, 3 at 256.  The two row
// groups of four wavefronts run one phase apart: one reads the fragments of its next slab and issues loads (spread
// between the reads), the other runs its MFMAs; two barriers a slab (the 256 x 256 core has four, with twice the MFMAs
// between them).
#pragma once

#include "gemm.hpp"

namespace skipffn {

constexpr int SLAB_THREADS = 512;
constexpr int SLAB_B_ROWS = 128;              // or 64, where tiles of 128 are too few
template <int A_ROWS, int B_ROWS = SLAB_B_ROWS>
constexpr int kSlabStage = (A_ROWS + B_ROWS) * 128;                      // bytes of a slab
template <int A_ROWS, int B_ROWS = SLAB_B_ROWS>
constexpr int kSlabStages = (160 * 1024) / kSlabStage<A_ROWS, B_ROWS>;
template <int A_ROWS, int B_ROWS = SLAB_B_ROWS>
constexpr int kSlabLds = kSlabStages<A_ROWS, B_ROWS> * kSlabStage<A_ROWS, B_ROWS>;       // dynamic LDS of the kernel
template <int A_ROWS>
constexpr int kSlabPiecesA = A_ROWS / 64;                                // 1 KB pieces of A each wavefront loads
template <int A_ROWS, int B_ROWS = SLAB_B_ROWS>
constexpr int kSlabPieces = kSlabPiecesA<A_ROWS> + B_ROWS / 64;          // and of both

// goff[l]: byte offset of the lane's 16 bytes of piece l at slab 0, or kOobOffset.  Wavefront w loads the 8-row pieces
// q = w * kSlabPiecesA + l of A, then q = 2 w, 2 w + 1 of B; (B_ROWS = 64: q = w); its lane takes row 8 q + lane / 8 and the chunk of 8 k
// (lane % 8) ^ ((row / 2) % 8).  Slabs kt0 .. kt0 + nk - 1 are summed, beginning at kt0 + rot (rot = 0: in order;
// otherwise every slab has to lie inside K); k past K count as zeros.
// acc[m][f], wavefront (wm, wn): A rows wm * A_ROWS / 2 + 16 m + lane % 16, B rows b_row + f * B_STRIDE + 4 (lane / 16) + r, f < B_ROWS / 64.
// All 512 threads call it with the same kt0, nk, rot, K.
//
// NORM: the rows of A are not normalised yet; their squares are added from the MFMA operands in registers, a fragment by one
// of the four wavefronts that hold it: ss[m] of a lane gathers k of row ... + 16 m + lane % 16, and the sum over the four lanes
// of a row in the four wavefronts of the row group is the row's.
template <int A_ROWS, int B_STRIDE, bool NORM = false, int B_ROWS = SLAB_B_ROWS>
__device__ __forceinline__ void slab_loop(const __amdgpu_buffer_rsrc_t ra, const __amdgpu_buffer_rsrc_t rb,
                                          const uint32_t (&goff)[kSlabPieces<A_ROWS, B_ROWS>], const int b_row, const int kt0,
                                          const int nk, const int rot, const int K, f32x4 (&acc)[A_ROWS / 32][B_ROWS / 64],
                                          float (&ss)[A_ROWS / 32]) {
    static_assert(A_ROWS % 64 == 0 && A_ROWS <= 256, "two row groups, whole pieces per wavefront");
    constexpr int NST = kSlabStages<A_ROWS, B_ROWS>, STAGE = kSlabStage<A_ROWS, B_ROWS>, B_BASE = A_ROWS * 128;
    constexpr int MI = A_ROWS / 32;           // row fragments of a wavefront
    constexpr int NLA = kSlabPiecesA<A_ROWS>, NL = kSlabPieces<A_ROWS, B_ROWS>;
    constexpr int NF = B_ROWS / 64;           // fragments and 1 KB pieces of B of a wavefront
    static_assert(B_ROWS == 64 || B_ROWS == 128, "four column groups");
    static_assert(NST >= 3, "two slabs in flight beside the one that is read");
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2;
    const int r16 = lane & 15, kq = lane >> 4;
    typedef __attribute__((address_space(3))) void* lds_void_ptr;
    auto lds_piece = [&](int stage, int l) {
        return smem + stage * STAGE + (l < NLA ? (wave * NLA + l) * 1024 : B_BASE + (wave * NF + (l - NLA)) * 1024);
    };
    auto slab_of = [&](int j) { const int jr = j + rot; return kt0 + (jr < nk ? jr : jr - nk); };
    // a slab that may reach past K: k past the end are zeros
    auto load_masked = [&](int j) {
        const int slab = slab_of(j);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int q = l < NLA ? wave * NLA + l : wave * NF + (l - NLA);
            const int row = 8 * q + (lane >> 3), kk = slab * BK + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
            const uint32_t off = goff[l] != kOobOffset && kk < K ? goff[l] + (uint32_t)slab * (BK * 2) : kOobOffset;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(l < NLA ? ra : rb, (lds_void_ptr)lds_piece(j % NST, l), 16, (int)off, 0, 0, 0);
        }
    };

#pragma unroll
    for (int m = 0; m < MI; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[m][f] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < MI; ++m) ss[m] = 0.0f;
    uint32_t a_rd[2], b_rd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        a_rd[ks] = lds_addr_of(smem) + kc_off(wm * MI * 16 + r16, 4 * ks + kq);
        b_rd[ks] = lds_addr_of(smem) + B_BASE + kc_off(b_row + r16, 4 * ks + kq);
    }
    auto phase_barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    bf16x8 af[2][MI], bfr[2][NF];
    int st_rd = 0, st_ld = NST - 1;                     // stages slab j is read from and slab j + NST - 1 loaded to
    // the memory phase of slab j: the loads of slab j + NST - 1 spread between the fragment reads
    auto memory_phase = [&](int j, auto steady) {
        constexpr bool STEADY = decltype(steady)::value;
        if (!STEADY && j + NST - 1 < nk) load_masked(j + NST - 1);
        const int step = STEADY ? slab_of(j + NST - 1) * (BK * 2) : 0;
        const uint32_t so = (uint32_t)(st_rd * STAGE);
        const uint32_t aa[2] = {a_rd[0] + so, a_rd[1] + so}, ba[2] = {b_rd[0] + so, b_rd[1] + so};
        constexpr int NR = 2 * (MI + NF);
        static_for<NR>([&](auto r) {
            if constexpr (STEADY)
                static_for<NL>([&](auto l) {
                    if constexpr (l * NR / NL == r)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(l < NLA ? ra : rb, (lds_void_ptr)lds_piece(st_ld, l), 16, (int)goff[l], step, 0, 0);
                });
            constexpr int ks = r / (MI + NF), i = r % (MI + NF);
            if constexpr (i < NF) bfr[ks][i] = ds_read_b128_imm<i * B_STRIDE * 128>(ba[ks]);
            else af[ks][i - NF] = ds_read_b128_imm<(i - NF) * 2048>(aa[ks]);
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
        if constexpr (NORM) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int m = 0; m < MI; ++m)
                    if (((ks * MI + m) & 3) == (wave & 3)) ss[m] = add_squares(af[ks][m], ss[m]);      // uniform
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int m = 0; m < MI; ++m)
#pragma unroll
                for (int fj = 0; fj < NF; ++fj) {
                    const int f = (m & 1) ? NF - 1 - fj : fj;
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
        const int full = (kt0 + nk) * BK <= K ? nk : nk - 1;  // slabs inside K (rot == 0 if the last one is not)
        for (; j + NST - 1 < full; ++j) iteration(j, std::true_type{});
        for (; j < nk; ++j) iteration(j, std::false_type{});
        if (wm == 0) phase_barrier();
    }
}

}  // namespace skipffn
