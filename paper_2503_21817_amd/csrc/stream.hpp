// The GEMM core as a stream: a workgroup runs a list of output tiles, and the K slabs of all of them pass through one
// pipeline; both operands K-contiguous.  (gemm.hpp: operand layouts, LDS swizzles, epilogue kinds, the ping-pong
// schedule.)  The GEMMs with an N-contiguous operand stay there, a tile at a time: their memory phases are the longer ones,
// and with the cursors of a stream in them dXn took 675 us instead of 640 at 4096 rows.
//
// With one tile per workgroup a tile costs 11.5 us beside its slabs (1.15 us each): the launch, the first loads, and an
// epilogue that goes through LDS in passes with barriers between them.  Here the loads of the next tile are under way
// before a tile's last slab is computed, and the sums leave from the registers while they fly; the stores are waited for
// a slab later.  What is left at the end of a tile is 2-4 us: the instructions of the epilogue, of which each row group
// hides only what fits under a compute phase of the other.
//
// dW_gate + dW_up (I = 14336, C = 4096, 1792 tiles, R the contraction), us, one tile per workgroup / stream:
// R = 64 69 / 52, 256 97 / 76, 368 120 / 99, 640 157 / 137, 1472 277 / 251, 2944 499 / 471.
#pragma once

#include "gemm.hpp"
#include "tilelists.hpp"

namespace skipffn {

constexpr int kStreamRingB = 3;               // slabs of B in LDS
template <int MI>
constexpr int kStreamRingA = (GEMM_LDS_BYTES - kStreamRingB * OPER_BYTES) / (MI * 4096) < 3 ? 2 : 3;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* base, uint32_t offset, uint32_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base) + offset;
    return make_rsrc(reinterpret_cast<const void*>((uint64_t)uniform((uint32_t)(p >> 32)) << 32 | uniform((uint32_t)p)), uniform(bytes));
}

// ---- epilogue --------------------------------------------------------------------------------------------
// acc[mi][ni][r] of wavefront (wm, wn) is C[m0 + wm * 16 MI + 16 mi + lane % 16][n0 + 16 ni' + 4 (lane / 16) + r].  A lane
// holds four consecutive columns of a row; exchanging a register of fragment 2 p + 1 with the neighbouring row of 16
// lanes (v_permlane16_swap) gives it eight: columns 8 (q / 2) .. + 7 of fragment 2 p + q % 2, q = lane / 16.  So every
// access is 16 bytes, four lanes cover 64 contiguous bytes of a row (bf16), and no LDS round trip is needed.
struct Cols8 { float v[8]; };
__device__ __forceinline__ Cols8 swap_cols(const f32x4& even, const f32x4& odd) {
    Cols8 c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(even[r]), __float_as_uint(odd[r]), false, false);
        c.v[r] = __uint_as_float(s[0]);
        c.v[4 + r] = __uint_as_float(s[1]);
    }
    return c;
}
__device__ __forceinline__ u32x4 pack_cols(const Cols8& c) {
    u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = pack_bf16x2(c.v[2 * k], c.v[2 * k + 1]);
    return v;
}

constexpr uint32_t kStoreOob = 0xFFFFFF00u;   // byte offset past every descriptor of an output block, also with 16 added to it

// The rows of a wavefront in an output matrix, 16 at a time.  Blocks whose rows all exist share a descriptor and step the
// lane's offset; others have one of their own that ends at the last row (stores past it are dropped, loads read zeros).
// Stores keep a zero scalar offset: of a store of 16 bytes a lane with its offset in a scalar register, the compiler lets
// the next instruction overwrite the data, and single words of some lanes then went out wrong.
struct OutRows {
    char* base; int64_t row_bytes; int rows;  // first row and column of the wavefront's part; how many rows exist
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t block(int mi) const {
        const int left = rows - 16 * mi;
        return make_rsrc(base + 16 * mi * row_bytes, left <= 0 ? 0u : (left >= 16 ? kStoreOob : (uint32_t)(left * row_bytes)));
    }
};
// f(desc, at, mi, whole) for the MI blocks of 16 rows: desc(o') the descriptor of the block in a matrix of the same shape,
// at(off) the lane's offset there; off: its offset in a block, or kStoreOob; whole: true_type where every row is known to exist
template <int MI, class F>
__device__ __forceinline__ void for_row_blocks(const OutRows& o, F&& f) {
    if (o.rows >= 16 * MI && 16 * MI * o.row_bytes < (int64_t)kOobOffset) {    // uniform
        const uint32_t step = (uint32_t)(16 * o.row_bytes);
        static_for<MI>([&](auto mi) {
            f([](const OutRows& m) { return make_rsrc(m.base, kOobOffset); },
              [&](uint32_t off) { return (off < kOobOffset ? off : kOobOffset) + mi * step; }, mi, std::true_type{});
        });
    } else {
        static_for<MI>([&](auto mi) {
            f([&](const OutRows& m) { return m.block(mi); }, [](uint32_t off) { return off; }, mi, std::false_type{});
        });
    }
}
__device__ __forceinline__ void buf_store(const u32x4& v, __amdgpu_buffer_rsrc_t d, uint32_t off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, d, (int)off, 0, 0);
}
__device__ __forceinline__ f32x4 buf_load_f32x4(__amdgpu_buffer_rsrc_t d, uint32_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(d, (int)off, 0, 0));
}

__device__ __forceinline__ void store_f32(const Cols8& c, __amdgpu_buffer_rsrc_t d, uint32_t off) {
    const f32x4 lo = {c.v[0], c.v[1], c.v[2], c.v[3]}, hi = {c.v[4], c.v[5], c.v[6], c.v[7]};
    buf_store(__builtin_bit_cast(u32x4, lo), d, off);
    buf_store(__builtin_bit_cast(u32x4, hi), d, off + 16);
}

// Transposition of 32 rows x 32 columns of bf16 inside a wavefront, through 2 KB of LDS of its own: 64 bytes a row, the two
// 32-byte halves of rows 8 - 15 and 24 - 31 exchanged (a transposing read takes 4 rows x 32 bytes per 16 lanes, two such
// groups, 8 rows apart, at a time).  No barrier: a wavefront's LDS operations are done in order.  Inline assembly, because
// the compiler would wait for every direct-to-LDS load in flight first.
struct TransposedBlock {
    uint32_t wr, rd;
    __device__ __forceinline__ TransposedBlock(uint32_t lds, int lane) {
        const int r16 = lane & 15, q = lane >> 4, half = (r16 >> 3) & 1;
        wr = lds + r16 * 64 + ((((q & 1) ^ half) << 1 | (q >> 1)) << 4);
        rd = lds + (8 * q + (r16 >> 2)) * 64 + ((q & 1) << 5) + (r16 & 3) * 8;
    }
    // the lane's 8 columns (chunk 2 (q % 2) + q / 2) of row 16 I + lane % 16
    template <int I>
    __device__ __forceinline__ void put(const u32x4& v) const {
        asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(wr), "v"(v), "n"(I * 1024) : "memory");
    }
    // rows 8 q .. 8 q + 7 of columns lane % 16 (c0) and 16 + lane % 16 (c1)
    __device__ __forceinline__ void get(u32x4& c0, u32x4& c1) const {
        u32x2 a, b, c, d;
        asm volatile("ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:256\n\t"
                     "ds_read_b64_tr_b16 %2, %5\n\tds_read_b64_tr_b16 %3, %5 offset:256\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d) : "v"(rd), "v"(rd ^ 32u) : "memory");
        c0 = u32x4{a[0], a[1], b[0], b[1]};
        c1 = u32x4{c[0], c[1], d[0], d[1]};
    }
};

// scratch: 4 KB of LDS of the wavefront's own
template <int MI, int EPI>
__device__ __forceinline__ void stream_epilogue(const GemmArgs& P, const StreamTile& t, const int Meff, const int row_base,
                                                f32x4 (&acc)[MI][4], const uint32_t scratch) {
    constexpr int WROWS = 16 * MI;
    const int lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = row_base + t.tm * (2 * WROWS) + (wave >> 2) * WROWS;           // first row of the wavefront
    const int lane_col = (q & 1) * 16 + (q >> 1) * 8;
    // byte offset of the lane's 8 columns, column pair p, in a 16-row block
    auto lane_offset = [&](int64_t row_bytes, int es, int col0, int p) {
        const int64_t o = r16 * row_bytes + (lane_col + 32 * p) * es;
        return col0 + lane_col + 32 * p < P.N && o < (int64_t)kStoreOob ? (uint32_t)o : kStoreOob;
    };
    if constexpr (EPI == EPI_STORE) {
        const int col0 = t.tn * BN + (wave & 3) * 64;
        const int es = P.out_f32 ? 4 : 2;
        OutRows o;
        o.row_bytes = (int64_t)P.ldo * es;
        o.base = static_cast<char*>(t.second ? P.out1 : P.out0) + row0 * o.row_bytes + col0 * es;
        o.rows = Meff - row0;
        const uint32_t off[2] = {lane_offset(o.row_bytes, es, col0, 0), lane_offset(o.row_bytes, es, col0, 1)};
        if (P.out_f32 && !P.accumulate) {
            for_row_blocks<MI>(o, [&](auto desc, auto at, auto mi, auto) {
                const __amdgpu_buffer_rsrc_t d = desc(o);
                static_for<2>([&](auto p) { store_f32(swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1]), d, at(off[p])); });
            });
        } else if (P.out_f32) {
            for_row_blocks<MI>(o, [&](auto desc, auto at, auto mi, auto) {
                const __amdgpu_buffer_rsrc_t d = desc(o);
                f32x4 old[4];
                static_for<4>([&](auto h) { old[h] = buf_load_f32x4(d, at(off[h >> 1]) + (h & 1) * 16); });
                static_for<2>([&](auto p) {
                    Cols8 c = swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) { c.v[k] += old[2 * p][k]; c.v[4 + k] += old[2 * p + 1][k]; }
                    store_f32(c, d, at(off[p]));
                });
            });
        } else if (!P.accumulate) {
            for_row_blocks<MI>(o, [&](auto desc, auto at, auto mi, auto) {
                const __amdgpu_buffer_rsrc_t d = desc(o);
                static_for<2>([&](auto p) { buf_store(pack_cols(swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1])), d, at(off[p])); });
            });
        } else {
            for_row_blocks<MI>(o, [&](auto desc, auto at, auto mi, auto) {
                const __amdgpu_buffer_rsrc_t d = desc(o);
                u32x4 old[2];
                static_for<2>([&](auto p) { old[p] = __builtin_amdgcn_raw_buffer_load_b128(d, (int)at(off[p]), 0, 0); });
                static_for<2>([&](auto p) {
                    Cols8 c = swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        c.v[2 * k] += bf16lo_to_f32(old[p][k]);
                        c.v[2 * k + 1] += bf16hi_to_f32(old[p][k]);
                    }
                    buf_store(pack_cols(c), d, at(off[p]));
                });
            });
        }
    } else if constexpr (EPI == EPI_PARTIAL) {
        const int col0 = t.tn * BN + (wave & 3) * 64;
        OutRows o;
        o.row_bytes = (int64_t)P.N * 4;
        o.base = reinterpret_cast<char*>(P.partial) + ((int64_t)t.z * P.M + row0) * o.row_bytes + col0 * 4;
        o.rows = Meff - row0;
        const uint32_t off[2] = {lane_offset(o.row_bytes, 4, col0, 0), lane_offset(o.row_bytes, 4, col0, 1)};
        for_row_blocks<MI>(o, [&](auto desc, auto at, auto mi, auto) {
            const __amdgpu_buffer_rsrc_t d = desc(o);
            static_for<2>([&](auto p) { store_f32(swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1]), d, at(off[p])); });
        });
    } else if constexpr (EPI == EPI_RESID_SCATTER) {
        // rows idx[row] of out and of the residual (the same tensor in place: a lane reads what it writes); below 2 GiB
        const int col0 = t.tn * BN + (wave & 3) * 64;
        const __amdgpu_buffer_rsrc_t res = make_rsrc(P.e0, kOobOffset), out = make_rsrc(P.out0, kOobOffset);
        uint32_t at[MI][2];
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int row = row0 + mi * 16 + r16;
            const uint32_t r = row < Meff ? (uint32_t)P.idx[row] * (uint32_t)P.ldo : 0u;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int col = col0 + lane_col + 32 * p;
                at[mi][p] = row < Meff && col < P.N ? (r + (uint32_t)col) * 2u : kOobOffset;
            }
        }
        static_for<(MI + 1) / 2>([&](auto h) {
            constexpr int n = 2 * h + 2 <= MI ? 4 : 2;       // the last row of an odd height stands alone
            u32x4 x[2][2];
            if (!P.no_residual)
                static_for<n>([&](auto k) { x[k >> 1][k & 1] = buf_load16(res, at[2 * h + (k >> 1)][k & 1]); });
            static_for<n>([&](auto k) {
                constexpr int mi = 2 * h + (k >> 1), p = k & 1;
                Cols8 c = swap_cols(acc[mi][2 * p], acc[mi][2 * p + 1]);
                if (!P.no_residual) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        c.v[2 * e] += bf16lo_to_f32(x[k >> 1][p][e]);
                        c.v[2 * e + 1] += bf16hi_to_f32(x[k >> 1][p][e]);
                    }
                }
                buf_store(pack_cols(c), out, at[mi][p]);
            });
        });
    } else if constexpr (EPI == EPI_SWIGLU) {
        // fragments 0, 1: 32 columns of gate, 2, 3: the same of up
        const int col0 = t.tn * (BN / 2) + (wave & 3) * 32;
        OutRows h;
        h.row_bytes = (int64_t)P.ldo * 2;
        h.base = static_cast<char*>(P.out0) + row0 * h.row_bytes + col0 * 2;
        h.rows = Meff - row0;
        OutRows g = h, u = h;
        g.base = static_cast<char*>(P.out1) + row0 * h.row_bytes + col0 * 2;
        u.base = static_cast<char*>(P.out2) + row0 * h.row_bytes + col0 * 2;
        const uint32_t off = lane_offset(h.row_bytes, 2, col0, 0);
        const bool saved = P.out1 != nullptr, transposed = P.outT0 != nullptr;
        const TransposedBlock tb(scratch, lane);
        // the lane's column and first row in the transposed copy, columns 16 further on for the second half
        bf16_t* to = static_cast<bf16_t*>(P.outT0) + (int64_t)(col0 + r16) * P.ldt + row0 + 8 * q;
        for_row_blocks<MI>(h, [&](auto desc, auto at, auto mi, auto whole) {
            const Cols8 gc = swap_cols(acc[mi][0], acc[mi][1]), uc = swap_cols(acc[mi][2], acc[mi][3]);
            Cols8 hc;
#pragma unroll
            for (int k = 0; k < 8; ++k) hc.v[k] = gc.v[k] * sigmoid_f(gc.v[k]) * uc.v[k];
            u32x4 hp = pack_cols(hc);
            buf_store(hp, desc(h), at(off));
            if (saved) {
                buf_store(pack_cols(gc), desc(g), at(off));
                buf_store(pack_cols(uc), desc(u), at(off));
            }
            if (transposed) {
                // zeros past the last row: the sums there are 0 * W, and that is NaN where W is not finite
                if (!whole && row0 + mi * 16 + r16 >= Meff) hp = u32x4{0u, 0u, 0u, 0u};
                tb.template put<mi & 1>(hp);
                if constexpr ((mi & 1) == 1) {
                    u32x4 c0, c1;
                    tb.get(c0, c1);
                    if (row0 + (mi - 1) * 16 + 8 * q < P.ldt) {
                        if (col0 + r16 < P.N) *reinterpret_cast<u32x4*>(to + (mi - 1) * 16) = c0;
                        if (col0 + 16 + r16 < P.N) *reinterpret_cast<u32x4*>(to + (int64_t)16 * P.ldt + (mi - 1) * 16) = c1;
                    }
                }
            }
        });
    }
}

// All 512 threads of the workgroup call it with the same arguments; tile rows count from row_base.  K of an operand whose rows are zero from Keff to the
// next multiple of 64 may be passed rounded up: only a slab that reaches past Keff masks its lanes.
template <int MI, int EPI, class Work>
__device__ __forceinline__ void stream_gemm(const GemmArgs& P, const Work work, const int Meff, const int Keff, const int row_base = 0) {
    constexpr bool GU = EPI == EPI_SWIGLU;   // B tile = 128 rows of W_gate + 128 of W_up
    constexpr int TM = 32 * MI, WROWS = 16 * MI;
    constexpr int STAGE_A = TM * 128, NSA = kStreamRingA<MI>, A_AHEAD = NSA - 1, B_BASE = NSA * STAGE_A;
    constexpr int AL0 = (MI + 1) / 2, AL1 = MI / 2;         // 1 KB regions of an A slab a wavefront of row group 0 / 1 loads
    constexpr bool ODD = AL0 != AL1;
    static_assert(B_BASE + kStreamRingB * OPER_BYTES <= GEMM_LDS_BYTES, "operand rings must fit in LDS");
    extern __shared__ __align__(16) char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const uint32_t lds0 = lds_addr_of(smem);
    typedef __attribute__((address_space(3))) void* lds_void_ptr;

    StreamTile tile;
    if (!work.get(0, tile)) return;                          // uniform over the workgroup

    // ---- per-lane offsets of the loads inside a tile (constant: the tile's place is in the descriptor, which also ends
    // at the last row, so that rows past it read zeros)
    const int region_a = wm == 0 ? wave * AL0 : 4 * AL0 + (wave - 4) * AL1;
    uint32_t a_goff[AL0], b_goff[4];
    auto lane_off = [](int64_t bytes) { return bytes < (int64_t)kOobOffset ? (uint32_t)bytes : kOobOffset; };
#pragma unroll
    for (int l = 0; l < AL0; ++l) {
        const int row = 8 * (region_a + l) + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        a_goff[l] = lane_off(((int64_t)row * P.lda + c * 8) * 2);
    }
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        const int qb = wave * 4 + l;
        const int row = 8 * qb + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        b_goff[l] = lane_off(((int64_t)(GU ? row & 127 : row) * P.ldb + c * 8) * 2);
    }

    // ---- load cursors: the next slab of A (of B) to fetch, A_AHEAD (2) slabs ahead of the one that is read.  Operands
    // are smaller than 2 GiB, so offsets of existing tiles fit 32 bits.  (Flags are kept as integers: as truth values
    // they travel in lane masks.)
    const int ktp = Keff > 0 ? (Keff + BK - 1) / BK : 1;     // slabs of K; K = 0: one slab of zeros (empty operands)
    const int ragged = Keff % BK != 0 ? 1 : 0;               // the last one reaches past K
    const uint32_t a_base = (uint32_t)row_base * (uint32_t)P.lda * 2u;
    const uint32_t a_tile = (uint32_t)TM * (uint32_t)P.lda * 2u, a_end = Keff > 0 ? (uint32_t)Meff * (uint32_t)P.lda * 2u : 0u;
    const uint32_t b_tile = (uint32_t)(GU ? BN / 2 : BN) * (uint32_t)P.ldb * 2u;
    const uint32_t b_end = Keff > 0 ? (uint32_t)P.N * (uint32_t)P.ldb * 2u : 0u;
    // *_left: slabs until the tile ends (0: the list has ended), of which the last *_mask reach past K
    int a_i = 0, a_kt = 0, a_left = 0, a_mask = 0, b_i = 0, b_kt = 0, b_left = 0, b_mask = 0;
    uint32_t a_step = 0, b_step = 0;
    StreamTile a_t = tile, b_t = tile;
    __amdgpu_buffer_rsrc_t a_src, b_src;
    auto begin_a = [&]() {                                   // tile a_t
        a_kt = a_t.kb;
        a_left = a_t.ke - a_t.kb;
        a_mask = ragged - (ktp - a_t.ke);
        a_mask = a_mask > 0 ? a_mask : 0;
        const uint32_t o = a_base + (uint32_t)a_t.tm * a_tile;
        a_src = uniform_rsrc(a_t.second ? P.A1 : P.A0, o, a_end > o ? a_end - o : 0u);
        a_step = (uint32_t)a_kt * (BK * 2u);
    };
    auto begin_b = [&]() {                                   // tile b_t
        b_kt = b_t.kb;
        b_left = b_t.ke - b_t.kb;
        b_mask = ragged - (ktp - b_t.ke);
        b_mask = b_mask > 0 ? b_mask : 0;
        const uint32_t o = (uint32_t)b_t.tn * b_tile;
        b_src = uniform_rsrc(GU && wave >= 4 ? P.B1 : P.B0, o, b_end > o ? b_end - o : 0u);       // GU: regions 16 .. = rows 128 ..
        b_step = (uint32_t)b_kt * (BK * 2u);
    };
    uint32_t a_ld = region_a * 1024, b_ld = B_BASE + wave * 4096;        // LDS offsets this wavefront loads to
    const uint32_t a_ld_end = NSA * STAGE_A + region_a * 1024, b_ld_end = B_BASE + kStreamRingB * OPER_BYTES + wave * 4096;
    // after a slab has been issued
    auto step_a = [&]() {
        a_ld += STAGE_A;
        if (a_ld == a_ld_end) a_ld -= NSA * STAGE_A;
        a_step += BK * 2u;
        ++a_kt;
        if (--a_left == 0) {
            if (work.get(++a_i, a_t)) begin_a();
        }
    };
    auto step_b = [&]() {
        b_ld += OPER_BYTES;
        if (b_ld == b_ld_end) b_ld -= kStreamRingB * OPER_BYTES;
        b_step += BK * 2u;
        ++b_kt;
        if (--b_left == 0) {
            if (work.get(++b_i, b_t)) begin_b();
        }
    };
    auto load_a1 = [&](auto l, uint32_t off) {
        if (ODD && l == AL0 - 1 && wm != 0) return;          // uniform
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a_src, (lds_void_ptr)(smem + a_ld + l * 1024), 16, (int)off, (int)a_step, 0, 0);
    };
    auto load_b1 = [&](auto l, uint32_t off) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b_src, (lds_void_ptr)(smem + b_ld + l * 1024), 16, (int)off, (int)b_step, 0, 0);
    };
    // a whole share; a slab that reaches past K masks its lanes (the mask has to be in the per-lane offset)
    auto load_a = [&]() {
        if (a_left == 0) return;                             // uniform
        if (a_left > a_mask) {
            static_for<AL0>([&](auto l) { load_a1(l, a_goff[l]); });
        } else {
            asm volatile("; K tail" ::: "memory");
            static_for<AL0>([&](auto l) {
                const int row = 8 * (region_a + l) + (lane >> 3), kk = a_kt * BK + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
                load_a1(l, kk < Keff ? a_goff[l] : kOobOffset);
            });
            asm volatile("; K tail end" ::: "memory");
        }
        step_a();
    };
    auto load_b = [&]() {
        if (b_left == 0) return;
        if (b_left > b_mask) {
            static_for<4>([&](auto l) { load_b1(l, b_goff[l]); });
        } else {
            asm volatile("; K tail" ::: "memory");
            static_for<4>([&](auto l) {
                const int qb = wave * 4 + l, row = 8 * qb + (lane >> 3);
                const int kk = b_kt * BK + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
                load_b1(l, kk < Keff ? b_goff[l] : kOobOffset);
            });
            asm volatile("; K tail end" ::: "memory");
        }
        step_b();
    };

    // ---- fragment reads: see gemm.hpp
    uint32_t a_rd[2], b_rd[2];
    const int b_row0 = GU ? wn * 32 : wn * 64;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        a_rd[ks] = lds0 + kc_off(wm * WROWS + (lane & 15), 4 * ks + (lane >> 4));
        b_rd[ks] = lds0 + B_BASE + kc_off(b_row0 + (lane & 15), 4 * ks + (lane >> 4));
    }
    uint32_t rd_a = 0, rd_b = 0;                             // byte offsets of the stages that are read
    f32x4 acc[MI][4];
    bf16x8 af[MI], bfr[4];
    // the reads of half slab KS; LOADS: with the loads of A (KS = 0) or B (KS = 1) spread between them
    auto read_frags = [&](auto ks, auto loads) {
        constexpr int KS = decltype(ks)::value;
        constexpr int NL = !decltype(loads)::value ? 0 : (KS == 0 ? AL0 : 4), NR = MI + 4;
        const uint32_t aa = a_rd[KS] + rd_a;
        const uint32_t ba = b_rd[KS] + rd_b;
        static_for<NR>([&](auto r) {
            static_for<NL>([&](auto l) {
                if constexpr (l * NR / (NL > 0 ? NL : 1) == r) {
                    if constexpr (KS == 0) load_a1(l, a_goff[l]); else load_b1(l, b_goff[l]);
                }
            });
            if constexpr (r < MI) {
                af[r] = ds_read_b128_imm<r * 2048>(aa);
            } else {
                constexpr int ni = r - MI;
                bfr[ni] = ds_read_b128_imm<GU ? (ni >> 1) * 16384 + (ni & 1) * 2048 : ni * 2048>(ba);
            }
        });
    };
    auto phase_barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    // FIRST: the sums begin here
    auto compute_phase = [&](auto first) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int nj = 0; nj < 4; ++nj) {
                const int ni = (mi & 1) ? 3 - nj : nj;
                acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ni], af[mi], decltype(first)::value ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : acc[mi][ni], 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    // slab j + 1 has landed; what slab j issued for slab j + 2 may still fly
    auto wait_next_slab = [&](int issued) {
        if (issued == 0) SKIPFFN_WAIT_VMCNT(0);
        else if (A_AHEAD == 1) SKIPFFN_WAIT_VMCNT(4);
        else if (!ODD || wm == 0) SKIPFFN_WAIT_VMCNT(4 + AL0);
        else SKIPFFN_WAIT_VMCNT(4 + AL1);
    };

    begin_a();
    begin_b();
    load_a();
    load_b();
    {
        const int two = b_left;
        if (A_AHEAD == 2) load_a();
        load_b();
        wait_next_slab(two);
    }
    phase_barrier();
    if (wm == 1) phase_barrier();                            // row group 1 runs one phase later
    const std::integral_constant<int, 0> k0{};
    const std::integral_constant<int, 1> k1{};
    // M(j, 1), C(j, 1)
    auto second_half = [&]() {
        const int issued = b_left;
        if (b_left > b_mask) {
            read_frags(k1, std::true_type{});
            step_b();
        } else {
            load_b();
            read_frags(k1, std::false_type{});
        }
        if (wm == 1) wait_next_slab(issued);
        SKIPFFN_WAIT_LGKMCNT0();
        phase_barrier();
        compute_phase(std::false_type{});
        if (wm == 0) wait_next_slab(issued);
        rd_a += STAGE_A; if (rd_a == NSA * STAGE_A) rd_a = 0;
        rd_b += OPER_BYTES; if (rd_b == kStreamRingB * OPER_BYTES) rd_b = 0;
        phase_barrier();
    };
    StreamTile done = tile;                                  // the tile whose sums are in acc
    // LDS for the epilogue: this wavefront's part of the stage that the tile's last slab of B was read from, which it
    // fills again itself, after the epilogue
    auto scratch = [&]() { return lds0 + B_BASE + wave * 4096 + (rd_b == 0 ? (kStreamRingB - 1) * OPER_BYTES : rd_b - OPER_BYTES); };
    for (int i = 0;;) {
        // M(0, 0): the tile before leaves while the loads for this one fly
        load_a();
        if (i > 0) {
            __builtin_amdgcn_sched_barrier(0);
            stream_epilogue<MI, EPI>(P, done, Meff, row_base, acc, scratch());
            __builtin_amdgcn_sched_barrier(0);
        }
        read_frags(k0, std::false_type{});
        SKIPFFN_WAIT_LGKMCNT0();
        phase_barrier();
        compute_phase(std::true_type{});
        phase_barrier();
        second_half();
        for (int j = tile.ke - tile.kb - 1; j > 0; --j) {
            if (a_left > a_mask) {
                read_frags(k0, std::true_type{});
                step_a();
            } else {
                load_a();
                read_frags(k0, std::false_type{});
            }
            SKIPFFN_WAIT_LGKMCNT0();
            phase_barrier();
            compute_phase(std::false_type{});
            phase_barrier();
            second_half();
        }
        done = tile;
        if (!work.get(++i, tile)) break;
    }
    if (wm == 0) phase_barrier();                            // balances group 1's extra barrier
    stream_epilogue<MI, EPI>(P, done, Meff, row_base, acc, scratch());
}

// Tiles over the rows [row_base, rows); `after` tiles have been dealt to the workgroups already
template <int MI, int EPI>
__device__ __forceinline__ void stream_grid(const GemmArgs& P, const int splits, const int block, const int workgroups, const int rows,
                                            const int Meff, const int Keff, const int row_base = 0, const int after = 0) {
    constexpr bool SPLIT = EPI == EPI_STORE || EPI == EPI_PARTIAL;
    const GridWork<SPLIT> w(block, workgroups, (rows - row_base + 32 * MI - 1) / (32 * MI), P.tiles_n, splits, P.batch,
                            Keff > 0 ? (Keff + BK - 1) / BK : 1, after);
    stream_gemm<MI, EPI>(P, w, Meff, Keff, row_base);
}

// 256-row tiles: workgroup `block` of `workgroups`
template <int EPI>
__device__ __forceinline__ void stream_tall(const GemmArgs& P, const int block, const int workgroups) {
    const int Meff = uniform(effective_rows(P.M, P.m_dev));
    int Keff = uniform(effective_rows(P.K, P.k_dev));
    if (EPI == EPI_STORE) Keff = (Keff + BK - 1) / BK * BK;  // the transposed copies are zero up to the next multiple of 64
    if (Meff > 0) stream_grid<8, EPI>(P, P.splits, block, workgroups, Meff, Meff, Keff);
}
template <int EPI>
__global__ __launch_bounds__(GEMM_THREADS) void stream_gemm_kernel(GemmArgs P) {
    stream_tall<EPI>(P, (int)blockIdx.x, (int)gridDim.x);
}

// Tiles of the heights that suit the row count: gate/up (streamk.hpp), and the down GEMM where its K range is cut evenly or not
// at all.  Down, 256-row tiles / these, us: 300 rows 59 / 51, 368 58 / 52, 420 58 / 54 (C = 4096, I = 14336; 480 to 512 rows
// even), 368 rows 173 / 154 (C = 8192, I = 28672), 1100 rows 50 / 46 (2048, 8192); with the residual in the epilogue 2300 rows
// 25 / 21, 4200 rows 43 / 34 (4096, 512).
template <int EPI>
__device__ __forceinline__ void stream_rows(const GemmArgs& P, const StreamRows plan, const int splits, const int b, const int nb) {
    const int Meff = uniform(effective_rows(P.M, P.m_dev)), Keff = uniform(effective_rows(P.K, P.k_dev));
    if (Meff <= 0) return;
    const int columns = P.tiles_n * splits;                  // tiles of a tile row
    int base = 0, after = 0;                                 // rows and tiles of the first of two parts
    if (plan.full > 0) {
        if constexpr (EPI == EPI_SWIGLU) {
            base = plan.full * 256 < Meff ? plan.full * 256 : Meff;
            after = plan.full * columns;
        }
        stream_grid<8, EPI>(P, splits, b, nb, EPI == EPI_SWIGLU ? base : Meff, Meff, Keff);
        if (EPI != EPI_SWIGLU || plan.mi == 0) return;
        lds_barrier();                                       // other stages, other parts of them
    }
    switch (plan.mi) {                                       // uniform
        case 4: stream_grid<4, EPI>(P, splits, b, nb, Meff, Meff, Keff, base, after); break;
        case 5: stream_grid<5, EPI>(P, splits, b, nb, Meff, Meff, Keff, base, after); break;
        case 6: stream_grid<6, EPI>(P, splits, b, nb, Meff, Meff, Keff, base, after); break;
        default: stream_grid<7, EPI>(P, splits, b, nb, Meff, Meff, Keff, base, after); break;
    }
}

// the plan of a row count on the device
template <int EPI>
__device__ __forceinline__ StreamRows stream_plan_of_count(const GemmArgs& P, const int splits, const int nb) {
    const int Meff = uniform(effective_rows(P.M, P.m_dev)), Keff = uniform(effective_rows(P.K, P.k_dev));
    const int slabs = ((Keff + BK - 1) / BK + splits - 1) / splits;
    const StreamRows plan = stream_rows_plan(Meff, P.tiles_n * splits, slabs, nb, P.outT0 != nullptr, EPI == EPI_SWIGLU);
    return StreamRows{uniform(plan.full), uniform(plan.mi)};
}
// plan: of a row count on the host; {0, 0}: the count is on the device
template <int EPI>
__global__ __launch_bounds__(GEMM_THREADS) void stream_gemm_rows_kernel(GemmArgs P, StreamRows plan) {
    if (plan.full == 0 && plan.mi == 0) plan = stream_plan_of_count<EPI>(P, P.splits, (int)gridDim.x);
    stream_rows<EPI>(P, plan, P.splits, (int)blockIdx.x, (int)gridDim.x);
}

// The balanced split-K of streamk.hpp into fp32 slabs: workgroup `block` of tiles_n * nbg
__device__ __forceinline__ void stream_balanced(const GemmArgs& P, const int block, const int tiles_n, const int nbg) {
    const int Meff = uniform(effective_rows(P.M, P.m_dev)), Keff = uniform(effective_rows(P.K, P.k_dev));
    const int g = (Meff + BM - 1) / BM, kt = (Keff + BK - 1) / BK;
    if (g == 0 || kt == 0) return;
    const StreamKPlan p = streamk_plan(g, kt, nbg);
    int tn, j;
    balanced_share(p, tiles_n, block, tn, j);
    stream_gemm<8, EPI_PARTIAL>(P, BalancedWork(p, tn, j), Meff, Keff);
}

}  // namespace skipffn
