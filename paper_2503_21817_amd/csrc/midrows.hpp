// The two forward GEMMs for up to 256 retained rows (decode batches, prefill of an image, small training batches), and
// for more rows of a narrow layer, in several row tiles.
//
// Bound by streaming the weights from HBM.  A tile is ALL rows (16 * MT of them) times up to 128 weight rows, so that every
// weight byte goes to one CU only and the tiles are many (I / 64 or more for gate/up, see gate_up_cols; C / 128 with K split for down, whose
// fp32 slabs a reducing kernel adds; gate/up splits K as well where I is so small that most CUs would have no tile).
// What limits a CU is the bytes it loads, weights and activations together, and the ends of its K range: 56-column gate/up tiles take 620 MB
// of both at 184 rows in 57 us (11 TB/s over the chip), down's parts of 28 slabs 294 MB in 37 (8 TB/s).  Hence both operands go to LDS by direct
// loads of whole 128-byte lines
// (weights straight to registers, 16 rows x 64 bytes a load: 65 instead of 57 us at 184 rows), and the rows are not
// padded further than to 64.
//
// Where rows are a multiple of 8 KB apart, workgroups of an XCD start at different slabs and wrap around: walking K in step they would all read the same few
// L2 and HBM channels (gate/up at 64 rows 52 -> 43 us).  At strides of 6, 4 and 28 KB it makes no difference, and K
// is summed in order.
//
// Measured at C = 4096, I = 14336 in a kernel trace (the loads of the weights alone: 41 + 21 us): gate/up 43 / 50 / 58 / 65
// us and down 26 / 32 / 37 / 43 us at 64 / 128 / 184 / 256 rows; 128-row tiles with the weights shared through L2: 73
// and 41 at 184.  Split gate/up and its reduction, 128 rows:  C = 8192, I = 512: 13.2 + 7.1 us;  C = 4096, I = 2048: 15.5 + 4.3.
//
// NORM: gate/up of up to 64 rows on the rows as they are in the hidden states, normalised beside the product (layout.hpp,
// norm_in_gate_up).  A fragment's squares are 16 vector operations of one of the four wavefronts that read it; with all
// four adding all fragments and a gain multiplied in, the loop becomes bound by them (C = 4096, 8 rows: 92 instead of 67 us a layer),
// and so it does on more rows (184: 122 instead of 106).
#pragma once

#include "kernels.hpp"
#include "slabloop.hpp"

namespace skipffn {

constexpr int MID_CHANNEL_K = 4096;           // rows this many k apart share their L2 channels

struct MidRowsArgs {
    int rows; const int32_t* r_dev;           // row bound, optional device count
    int N, K;                                 // output columns, contraction length (multiples of 8)
    const bf16_t* A; uint32_t a_bytes;        // [rows][K]
    const bf16_t* B0; const bf16_t* B1; uint32_t b_bytes;   // [N][K]; gate/up: W_gate, W_up
    int splits;
    int cols;                                 // gate/up: columns of a tile (gate_up_cols)
    // gate/up: 16-byte chunk c (8 columns) of row r of H at byte r * h_row + c * h_chunk; G, U [rows][N], optional
    bf16_t* H; uint32_t h_row, h_chunk; bf16_t* G; bf16_t* U;
    float* partial;                           // down: [splits][rows][N]; gate/up with splits > 1: [splits][rows][2][N]
    // gate/up that normalises its rows itself: A = hidden [T][K], of which the rows idx are taken
    const int32_t* idx; float eps;
    const float* rstd;                        // gate/up of up to 64 rows, optional: A holds rows yet to be multiplied by this
};

// chunk_major_h: H is [N / 8][rows][8], splits 1, whole rows
MidRowsArgs mid_rows_gate_up_args(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                  const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major_h, int cols);
MidRowsArgs mid_rows_down_args(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down, int splits,
                               float* partial);

// workgroup `block` of the tiles' (MT fragments of 16 rows high), all 512 threads
// (SCALE: P.rstd may be given)
template <int MT, bool GATE_UP, bool NORM = false, bool SCALE = false>
__device__ __forceinline__ void mid_rows_tile(const MidRowsArgs& P, const int block) {
    constexpr int MI = MT / 2;                // row fragments of a wavefront
    constexpr int NLA = kSlabPiecesA<16 * MT>, NL = kSlabPieces<16 * MT>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;  // row group, column quarter
    const int R = effective_rows(P.rows, P.r_dev);
    if (R <= 0) return;                       // uniform
    // row tile by row tile, in each the column tiles, in each the K splits
    const int cols = GATE_UP ? P.cols : SLAB_B_ROWS;
    const int per_m = (P.N + cols - 1) / cols * P.splits;
    const int tm = block / per_m, b = block - tm * per_m;
    const int z = b % P.splits;
    const int m0 = tm * 16 * MT, n0 = b / P.splits * cols;
    if (m0 >= R) return;                      // uniform: the bound of a device count
    const int r16 = lane & 15, kq = lane >> 4;

    const int ktiles = (P.K + BK - 1) / BK, per = (ktiles + P.splits - 1) / P.splits;
    const int kt0 = z * per, kt1 = kt0 + per < ktiles ? kt0 + per : ktiles;
    const int nk = kt1 > kt0 ? kt1 - kt0 : 0;
    // where in its K range the workgroup starts (blocks b, b + 8, ... share an XCD); see the note above
    const int rot = nk > 0 && P.K % MID_CHANNEL_K == 0 ? (b >> 3) * 2 % nk : 0;

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(P.A, P.a_bytes),
                                 rb = make_rsrc(GATE_UP && wave >= 4 ? P.B1 : P.B0, P.b_bytes);
    // piece q of an operand slab = its rows 8 q .. 8 q + 7: lane -> row 8 q + lane / 8, the chunk whose swizzled
    // home is slot lane % 8
    uint32_t goff[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int q = l < NLA ? wave * NLA + l : wave * 2 + (l - NLA);
        const int row = 8 * q + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        int gr = l < NLA ? m0 + row : n0 + (GATE_UP ? row & 63 : row);
        const bool in = l < NLA ? gr < R : gr < P.N && (!GATE_UP || (row & 63) < cols);
        if (NORM && l < NLA && in) gr = P.idx[gr];
        goff[l] = in ? (uint32_t)(((int64_t)gr * P.K + c * 8) * 2) : kOobOffset;
    }
    f32x4 acc[MI][2];
    float ss[MI];
    slab_loop<16 * MT, GATE_UP ? 64 : 16, NORM>(ra, rb, goff, wn * (GATE_UP ? 16 : 32), kt0, nk, rot, P.K, acc, ss);

    __shared__ float sq[NORM ? 8 : 1][MI][64];
    if (NORM) {
#pragma unroll
        for (int m = 0; m < MI; ++m) sq[wave][m][lane] = ss[m];
        __syncthreads();
    }
#pragma unroll
    for (int m = 0; m < MI; ++m) {
        const int row = m0 + (wm * MI + m) * 16 + r16;
        float rstd = 1.0f;
        if (NORM) {
            const int w0 = wm * 4;
            rstd = rstd_of_lanes((sq[w0][m][lane] + sq[w0 + 1][m][lane]) + (sq[w0 + 2][m][lane] + sq[w0 + 3][m][lane]), P.K, P.eps);
        }
        if (row >= R) continue;
        if (GATE_UP) {
            const int n = n0 + wn * 16 + 4 * kq;
            if (n >= P.N || n >= n0 + cols) continue;
            f32x4 g = acc[m][0], u = acc[m][1];
            if (SCALE && P.rstd != nullptr) rstd = P.rstd[row];
            if (NORM || SCALE) {
                g *= rstd;
                u *= rstd;
            }
            if (P.splits > 1) {               // uniform
                float* p = P.partial + ((int64_t)z * P.rows + row) * 2 * P.N + n;
                *reinterpret_cast<f32x4*>(p) = g;
                *reinterpret_cast<f32x4*>(p + P.N) = u;
                continue;
            }
            float h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = g[j] * sigmoid_f(g[j]) * u[j];
            *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(P.H) + (uint32_t)row * P.h_row + (uint32_t)(n >> 3) * P.h_chunk +
                                      (n & 4) * 2) = u32x2{pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
            if (P.G != nullptr) {
                const int64_t o = (int64_t)row * P.N + n;
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

}  // namespace skipffn
