// Host-side planning of the Skip-FFN block: how the `saved` buffer and the workspaces are carved
// into sections, and how the K range of a GEMM is cut over the compute units.  Plain C++ (no HIP
// constructs), shared by the library's entry points and by a host test that is built with the
// address and undefined-behaviour sanitizers.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "streamk.hpp"

namespace skipffn {

constexpr int BM = 256, BN = 256, BK = 64;          // output tile and K slab of the GEMM core
constexpr int GAIN_STRIP = 4;                        // rows per workgroup of the gain-gradient pass

inline size_t align_up(size_t v, size_t a = 256) { return (v + a - 1) / a * a; }
// bytes of the gain-gradient scratch (one fp32 row of C per strip of rows)
inline size_t gain_partial_bytes(int64_t R, int64_t C) {
    return (size_t)((R + GAIN_STRIP - 1) / GAIN_STRIP) * (size_t)C * 4;
}

constexpr int kMaxSplits = 8;
constexpr int kMaxSplitsNarrow = 16;     // up to 256 rows: small fp32 slabs, and every CU has to stream weights

// How the K range of a GEMM with tiles_m x tiles_n output tiles and `ktiles` K slabs is cut
// on `ncu` CUs (one workgroup per CU).  Costs are in units of one K slab of one tile: every
// round of `ncu` workgroups costs its slab count plus a fixed prologue/epilogue, partial tiles
// cost a write now and a read in the reducing kernel.
// A split of fewer than 4 slabs would be all prologue (at least 8 before: the dXn GEMM of the 32-row, C = 256 layer, 22
// slabs on 2 workgroups, ended its training step at 65.1 us, on 5 at 61.3).
//   splits == 1, sk_nbg == 0 : K whole; the epilogue of the down GEMM adds the residual, dXn leaves as one fp32 slab
//   splits  > 1, sk_nbg == 0 : plain split-K into `splits` fp32 slabs
//   sk_nbg  > 0              : balanced split (down: stream_gemm_balanced_kernel, dXn: gemm_bf16_streamk_kernel), sk_nbg
//                              workgroups per n-tile group (with more m-tiles than workgroups in a group, every
//                              workgroup first runs whole tiles of its own; the rest is split)
// Both GEMMs are planned in 256-row tiles.  The down GEMM then lowers them where K is not balanced (stream_rows_plan).
struct KPartition { int splits; int sk_nbg; };
// `slab`: the cost of writing a tile's slab and reading it back
inline double k_partition_cost(KPartition k, int tiles_m, int tiles_n, int ktiles, int ncu, double slab = 0.04) {
    const int tiles = tiles_m * tiles_n, s = k.splits;
    if (k.sk_nbg == 0) {
        const int per = (ktiles + s - 1) / s, rounds = (tiles * s + ncu - 1) / ncu;
        return rounds * (per + 8.0 + (s > 1 ? 8.0 : 0.0)) + (s > 1 ? slab * s * tiles : 0.0);
    }
    const StreamKPlan p = streamk_plan(tiles_m, ktiles, k.sk_nbg);
    double slabs = 0.0;
    for (int i = 0; i < tiles_m; ++i) slabs += streamk_count(p, i);
    // an aligned chunk is one segment; a remainder piece runs one segment (with its own
    // prologue and epilogue: about 5 slabs' worth, measured) per tile it touches; with more
    // tiles than workgroups in a group, whole tiles come first
    const double aligned = p.a > 0 ? p.q + 16.0 : 0.0;
    const double pieces = p.nr > 0 ? p.qr + 16.0 + 5.0 * (p.qr / p.rem) : 0.0;
    return p.full * (ktiles + 16.0) + std::max(aligned, pieces) + slab * slabs * tiles_n;
}
inline KPartition choose_k_partition(int tiles_m, int tiles_n, int ktiles, bool force_balanced, int ncu, double* cost_of = nullptr) {
    KPartition best{1, 0};
    double best_cost = 1e30;
    auto consider = [&](KPartition k) {
        const double cost = k_partition_cost(k, tiles_m, tiles_n, ktiles, ncu);
        if (cost < best_cost - 1e-9) { best_cost = cost; best = k; }
    };
    for (int s = 1; s <= kMaxSplits; ++s) {
        if (s > 1 && (ktiles + s - 1) / s < 4) break;
        consider(KPartition{s, 0});
    }
    const int nbg = tiles_n > 0 ? ncu / tiles_n : 0;
    if (nbg >= 1 && tiles_m * tiles_n > 0) {
        if (force_balanced) return KPartition{1, nbg};
        const StreamKPlan p = streamk_plan(tiles_m, ktiles, nbg);
        if (p.gr > 0 && p.q >= 8) consider(KPartition{1, nbg});
    }
    if (cost_of != nullptr) *cost_of = best_cost;
    return best;
}

// dXn and dW_gate, dW_up both wait for dG and dU only.  Up to some hundred rows they share a launch: dXn, cut into fewer and
// longer parts, on the first n0 workgroups (a multiple of 8), lists of dW's tiles on dw_workgroups others, all on the chip at
// once (added gradients apart, see below).  The ends of dXn's parts and the stores of dW then fall into each other's K slabs, and dXn leaves fewer fp32 slabs.
// dw_workgroups = 0: two launches, each with the chip to itself, which many rows of a wide layer fill as well.  Costs in slabs of
// dXn; a slab of dW, alone or not, takes 1.15 of one, and the end of a tile 2.5, as bf16 stores do: the type of dW and whether it is
// added to choose no plan, so that they change no bit of the gradients.  Backward of a layer, us, two launches / one (parts of dXn), bf16 dW:  C = 4096, I = 14336: 32 rows 226 / 197
// (8), 184 rows 277 / 248 (7), 256 rows 304 / 274 (6), 368 rows 326 / 314 (4), 600 rows 443 / 451 (3);  C = 3072, I = 10752:
// 184 rows 210 / 184 (8), 368 rows 225 / 210 (5), 640 rows 272 / 278 (4);  C = 2048, I = 7168: 184 rows 123 / 102 (8), 640 rows
// 167 / 150 (6), 1024 rows 209 / 196 (4), 1472 rows 295 / 277 (3);  C = 1024, I = 3584: 64 rows 69 / 59 (8), 368 rows 90 / 75
// (8), 2944 rows 198 / 165 (3).  With less than 8 % to gain by these costs it measured from 6 % faster to 5 %
// slower, and is left.
// Gradients that are added to are read at the end of a tile before they are written, and dXn's workgroups are through long before
// lists on the rest of the chip.  There every tile of dW is a workgroup, so that the CUs of dXn take their part (the same sums).  Two launches /
// lists / a workgroup a tile, added to fp32 gradients:  C = 5120, I = 17920, 1 row 762 / 931 / 725;  C = 4096, I = 14336: 100 rows
// 496 / 551 / 477, 256 rows 552 / 548 / 511;  C = 8192, I = 8192, 184 rows 613 / 618 / 615;  C = 2048, I = 7168, 600 rows 232 / 234 /
// 210, to bf16 ones 191 / 179 / 172.  Overwritten gradients are faster in lists, whose stores overlap:  C = 4096, I = 14336, 184 rows,
// bf16 272 / 235 / 254, fp32 350 / 315 / 328.
// A count on the device, far below its bound as a rule, leaves most of dXn's workgroups without work and the others a chain as long as
// the bound's plan made it; so one launch has to gain at every row of tiles below the bound.  Two launches / one by the bound alone / now:
// C = 1024: I = 1024, bound 2112, 264 rows 84 / 90 / 76, I = 3584, bound 7248, 906 rows 152 / 180 / two launches again;  C = 512,
// I = 1024, bound 4160, 520 rows 80 / 83 / 68;  C = 256, I = 896, bound 2720, 340 rows 62 / 71 / 57.
constexpr double kDwTileEnd = 2.5;
struct DxnPlan { KPartition k; int n0, dw_workgroups; };
inline DxnPlan plan_dxn(int64_t rows, int64_t C, int64_t I, bool balanced, bool count_on_device, bool accumulate, int ncu) {
    const int tiles_m = (int)((rows + BM - 1) / BM), tiles_n = (int)((C + BN - 1) / BN);
    const int tiles = tiles_m * tiles_n, ktiles = 2 * (int)((I + BK - 1) / BK);
    double cost = 0.0;
    DxnPlan p{choose_k_partition(tiles_m, tiles_n, ktiles, balanced, ncu, &cost), 0, 0};
    if (balanced || tiles <= 0) return p;
    const int dw_tiles = (int)((I + BM - 1) / BM) * tiles_n * 2, dw_slabs = (int)((rows + BK - 1) / BK);
    const int whole = (dw_tiles + 7) / 8 * 8;                // a workgroup for every tile
    auto dw_cost = [&](int workgroups, int slabs) {
        return 1.15 * ((dw_tiles + workgroups - 1) / workgroups * (slabs + kDwTileEnd) + 8.0);
    };
    // whether any count below the bound, by these costs, gains less than that over two launches
    const KPartition two = p.k;
    auto longer_below = [&](int s, int n1) {
        for (int t = 1; t < tiles_m; ++t) {
            const int slabs = t * (BM / BK);
            const double one = std::max((ktiles + s - 1) / s + (s > 1 ? 16.0 : 8.0) + 0.04 * s * t * tiles_n, dw_cost(n1, slabs));
            if (one > 0.92 * (k_partition_cost(two, t, tiles_n, ktiles, ncu) + dw_cost(std::min(whole, ncu), slabs))) return true;
        }
        return false;
    };
    double best = 0.92 * (cost + dw_cost(std::min(whole, ncu), dw_slabs));
    for (int s = 1; s <= kMaxSplits; ++s) {
        const int per = (ktiles + s - 1) / s, n0 = (tiles * s + 7) / 8 * 8;
        if ((s > 1 && per < 4) || n0 > ncu - 8) break;
        if ((s - 1) * per >= ktiles) continue;
        const int n1 = std::min((ncu - n0) / 8 * 8, whole);
        if (count_on_device && n1 < whole) continue;         // the rows there are may leave dXn's workgroups without work
        const double c = std::max(per + (s > 1 ? 16.0 : 8.0) + 0.04 * s * tiles, dw_cost(n1, dw_slabs));
        if (count_on_device && longer_below(s, n1)) continue;
        if (c < best - 1e-9) { best = c; p = DxnPlan{KPartition{s, 0}, n0, accumulate ? whole : n1}; }
    }
    return p;
}

// Parts of K of the dH GEMM (K = C), which shares its grid with dW_down: with few rows its tiles are few and each is a chain of C / 64
// slabs and a long epilogue, behind which the rest of the chip idles once dW_down is done.  Cut, they leave fp32 slabs, and the
// SwiGLU backward and its transposed copies are a kernel of their own.  Costs in slabs as above: the longest tile of either, or all of
// them on the chip, and the bytes of that kernel at 4.5 TB/s.  Backward of a layer, us, whole / parts (how many):  C = 1024,
// I = 3584: 32 rows 56 / 47 (2), 184 rows 70 / 57 (2), 368 rows 75 / 62 (2), 768 rows 80 / 72 (2);  C = 2048, I = 7168: 184 rows
// 102 / 83 (2), 368 rows 124 / 106 (2);  C = 4096, I = 2048: 184 rows 118 / 66 (4);  C = 4096, I = 8192: 184 rows 194 / 146 (3),
// 368 rows 236 / 204 (2);  C = 3072, I = 10752: 184 rows 188 / 156 (2);  C = 4096, I = 14336: 64 rows 203 / 180 (2), 184 rows
// 254 / 233 (2), 256 rows 282 / 263 (2);  C = 8192, I = 8192: 184 rows 355 / 263 (3).  Past the line: C = 4096, I = 14336, 368
// rows 317 / 331 (2);  C = 2048, I = 1024, 3000 rows, where dW_down's tiles are as long, 131 / 136 (2).
constexpr int kDhSplits = 4;
inline int dh_splits(int64_t rows, int64_t C, int64_t I, bool balanced, int ncu) {
    if (balanced || rows <= 0) return 1;
    const int tiles_i = (int)((I + BN - 1) / BN), tiles = (int)((rows + BM - 1) / BM) * tiles_i, ktiles = (int)((C + BK - 1) / BK);
    const double dw_tile = 1.15 * ((rows + BK - 1) / BK + kDwTileEnd), dw = (double)((C + BM - 1) / BM) * tiles_i * dw_tile;
    auto cost = [&](int s) {
        const double tile = (ktiles + s - 1) / s + (s > 1 ? 14.0 : 24.0);
        return std::max({tile, dw_tile + 8.0, (tiles * s * tile + dw) / ncu + 8.0}) + (s > 1 ? 4.0 + (double)rows * I * (4 * s + 12) / 5.4e6 : 0.0);
    };
    int splits = 1;
    double best = 0.92 * cost(1);
    for (int s = 2; s <= kDhSplits; ++s) {
        const int per = (ktiles + s - 1) / s;
        if (per < 4 || s * I > kMaxSplits * C) break;        // its slabs lie where dXn's will (bwd_ws)
        if ((s - 1) * per >= ktiles) continue;
        const double c = cost(s);
        if (c < best - 1e-9) { best = c; splits = s; }
    }
    return splits;
}

// Up to 256 rows the forward GEMMs are bound by streaming the 6 * C * I bytes of weights.  They run on tiles of ALL
// rows and 128 weight rows (midrows.hip), the down GEMM with its K range split into fp32 slabs.  Layer forward, us,
// against 128-row tiles that shared the weights through L2:  C = 4096: 64 rows 77 / 104, 184 rows 102 / 117,
// 256 rows 117 / 128;  C = 3072: 128 rows 70 / 76;  C = 2048: 128 rows 49 / 56;  C = 1024: 128 rows 30 / 38.
// Beyond 256 rows a second row of tiles reads the weights again, from L2, and pays where it finds idle CUs: a narrow
// layer whose gate/up tiles all fit on the chip at once (the general core gives such a layer a few dozen 256-row
// tiles).  C = 2048: 300 rows 55 / 79, 512 rows 67 / 86;  C = 1024: 300 rows 34 / 51, 1024 rows 47 / 58;  C = 256: 1024 rows
// 30 / 41;  C = 3072, I = 8192: 512 rows 105 / 112.  One tile more than the chip holds (1500 rows, C = 1024) is even, and
// so are, at C = 8192 and I = 512, 6144 rows on 192 tiles; 7168 rows take 323 / 313 (the larger tiles read less).
inline int mid_row_tiles(int64_t rows) { return (int)((rows + 255) / 256); }
inline bool mid_rows(int64_t rows, int64_t C, int64_t I, int ncu) {
    return rows <= 256 || (mid_row_tiles(rows) * ((I + 63) / 64) <= ncu && (rows <= 6144 || C <= 4096));
}
// The down GEMM of such a layer follows with its own tiles.  Where I is below C these are many and their K range is short:
// once they are more than the chip holds, writing fp32 slabs (of the one split that is left) and reading them back
// costs more than the general core with its fused epilogue.  Layer forward, us, core / slabs:  I = 512, C = 4096: 2300
// rows 76 / 89, 4096 rows 86 / 122;  C = 8192: 2048 rows 135 / 155;  I = 64, C = 4096: 4096 rows 74 / 91.  With tiles
// that fit:  C = 2048, I = 512: 2048 rows 54 / 50;  C = 4096, I = 2048: 2048 rows 119 / 114.
inline bool mid_rows_down(int64_t rows, int64_t C, int ncu) {
    return rows <= 256 || mid_row_tiles(rows) * ((C + 127) / 128) <= ncu;
}
// plain split-K into at most max_splits slabs: fill the CUs, keep at least 4 K slabs per workgroup (see
// choose_k_partition).  max_splits bounds the search itself: 33 K slabs cut for 9 splits and then held to 8 would
// leave the eighth without any, where the search up to 8 takes 7 splits of 5.
inline int choose_k_split(int tiles, int ktiles, int max_splits, int ncu) {
    int best = 1;
    double best_cost = 1e30;
    for (int s = 1; s <= max_splits; ++s) {
        const int per = (ktiles + s - 1) / s;
        if (s > 1 && per < 4) break;
        const int rounds = (tiles * s + ncu - 1) / ncu;
        const double cost = rounds * (per + 8.0 + (s > 1 ? 8.0 : 0.0)) + (s > 1 ? 0.02 * s * tiles : 0.0);
        if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
    return best;
}

// A handful of rows: the weights go straight to registers (fewrows.hip), complete sums and a fused epilogue in one launch.
// Every 16 columns read all activations again, a time that grows with rows * C * I, and a wavefront walks its share
// of K in a chain of loads whose length K sets, one, two or four row fragments (16, 32, 64 rows) wide; the tiles above
// cut K instead.  Row-major activations (a saved buffer) cost more to read, the more the more rows.  Each of the two GEMMs
// chooses for itself; measured as registers minus tiles, us of a layer forward, saved buffer in brackets:
//   gate/up (K = C)   C = 256, I = 688: -2 at any rows;  C = 1024, I = 3584: -4 at 16 rows, -2.7 (-1.7) at 64;  C = 2048,
//     I = 7168: -3 (-1.3) at 16, -3 (0) at 32, -1.3 (6) at 64;  C = 4096, I = 4096: -3.5 at 16, 0.5 (2.7) at 32, 5 (10) at
//     64;  C = 8192, I = 512: 11 at 16;  C = 4096, I = 14336 (above 24 Mi weights): 5 to 49
//   down (K = I)      C = 256, I = 688: -6.5;  C = 2048, I = 2048: -4.8 (-3.9) at 16, -3.7 (-0.8) at 64;  C = 1024, I = 3584:
//     -2.9 (-1.9) at 16, 0.7 (6) at 64;  C = 512, I = 8192: 0.4 (4) at 16, 5 (12) at 32, 11 (27) at 64;  I = 32768: 21 to
//     133.  With a column block for every CU (C = 4096) the tiles are slower too: I = 14336: -3.3 at 1 row, -0.2 at 16.
// Without a saved buffer and a gain the tiles normalise their rows themselves (norm_in_gate_up), and they are no wider than
// the chip needs (gate_up_cols):  C = 2048, I = 7168, registers / tiles: 17 rows 34.6 / 33.9, 32 rows 35.9 / 34.5, with a
// gain 36.2 / 36.6, 33 rows with a gain 40.1 / 37.1;  C = 3072, I = 7168: 17 rows 45.4 / 42.1, with a gain 46.2 / 43.0;
// C = 1024, I = 3584: 32 rows 15.2 / 19.3, 64 rows 20.4 / 22.6.  Below 12 Mi weights the tiles of C = 2048 have nothing to gain (a split K
// range, which needs a launch that adds its parts, or 16 columns).  Kernels of a layer, weights from memory, us:  I = 4096: 20 rows
// 25.5 / 28.1, 32 rows 26.7 / 29.5;  I = 3072: 32 rows 25.4 / 30.2, 64 rows 32.5 / 33.1;  I = 2048: 32 rows 22.6 / 25.6, 64 rows
// 28.1 / 29.4;  I = 6144: 32 rows 34.0 / 33.6;  I = 1024: 40 rows 25.6 / 25.1;  I = 512: 40 rows 24.6 / 20.9;  C = 3072,
// I = 3072: 20 rows 29.2 / 30.7;  I = 4608: 20 rows 38.2 / 34.0.
constexpr int64_t kFewRowsMax = 64;
inline bool few_rows_gate_up(int64_t rows, int64_t C, int64_t I, bool has_saved, bool has_gain) {
    const int64_t weight = C * I, limit = (int64_t)40 * 2048 * 7168;
    if (rows > kFewRowsMax || weight > (int64_t)24 << 20 || rows * weight > (has_saved ? limit / 2 : limit)) return false;
    if (rows <= 16) return C <= 4096;
    if (weight <= (int64_t)12 << 20) {
        if (C <= 2048 && (rows <= 32 || (!has_saved && I >= 2048))) return true;
        if (C <= 3072 && I >= C && rows <= 32 && !has_saved) return true;
    }
    return C <= (rows <= 32 && (has_saved || has_gain) ? 2048 : 1536);
}
inline bool few_rows_down(int64_t rows, int64_t C, int64_t I, bool has_saved, int ncu) {
    if (rows > kFewRowsMax || rows * C * I > (int64_t)1 << (has_saved ? 29 : 30)) return false;
    // time of a step of the chain, in units of the one-fragment step: 8192 k of those take what the tiles' split costs
    const double step = has_saved ? (rows <= 8 ? 1.0 : 0.8 + 0.05 * rows) : rows <= 16 ? 1.0 : rows <= 32 ? 1.6 : 2.0;
    if (I * step <= 8192.0) return true;
    return !has_saved && rows <= 16 && I * ncu <= 14336 * std::min<int64_t>((C + 15) / 16, ncu);
}

// The gate/up GEMM has I / 64 workgroups a row tile, each walking the whole K range: a layer of small I leaves most of
// the chip idle for C / 64 slabs.  Where three fifths or more of it would be idle, up to 256 rows split K as well; the SwiGLU
// then waits for a reducing kernel, which costs about 16 slabs' time and the traffic of the fp32 sums.  Layer forward, us,
// split / whole:  C = 8192, I = 512: 16 rows 29 / 61, 128 rows 40 / 88;  C = 4096, I = 2048: 64 rows 36 / 49, 128 rows
// 45 / 59;  C = 4096, I = 4096: 256 rows 61 / 82;  C = 16384, I = 512: 64 rows 41 / 124;  C = 8192, I = 6400: 128 rows
// 99 / 115.  Past the line:  C = 8192, I = 8192 (half the chip idle): 128 rows 133 / 128;  C = 1024, I = 2048 (16
// slabs): 256 rows 42 / 35.
inline int gate_up_splits(int64_t C, int64_t I, int ncu) {
    const int tiles = (int)((I + 63) / 64), ktiles = (int)((C + BK - 1) / BK);
    if (tiles * 5 > 2 * ncu) return 1;
    int best = 1;
    double best_cost = ktiles + 8.0;
    for (int s = 2; s <= kMaxSplitsNarrow && s * tiles <= ncu; ++s) {
        const int per = (ktiles + s - 1) / s;
        if (per < 4) break;
        const double cost = per + 8.0 + 8.0 + 0.08 * s * tiles;
        if (cost < best_cost - 1e-9) { best_cost = cost; best = s; }
    }
    return best;
}

// The columns of gate (and of up) that a tile takes where K is whole: 64, or fewer where these need no more rounds of the chip.
// A slab of such a tile is fewer bytes of weights, and CUs that would be idle take part; 64 columns of I = 14336 are 224 tiles, 56
// are 256.  Layer forward, us, 64 columns / these:  C = 4096, I = 14336 (56): 8 rows 68.2 / 66.9, 184 rows 106.5 / 105.6;
// C = 3072, I = 10752 (48): 64 rows 57.0 / 53.6, 184 rows 81.8 / 79.8;  C = 2048, I = 7168 (32): 64 rows 39.7 / 36.2, 184
// rows 56.1 / 54.2;  C = 1024, I = 3584 (16): 250 rows 38.0 / 36.7.  One more round than needed: 184 rows, C = 4096, 48
// columns 141.5.
// Only where the tiles are of all rows: in several row tiles every column tile loads its 256 rows again, and those bytes, not the
// weights, bound it.  Gate/up kernel, us, 64 columns / as few as fit the chip:  C = 4096: I = 512, 1500 rows 42 / 48, 4200 rows 48 /
// 54, I = 2048, 400 rows 43 / 49;  C = 8192: I = 1024, 2944 rows 92 / 107, I = 4096, 400 rows 83 / 93;  C = 2048, I = 2048, 512 rows
// 25.0 / 27.5;  no shape was faster with fewer.
inline int gate_up_cols(int64_t rows, int64_t I, int ncu) {
    if (rows > 256) return 64;
    const int64_t room = ((I + 63) / 64 + ncu - 1) / ncu * ncu;
    int cols = 16;
    while (cols < 64 && (I + cols - 1) / cols > room) cols += 8;
    return cols;
}

// Without a saved buffer nothing but the gate/up GEMM reads the normalised rows, and 1 / rms can be applied to its sums: the
// squares of a row are added beside the product, the gain is multiplied into the rows.  It saves a launch, and the rounding of
// the normalised rows: error of a layer against 64 bits 2.3e-3 instead of 3.5e-3.  On registers (row-major rows then) it
// pays where these are few or narrow, on tiles for 64 rows without a gain, whose product every wavefront would have to form for all
// rows.  Layer forward, us, in the GEMM / before it:  registers  C = 256, I = 688: 11.4 / 14.3;  C = 1024, I = 3584: 8 rows 14.9 /
// 17.7, 64 rows 24.4 / 27.2 (with a gain 26.4 / 27.3);  C = 2048, I = 7168: 8 rows 28.0 / 29.8, 16 rows 31.3 / 32.2, 32 rows 36.0
// / 34.6;  C = 4096, I = 4096: 16 rows 26.2 / 29.7;  tiles  C = 4096, I = 14336: 8 rows 67.4 / 70.5, 64 rows 74.0 / 76.3 (with
// a gain 92.1 / 71.2 and 98.8 / 76.7);  C = 3072, I = 10752: 8 rows 45.6 / 48.9, 64 rows 57.1 / 59.4.
// From 33 rows only while all workgroups of 16 columns run at once, each of which forms the squares and the gain's products of all
// rows:  C = 1024, I = 7168, before it / in the GEMM: 64 rows 30.3 / 31.2, with a gain 30.5 / 36.1, 40 rows with a gain 30.3 / 33.7.
// Where skipped rows are copied, the kernel before the GEMM is launched for them anyway and normalises beside it; the tiles then gain nothing
// by doing it themselves, and lose where they are narrow.  8 of 64 rows, before it / in the GEMM:  C = 4096: I = 14336 68.6 / 68.8, I = 8192
// 44.0 / 47.3;  C = 5120, I = 8192 60.9 / 64.0;  C = 8192: I = 14336 134.5 / 135.5, I = 8192 81.0 / 86.7 (a launch of its own for the norm: 83);
// 64 of 616: C = 4096, I = 14336 77.6 / 76.2.
// Where the launch before the GEMM forms the norms of so few rows and there is no gain, it leaves the rows as they are, beside 1 / rms
// (scale_in_gate_up): the sums are multiplied by it, so the rounding of the normalised rows is saved there too.  Error against 64 bits, rounded
// rows / this:  C = 2048, I = 4096, 20 rows 3.5e-3 / 2.3e-3;  C = 8192, I = 8192, 8 of 64 rows 3.4e-3 / 2.4e-3;  time up to 0.3 us more.
constexpr int64_t kNormInMidRows = 64;
inline bool norm_in_gate_up(int64_t rows, int64_t C, int64_t I, bool has_gain, bool copies_skipped, bool registers, int ncu) {
    if (!registers) return rows <= kNormInMidRows && !has_gain && !copies_skipped;
    return rows <= 16 || (C <= 1024 && (rows <= 32 || (I + 15) / 16 <= ncu));
}

// Which kernels a forward call launches.
enum FwdKernel { FWD_FEW, FWD_MID, FWD_CORE };           // fewrows.hip, midrows.hip, stream.hpp
struct ForwardPlan {
    FwdKernel gate_up, down;
    bool norm_in_gate_up;                                // the rows are normalised by the gate/up GEMM, not before it
    bool scale_in_gate_up;                               // their 1 / rms is formed before it and applied to its sums
    int gate_up_splits, gate_up_cols;                    // FWD_MID
    KPartition k_down;                                   // FWD_MID: plain split; FWD_CORE: as choose_k_partition; FWD_FEW: none
};
// most fp32 slabs the down GEMM of `rows` rows may write (fwd_ws has room for them)
inline int max_down_splits(int64_t rows) { return rows <= 256 ? kMaxSplitsNarrow : kMaxSplits; }
inline ForwardPlan plan_forward(int64_t rows, int64_t C, int64_t I, bool has_saved, bool balanced, int ncu,
                                bool has_gain = false, bool copies_skipped = false) {
    ForwardPlan p{FWD_CORE, FWD_CORE, false, false, 1, 64, KPartition{1, 0}};
    if (!balanced && mid_rows(rows, C, I, ncu)) {
        p.gate_up = few_rows_gate_up(rows, C, I, has_saved, has_gain) ? FWD_FEW : FWD_MID;
        if (p.gate_up == FWD_MID && rows <= 256) p.gate_up_splits = gate_up_splits(C, I, ncu);
        if (p.gate_up_splits == 1) p.gate_up_cols = gate_up_cols(rows, I, ncu);
        p.norm_in_gate_up = !has_saved && p.gate_up_splits == 1 && norm_in_gate_up(rows, C, I, has_gain, copies_skipped, p.gate_up == FWD_FEW, ncu);
        p.scale_in_gate_up = !has_saved && !has_gain && rows <= kNormInMidRows && p.gate_up_splits == 1 && !p.norm_in_gate_up;
        p.down = few_rows_down(rows, C, I, has_saved, ncu) ? FWD_FEW : mid_rows_down(rows, C, ncu) ? FWD_MID : FWD_CORE;
    }
    const int ktiles = (int)((I + BK - 1) / BK);
    if (p.down == FWD_MID)
        p.k_down.splits = choose_k_split(mid_row_tiles(rows) * (int)((C + 127) / 128), ktiles, max_down_splits(rows), ncu);
    if (p.down == FWD_CORE)
        p.k_down = choose_k_partition((int)((rows + BM - 1) / BM), (int)((C + BN - 1) / BN), ktiles, balanced, ncu);
    return p;
}

// A row count on the device, below a bound for which the core runs the down GEMM: the plan of every row of tiles, so that the kernels
// take that of the rows there are.  Up to 256 rows `mid_splits` parts on tiles of all rows (zstride: 256 rows).
// A count takes its own plan only where that is cheaper than the bound's with slabs at 0.12 for the rows that its tiles have at least:
// the 0.04 that choose_k_partition prices them at is what they cost with the chip's cache to themselves, and a count's plan of many parts
// lost to the bound's of few.  Layer forward, us, plan of the bound / of the count at 0.04 / of the two:  C = 1024, I = 3584: bound
// 4200, 2100 rows 73.6 / 79.7 / 73;  bound 4928, 2464 rows 85 / 91 / 84;  C = 512, I = 2048: bound 4928, 2464 rows 45.3 / 49.5 / 45;
// C = 4096, I = 4096: bound 9856, 4928 rows, with a saved buffer 473 / 490 / 472;  C = 4096, I = 14336: bound 2944, 736 rows 260 / 240 / 240.
// Where the tiles fill half the chip, plans that do not balance K are priced with their lowered tiles, 3 % of doubt apart (fewer tiles
// do not shorten a call by being lower: counted there too, a bound's whole K lost up to 25 %).  Layer forward, us, plan of the bound / of the count
// without / with it:  C = 3072: I = 12288, bound 4239, 3261 rows 554 / 587 / 560, I = 10752, bound 4048, 3114 rows 496 / 524 / 497;  C = 8192,
// I = 4096, bound 2963, 898 rows now 201, without 209.
// sum_rows: the most rows whose plan leaves slabs, 256 at least (their tiles always do).  A reducing launch for the bound cost
// up to 9 us of workgroups without work:  C = 8192, I = 1024: bound 9856, 4928 rows, with a saved buffer 360 / 370 / 358.  0 where no
// plan of more than 256 rows leaves slabs: the core adds to the rows itself and nothing follows it, as without these plans.  A reducing
// launch that has nothing to do took 4.6 us, more than the tiles of all rows save up to 256:  C = 4096, I = 512, bound 4200, of the
// count with it / without any: 1000 rows 68.5 / 63.4, 3800 rows 91.6 / 84.6, 200 rows 62.7 / 59.6, 60 rows 57.0 / 56.0;  C = 512,
// I = 512, bound 12000, 2442 rows 40.1 / 35.7, 200 rows 30.3 / 30.5.
constexpr int kRowPlans = 64;                            // 16384 rows; the bound's plan beyond
constexpr uint16_t kRowPlanBalanced = 0x8000;
// Two plans a word, which the kernels read by a scalar load; half a word would be a vector load, and a wait for all loads before it.
struct RowPlans { int mid_splits; uint32_t beyond, down[kRowPlans / 2]; };
SKIPFFN_HD inline KPartition row_plan(const RowPlans& p, int tiles_m) {
    const uint32_t word = tiles_m <= kRowPlans ? p.down[(tiles_m - 1) >> 1] >> ((tiles_m - 1) & 1) * 16 : p.beyond;
    const int v = (int)(word & 0xffffu);
    return v & kRowPlanBalanced ? KPartition{1, v & ~kRowPlanBalanced} : KPartition{v, 0};
}
inline RowPlans plan_rows(int64_t bound, int64_t C, int64_t I, int ncu, int64_t* sum_rows = nullptr) {
    RowPlans p{};
    const int ktiles = (int)((I + BK - 1) / BK), tiles_m = (int)((bound + BM - 1) / BM), tiles_n = (int)((C + BN - 1) / BN);
    p.mid_splits = choose_k_split((int)((C + 127) / 128), ktiles, kMaxSplitsNarrow, ncu);
    const KPartition of_bound = choose_k_partition(tiles_m, tiles_n, ktiles, false, ncu);
    int last = 1;                                        // row of tiles with slabs
    auto half_full = [&](int t) { return 2 * t * tiles_n >= ncu; };
    auto cost_at = [&](KPartition k, int t) {
        const double c = k_partition_cost(k, t, tiles_n, ktiles, ncu, 0.12 * (t - 1) / t);
        const int n = t * tiles_n * k.splits, tall = (n + ncu - 1) / ncu * stream_tile_cost(8) + n / 16 * stream_tile_cost(8) / ncu;
        int low = tall;
        if (k.sk_nbg == 0 && half_full(t))
            stream_rows_plan(t * BM - BM / 2, tiles_n * k.splits, (ktiles + k.splits - 1) / k.splits, ncu, false, false, &low);
        return c * low / tall;
    };
    auto code = [&](int t) {
        KPartition k = choose_k_partition(t, tiles_n, ktiles, false, ncu);
        const bool same = k.splits == of_bound.splits && k.sk_nbg == of_bound.sk_nbg;
        if (!same && cost_at(of_bound, t) <= (half_full(t) ? 0.97 : 1.0) * cost_at(k, t)) k = of_bound;
        if (k.sk_nbg > 0 || k.splits > 1) last = t;
        return (uint16_t)(k.sk_nbg > 0 ? kRowPlanBalanced | k.sk_nbg : k.splits);
    };
    for (int t = 1; t <= kRowPlans; ++t)                 // (t = 1: tiles of all rows)
        p.down[(t - 1) >> 1] |= (uint32_t)(t > 1 && t <= tiles_m ? code(t) : 1) << ((t - 1) & 1) * 16;
    p.beyond = tiles_m > kRowPlans ? code(tiles_m) : 1;
    if (sum_rows != nullptr) *sum_rows = last > 1 ? std::min<int64_t>(bound, (int64_t)last * BM) : 0;
    return p;
}

// The tile of the token merge's products, dropped rows x kept rows, an index into kMergeTiles: rounds of the chip's CUs times the time of a
// slab, which the rows of its operands set (in units of 3.5 cycles a row).  Whole merges of 240 drawn sizes (1 to 64 sets of 60 to 3000
// tokens, 256 to 4096 columns) are within 1.3 % of the best of the three, 0.02 % in the mean; always 128 x 128: 8.8 % in the mean,
// 64 x 128: 6.6, 64 x 64: 8.0.
constexpr int kMergeTiles[3][2] = {{128, 128}, {64, 128}, {64, 64}};
inline int merge_target_tile(int64_t dropped, int64_t kept, int64_t sets, int ncu) {
    int best = 0;
    int64_t best_cost = 0;
    for (int q = 0; q < 3; ++q) {
        const int a = kMergeTiles[q][0], b = kMergeTiles[q][1];
        const int64_t tiles = (dropped + a - 1) / a * ((kept + b - 1) / b) * sets, cost = (tiles + ncu - 1) / ncu * (60 + a + b);
        if (q == 0 || cost < best_cost) { best = q; best_cost = cost; }
    }
    return best;
}

// Leading dimension of the transposed copies ([columns][rows]): rows rounded up to 64 elements, so that every
// row of a copy starts on a 128-byte line (with a multiple of 8 only, each 128-byte piece the GEMMs load
// straddles two lines: the weight-gradient GEMMs ran 11-23 % slower at such row counts).
inline int64_t ld_transposed(int64_t R) { return (R + 63) / 64 * 64; }

struct SavedLayout { size_t off[8]; size_t total; };
inline SavedLayout saved_layout(int64_t R, int64_t C, int64_t I) {
    SavedLayout L;
    size_t o = 0;
    L.off[0] = o; o += align_up((size_t)R * C * 2);
    L.off[1] = o; o += align_up((size_t)R * C * 2);
    L.off[2] = o; o += align_up((size_t)R * 4);
    L.off[3] = o; o += align_up((size_t)R * I * 2);
    L.off[4] = o; o += align_up((size_t)R * I * 2);
    L.off[5] = o; o += align_up((size_t)R * I * 2);
    L.off[6] = o; o += align_up((size_t)C * ld_transposed(R) * 2);
    L.off[7] = o; o += align_up((size_t)I * ld_transposed(R) * 2);
    L.total = o;
    return L;
}

struct FwdWs { size_t xn, rstd, h, partial, status, total; };
inline FwdWs fwd_ws(int64_t R, int64_t C, int64_t I, bool has_saved, int ncu) {
    FwdWs w; size_t o = 0;
    w.xn = o;   if (!has_saved) o += align_up((size_t)R * C * 2);
    w.rstd = o; if (!has_saved) o += align_up((size_t)R * 4);
    w.h = o;    if (!has_saved) o += align_up((size_t)R * I * 2);
    // a buffer sized for R_max rows must do for every smaller count: up to 256 rows may use more slabs
    const size_t slab_rows = std::max<size_t>((size_t)kMaxSplits * R, (size_t)kMaxSplitsNarrow * std::min<int64_t>(R, 256));
    const size_t gate_up_slabs = (size_t)gate_up_splits(C, I, ncu) * std::min<int64_t>(R, 256) * 2 * I;
    w.partial = o; o += align_up(std::max<size_t>(slab_rows * C, gate_up_slabs) * 4);       // one GEMM after the other
    w.status = o; o += 256;              // verdict of SKIPFFN_FLAG_VALIDATE_IDX
    w.total = o;
    return w;
}

struct BwdWs { size_t dy, dyT, dg, du, dgT, duT, partial, gainp, status, total; };
inline BwdWs bwd_ws(int64_t R, int64_t C, int64_t I) {
    BwdWs w; size_t o = 0;
    w.dy = o; o += align_up((size_t)R * C * 2);
    w.dyT = o; o += align_up((size_t)C * ld_transposed(R) * 2);
    w.dg = o; o += align_up((size_t)R * I * 2);
    w.du = o; o += align_up((size_t)R * I * 2);
    w.dgT = o; o += align_up((size_t)I * ld_transposed(R) * 2);
    w.duT = o; o += align_up((size_t)I * ld_transposed(R) * 2);
    w.partial = o; o += align_up((size_t)kMaxSplits * R * C * 4);          // dXn's slabs, before it dH's
    w.gainp = o; o += align_up(gain_partial_bytes(R, C));
    w.status = o; o += 256;              // verdict of SKIPFFN_FLAG_VALIDATE_IDX
    w.total = o;
    return w;
}

}  // namespace skipffn
