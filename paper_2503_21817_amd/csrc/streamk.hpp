// Balanced split of the K range of a GEMM whose result leaves through fp32 partial slabs.
// Plain C++ (no HIP constructs): shared by the GEMM kernel, the reducing kernels and the host.
//
// When a GEMM has fewer output tiles than the chip has CUs, the K range of its tiles is cut so
// that every workgroup gets the same number of slabs, instead of an integer split factor that
// leaves CUs idle.  All m-tiles of one n-tile form a group served by `nbg` workgroups; a group
// of g tiles with kt slabs each is cut into
//   * `a` aligned chunks of q slabs per tile (workgroups 0 .. a*g-1 of the group: the g tiles of
//     a chunk walk the same K range at the same time, so they share the streamed operand in
//     L2), and
//   * the rest [a*q, kt) of every tile, laid end to end (g * rem slabs) and cut into nr pieces
//     of qr >= rem slabs (workgroups a*g .. a*g+nr-1); a piece runs one segment per tile it
//     touches.
// Tile i of a group receives streamk_count() partial slabs: slots 0..a-1 from the aligned
// chunks, then one or two from the remainder pieces.  The reducing kernels add exactly those.
//
// A group with more tiles than workgroups (g > nbg) first gives every workgroup `full` = g / nbg
// whole tiles (workgroup j: tiles j, j + nbg, ...: one partial slab each, and the nbg tiles of a
// round walk the K range together); the scheme above then applies to the gr = g - full * nbg tiles
// that are left.  (Letting every workgroup walk an equal share of all g tiles end to end balances
// just as well, but puts the workgroups of a group at different K positions: the streamed operand
// is then fetched once per workgroup instead of once per group - measured 13-20 % slower on the
// down and dXn GEMMs at 17 and 33 tile rows.)
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define SKIPFFN_HD __host__ __device__
#else
#define SKIPFFN_HD
#endif

namespace skipffn {

struct StreamKPlan { int g, kt, nbg, q, a, rem, nr, qr, full, base, gr; };
constexpr int kStreamKMaxAligned = 6;            // at most 6 + 2 partial slabs per tile

SKIPFFN_HD inline StreamKPlan streamk_plan(int g, int kt, int nbg) {
    StreamKPlan p;
    p.g = g; p.kt = kt; p.nbg = nbg;
    p.full = g > nbg ? g / nbg : 0;
    p.base = p.full * nbg;
    p.gr = g - p.base;
    g = p.gr;                                                // the split applies to these tiles
    if (g == 0) { p.q = kt > 0 ? kt : 1; p.a = 0; p.rem = 0; p.nr = 0; p.qr = 1; return p; }
    const int q_bal = (g * kt + nbg - 1) / nbg;
    const int q_min = (kt + kStreamKMaxAligned - 1) / kStreamKMaxAligned;
    p.q = q_bal > q_min ? q_bal : q_min;
    if (p.q < 1) p.q = 1;
    p.a = kt / p.q;                                          // a * g <= nbg
    p.rem = kt - p.a * p.q;
    if (p.rem > 0) {
        const int want = (g * p.rem + p.q - 1) / p.q;       // <= g
        const int have = nbg - p.a * g;                      // >= 1 when rem > 0
        p.nr = want < have ? want : have;
        p.qr = (g * p.rem + p.nr - 1) / p.nr;                // rem <= qr <= q
    } else {
        p.nr = 0; p.qr = 1;
    }
    return p;
}

// number of partial slabs tile i (0 <= i < g) of a group receives
SKIPFFN_HD inline int streamk_count(const StreamKPlan& p, int i) {
    if (i < p.base) return 1;
    i -= p.base;
    int c = p.a;
    if (p.rem > 0) c += ((i + 1) * p.rem - 1) / p.qr - (i * p.rem) / p.qr + 1;
    return c;
}

// The work of workgroup j (0 <= j < nbg) of a group, one segment at a time:
//   StreamKIter it = streamk_begin(p, j);  StreamKSeg s;  while (streamk_next(p, it, s)) ...
// A segment is K slabs [kb, ke) of tile i, accumulated into partial slab `slot` of that tile.
struct StreamKSeg { int i, kb, ke, slot; };
struct StreamKIter { int j, u, u_end, f; };
SKIPFFN_HD inline StreamKIter streamk_begin(const StreamKPlan& p, int j) {
    StreamKIter it;
    it.j = j;
    it.f = 0;                            // whole tiles done so far
    if (j < p.a * p.gr) {                // aligned chunk: one pseudo-unit
        it.u = 0; it.u_end = 1;
    } else {
        const int rj = j - p.a * p.gr;
        if (rj >= p.nr) { it.u = 0; it.u_end = 0; return it; }
        it.u = rj * p.qr;
        it.u_end = it.u + p.qr;
        if (it.u_end > p.gr * p.rem) it.u_end = p.gr * p.rem;
    }
    return it;
}
SKIPFFN_HD inline bool streamk_next(const StreamKPlan& p, StreamKIter& it, StreamKSeg& s) {
    if (it.f < p.full) {                 // a whole tile of this workgroup's own
        s.i = it.f * p.nbg + it.j;
        s.kb = 0; s.ke = p.kt; s.slot = 0;
        ++it.f;
        return true;
    }
    if (it.u >= it.u_end) return false;
    if (it.j < p.a * p.gr) {
        const int c = it.j / p.gr;
        s.i = p.base + it.j - c * p.gr;
        s.kb = c * p.q;
        s.ke = s.kb + p.q;
        s.slot = c;
        it.u = it.u_end;
        return true;
    }
    const int rj = it.j - p.a * p.gr;
    const int ir = it.u / p.rem;         // index among the tiles that are split
    s.i = p.base + ir;
    const int k0 = it.u - ir * p.rem;
    int len = p.rem - k0;
    if (len > it.u_end - it.u) len = it.u_end - it.u;
    s.slot = p.a + rj - (ir * p.rem) / p.qr;
    s.kb = p.a * p.q + k0;
    s.ke = s.kb + len;
    it.u += len;
    return true;
}

// Output tiles of a GEMM with `rows` rows, `columns` tile columns (times the parts its K range is cut into) and `slabs` K
// slabs a tile on `cus` workgroups: `full` rows of tiles of 256 rows, then one row of tiles of 32 * mi rows (mi = 4 .. 7)
// over the rest, if any (two_parts); or (full = 0) tiles of 32 * mi rows throughout.  (The kernels plan with the row count on
// the device.)
//
// A round of tiles costs 34 + 6.5 mi us (measured, gate/up at C = 4096, I = 14336, 64 slabs: 60, 67, 74, 79, 86 a round for
// mi = 4 .. 8 on 448 to 2944 rows; a slab's phases and loads do not shrink with the rows).  So tall tiles win unless others
// leave fewer rows empty or save a round, or a last row of lower tiles fits where tall ones end unevenly: 368 rows 93 us on
// 192-row tiles, 102 on 256; 640 rows 139 on 160, 163; 768 rows 148 on 192, 165; 1200 rows 245 on 224, 250; 940, 1472 and 2048
// rows best on 256.  A sixteenth of the work in all decides between equal makespans.  even: heights of 64 rows only
// (transposed copies are zero up to a multiple of 64 rows).
//
// Two parts are the gate/up GEMM's: in the down GEMM they gave nothing (0.93 to 1.05 of the best single height, 1.00 on average,
// at 5000 to 10500 rows, C = 11520 to 15360, I = 256 to 3072).  Between the two the pipeline drains, about 5 us whatever K.  And the low tiles read the weights again, alone: rows of
// tiles that run together share them, but a row of its own is no faster than its 32 KB a slab and tile come from memory (5 TB/s).
// Gate/up with saved buffers, two parts / one height, us:  C = 8192, I = 28672: 420 rows 400 / 351, 580 rows 528 / 489, 700 rows
// 562 / 519;  C = 1024, I = 32768: 640 rows 104 / 97, 1472 rows 218 / 201;  without:  C = 8192, I = 28672: 396 rows 1.18 times as
// long.  Where the low tiles fit into a round that the tall ones leave uneven, two parts stay the better ones:  C = 8192, I = 14336:
// 420 rows 163 / 174;  C = 4096, I = 14336, without: 5149 rows 4 % shorter.
//
// With saved buffers (even) a tile column stores 1 KB a row.  Where K is so short that a round takes no longer than its stores (a
// tall tile's 256 KB about 26 us, its slabs 1.35 us each) and all stores are more than the last-level cache of 256 MB takes in,
// low tiles only shorten the runs in which the transposed copy is written.  C = 520, I = 28672 (9 slabs), 192-row tiles / 256, us:
// 1300 rows 162 / 147, 1700 rows 216 / 174, 2000 rows 279 / 191; below that size 300 rows 41 / 47.  16 slabs (C = 1024) are even.
// cost_of: what all rounds of the best one cost, in units of 0.5 us a tile of 64 slabs.
struct StreamRows { int full, mi; };
SKIPFFN_HD inline int stream_tile_cost(int mi) { return 68 + 13 * mi; }       // 64 slabs, in units of 0.5 us
SKIPFFN_HD inline StreamRows stream_rows_plan(int rows, int columns, int slabs, int cus, bool even, bool two_parts, int* cost_of = nullptr) {
    const int tall = stream_tile_cost(8);
    StreamRows best{(rows + 255) / 256, 0};
    int n = best.full * columns;
    int best_cost = (n + cus - 1) / cus * tall + n / 16 * tall / cus;
    if (cost_of != nullptr) *cost_of = best_cost;
    if (even && slabs <= 12 && (int64_t)rows * columns > 256 * 1024) return best;
    for (int mi = 7; mi >= 4; --mi) {
        if (even && (mi & 1)) continue;
        n = (rows + 32 * mi - 1) / (32 * mi) * columns;
        const int cost = (n + cus - 1) / cus * stream_tile_cost(mi) + n / 16 * stream_tile_cost(mi) / cus;
        if (cost < best_cost) { best = StreamRows{0, mi}; best_cost = cost; }
    }
    const int full = rows / 256, rest = rows - full * 256;
    int mi = (rest + 31) / 32;
    mi = mi < 4 ? 4 : (even ? (mi + 1) / 2 * 2 : mi);
    if (two_parts && full > 0 && rest > 0 && mi < 8) {
        // the tall tiles go round the workgroups, the low ones on from there
        const int low = stream_tile_cost(mi), read = columns * 5 / 6, q = full * columns / cus, r = full * columns - q * cus;
        const int last = r + columns;                        // low tiles end here, counted from the first workgroup of the last round
        int head = q * tall + (r > 0 ? tall : 0), tail = 0;
        if (r == 0 || last > cus) {
            tail = (last - (r > 0 ? cus : 0) + cus - 1) / cus * low;
            tail = tail > read ? tail : read;
            if (full == 1) head = head > read ? head : read;
        }
        const int cost = head + tail + 640 / (slabs > 0 ? slabs : 1) + (full * columns / 16 * tall + columns / 16 * low) / cus;
        if (cost < best_cost) { best = StreamRows{full, mi}; best_cost = cost; }
    }
    if (cost_of != nullptr) *cost_of = best_cost;
    return best;
}

}  // namespace skipffn
