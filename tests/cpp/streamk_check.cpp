// Brute-force check of the balanced K split (csrc/streamk.hpp): for every (g, kt, nbg) in a
// range, every K slab of every tile is covered exactly once, slot numbers of a tile are
// 0..count-1 without repeats, counts stay within the partial-slab budget, and no workgroup
// gets more than q slabs beyond its whole tiles.  Prints "ok <cases>" or the first violation.
#include <cstdio>
#include <vector>
#include "../../paper_2503_21817_amd/csrc/streamk.hpp"
using namespace skipffn;

int main() {
    long cases = 0;
    for (int g = 1; g <= 40; ++g)
        for (int nbg = 1; nbg <= 40; ++nbg)
            for (int kt = 1; kt <= 300; kt += (kt < 70 ? 1 : 7)) {
                const StreamKPlan p = streamk_plan(g, kt, nbg);
                if (p.base + p.gr != g || p.gr < 0 || (g > nbg && p.gr >= nbg) || (g <= nbg && p.full != 0) ||
                    p.a * p.gr > nbg || p.a > kStreamKMaxAligned || (p.rem > 0 && (p.nr < 1 || p.a * p.gr + p.nr > nbg)) ||
                    (p.rem > 0 && p.qr < p.rem)) {
                    printf("bad plan g=%d kt=%d nbg=%d: q=%d a=%d rem=%d nr=%d qr=%d\n", g, kt, nbg, p.q, p.a, p.rem, p.nr, p.qr);
                    return 1;
                }
                std::vector<int> cover(g * kt, 0);
                std::vector<std::vector<int>> slots(g);
                for (int j = 0; j < nbg; ++j) {
                    StreamKIter it = streamk_begin(p, j);
                    StreamKSeg s;
                    int work = 0;
                    while (streamk_next(p, it, s)) {
                        if (s.i < 0 || s.i >= g || s.kb < 0 || s.ke > kt || s.kb >= s.ke) {
                            printf("bad segment g=%d kt=%d nbg=%d j=%d: i=%d [%d,%d)\n", g, kt, nbg, j, s.i, s.kb, s.ke);
                            return 1;
                        }
                        for (int k = s.kb; k < s.ke; ++k) cover[s.i * kt + k]++;
                        slots[s.i].push_back(s.slot);
                        work += s.ke - s.kb;
                    }
                    if (work > p.full * kt + (p.gr > 0 ? p.q : 0)) { printf("overload g=%d kt=%d nbg=%d j=%d: %d > q=%d\n", g, kt, nbg, j, work, p.q); return 1; }
                }
                for (int x = 0; x < g * kt; ++x)
                    if (cover[x] != 1) { printf("coverage g=%d kt=%d nbg=%d tile %d slab %d: %d\n", g, kt, nbg, x / kt, x % kt, cover[x]); return 1; }
                for (int i = 0; i < g; ++i) {
                    const int c = streamk_count(p, i);
                    if (c > kStreamKMaxAligned + 2 || (int)slots[i].size() != c) { printf("count g=%d kt=%d nbg=%d tile %d: count %d, segments %zu\n", g, kt, nbg, i, c, slots[i].size()); return 1; }
                    std::vector<int> seen(c, 0);
                    for (int sl : slots[i]) {
                        if (sl < 0 || sl >= c || seen[sl]) { printf("slot g=%d kt=%d nbg=%d tile %d: slot %d of %d\n", g, kt, nbg, i, sl, c); return 1; }
                        seen[sl] = 1;
                    }
                }
                ++cases;
            }
    // tile rows of the row plan: all rows covered, no tile row without rows, the heights that exist
    for (int even = 0; even < 2; ++even)
        for (int tiles_n : {1, 6, 17, 56, 65, 112, 300})
            for (int rows = 1; rows <= 3000; rows += rows < 700 ? 1 : 13) {
                const int slabs = 1 + rows % 3 * 63;
                const StreamRows p = stream_rows_plan(rows, tiles_n, slabs, 256, even != 0, rows % 2 != 0);
                const int base = p.full * 256, step = 32 * p.mi;
                const bool low = p.mi >= 4 && p.mi <= 7 && (!even || p.mi % 2 == 0);
                if ((p.mi == 0 && (base < rows || base - rows >= 256)) || (p.mi != 0 && (!low || base >= rows)) ||
                    (p.full > 0 && p.mi != 0 && (rows - base > step || rows % 2 == 0))) {
                    printf("rows=%d tiles_n=%d even=%d: full=%d mi=%d\n", rows, tiles_n, even, p.full, p.mi);
                    return 1;
                }
                ++cases;
            }
    // A row of low tiles that starts when the tall ones are done reads the weights again, and the pipeline drains in between:
    // one height was measured the faster one here (gate/up of C = 8192, I = 28672; of C = 1024, I = 32768) ...
    const struct { int rows, tiles_n, slabs; bool even, two; } measured[] = {
        {396, 224, 128, true, false}, {420, 224, 128, true, false}, {580, 224, 128, true, false}, {700, 224, 128, true, false},
        {396, 224, 128, false, false}, {405, 224, 128, false, false}, {2465, 224, 128, false, false},
        {700, 256, 16, true, false}, {900, 256, 16, true, false}, {1472, 256, 16, true, false}, {2465, 224, 9, false, false},
        // ... and two parts here (C = 8192 or 4096, I = 14336)
        {2944, 112, 128, true, true}, {2465, 112, 64, false, true}, {5149, 112, 64, false, true}};
    for (const auto& m : measured) {
        const StreamRows p = stream_rows_plan(m.rows, m.tiles_n, m.slabs, 256, m.even, true);
        if ((p.full > 0 && p.mi != 0) != m.two) {
            printf("rows=%d tiles_n=%d slabs=%d even=%d: full=%d mi=%d\n", m.rows, m.tiles_n, m.slabs, m.even, p.full, p.mi);
            return 1;
        }
        ++cases;
    }
    // a short K and more to store than the last-level cache takes in: 256-row tiles (measured, C = 520, I = 28672)
    for (int rows : {1300, 1625, 1700, 2000, 2121}) {
        const StreamRows p = stream_rows_plan(rows, 224, 9, 256, true, true);
        if (p.mi != 0) { printf("rows=%d short K: full=%d mi=%d\n", rows, p.full, p.mi); return 1; }
        ++cases;
    }
    printf("ok %ld\n", cases);
    return 0;
}
