// Brute-force check of the balanced K split (csrc/streamk.hpp): for every (g, kt, nbg) in a
// range, every K slab of every tile is covered exactly once, slot numbers of a tile are
// 0..count-1 without repeats, counts stay within the partial-slab budget, and no workgroup
// gets more than q slabs beyond its whole tiles.  Then the lists of tiles that the kernels run (csrc/tilelists.hpp): the
// balanced lists are the segments of streamk_next, the lists of a plain grid cover every tile and K slab once, and the
// launch order hands out every share once.  Prints "ok <cases>" or the first violation.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
#include "../../paper_2503_21817_amd/csrc/layout.hpp"
#include "../../paper_2503_21817_amd/csrc/tilelists.hpp"
using namespace skipffn;

// the lists of all workgroups of one grid
template <bool SPLIT>
static const char* check_grid(int workgroups, int tiles_m, int tiles_n, int splits, int batch, int ktiles, int after) {
    std::vector<int> cover((size_t)tiles_m * tiles_n * batch * ktiles, 0);
    long total = 0, most = 0;
    for (int b = 0; b < workgroups; ++b) {
        const GridWork<SPLIT> w(b, workgroups, tiles_m, tiles_n, splits, batch, ktiles, after);
        StreamTile t{};
        long n = 0;
        for (; w.get((int)n, t); ++n) {
            if (t.tm < 0 || t.tm >= tiles_m || t.tn < 0 || t.tn >= tiles_n || t.z < 0 || t.z >= splits || (t.second && batch == 1))
                return "tile out of range";
            if (t.kb < 0 || t.kb >= t.ke || t.ke > ktiles) return "K range";
            const size_t tile = ((size_t)(t.second ? 1 : 0) * tiles_m + t.tm) * tiles_n + t.tn;
            for (int k = t.kb; k < t.ke; ++k) cover[tile * ktiles + k]++;
        }
        if (w.get((int)n + 1, t)) return "a list that goes on after its end";
        total += n;
        most = std::max(most, n);
    }
    for (int c : cover) if (c != 1) return "coverage";
    if (total != (long)tiles_m * tiles_n * splits * batch) return "number of tiles";
    if (most > (total + workgroups - 1) / workgroups + 1) return "balance";
    return nullptr;
}

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
                    const BalancedWork list(p, 3, j);
                    StreamTile t{};
                    int work = 0, i = 0;
                    while (streamk_next(p, it, s)) {
                        if (!list.get(i++, t) || t.tm != s.i || t.kb != s.kb || t.ke != s.ke || t.z != s.slot || t.tn != 3 || t.second) {
                            printf("list g=%d kt=%d nbg=%d j=%d segment %d\n", g, kt, nbg, j, i - 1);
                            return 1;
                        }
                        if (s.i < 0 || s.i >= g || s.kb < 0 || s.ke > kt || s.kb >= s.ke) {
                            printf("bad segment g=%d kt=%d nbg=%d j=%d: i=%d [%d,%d)\n", g, kt, nbg, j, s.i, s.kb, s.ke);
                            return 1;
                        }
                        for (int k = s.kb; k < s.ke; ++k) cover[s.i * kt + k]++;
                        slots[s.i].push_back(s.slot);
                        work += s.ke - s.kb;
                    }
                    if (list.get(i, t)) { printf("list too long g=%d kt=%d nbg=%d j=%d\n", g, kt, nbg, j); return 1; }
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
    // every share of a balanced split is taken by one workgroup
    for (int tiles_n : {1, 2, 3, 5, 8, 12, 16, 31})
        for (int nbg : {1, 2, 5, 8, 16, 21, 64})
            for (int g : {1, 3, 6, 17, 70})
                for (int kt : {1, 9, 64, 224}) {
                    const StreamKPlan p = streamk_plan(g, kt, nbg);
                    std::vector<int> seen(tiles_n * nbg, 0);
                    for (int b = 0; b < tiles_n * nbg; ++b) {
                        int tn = -1, j = -1;
                        balanced_share(p, tiles_n, b, tn, j);
                        if (tn < 0 || tn >= tiles_n || j < 0 || j >= nbg || seen[tn * nbg + j]++) {
                            printf("order g=%d kt=%d nbg=%d tiles_n=%d b=%d: tn=%d j=%d\n", g, kt, nbg, tiles_n, b, tn, j);
                            return 1;
                        }
                    }
                    ++cases;
                }
    // divisions of tile counts, at the multiples and one below, up to the largest count
    for (int d = 1; d < 70000; d += d < 300 ? 1 : 997)
        for (int64_t n = d; n <= 0x7fffffff; n = n < 50 * (int64_t)d ? n + d : n / d * 2 * d + d)
            for (const int64_t m : {n - 1, n, std::min<int64_t>(n + d - 1, 0x7fffffff)})
                if (TileDiv(d).div((int)m) != m / d) { printf("%ld / %d = %d\n", (long)m, d, TileDiv(d).div((int)m)); return 1; }
    // plain grids: one or two problems, K whole or cut as the planner cuts it, fewer than 256 workgroups too, and the second
    // part of a launch, which goes on where the first ended
    std::mt19937 rng(1);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    for (int n = 0; n < 4000; ++n) {
        const int workgroups = 8 * pick(1, 32), tiles_m = pick(1, n % 4 ? 12 : 40), tiles_n = pick(1, n % 3 ? 20 : 120), ktiles = pick(1, 70);
        const int after = n % 2 ? pick(0, 3000) : 0;
        const int splits = choose_k_split(tiles_m * tiles_n, ktiles, kMaxSplits, workgroups), batch = splits == 1 ? pick(1, 2) : 1;
        const char* bad = check_grid<true>(workgroups, tiles_m, tiles_n, splits, batch, ktiles, after);
        if (bad == nullptr) bad = check_grid<false>(workgroups, tiles_m, tiles_n, 1, 1, ktiles, after);
        if (bad != nullptr) {
            printf("%s: workgroups=%d tiles %d x %d splits=%d batch=%d ktiles=%d after=%d\n", bad, workgroups, tiles_m, tiles_n, splits, batch,
                   ktiles, after);
            return 1;
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
