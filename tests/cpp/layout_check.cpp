// Host check of the buffer carving and K-split planning (csrc/layout.hpp), meant to be built with
// -fsanitize=address,undefined: every section of `saved` and of the two workspaces is 256-byte
// aligned, the sections are disjoint, in order and large enough for what the kernels put there,
// totals never decrease as the row bound grows, and every K partition the planner picks - for a forward
// call the very plan it launches - stays within the partial-slab budget the workspaces are sized for.  A byte map of each buffer is
// painted section by section, so an overlap or an overrun is also a sanitizer report.
// Prints "ok <cases>" or the first violation.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "../../paper_2503_21817_amd/csrc/layout.hpp"
using namespace skipffn;

static int fail(const char* what, long R, long C, long I, int ncu) {
    printf("%s at R=%ld C=%ld I=%ld ncu=%d\n", what, R, C, I, ncu);
    return 1;
}

// paint [off, off + bytes) of a map scaled down by `unit` bytes per cell; returns false on overlap
static bool paint(std::vector<unsigned char>& map, size_t off, size_t bytes, size_t unit) {
    if (bytes == 0) return true;
    const size_t a = off / unit, b = (off + bytes - 1) / unit;
    for (size_t i = a; i <= b; ++i) {
        if (map.at(i)) return false;
        map[i] = 1;
    }
    return true;
}

// what is wrong with the down GEMM's plans of all counts below a bound of more than 256 rows, or null
static const char* check_row_plans(long bound, long C, long I, int ncu) {
    int64_t sum_rows = 0;
    const RowPlans p = plan_rows(bound, C, I, ncu, &sum_rows);
    const int ktiles = (int)((I + BK - 1) / BK), tiles_m = (int)((bound + BM - 1) / BM), tiles_n = (int)((C + BN - 1) / BN);
    for (int hs = 0; hs < 2; ++hs) {
        const FwdWs W = fwd_ws(bound, C, I, hs != 0, ncu);
        const size_t room = W.status - W.partial, slab = (size_t)bound * C * 4;
        if (p.mid_splits < 1 || (size_t)p.mid_splits * 256 * C * 4 > room) return "the slabs of up to 256 rows do not fit";
        if ((size_t)kMaxSplits * slab > room) return "the slabs of a count do not fit";
    }
    if ((p.mid_splits - 1) * ((ktiles + p.mid_splits - 1) / p.mid_splits) >= ktiles) return "an empty part of up to 256 rows";
    if (sum_rows != 0 && (sum_rows < 256 || sum_rows > bound)) return "rows of the reducing launch";
    bool slabs = false;
    for (int t = 2; t <= tiles_m; ++t) {
        const KPartition k = row_plan(p, t);
        slabs = slabs || k.sk_nbg > 0 || k.splits > 1;
        if (k.sk_nbg > 0 || k.splits > 1)
            if (sum_rows < std::min<long>(bound, (long)t * BM)) return "slabs past the rows of the reducing launch";
        if (t > kRowPlans && t < tiles_m) {
            const KPartition b = row_plan(p, tiles_m);
            if (k.splits != b.splits || k.sk_nbg != b.sk_nbg) return "a count past the table has the bound's plan";
        }
        if (k.sk_nbg > 0) {
            if (k.splits != 1 || k.sk_nbg * tiles_n > ncu) return "balanced split of a count larger than the chip";
            const StreamKPlan sk = streamk_plan(t, ktiles, k.sk_nbg);
            for (int i = 0; i < t; ++i)
                if (streamk_count(sk, i) > kMaxSplits) return "slabs of a balanced split of a count";
        } else if (k.splits < 1 || k.splits > kMaxSplits || (k.splits - 1) * ((ktiles + k.splits - 1) / k.splits) >= ktiles) {
            return "split of a count";
        }
    }
    if (slabs != (sum_rows > 0)) return "a reducing launch without slabs, or slabs without one";
    const KPartition own = choose_k_partition(tiles_m, tiles_n, ktiles, false, ncu), b = row_plan(p, tiles_m);
    return b.splits != own.splits || b.sk_nbg != own.sk_nbg ? "the bound's own plan" : nullptr;
}

// what is wrong with the forward plan, or null
static const char* check_plan(long R, long C, long I, bool hs, bool balanced, int ncu) {
    const ForwardPlan p = plan_forward(R, C, I, hs, balanced, ncu);
    const FwdWs W = fwd_ws(R, C, I, hs, ncu);
    const size_t room = W.status - W.partial, slab = (size_t)R * C * 4;
    const int ktiles = (int)((I + BK - 1) / BK);
    if (balanced && (p.gate_up != FWD_CORE || p.down != FWD_CORE)) return "the balanced split is the core's";
    if (p.gate_up_splits != 1) {
        const int kt = (int)((C + BK - 1) / BK), per = (kt + p.gate_up_splits - 1) / p.gate_up_splits;
        if (p.gate_up != FWD_MID || R > 256 || (p.gate_up_splits - 1) * per >= kt) return "split of the gate/up GEMM";
        if ((size_t)p.gate_up_splits * R * 2 * I * 4 > room) return "the slabs of the gate/up GEMM do not fit";
    }
    // whole 16-byte chunks of H, and no more rounds of the chip than tiles of 64 columns take
    const long row_tiles = (R + 255) / 256, cols = p.gate_up_cols;
    if (cols % 8 || cols < 16 || cols > 64) return "columns of a gate/up tile";
    if (R > 256 && cols != 64) return "narrow gate/up tiles load the rows of several row tiles again";
    if (p.gate_up == FWD_MID && (row_tiles * ((I + cols - 1) / cols) + ncu - 1) / ncu > (row_tiles * ((I + 63) / 64) + ncu - 1) / ncu)
        return "narrow gate/up tiles take another round";
    // where two thirds of the chip are idle, no workgroup walks more than 48 K slabs
    if (p.gate_up == FWD_MID && R <= 256 && 3 * ((I + 63) / 64) * p.gate_up_splits <= ncu &&
        (C + BK - 1) / BK > 48 * p.gate_up_splits)
        return "a long K range on an idle chip";
    if ((p.gate_up == FWD_FEW || p.down == FWD_FEW) && R > kFewRowsMax) return "too many rows for the register path";
    if (p.gate_up == FWD_MID && plan_forward(R, C, I, hs, balanced, ncu, false, true).norm_in_gate_up)
        return "tiles form the norms beside a launch that could";
    if (p.gate_up == FWD_FEW && p.norm_in_gate_up && R > 32 && (I + 15) / 16 > ncu) return "more workgroups form the norms than run at once";
    // a layer of the widths that the register path takes, too small for tiles of their own: no split K range instead
    if (!hs && !balanced && ncu == 256 && R > 16 && C == 2048 && I >= 2048 && I <= 6144 && R <= kFewRowsMax && p.gate_up != FWD_FEW)
        return "tiles for a small layer";
    // its workgroups walk all of K: a chain of loads, twice as long with four row fragments
    if (p.gate_up == FWD_FEW && C > 4096) return "a long K range of the gate/up GEMM on the register path";
    if (p.down == FWD_FEW && I * (R > 32 ? 2 : 1) > (R > 16 || hs ? 8192 : 14336))
        return "a long K range of the down GEMM on the register path";
    if (p.down == FWD_FEW) return nullptr;
    if (p.down == FWD_MID) {
        if (p.k_down.splits < 1 || p.k_down.sk_nbg != 0) return "split of the tiles of all rows";
        if (R > 256 && ((R + 255) / 256) * ((C + 127) / 128) > ncu) return "slabs of more tiles than the chip holds";
        if (p.k_down.splits * slab > room) return "the slabs of the tiles of all rows do not fit";
        const int per = (ktiles + p.k_down.splits - 1) / p.k_down.splits;
        if ((p.k_down.splits - 1) * per >= ktiles) return "an empty split";
        return nullptr;
    }
    const int tiles_m = (int)((R + BM - 1) / BM), tiles_n = (int)((C + BN - 1) / BN);
    if (p.k_down.sk_nbg > 0) {
        const StreamKPlan sk = streamk_plan(tiles_m, ktiles, p.k_down.sk_nbg);
        if (p.k_down.sk_nbg * tiles_n > ncu) return "balanced split larger than the chip";
        for (int i = 0; i < tiles_m; ++i)
            if (streamk_count(sk, i) * slab > room) return "the slabs of the balanced split do not fit";
    } else {
        const int s = p.k_down.splits;
        if (s > 1 && s * slab > room) return "the slabs of the core do not fit";
        if ((s - 1) * ((ktiles + s - 1) / s) >= ktiles) return "a split of the core without slabs";
    }
    return nullptr;
}

int main() {
    long cases = 0;
    const long Cs[] = {8, 256, 264, 4096}, Is[] = {8, 688, 14336};
    const long Rs[] = {0, 1, 7, 8, 31, 128, 129, 184, 256, 257, 1000, 1472, 2560, 2944, 9623, 16384};
    const int ncus[] = {256, 304, 64, 1};
    for (int ncu : ncus)
        for (long C : Cs)
            for (long I : Is) {
                size_t prev_sv = 0, prev_fw[2] = {0, 0}, prev_bw = 0;
                for (long R : Rs) {
                    const size_t unit = 256;
                    // ---- saved
                    const SavedLayout L = saved_layout(R, C, I);
                    const size_t need[8] = {(size_t)R * C * 2, (size_t)R * C * 2, (size_t)R * 4, (size_t)R * I * 2,
                                            (size_t)R * I * 2, (size_t)R * I * 2, (size_t)C * ld_transposed(R) * 2,
                                            (size_t)I * ld_transposed(R) * 2};
                    std::vector<unsigned char> map(L.total / unit + 2, 0);
                    for (int k = 0; k < 8; ++k) {
                        if (L.off[k] % 256) return fail("saved section not aligned", R, C, I, ncu);
                        if (L.off[k] + need[k] > L.total) return fail("saved section past the end", R, C, I, ncu);
                        if (!paint(map, L.off[k], need[k], unit)) return fail("saved sections overlap", R, C, I, ncu);
                    }
                    if (ld_transposed(R) % 64 || ld_transposed(R) < R) return fail("transposed leading dimension", R, C, I, ncu);
                    if (L.total < prev_sv) return fail("saved size decreases", R, C, I, ncu);
                    prev_sv = L.total;
                    // ---- forward workspace, with and without a saved buffer
                    for (int hs = 0; hs < 2; ++hs) {
                        const FwdWs W = fwd_ws(R, C, I, hs != 0, ncu);
                        std::vector<unsigned char> m2(W.total / unit + 2, 0);
                        const size_t slab_rows = std::max<size_t>((size_t)kMaxSplits * R, (size_t)kMaxSplitsNarrow * std::min<long>(R, 256));
                        const size_t offs[5] = {W.xn, W.rstd, W.h, W.partial, W.status};
                        const size_t sz[5] = {hs ? 0 : (size_t)R * C * 2, hs ? 0 : (size_t)R * 4, hs ? 0 : (size_t)R * I * 2,
                                              slab_rows * C * 4, 8};
                        for (int k = 0; k < 5; ++k) {
                            if (offs[k] % 256) return fail("forward workspace section not aligned", R, C, I, ncu);
                            if (offs[k] + sz[k] > W.total) return fail("forward workspace section past the end", R, C, I, ncu);
                            if (!paint(m2, offs[k], sz[k], unit)) return fail("forward workspace sections overlap", R, C, I, ncu);
                        }
                        if (W.total < prev_fw[hs]) return fail("forward workspace size decreases", R, C, I, ncu);
                        prev_fw[hs] = W.total;
                    }
                    // ---- backward workspace
                    {
                        const BwdWs W = bwd_ws(R, C, I);
                        std::vector<unsigned char> m3(W.total / unit + 2, 0);
                        const size_t offs[9] = {W.dy, W.dyT, W.dg, W.du, W.dgT, W.duT, W.partial, W.gainp, W.status};
                        const size_t sz[9] = {(size_t)R * C * 2, (size_t)C * ld_transposed(R) * 2, (size_t)R * I * 2, (size_t)R * I * 2,
                                              (size_t)I * ld_transposed(R) * 2, (size_t)I * ld_transposed(R) * 2,
                                              (size_t)kMaxSplits * R * C * 4, gain_partial_bytes(R, C), 8};
                        for (int k = 0; k < 9; ++k) {
                            if (offs[k] % 256) return fail("backward workspace section not aligned", R, C, I, ncu);
                            if (offs[k] + sz[k] > W.total) return fail("backward workspace section past the end", R, C, I, ncu);
                            if (!paint(m3, offs[k], sz[k], unit)) return fail("backward workspace sections overlap", R, C, I, ncu);
                        }
                        if (W.total < prev_bw) return fail("backward workspace size decreases", R, C, I, ncu);
                        prev_bw = W.total;
                    }
                    // ---- K partitions of the down GEMM (K = I) and of the dXn GEMM (K = 2 I)
                    if (R > 0) {
                        const int tiles_n = (int)((C + BN - 1) / BN);
                        for (int pairs = 1; pairs <= 2; ++pairs)
                            for (int forced = 0; forced < 2; ++forced) {
                                const int tiles_m = (int)((R + BM - 1) / BM), ktiles = pairs * (int)((I + BK - 1) / BK);
                                const KPartition kp = choose_k_partition(tiles_m, tiles_n, ktiles, forced != 0, ncu);
                                if (kp.splits < 1 || kp.splits > kMaxSplits) return fail("split factor out of range", R, C, I, ncu);
                                if ((kp.splits - 1) * ((ktiles + kp.splits - 1) / kp.splits) >= ktiles) return fail("a split without slabs", R, C, I, ncu);
                                if (kp.sk_nbg > 0) {
                                    if (kp.sk_nbg * tiles_n > ncu) return fail("balanced split larger than the chip", R, C, I, ncu);
                                    const StreamKPlan p = streamk_plan(tiles_m, ktiles, kp.sk_nbg);
                                    for (int i = 0; i < tiles_m; ++i)
                                        if (streamk_count(p, i) > kMaxSplits) return fail("more partial slabs than the workspace holds", R, C, I, ncu);
                                }
                            }
                    }
                    ++cases;
                }
            }
    // the plan that a forward call launches: widths in both orders
    const long widths[] = {8, 64, 256, 264, 512, 688, 1024, 2048, 2112, 4096, 7168, 8192, 14336, 32768};
    for (int ncu : ncus)
        for (long C : widths)
            for (long I : widths)
                for (long R = 1; R <= 16384; R += R < 300 ? 1 : R / 16)
                    for (int variant = 0; variant < 4; ++variant) {
                        if (const char* what = check_plan(R, C, I, variant & 1, variant & 2, ncu)) return fail(what, R, C, I, ncu);
                        ++cases;
                    }
    // the plans of a count on the device
    for (int ncu : ncus)
        for (long C : widths)
            for (long I : widths)
                for (long bound : {257L, 300L, 512L, 616L, 1232L, 2944L, 4928L, 9856L, 16384L, 16385L, 20000L}) {
                    if (const char* what = check_row_plans(bound, C, I, ncu)) return fail(what, bound, C, I, ncu);
                    ++cases;
                }
    // tiles of the token merge: no other one is as few rounds of the chip with fewer rows
    for (int ncu : ncus)
        for (long dropped : {1L, 64L, 65L, 128L, 129L, 800L, 1728L, 4095L})
            for (long kept : {1L, 64L, 65L, 129L, 256L, 1000L, 4095L})
                for (long sets : {1L, 3L, 8L, 64L}) {
                    auto rounds = [&](int q) {
                        const long a = kMergeTiles[q][0], b = kMergeTiles[q][1];
                        return ((dropped + a - 1) / a * ((kept + b - 1) / b) * sets + ncu - 1) / ncu;
                    };
                    const int best = merge_target_tile(dropped, kept, sets, ncu);
                    if (best < 0 || best > 2) return fail("tile of the merge", dropped, kept, sets, ncu);
                    for (int q = best + 1; q < 3; ++q)
                        if (rounds(q) <= rounds(best)) return fail("a taller tile of the merge in as many rounds", dropped, kept, sets, ncu);
                    ++cases;
                }
    // dXn beside dW_gate and dW_up: all workgroups on the chip at once (a workgroup a tile where gradients are added to), every part of K with
    // slabs, no more of them than the workspace holds
    for (int ncu : ncus)
        for (long C : widths)
            for (long I : widths)
                for (long R = 1; R <= 16384; R += R < 300 ? 1 : R / 16)
                    for (int variant = 0; variant < 8; ++variant) {
                        const bool forced = variant & 1, on_device = variant & 2, added = variant & 4;
                        const DxnPlan p = plan_dxn(R, C, I, forced, on_device, added, ncu);
                        const long tiles = (R + BM - 1) / BM * ((C + BN - 1) / BN), dw = (I + BM - 1) / BM * ((C + BN - 1) / BN) * 2;
                        const int ktiles = 2 * (int)((I + BK - 1) / BK), s = p.k.splits;
                        if (s < 1 || s > kMaxSplits || (s - 1) * ((ktiles + s - 1) / s) >= ktiles) return fail("split of dXn", R, C, I, ncu);
                        const BwdWs W = bwd_ws(R, C, I);
                        const int d = dh_splits(R, C, I, forced, ncu), kc = (int)((C + BK - 1) / BK);
                        if (d < 1 || d > kDhSplits || (d - 1) * ((kc + d - 1) / d) >= kc) return fail("split of dH", R, C, I, ncu);
                        if (d > 1 && (forced || (size_t)d * R * I * 4 > W.gainp - W.partial)) return fail("the slabs of dH do not fit", R, C, I, ncu);
                        if (p.dw_workgroups > 0) {
                            if (forced || p.k.sk_nbg != 0) return fail("the balanced split shares no launch", R, C, I, ncu);
                            if (p.n0 % 8 || p.n0 < tiles * s || p.dw_workgroups % 8 || (!added && p.n0 + p.dw_workgroups > ncu))
                                return fail("workgroups of dXn and dW", R, C, I, ncu);
                            if (added && p.dw_workgroups < dw) return fail("lists of gradients that are added to", R, C, I, ncu);
                            const DxnPlan q = plan_dxn(R, C, I, forced, on_device, false, ncu);
                            if (q.k.splits != p.k.splits || q.n0 != p.n0) return fail("the sums of dXn by the type of dW", R, C, I, ncu);
                            const int slabs = std::min<int>(BM, R) / BK + 3, n = (int)((C + BN - 1) / BN);
                            const KPartition two = choose_k_partition((int)((R + BM - 1) / BM), n, ktiles, false, ncu);
                            if (on_device && (ktiles + s - 1) / s > k_partition_cost(two, 1, n, ktiles, ncu) + 1.15 * ((dw + ncu - 1) / ncu * slabs + 8))
                                return fail("a chain of dXn as the bound's rows have it, for few rows", R, C, I, ncu);
                            if (on_device && p.dw_workgroups < dw) return fail("lists of dW by the bound of the rows", R, C, I, ncu);
                        }
                        ++cases;
                    }
    printf("ok %ld\n", cases);
    return 0;
}
