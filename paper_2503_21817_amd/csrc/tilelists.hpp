// Lists of output tiles that a workgroup of the stream of tiles (stream.hpp) runs, and the order in which the workgroups of a
// balanced split take their shares.  Plain C++ but for the qualifiers: the kernels and a host test walk the same code.
#pragma once

#include "streamk.hpp"

#if defined(__HIPCC__)
#define SKIPFFN_LIST __device__ __forceinline__
#else
#define SKIPFFN_LIST inline
#endif

namespace skipffn {

constexpr int PANEL_M = 8;                          // tile-order panel width (L2 locality)

// A value that is the same in all lanes, in a scalar register.  Divisions and loads of the row count leave their
// results in vector registers, and a descriptor that comes from there turns every load into a loop over the lanes (dW at
// 1472 rows 250 -> 320 us).
#if defined(__HIPCC__)
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint32_t mul_hi(uint32_t a, uint32_t b) { return __umulhi(a, b); }
#else
inline int uniform(int v) { return v; }
inline uint32_t uniform(uint32_t v) { return v; }
inline uint32_t mul_hi(uint32_t a, uint32_t b) { return (uint32_t)((uint64_t)a * b >> 32); }
#endif

struct StreamTile { int tm, tn, z, kb, ke; bool second; };

// n / d of tile counts by a multiplication: the tile lists are read in the middle of the pipeline, where a division by a
// variable costs as much as a memory phase.  m >= 2^32 / d, so the product is at most one too large.
struct TileDiv {
    uint32_t d, m;
    SKIPFFN_LIST explicit TileDiv(int v) : d((uint32_t)v), m(uniform(0xFFFFFFFFu / (uint32_t)(v > 1 ? v : 2) + 1)) {}
    SKIPFFN_LIST int div(int n) const {
        if (d == 1) return n;
        const uint32_t q = mul_hi((uint32_t)n, m);
        return (int)(q * d > (uint32_t)n ? q - 1 : q);
    }
};

// Tiles of a plain grid, dealt to `workgroups` workgroups in the XCD-aware order of tile_of_block: get(i) is the i-th tile
// of workgroup `block` (a multiple of 8 workgroups).  SPLIT: the K range is cut into `splits`, or the grid holds two problems
// (batch), one after the other.  Every part of the K range has slabs: (splits - 1) * ceil(ktiles / splits) < ktiles.  To the
// pipeline a tile without slabs would be the end of the list.
template <bool SPLIT>
struct GridWork {
    int tiles_m, ktiles;
    int first, count, step;                   // tile i of this workgroup: number first + i * step of the order, i * step < count
    TileDiv panel_tiles, last_panel, split_tiles;
    int splits, per_k;
    // after: tiles that these workgroups have been dealt before, in the same order
    SKIPFFN_LIST GridWork(int block, int workgroups, int tiles_m_, int tiles_n, int splits_, int batch, int ktiles_, int after = 0)
        : tiles_m(tiles_m_), ktiles(ktiles_), panel_tiles(PANEL_M * tiles_n),
          last_panel(tiles_m_ % PANEL_M != 0 ? tiles_m_ % PANEL_M : PANEL_M), split_tiles(SPLIT ? tiles_m_ * tiles_n : 1),
          splits(SPLIT ? splits_ : 1), per_k(SPLIT ? (ktiles_ + splits_ - 1) / splits_ : ktiles_) {
        const int nb = tiles_m * tiles_n * (SPLIT ? splits * batch : 1), xcd = block & 7, q = nb >> 3, rem = nb & 7;
        per_k = uniform(per_k);
        step = workgroups >> 3;
        const int before = (after >> 3) + (xcd < (after & 7) ? 1 : 0);               // of this XCD
        int slot = (block >> 3) - before % step;
        slot = uniform(slot < 0 ? slot + step : slot);
        first = xcd * q + (xcd < rem ? xcd : rem) + slot;
        count = q + (xcd < rem ? 1 : 0) - slot;
    }
    SKIPFFN_LIST bool get(const int i, StreamTile& t) const {
        if (i * step >= count) return false;
        int L = first + i * step, z = 0;
        if (SPLIT) {
            z = split_tiles.div(L);
            L -= z * (int)split_tiles.d;
        }
        const int p = panel_tiles.div(L), in_panel = L - p * (int)panel_tiles.d;
        if ((p + 1) * PANEL_M <= tiles_m) {
            t.tn = in_panel / PANEL_M;
            t.tm = p * PANEL_M + in_panel % PANEL_M;
        } else {
            t.tn = last_panel.div(in_panel);
            t.tm = p * PANEL_M + (in_panel - t.tn * (int)last_panel.d);
        }
        t.second = SPLIT && z >= splits;
        t.z = t.second ? z - splits : z;
        t.kb = t.z * per_k;
        t.ke = SPLIT && t.kb + per_k >= ktiles ? ktiles : t.kb + per_k;
        return true;
    }
};

// The share of a workgroup in the balanced split of streamk.hpp (the segments streamk_next yields, by index): workgroup j of
// the group of tile column tn.
struct BalancedWork {
    int tn, j, nbg, full, base, kt, ke_whole;
    int aligned, tile0, kb0, ke0, slot0;      // an aligned chunk: one segment after the whole tiles
    int rem, u0, u_end, ir0, a, rj; TileDiv qr;           // or pieces [u0, u_end) of the remainders laid end to end
    SKIPFFN_LIST BalancedWork(const StreamKPlan& p, int tn_, int j_)
        : tn(tn_), j(j_), nbg(p.nbg), full(p.full), base(p.base), kt(p.kt), ke_whole(p.kt), aligned(j_ < p.a * p.gr ? 1 : 0),
          tile0(0), kb0(0), ke0(0), slot0(0), rem(p.rem), u0(0), u_end(0), ir0(0), a(p.a), rj(j_ - p.a * p.gr), qr(p.qr) {
        if (aligned) {
            slot0 = j / p.gr;
            tile0 = base + j - slot0 * p.gr;
            kb0 = slot0 * p.q;
            ke0 = kb0 + p.q;
        } else if (rj < p.nr) {
            u0 = rj * p.qr;
            u_end = u0 + p.qr < p.gr * rem ? u0 + p.qr : p.gr * rem;
            ir0 = u0 / rem;
        }
        tn = uniform(tn); j = uniform(j); full = uniform(full); base = uniform(base); aligned = uniform(aligned);
        tile0 = uniform(tile0); kb0 = uniform(kb0); ke0 = uniform(ke0); slot0 = uniform(slot0);
        rem = uniform(rem); u0 = uniform(u0); u_end = uniform(u_end); ir0 = uniform(ir0); a = uniform(a); rj = uniform(rj);
        qr.d = uniform(qr.d);
    }
    SKIPFFN_LIST bool get(const int i, StreamTile& t) const {
        t.tn = tn;
        t.second = false;
        if (i < full) {
            t.tm = i * nbg + j; t.z = 0; t.kb = 0; t.ke = ke_whole;
            return true;
        }
        const int k = i - full;
        if (aligned) {
            t.tm = tile0; t.z = slot0; t.kb = kb0; t.ke = ke0;
            return k == 0;
        }
        const int ir = ir0 + k, first = ir * rem, u = first > u0 ? first : u0;
        if (u >= u_end) return false;
        t.tm = base + ir;
        t.z = a + rj - qr.div(first);
        t.kb = kt - rem + u - first;
        t.ke = kt - rem + (first + rem < u_end ? rem : u_end - first);
        return true;
    }
};

// The share of workgroup b in the launch order of a balanced split: workgroup j of the group of tile column tn.
// Workgroups are dealt round-robin to the 8 XCDs, and each XCD gets a contiguous range of this order: aligned chunks first,
// chunk-major, then tile column, then tile row - so an XCD works on ONE K range of many tile columns (the tile rows of a
// column share the weight slabs, the columns share the activation slabs, and no XCD streams the whole K extent of the
// activations); the remainder pieces follow.
SKIPFFN_HD inline void balanced_share(const StreamKPlan& p, int tiles_n, int b, int& tn, int& j) {
    const int nb = tiles_n * p.nbg;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int gr = p.gr, aligned_total = p.a * gr * tiles_n;
    if (b < aligned_total) {
        const int c = b / (tiles_n * gr), r = b - c * (tiles_n * gr);
        tn = r / gr;
        j = c * gr + (r - tn * gr);
    } else {
        const int per = p.nbg - p.a * gr;         // workgroups per group left for the remainder
        const int r = b - aligned_total;
        tn = r / per;
        j = p.a * gr + (r - tn * per);
    }
}

}  // namespace skipffn
