// How the tiles of the persistent prefill kernels are numbered, shared out among the XCDs, cut along the reduction and cut
// narrower.  Plain C++ (compiles on the host as well, where tests look at what every tile and piece gets).
#pragma once
#include <cstddef>
#include "bm_device_shape.h"
#include "bm_tile_dealer.h"

namespace bm {

// Logical tile id -> (row tile, column tile).  The 32 workgroups that run together on one XCD (its
// 32 compute units take consecutive ids) form a block of GM row tiles x 32/GM column tiles, so they
// share GM activation tiles and 32/GM weight panels in that XCD's L2 instead of 32 + 1.
constexpr int G_GM = 4;
BM_HOST_DEVICE void tile_of(int lid, int n_mt, int n_nt, int &mt, int &nt) {
    const int per_group = G_GM * n_nt;
    const int group = lid / per_group, in_group = lid - group * per_group;
    const int first = group * G_GM;
    const int gsize = n_mt - first < G_GM ? n_mt - first : G_GM;
    nt = in_group / gsize;
    mt = first + (in_group - nt * gsize);
}

// One XCD's share of a launch that runs both tile heights.  Its workgroups (XCD_WGS of them) take its 256-row tiles round by
// round, then its 128-row tiles (SmallTileDealer).  SPLIT: the 256-row tiles that do not fill a round (R of them) and the
// 128-row tiles are cut along the reduction into S pieces each, so that the last round is short; the pieces
// leave fp32 partial tiles in scratch memory and split_fixup_kernel adds them up.  All tiles are cut at the same places and
// first pieces go out before second ones, because workgroups that run together share panels in the XCD's L2 only
// while they are at the same k: pieces of equal cost laid end to end (every workgroup at a k of its own)
// fetch 64 KB a k-step from outside the XCD, 2.4 us at the 28 GB/s that a unit gets there.
constexpr int XCD_WGS = K64_CUS / K64_XCDS;            // workgroups of a launch that an XCD gets
constexpr int SPLIT_COST = 160, SPLIT_COST_PART = 40;   // of partial tiles and their sums, in twentieths of a 256-row k-step
constexpr int SPLIT_MAX = 8;                           // most pieces of a tile
constexpr int SPLIT_TILE_FLOATS = 256 * 256;           // a partial 256-row tile; a 128-row tile takes half
constexpr int SPLIT_XCD_TILES = XCD_WGS;               // partial 256-row tiles that an XCD has scratch for
// most cut tiles of an XCD, 2 to 8 pieces each: in a launch of both heights, of 256-row tiles alone
constexpr int FIXUP_TILES = SPLIT_XCD_TILES, FIXUP_TILES_256 = SPLIT_XCD_TILES / 2;
struct XcdWork {
    int big0, small0;    // first 256-row and 128-row tile of this XCD
    int nb, ns;          // number of either
    int full;            // 256-row tiles that are not cut
    int S;               // pieces of the others and of the 128-row tiles
    int KT;              // k-steps of the reduction
    BM_HOST_DEVICE void init(int total_big, int total_small, int KT_, int xcd, bool split) {
        big0 = total_big * xcd / K64_XCDS; nb = total_big * (xcd + 1) / K64_XCDS - big0;
        small0 = total_small * xcd / K64_XCDS; ns = total_small * (xcd + 1) / K64_XCDS - small0;
        full = nb;
        S = 1;
        KT = KT_;
        if (split) cut(choose());
    }
    BM_HOST_DEVICE void cut(int pieces) {
        S = pieces;
        full = S > 1 ? nb / XCD_WGS * XCD_WGS : nb;
    }
    BM_HOST_DEVICE int choose() const {
        const int R = nb % XCD_WGS;
        int S = 1;
        int best = 1 << 30;
        // (unrolled, and with a constant number of workgroups, so that it divides by constants: it runs before a launch's first load)
        BM_UNROLL for (int s = 1; s <= SPLIT_MAX && KT / s >= 16 && R * s + (ns * s + 1) / 2 <= SPLIT_XCD_TILES; ++s) {
            // load of the lighter and the heavier workgroups once the pieces are dealt out; a k-step of 256 rows counts 20, of 128 rows 13
            const int n = R * s, h = n % XCD_WGS, l = XCD_WGS - h;
            int light = n / XCD_WGS * 20, heavy = light + (h ? 20 : 0);
            for (int left = ns * s; left > 0;) {
                if (h == 0 || light <= heavy) { light += 13; left -= l; }
                else { heavy += 13; left -= h; }
            }
            const int t = (light > heavy ? light : heavy) * (KT / s) + (s > 1 ? SPLIT_COST + SPLIT_COST_PART * s : 0);
            if (t < best) { best = t; S = s; }
        }
        return S;
    }
    // first pieces of all tiles go out before second ones: the piece that item idx (from full on) of the 256-row tiles is, and
    // that item of the 128-row tiles is
    BM_HOST_DEVICE int big_piece(int idx) const { return (idx - full) / (nb - full); }
    BM_HOST_DEVICE int small_piece(int item) const { return item / ns; }
    // the k-steps of piece c of a cut tile, and back: the piece that starts at k-step kbeg
    BM_HOST_DEVICE void piece(int c, int &kbeg, int &kend) const { kbeg = c * KT / S; kend = (c + 1) * KT / S; }
    BM_HOST_DEVICE int piece_at(int kbeg) const { return (kbeg * S + KT - 1) / KT; }
    // where piece c of the cut tile t of an XCD lies in the XCD's scratch, 256-row tiles first (floats)
    BM_HOST_DEVICE size_t partial_offset(int t, int c) const {
        const int R = nb - full;
        return t < R ? (size_t)(t * S + c) * SPLIT_TILE_FLOATS : (size_t)(2 * R * S + (t - R) * S + c) * (SPLIT_TILE_FLOATS / 2);
    }
};

// Column tiles of the 128-row tiles.  A launch of fewer tiles than units - few live groups, narrow matrices - cuts 256-row
// tiles into halves and every tile into as many column tiles, 16 (DUAL) or 32 columns up, as give each unit one: a k-step
// takes as long as its loads, and tiles of at most half the width have a loop of their own whose k-step is 32 KB instead of 48
// and four deep (the shortest reductions, which are over before it gets going, keep the wide one).  Kernel times, us, tiles of
// full width | narrower | with the narrow loop: 495 tokens, 5 experts of d = 1792, F = 256 38 + 12 | 25 + 9 | 17 + 9; 900 tokens,
// 12 experts of d = 1024, F = 512 28 + 17 | 20 + 12 | 14 + 9; 300 tokens, 3 experts of d = 3072, F = 1024 59 + 25 | 42 + 18 | 28 +
// 13; DeepSeek-shaped 17 / 32 / 128 tokens, down projection 30 30 34 | 24 25 28 | 19 25 28.  Twice as many tiles as units were
// no better cut (Qwen3-shaped, 512 tokens: 378 tiles 80 us, 504 narrower ones 88).
struct SmallPlan {
    int halved;          // 256-row tiles cut into halves: all or none of them
    int cols;            // column tiles
    bool narrow;         // they are at most half as wide as a tile can be
    BM_HOST_DEVICE SmallPlan(int n_big, int n_small, int n_nt, int n_blk, int KT, int units, bool may) {
        const int tiles = 2 * n_big + n_small;
        halved = 0; cols = n_nt; narrow = false;
        if (may && tiles > 0 && tiles * n_nt <= units) {
            halved = n_big;
            cols = units / tiles < n_blk ? units / tiles : n_blk;
            narrow = n_blk <= 4 * cols && KT >= 6;
        }
    }
};

}  // namespace bm
