// The 4-wave tile and reduction splits of a pass (gemm_mfma_dispatch.h), on the
// host: sizes only, no device code.
#pragma once

#include "dyad_internal.h"

namespace dyad {

constexpr int kPlanK = 32;   // reduction indices per stage

// Splits of the reduction for a launch of `tiles` output tiles: none when the
// tiles alone fill the GPU; otherwise the fewest that give about 384 work
// items, each split keeping at least `min_stages` stages per component, and no
// more than keep the fp32 partial sums (written and read once) within the
// bytes of the two weight tensors.
inline int gemm_splits(const GemmPass &p, int64_t tiles, int min_stages) {
    if (tiles >= 192) return 1;
    const int ks = (int)(p.bk / kPlanK);
    const int64_t wbytes = 4 * p.D * p.bn * p.bk;
    int best = 1;
    for (int sp = 2; sp * min_stages <= ks; ++sp) {
        if (ks % sp != 0) continue;
        if ((int64_t)sp * p.M * p.Nout * 8 > wbytes) break;
        best = sp;
        if (tiles * sp >= 384) break;
    }
    return best;
}

// The 4-wave tile and reduction splits of a pass, from two plans.
//
// The wide plan is the largest tile that divides the blocks, its reduction split
// as often as fills the GPU (gemm_splits).  The filling plan, largest tile first:
//   - a tile that gives the GPU 256 workgroups by itself (384 where the
//     reduction is short, under 12 stages a component, and the epilogue wants a
//     second workgroup on the CU to hide behind; 128 at n_dyad 8 and 16 with an
//     input transpose, where every column tile reads whole spans of the input);
//   - untransposed weights: 64 x 64 alone from 192, then the largest tile that
//     reaches 192 with up to 4 splits of at least 4 stages;
//   - weights read transposed: the largest tile that reaches 144 alone or 192
//     with up to 4 splits (narrow tiles leave most threads without a weight
//     block to transpose), then 64 x 64 alone;
//   - else 64 x 64 with up to 8 splits.
// It wins where the wide plan leaves CUs idle (OPT-125m fc2 forward 42 -> 12 us at
// 256 tokens, 41 -> 24 at 2047 (64 x 64), 42 -> 31 at 4096 (64 x 192); fc1 input
// gradient of Dyad-IT 44 -> 26 at 2047 (128 x 192, 4 splits)), and loses where a long
// reduction lets the wide plan split (32768 -> 8192, n_dyad 8, 64 tokens, forward:
// 64 x 256 with 16 splits 48 us, 64 x 64 147).  wide_wins() draws the line by the
// work items of both; measured over 27 000 passes of 33 to 9000 tokens, widths 768
// to 32768, n_dyad 2 to 16: 0.78x the wide plan's time in all, 0.98x the filling
// plan's, 1.01x the better of the two.
struct TilePlan {
    int bm = 0, bn = 0, splits = 1;
    int64_t items = 0;
};

struct TileChoice {
    int bm = 0, bn = 0, splits = 1;
    TilePlan wide, fill;
    int rank = 0;

    void consider(const GemmPass &p, int tm, int tn) {
        if (p.bn % tn != 0) return;
        const int64_t tiles = (p.M + tm - 1) / tm * (p.Nout / tn);
        const int ks = (int)(p.bk / kPlanK);
        if (wide.bm == 0) {
            const int sp = gemm_splits(p, tiles, 1);
            wide = TilePlan{tm, tn, sp, tiles * sp};
        }
        if (tm == 128 && tn == 64) return;   // in the wide plan alone, of blocks that nothing wider divides
        const bool smallest = tm == 64 && tn == 64;
        const int enough = p.D >= 8 && p.in_t ? 128 : ks < 12 ? 384 : p.w_t ? 144 : 256;
        int r = 1, sp = 1;
        if (tiles >= enough && !(smallest && p.w_t)) {
            r = 4;
        } else if (smallest && tiles >= 192) {
            r = p.w_t ? 2 : 3;
        } else {
            for (int k = 2; k <= 8 && tiles * sp < 192; ++k)
                if (ks % k == 0 && ks / k >= 4 && (int64_t)k * p.M * p.Nout * 4 <= ((int64_t)64 << 20)) sp = k;
            if (tiles * sp >= 192 && sp <= 4) r = p.w_t ? 4 : 2;
        }
        // ties go to the earlier, larger tile, except that the smallest is
        // taken where none reaches 192 workgroups
        if (r > rank || (r == 1 && rank == 1)) {
            fill = TilePlan{tm, tn, sp, tiles * sp};
            rank = r;
        }
    }

    // Whether the wide plan is the faster: it has work for most CUs.
    bool wide_wins(const GemmPass &p) const {
        const int ks = (int)(p.bk / kPlanK);
        const int64_t w = wide.items, f = fill.items;
        // a split of a short reduction costs more than it fills
        if (fill.splits > 1 && wide.splits == 1 && ks < 16 && w >= 80) return true;
        // half of a 128-row tile would be padding: only the longest reductions carry that
        if (p.M <= 64 && wide.bm == 128) return p.w_t && w >= 256 && ks > 96;
        // one row of tiles: below n_dyad 8 and the longest reductions, many splits of
        // the wide ones beat only a filling plan of few work items or few splits
        if (p.M <= 64 && !p.w_t && wide.splits > 1)
            return w > 224 && (f <= 192 || fill.splits <= 2 || ks > 128 || p.D >= 8);
        // a long reduction in 64 x 64 tiles reads its operands most often
        if (fill.bm == 64 && fill.bn == 64 && ks >= 48 && w >= 128) return true;
        if (p.w_t) return w >= 192 || (w >= 160 && 2 * w >= f);
        if (wide.bm == 128 && wide.bn == 64 && w >= 256) return true;
        return (w >= 128 && w >= f) || (w >= 256 && f < 512);
    }

    void settle(const GemmPass &p) {
        const TilePlan &t = wide_wins(p) ? wide : fill;
        bm = t.bm; bn = t.bn; splits = t.splits;
    }
};

}  // namespace dyad
