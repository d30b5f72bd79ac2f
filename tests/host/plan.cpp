// Host-side plans and load offsets of the large passes behind C names, for
// test_plan_cpu.py.
#include "gemm_mfma_dispatch.h"
#include "pp_core.h"
#include "pp_plan.h"

using dyad::GemmPass;

// The pass that the C-ABI describes to the kernels: forward, or with dx the
// input gradient; epilogue and stash as there.
static GemmPass pass(int variant, int64_t n_in, int64_t n_out, int64_t D, int64_t M, int dx, int act, int stash) {
    GemmPass p{};
    const bool it = variant == 0 || variant == 2, ot = variant == 1 || variant == 2;
    p.M = M; p.D = D;
    p.Kin = dx ? n_out : n_in; p.Nout = dx ? n_in : n_out;
    p.bk = (p.Kin + D - 1) / D; p.bn = (p.Nout + D - 1) / D;
    p.in_t = dx ? ot : it; p.out_t = dx ? it : ot; p.w_t = dx != 0;
    p.dtype = dyad::kBF16;
    p.epilogue = !act ? dyad::kEpiBias : dx ? dyad::kEpiGeluGrad : dyad::kEpiBiasGelu;
    static char any[16];
    if (stash) p.h_out = any;
    if (act && dx) p.h_in = any;
    return p;
}

extern "C" {

int pp_pays(int variant, int64_t n_in, int64_t n_out, int64_t D, int64_t M, int dx, int act, int stash) {
    return dyad::pp_pays(pass(variant, n_in, n_out, D, M, dx, act, stash));
}

// The form the pass takes (PPForm; 0: none) and its token chunk.
int pp_plan(int variant, int64_t n_in, int64_t n_out, int64_t D, int64_t M, int dx, int act, int stash, int64_t *chunk) {
    const dyad::PPPlan pl = dyad::pp_plan(pass(variant, n_in, n_out, D, M, dx, act, stash));
    *chunk = pl.chunk;
    return pl.form;
}

int padded_fused(int variant, int64_t n_in, int64_t n_out, int64_t D, int64_t M, int dx) {
    const GemmPass p = pass(variant, n_in, n_out, D, M, dx, 0, 0);
    return dyad::padded_fused(p, dyad::pad_up(p.bk, 32));
}

// The 4-wave tile of the pass: bm, bn, splits, and the two plans' work items.
void tile_choice(int variant, int64_t n_in, int64_t n_out, int64_t D, int64_t M, int dx, int64_t *out) {
    const GemmPass p = pass(variant, n_in, n_out, D, M, dx, 0, 0);
    dyad::TileChoice t;
    auto pick = [&](auto d) {
        constexpr int kD = decltype(d)::value;
        t = p.out_t ? dyad::choose_tile<kD, true>(p) : dyad::choose_tile<kD, false>(p);
    };
    switch (D) {
    case 2: pick(std::integral_constant<int, 2>{}); break;
    case 3: pick(std::integral_constant<int, 3>{}); break;
    case 4: pick(std::integral_constant<int, 4>{}); break;
    case 6: pick(std::integral_constant<int, 6>{}); break;
    case 8: pick(std::integral_constant<int, 8>{}); break;
    case 16: pick(std::integral_constant<int, 16>{}); break;
    default: break;
    }
    out[0] = t.bm; out[1] = t.bn; out[2] = t.splits; out[3] = t.wide.items; out[4] = t.fill.items;
}

// Loads of one unit k of a side (N rows of 2 * bk bytes, or with tr bk rows of N
// columns).  Returns how many lanes read outside those bytes, with the unit
// starting at pp_unit_step (or stepping back in a reduction of one step), or with
// plain != 0 at step 2 k.  wrong: lanes of a step that is multiplied whose bytes
// are not that step's.
int pp_outside(int n, int tr, int64_t bk, int64_t k, int plain, int *wrong) {
    int bad = 0;
    *wrong = 0;
    auto side = [&](auto N, auto TR) {
        constexpr int kN = decltype(N)::value;
        constexpr bool kTR = decltype(TR)::value;
        using S = dyad::PPSide<kN, kTR>;
        const int64_t pitch = kTR ? 2 * kN : 2 * bk, step = kTR ? dyad::kStageK * pitch : 2 * dyad::kStageK;
        const int ks = (int)(bk / dyad::kStageK);
        const bool one = ks == 1, both = 2 * k + 1 < ks;
        const int64_t start = (plain ? 2 * k : one ? 0 : dyad::pp_unit_step((int)k, ks)) * step;
        for (int wave = 0; wave < dyad::kPPWaves; ++wave)
            for (int q = 0; q < S::kPer; ++q)
                for (int lane = 0; lane < 64; ++lane) {
                    int row, byte;
                    const int i = dyad::pp_instr(wave, q);
                    dyad::pp_source<kN, kTR>(i, lane, row, byte);
                    const int64_t back = one && !plain ? dyad::pp_back<kN, kTR>(i, lane, (uint32_t)pitch) : 0;
                    const int64_t at = row * pitch + byte - back + start;
                    const int64_t lo = kTR ? 0 : row * pitch, hi = kTR ? bk * pitch : lo + 2 * bk;
                    bad += at < lo || at + 16 > hi;
                    // the loop multiplies both steps, or the second alone: step 2 k + h, or the last
                    const int h = kTR ? row / dyad::kStageK : byte / (2 * dyad::kStageK);
                    if (!both && h == 0) continue;
                    const int64_t want = both ? 2 * k + h : ks - 1;
                    *wrong += (kTR ? at / pitch / dyad::kStageK : (at - lo) / (2 * dyad::kStageK)) != want;
                }
    };
    auto with = [&](auto TR) {
        if (n == 256) side(std::integral_constant<int, 256>{}, TR);
        else if (n == 192) side(std::integral_constant<int, 192>{}, TR);
        else if (n == 128) side(std::integral_constant<int, 128>{}, TR);
        else if (n == 64) side(std::integral_constant<int, 64>{}, TR);
        else bad = -1;
    };
    if (tr) with(std::true_type{});
    else with(std::false_type{});
    return bad;
}

}  // extern "C"
