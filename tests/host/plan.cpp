// Host-side plans and load offsets of the large passes behind C names, for
// test_plan_cpu.py.
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

// Loads of one unit k of a side (N rows of 2 * bk bytes, or with tr bk rows of N
// columns): how many lanes read outside those bytes, stepping back in a unit of
// one step or (back == 0) not, and how many first-step lanes step back at all.
int pp_outside(int n, int tr, int64_t bk, int64_t k, int back, int *moved) {
    int bad = 0;
    *moved = 0;
    auto side = [&](auto N, auto TR) {
        constexpr int kN = decltype(N)::value;
        constexpr bool kTR = decltype(TR)::value;
        using S = dyad::PPSide<kN, kTR>;
        const int64_t pitch = kTR ? 2 * kN : 2 * bk, ks = bk / dyad::kStageK;
        const bool one = 2 * k + 1 >= ks;
        for (int wave = 0; wave < dyad::kPPWaves; ++wave)
            for (int q = 0; q < S::kPer; ++q)
                for (int lane = 0; lane < 64; ++lane) {
                    int row, byte;
                    const int i = dyad::pp_instr(wave, q);
                    dyad::pp_source<kN, kTR>(i, lane, row, byte);
                    const int64_t step = one && back ? dyad::pp_back<kN, kTR>(i, lane, (uint32_t)pitch) : 0;
                    const bool first = kTR ? row < dyad::kStageK : byte < 2 * dyad::kStageK;
                    *moved += first && step != 0;
                    const int64_t at = row * pitch + byte - step + k * (kTR ? dyad::kPPK * pitch : 2 * dyad::kPPK);
                    const int64_t lo = kTR ? 0 : row * pitch, hi = kTR ? bk * pitch : lo + 2 * bk;
                    bad += at < lo || at + 16 > hi;
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
