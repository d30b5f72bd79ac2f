// Host-side plans of the large passes behind C names, for test_plan_cpu.py.
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

}  // extern "C"
