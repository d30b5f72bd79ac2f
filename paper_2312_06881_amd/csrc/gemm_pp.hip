// Tile choice and instances of the grouped GEMM on block-ordered operands
// (gemm_pp.h).
#include "gemm_pp.h"
#include "pp_plan.h"

namespace dyad {
namespace {

// The tile of a launch: columns in a run of w (an output block, or one block
// and residue).  256-wide rows of the output fill the matrix cores best where
// they fill the GPU.  Two workgroups of the tiles under 128 x 128 share a CU
// and hide each other's epilogues, which wins for short reductions and for
// slices staged through LDS (768 -> 3072, n_dyad 5, 8192 tokens, GELU forward:
// pair 92 -> 83 us, slice 171 -> 143; 3072 -> 768 at 640 a block 76 -> 72 the
// other way; 8192 -> 32768, n_dyad 16, 4096 tokens, 512 a block 495 -> 529).
//   - Padded blocks that add a slice take no tile above 128 x 128 that divides
//     them: the larger ones hold more than a wave's registers (768 -> 3072,
//     n_dyad 12: 0.65-0.75x of the fused-stage tiles, 128 x 128 1.17x).
//   - 192-wide tiles that fill only part of the GPU beat 64-wide ones in more
//     than one round (1536 -> 6144, n_dyad 8, 3328 tokens, input gradient 0.75x
//     -> 1.02x of the earlier tiles).
//   - Of the 64-wide tiles the tall one pays only with untransposed weights and
//     no slice to add (padded 2048 -> 2048, n_dyad 3, input gradient 0.88 -> 1.0x).
template <bool W_T, int FORM>
hipError_t launch_form(const GemmArgs &a, hipStream_t s) {
    const int64_t tm = (a.M + 255) / 256;
    const int64_t w = FORM == kPPRes && a.bn % a.D == 0 ? a.bn / a.D : a.bn;
    constexpr bool add = FORM == kPPAdd || FORM == kPPPadAdd;
    auto fills = [&](int bn) { return tm * (a.Nout / bn) >= 192; };
    if constexpr (FORM == kPPPadAdd) {
        if (w % 128 == 0) return launch_pp_tile<128, 128, 2, 4, W_T, FORM>(a, s);
    } else {
        if (w % 256 == 0 && fills(256)) return launch_pp_tile<256, 256, 2, 4, W_T, FORM>(a, s);
    }
    if (w % 192 == 0 && (fills(192) || (FORM == kPPPair && w % 128 != 0 && tm * (a.Nout / 64) > 256)))
        return launch_pp_tile<256, 192, 4, 2, W_T, FORM>(a, s);
    if (w % 128 == 0 && (add || a.bk < 512 || !fills(128))) return launch_pp_tile<128, 128, 2, 4, W_T, FORM>(a, s);
    if constexpr (!add)
        if (w % 128 == 0) return launch_pp_tile<256, 128, 4, 2, W_T, FORM>(a, s);
    if (w % 64 == 0 && (add || W_T || a.bk < 512 || !fills(64))) return launch_pp_tile<128, 64, 4, 2, W_T, FORM>(a, s);
    if constexpr (!add && !W_T)
        if (w % 64 == 0) return launch_pp_tile<256, 64, 4, 2, W_T, FORM>(a, s);
    return hipErrorNotSupported;
}

template <bool W_T>
hipError_t launch_w(int form, const GemmArgs &a, hipStream_t s) {
    switch (form) {
    case kPPPair:
        // one step a component: epilogues all but alone, two workgroups a CU
        if (a.bk < kPPK)
            return a.bn % 128 == 0 ? launch_pp_tile<128, 128, 2, 4, W_T, kPPPairOne>(a, s)
                                   : launch_pp_tile<128, 64, 4, 2, W_T, kPPPairOne>(a, s);
        return launch_form<W_T, kPPPair>(a, s);
    case kPPSlice: return launch_form<W_T, kPPSlice>(a, s);
    case kPPAdd: return launch_form<W_T, kPPAdd>(a, s);
    case kPPPadAdd: return launch_form<W_T, kPPPadAdd>(a, s);
    case kPPPadPair: return launch_form<W_T, kPPPadPair>(a, s);
    case kPPRes: return launch_form<W_T, kPPRes>(a, s);
    default: return hipErrorNotSupported;
    }
}

}  // namespace

hipError_t launch_pp(int form, bool w_t, const GemmArgs &a, hipStream_t s) {
    return w_t ? launch_w<true>(form, a, s) : launch_w<false>(form, a, s);
}

// The inverse of deinterleave_kernel: out[n][t*D + r] = in[n][r*W + t] for
// rows of D*W values.  4*D threads move 32 columns of every residue: 16-byte
// loads along a residue, transposed in LDS, 16-byte stores.
__global__ void __launch_bounds__(256) interleave_kernel(const uint16_t *in, uint16_t *out, int64_t M, int W, int D) {
    __shared__ uint4 buf[256];
    const int tid = threadIdx.x, per = 4 * D;
    const int c = tid / per, pc = tid % per;
    const int spans = W / 32;
    const int64_t gc = (int64_t)blockIdx.x * (256 / per) + c;
    const bool ok = c < 256 / per && gc < M * spans;
    const int64_t n = ok ? gc / spans : 0, kc = ok ? gc % spans : 0;
    const int64_t N = (int64_t)W * D;
    uint16_t *span = reinterpret_cast<uint16_t *>(buf + c * per);
    if (ok) {
        const int r = pc / 4, t0 = (pc % 4) * 8;
        const uint4 v = *reinterpret_cast<const uint4 *>(in + n * N + (int64_t)r * W + kc * 32 + t0);
#pragma unroll
        for (int e = 0; e < 8; ++e) span[(t0 + e) * D + r] = (uint16_t)(word_of(v, e >> 1) >> (16 * (e & 1)));
    }
    __syncthreads();
    if (ok) *reinterpret_cast<uint4 *>(out + n * N + kc * 32 * D + pc * 8) = buf[c * per + pc];
}

hipError_t launch_interleave(const uint16_t *in, uint16_t *out, int64_t M, int64_t W, int D, hipStream_t s) {
    if (D < 1 || D > 64 || W % 32 != 0 || M < 0) return hipErrorNotSupported;
    if (M == 0) return hipSuccess;
    const int64_t groups = M * (W / 32), per_block = 256 / (4 * D);
    const int64_t blocks = (groups + per_block - 1) / per_block;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorNotSupported;
    interleave_kernel<<<(unsigned)blocks, 256, 0, s>>>(in, out, M, (int)W, D);
    return hipGetLastError();
}

hipError_t launch_permuted_pp(const GemmPass &p, hipStream_t s) {
    const PPPlan pl = pp_plan(p);
    if (!pl.form) return hipErrorNotSupported;
    const int D = (int)p.D;
    const bool res = pl.form == kPPRes, slices = pl.form == kPPSlice;
    const int64_t mc = pl.chunk;
    void *ws = nullptr;
    if (split_workspace(s, pl.per_tok * (size_t)mc + pl.wcopy, &ws) != hipSuccess) {
        (void)hipGetLastError();
        return hipErrorNotSupported;
    }
    float *slice = static_cast<float *>(ws);
    uint16_t *yp = reinterpret_cast<uint16_t *>(slice + (slices ? mc * p.Nout : 0));
    uint16_t *xp = yp + (res ? mc * p.Nout : 0);
    uint16_t *w1d = xp + (p.in_t ? mc * p.Kin : 0);
    GemmArgs a{};
    a.Kin = p.Kin; a.Nout = p.Nout; a.bk = p.bk; a.bn = p.bn; a.D = p.D;
    a.bias = static_cast<const uint16_t *>(p.bias);
    a.epilogue = p.epilogue;
    a.W1 = static_cast<const uint16_t *>(p.W1);
    a.W2 = static_cast<const uint16_t *>(p.W2);
    hipError_t e = hipSuccess;
    if (pl.wcopy) {
        e = launch_deinterleave(a.W1, w1d, p.D * p.bk, p.bn / p.D, D, s);
        a.W1 = w1d;
    }
    for (int64_t m0 = 0; m0 < p.M && e == hipSuccess; m0 += mc) {
        a.M = p.M - m0 < mc ? p.M - m0 : mc;
        a.in = static_cast<const uint16_t *>(p.in) + m0 * p.Kin;
        a.in2 = a.in;
        uint16_t *out = static_cast<uint16_t *>(p.out) + m0 * p.Nout;
        a.out = out;
        a.h_out = p.h_out ? static_cast<uint16_t *>(p.h_out) + m0 * p.Nout : nullptr;
        a.h_in = p.h_in ? static_cast<const uint16_t *>(p.h_in) + m0 * p.Nout : nullptr;
        if (p.in_t) {
            e = launch_deinterleave(a.in, xp, a.M, p.bk, D, s);
            a.in2 = xp;
        }
        if (res) {
            a.out = yp;
            if (e == hipSuccess) e = launch_pp(kPPRes, p.w_t, a, s);
            if (e == hipSuccess) e = launch_interleave(yp, out, a.M, p.Nout / D, D, s);
        } else if (!slices) {
            if (e == hipSuccess) e = launch_pp(kPPPair, p.w_t, a, s);
        } else {
            GemmArgs c2 = a;
            c2.in = a.in2; c2.W1 = a.W2;
            c2.bias = nullptr; c2.h_in = nullptr; c2.out = nullptr; c2.h_out = nullptr; c2.epilogue = kEpiBias;
            c2.part = slice; c2.unperm = 0;
            if (e == hipSuccess) e = launch_pp(kPPSlice, p.w_t, c2, s);
            a.part = slice; a.unperm = 1;
            if (e == hipSuccess) e = launch_pp(kPPAdd, p.w_t, a, s);
        }
    }
    return e;
}

}  // namespace dyad
