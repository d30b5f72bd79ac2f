// Which passes take the plain-block form on the large tiles (gemm_pp.h), on the
// host: sizes only, no device code.
#pragma once

#include "dyad_internal.h"

namespace dyad {

// Forms of a launch of the large tiles (gemm_pp.h).
enum PPForm { kPPNone = 0, kPPPair = 1, kPPSlice = 2, kPPAdd = 3, kPPPadAdd = 4, kPPPadPair = 5, kPPRes = 6, kPPPairOne = 7 };

// Whether the 32-bit byte offsets of a tile of BM token rows reach all of it:
// its input and output panels (fp32 sums included) and one weight tensor of
// `weights` entries.  The tiles of the other matrix-core kernels have the same
// bound; past it the vector kernel, which counts in 64 bits, takes the pass.
inline bool pp_fits(int64_t BM, int64_t Kin, int64_t Nout, int64_t weights) {
    const int64_t lim = (int64_t)1 << 31;
    return BM * Kin * 2 < lim && BM * Nout * 4 < lim && 2 * weights < lim;
}

// Residue-major columns in whole tiles: every (block, residue) pair of the
// output holds a multiple of 128 or 192 columns (64-column tiles lost to the
// slice: n_dyad 8, 4096 tokens, 16384 -> 4096 input gradient with 64 columns
// a pair 397 against 299 us).
inline bool pp_res_columns(const GemmPass &p) {
    return p.out_t && p.bn % p.D == 0 && (p.bn / p.D % 128 == 0 || p.bn / p.D % 192 == 0);
}

// Whether a pass takes the plain-block form on the large tiles rather than
// the fused tiles (or, at n_dyad 16, the earlier plain-block tiles).  The form
// pays for its copies in HBM traffic, so it wants reductions long enough, and
// blocks wide enough, for the faster multiply to earn that back.  Measured on
// gfx950 per call against those, M = 2048 to 16384 tokens:
//   no output transpose: n_dyad 8 from blocks of 256 1.35-2.1x (2048 -> 8192,
//     8192 tokens: 242 -> 120 us; under 2560 tokens from 512, below 0.9-1.05x), n_dyad 16
//     1.2-1.7x; n_dyad 2 and 4 from blocks of 512 both ways 1.2-1.6x (4096 ->
//     4096, n_dyad 4: 187 -> 149 us; blocks of 256 0.8x).
//   output transpose, residue-major: n_dyad 8 and 16 from reduction blocks of
//     256 1.1-1.5x without a stashed pre-activation or GELU' (whose extra
//     copies take the gain: 0.85-1.0x); n_dyad 4 from 512 (with an input copy as
//     well, and at n_dyad 2, from 1024) 1.04-1.6x (4096 -> 4096, n_dyad 4: 241 -> 153 us).
//   output transpose, slice: n_dyad 8 from reduction blocks of 512 and output
//     blocks of 256 1.4-1.7x (8192 -> 2048: 196 -> 118 us), n_dyad 2 and 4
//     without an input copy from 1024 1.15-1.25x; n_dyad 16 0.9-1.0x.
// n_dyad 2 and 4 also want 192 tiles of 256 x 256: with fewer, the fused
// tiles' smaller ones fill the GPU better (0.94x at 128 tiles).
inline bool pp_pays(const GemmPass &p) {
    if (p.M <= 1024 || p.bk % 32 != 0 || p.bn % 64 != 0) return false;
    if (!pp_fits(256, p.Kin, p.Nout, p.D * p.bn * p.bk)) return false;
    const bool h = p.h_out != nullptr || p.epilogue == kEpiGeluGrad;
    const bool res = pp_res_columns(p);
    if (p.D >= 8) {
        if (!p.out_t) return p.D >= 16 || p.bk >= 512 || (p.bk >= 256 && p.M >= 2560);
        if (res) return !h && p.bk >= 256;
        return p.D == 8 && p.bn >= 256 && p.bk >= 512;
    }
    if ((p.M + 255) / 256 * (p.Nout / 256) < 192) return false;
    if (!p.out_t) return p.bk >= 512 && p.bn >= 512;
    if (res) return !h && p.bk >= (p.in_t || p.D == 2 ? 1024 : 512);
    return !p.in_t && p.bn >= 256 && p.bk >= 1024;
}

// Whether a zero-padded form (padded_mfma.h) runs on the fused-stage tiles
// instead of the large ones; bkp: reduction block rounded up to 32.
//   Output transpose, short reductions: a tile is mostly epilogue, where the
//   fused-stage tiles' staged stores beat a second pass over the slice in LDS.
//     - blocks of a multiple of 8 columns, reductions up to 256 (768 -> 3072,
//       n_dyad 16, 16384 tokens, forward 194 against 265 us; n_dyad 12 at blocks
//       of 64 to 256 0.89-0.96x on the large tiles), while blocks that start
//       anywhere win 1.1-1.2x there from reductions of 96;
//     - blocks that only 64- or 192-column tiles divide: up to 64, and under 512
//       where 192-column tiles fill the GPU (1024 -> 1024, n_dyad 5, 0.91-0.96x).
//   Weights read transposed, blocks that only 64-column tiles divide, reductions
//   from 1024: 0.91-0.98x on the large tiles.
inline bool padded_fused(const GemmPass &p, int64_t bkp) {
    const int64_t w = pad_up(p.bn, 64);
    if (!p.out_t) return p.w_t && bkp >= 1024 && w % 128 != 0 && w % 192 != 0;
    if (p.bn % 8 == 0) return bkp <= 256;
    if (w % 128 == 0) return false;
    return bkp <= 64 || (bkp < 512 && w % 192 == 0 && (p.M + 255) / 256 * (p.D * w / 192) >= 192);
}

}  // namespace dyad
