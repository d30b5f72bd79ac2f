// Which passes take the plain-block form on the large tiles (gemm_pp.h), and
// how, on the host: sizes only, no device code.
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

// Whether the 256 x 256 tiles of M x N outputs use at least `percent` of the
// places that their rounds over the GPU's 256 CUs have.
inline bool pp_rounds_filled(int64_t M, int64_t N, int percent) {
    const int64_t tiles = (M + 255) / 256 * (N / 256);
    return 100 * tiles >= percent * 256 * ((tiles + 255) / 256);
}

// Whether a pass takes the plain-block form on the large tiles rather than
// the fused tiles (or, at n_dyad 8 and 16, the earlier plain-block tiles).  The
// form pays for its copies in HBM traffic, so it wants reductions long enough,
// and blocks wide enough, for the faster multiply to earn that back.  Measured
// on gfx950 per call against those, widths 640 to 32768, M = 1025 to 16896 (x:
// their time over this form's):
//   no output transpose:
//     n_dyad 16 1.2-1.9x; n_dyad 8 from blocks of 256 1.35-2.1x (2048 -> 8192,
//       8192 tokens: 242 -> 120 us; under 2560 tokens from 512, below 0.9-1.05x);
//     n_dyad 4 from blocks of 512 both ways 1.2-1.6x (4096 -> 4096: 187 -> 149 us;
//       blocks of 256 0.8x); with both blocks under 1024 where the rounds are
//       filled, else 0.9-1.05x;
//     n_dyad 2 from reduction blocks of 512 with output blocks of 2048 1.06-1.7x
//       (GELU' with unfilled rounds 0.91-0.97x), of 1024 both ways 1.05-1.2x (read
//       transposed with unfilled rounds from 2048); narrower 0.76-1.15x;
//   output transpose, residue-major, without a stashed pre-activation or GELU'
//   (whose extra copies take the gain: 0.85-1.0x):
//     n_dyad 8 and 16 from reduction blocks of 256 1.1-1.7x;
//     n_dyad 4 from blocks of 512, one of them from 1024, 1.04-1.9x (2048 -> 2048,
//       both 512, 0.8-1.0x), with an input copy as well both from 1024, or with
//       weights read transposed the reduction's, 1.04-1.7x (8192 -> 2048 forward,
//       8192 tokens 0.77x);
//     n_dyad 2 from 1024, output blocks from 2048 1.04-1.4x; narrower ones without
//       an input copy 1.1-1.5x (read transposed with unfilled rounds from 2048),
//       with one only from 4096 and 1024 1.0-1.6x, else 0.76-1.2x;
//   output transpose, slice:
//     n_dyad 8, output blocks from 256, reduction blocks from 1024 1.2-2x (8192 ->
//       2048: 196 -> 118 us; an untransposed pass without an input copy wants 64
//       tiles, below 0.92x), from 512 up to 2048 tokens 1.1-1.8x (beyond, against
//       the earlier tiles, 0.75-0.95x); n_dyad 16 0.9-1.0x;
//     n_dyad 2 and 4 without an input copy from 1024 with output blocks over 256,
//       or read transposed, 1.04-1.25x (4096 -> 1024, 16384 tokens, forward 0.89x).
// n_dyad 2 and 4 also want 192 tiles of 256 x 256: with fewer, the fused
// tiles' smaller ones fill the GPU better (0.94x at 128 tiles).
inline bool pp_pays(const GemmPass &p) {
    if (p.M <= 1024 || p.bk % 32 != 0 || p.bn % 64 != 0) return false;
    if (!pp_fits(256, p.Kin, p.Nout, p.D * p.bn * p.bk)) return false;
    const bool h = p.h_out != nullptr || p.epilogue == kEpiGeluGrad;
    const bool res = pp_res_columns(p);
    const int64_t tiles = (p.M + 255) / 256 * (p.Nout / 256);
    if (p.D >= 8) {
        if (!p.out_t) return p.D >= 16 || p.bk >= 512 || (p.bk >= 256 && p.M >= 2560);
        if (res) return !h && p.bk >= 256;
        if (p.D != 8 || p.bn < 256 || p.bk < 512) return false;
        if (p.bk < 1024) return p.M <= 2048;
        return p.in_t || p.w_t || tiles >= 64;
    }
    if (tiles < 192) return false;
    // a long reduction carries rounds that leave CUs idle
    const bool fed = !p.w_t || p.bk >= 2048 || pp_rounds_filled(p.M, p.Nout, 75);
    if (!p.out_t) {
        if (p.bk < 512 || p.bn < 512) return false;
        if (p.D == 4) return p.bk >= 1024 || p.bn >= 1024 || pp_rounds_filled(p.M, p.Nout, 75);
        if (p.bn >= 2048)
            return p.epilogue != kEpiGeluGrad || p.bn >= 4096 || p.bk >= 1024 || pp_rounds_filled(p.M, p.Nout, 80);
        return p.bk >= 1024 && p.bn >= 1024 && fed;
    }
    if (res) {
        if (h) return false;
        if (p.D == 2) {
            if (p.bk < 1024) return false;
            return p.bn >= 2048 || (p.in_t ? p.bk >= 4096 && p.bn >= 1024 : fed);
        }
        if (p.in_t) return p.bk >= 1024 && (p.w_t || p.bn >= 1024);
        return p.bk >= 512 && (p.bk >= 1024 || p.bn >= 1024);
    }
    return !p.in_t && p.bk >= 1024 && (p.bn > 256 || (p.w_t && p.bn == 256));
}

// The plain-block form of a large batch with a transpose.  An input transpose
// first de-interleaves the input (residue g's columns k*D + g become the
// contiguous block g).  Without an output transpose both components then run in
// one loop (kPPPair).  With one:
//   - where every (block, residue) pair of the output has whole tiles of
//     columns, both components still run in one loop over residue-major
//     columns (kPPRes), and a copy interleaves the bf16 results (4 bytes an
//     output);
//   - else component 2's sums go to an fp32 slice in block order, which
//     component 1's epilogue adds at the block-order place of each output
//     column (kPPSlice; 8 bytes an output and a second pass, but with output
//     blocks that narrow the outputs are few against the reduction).
// The tokens run in chunks of whole rounds of tiles over the GPU, kept short
// enough that what passes between the kernels stays in the 256 MB MALL
// (Dyad-DT 8192 -> 32768, n_dyad 16, 8192 tokens, forward: 1335 us in one
// chunk, 1138 in chunks of 160 MB).
constexpr size_t kPPChunkBytes = (size_t)160 << 20;

struct PPPlan {
    int form = kPPNone;       // kPPPair, kPPRes or kPPSlice; kPPNone: the pass stays with the other tiles
    int64_t chunk = 0;        // tokens per chunk
    size_t per_tok = 0;       // workspace bytes per token of a chunk
    size_t wcopy = 0;         // and for the copy of W1
};

inline PPPlan pp_plan(const GemmPass &p) {
    PPPlan pl;
    if ((!p.in_t && !p.out_t) || !pp_pays(p)) return pl;
    const int form = !p.out_t ? kPPPair : pp_res_columns(p) ? kPPRes : kPPSlice;
    pl.per_tok = (p.in_t ? (size_t)p.Kin * 2 : 0) + (form == kPPSlice ? (size_t)p.Nout * sizeof(float) : 0) +
                 (form == kPPRes ? (size_t)p.Nout * 2 : 0);
    pl.wcopy = form == kPPRes && p.w_t ? (size_t)(p.D * p.bn * p.bk) * 2 : 0;
    const int64_t round = 256 * ((256 * 256 + p.Nout - 1) / p.Nout);   // 256 tiles of 256 x 256
    const int64_t fit = (int64_t)(kPPChunkBytes / pl.per_tok) / round * round;
    pl.chunk = fit > round ? fit : round;
    if (pl.chunk > p.M) pl.chunk = p.M;
    if (pl.per_tok * (size_t)pl.chunk + pl.wcopy <= ((size_t)2 << 30)) pl.form = form;
    return pl;
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
