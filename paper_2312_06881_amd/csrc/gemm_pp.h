// The grouped GEMM on block-ordered operands, large tiles (pp_core.h): the
// large-batch and zero-padded forms of the forward pass and the input
// gradient, whose operands are plain blocks (a strided one de-interleaved into
// a copy beforehand).
//
// A tile lies in one output block g.  FORM:
//   kPPPair   both components in one loop, component 2 reading in2 (the
//             de-interleaved copy, or in) at the first's places; epilogue
//   kPPPairOne  the same for reduction blocks of one step (32 indices)
//   kPPSlice  component 1's sums into fp32 slice a.slice0 of a.part
//   kPPAdd    component 1, plus the slice's sums (at the block-order place of
//             each column with a.unperm); epilogue
//   kPPPadAdd, kPPPadPair   those two forms on zero-padded blocks
//             (pp_epilogue, PAD)
//   kPPRes    an output transpose in one loop, columns kept residue-major: the
//             tile takes columns g*bn + r + D*t of one output block g and one
//             residue r, so both components are plain blocks (component 1:
//             block g of the input, every D-th weight row; component 2: block
//             r of in2, consecutive rows of weight group r).  Its outputs (and
//             h_out, h_in) are rows of r*(Nout/D) + t columns, which a copy
//             before or after the pass puts in order.  With W_T the columns of
//             W1 come de-interleaved within each block (r*(bn/D) + t).
#pragma once

#include "gemm_common.h"
#include "pp_core.h"
#include "pp_plan.h"

namespace dyad {

template <int BM, int BN, int WGM, int WGN, bool W_T>
struct PPCfg {
    static constexpr int WM = BM / WGM, WN = BN / WGN;
    static constexpr int kSubM = WM / 16, kSubN = WN / 16;
    using A = PPSide<BM, false>;
    using B = PPSide<BN, W_T>;
    // three slots a side where they fit, the B side two where not; small tiles
    // take two, so that two workgroups share a CU
    static constexpr bool kTwo = BM * BN <= 128 * 128;
    static constexpr int kSlotA = kTwo ? 2 : 3;
    static constexpr int kSlotB = !kTwo && 3 * (A::kBytes + B::kBytes) <= 160 * 1024 ? 3 : 2;
    static constexpr int kOffB = kSlotA * A::kBytes;
    static constexpr int kLds = kOffB + kSlotB * B::kBytes;
    static_assert(WGM * WGN == kPPWaves && kLds <= 160 * 1024, "eight waves, LDS budget");
    static_assert(kSubN % 2 == 0, "the epilogue pairs column blocks");
};

// Swaps the odd 16-lane rows of a with the even ones of b.
__device__ __forceinline__ void swap_rows(uint32_t &a, uint32_t &b) {
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
    const u32x2_t r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r.x;
    b = r.y;
}

// Zero columns in front of padded block g of b real columns.
__host__ __device__ constexpr int pp_pad_shift(int64_t g, int64_t b) { return (int)(g * b & 7); }

// Slice columns per residue that a tile of BN consecutive real columns touches,
// and the pitch (floats) of a staged token row of all D residues.
__host__ __device__ constexpr int64_t pp_slice_span(int64_t D, int BN) { return (BN + 2 * D - 2) / D; }
__host__ __device__ constexpr int64_t pp_slice_pitch(int64_t D, int BN) {
    return (D * pp_slice_span(D, BN) + 63) / 64 * 64 + 4;
}

// Epilogue of a wave's WM x WN block straight from the accumulators.  The
// weights are the first MFMA operand, so lane l holds, of token l % 16 of
// block row i, columns 4 (l / 16) + v of column block j: four consecutive
// outputs.  Two column blocks packed to bf16 trade their odd and even lane
// rows (v_permlane16_swap), after which every lane holds 8 consecutive outputs
// and a 16-lane row's 16-byte pieces fill whole 64-byte sectors: no staging
// through LDS and no barrier, so the waves drain independently.
//   SLICE: fp32 sums to slice a.slice0 of a.part, no epilogue.
//   ADD:   each sum first gets component 2's from that slice; with a.unperm it
//          sits at the block-order place of the column (c % D) * bn + c / D,
//          and the tile's share of the slice goes through LDS (pp_stage_slice),
//          where the permuted reads are cheap.
//   PAD:   zero-padded blocks: block g's a.bn_r real columns sit behind
//          pp_pad_shift(g, a.bn_r) columns of zeros, which makes 8-column pieces
//          aligned in the padded block aligned in the real row of a.Nout_r
//          columns as well (16-byte pieces at 2-byte aligned addresses cost
//          the OPT-125m n_dyad 5 GELU forward 82 us against 60).  Columns
//          outside the real ones are dropped, element by element in the
//          pieces at a block's ends.
//   RES:   the tile's outputs are columns n0.. of residue-major rows; its real
//          columns (for the bias) are c_real + a.D * t.
template <class C, int BM, int BN, bool SLICE, bool ADD, bool PAD, bool RES>
__device__ __forceinline__ void pp_epilogue(const GemmArgs &a, unsigned char *smem,
                                            const f32x4_t (&acc)[C::kSubM][C::kSubN], int64_t m0, int n0, int g, int jb,
                                            int64_t rows_left, int lane, int wave, int wm0, int wn0, int c_real) {
    constexpr int SM = C::kSubM, SN = C::kSubN;
    const int lr = lane & 15, lg = lane >> 4;
    const uint32_t rows_t = (uint32_t)(rows_left < BM ? rows_left : BM);
    if constexpr (SLICE) {
        const __amdgpu_buffer_rsrc_t rP =
            buffer_rsrc(a.part + ((int64_t)a.slice0 * a.M + m0) * a.Nout, rows_t * (uint32_t)a.Nout * 4u);
#pragma unroll
        for (int i = 0; i < SM; ++i)
#pragma unroll
            for (int j = 0; j < SN; ++j) {
                const u32x4_t v = __builtin_bit_cast(u32x4_t, acc[i][j]);
                const uint32_t vo = ((uint32_t)(wm0 + 16 * i + lr) * (uint32_t)a.Nout + (uint32_t)(n0 + wn0 + 16 * j + 4 * lg)) * 4u;
                __builtin_amdgcn_raw_buffer_store_b128(v, rP, (int)vo, 0, 0);
            }
        return;
    }
    const bool grad = a.epilogue == kEpiGeluGrad;
    const bool act = a.epilogue == kEpiBiasGelu;
    const bool keep_h = act && a.h_out != nullptr;
    const uint32_t Nr = (uint32_t)(PAD ? a.Nout_r : a.Nout);
    // real column of the tile's first, and its real columns lo .. nt - 1
    const int sh = PAD ? pp_pad_shift(g, a.bn_r) : 0;
    const int cb = PAD ? g * (int)a.bn_r - sh + jb : n0;
    const int lo = PAD && sh > jb ? sh - jb : 0;
    int nt = BN;
    if constexpr (PAD) {
        nt = (int)a.bn_r + sh - jb < nt ? (int)a.bn_r + sh - jb : nt;
        nt = (int)Nr - cb < nt ? (int)Nr - cb : nt;
    }
    const bool rows16 = !PAD || Nr % 8 == 0;               // pieces are 16-byte aligned
    const __amdgpu_buffer_rsrc_t rO = buffer_rsrc(a.out + m0 * Nr, rows_t * Nr * 2u);
    const uint16_t *hbase = grad ? a.h_in : a.h_out;
    const __amdgpu_buffer_rsrc_t rH = buffer_rsrc((hbase ? hbase : a.out) + m0 * Nr, rows_t * Nr * 2u);

    float bias[SN][4];
#pragma unroll
    for (int j = 0; j < SN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) bias[j][v] = 0.f;
    if (a.bias != nullptr && !grad) {
#pragma unroll
        for (int j = 0; j < SN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = wn0 + 16 * j + 4 * lg + v;
                if (!PAD || (t >= lo && t < nt)) bias[j][v] = bf16_to_f32(a.bias[RES ? c_real + (int)a.D * t : cb + t]);
            }
    }
    // this lane's 16-byte piece of a column block pair, after the row swap
    const int piece = (lg & 1) * 16 + (lg >> 1) * 8;
    // default cache policy: a lane row's 64 bytes are half a line, which the L2
    // completes (streamed, 8192 tokens of 4096 -> 4096 took 150 us against
    // 142, and padded blocks, whose pieces straddle lines, 122 against 92)
    constexpr int kStore = 0;
    // WHOLE: every column of the tile is real and pieces are 16-byte aligned
    auto load_h = [&](auto whole, int i, int jp) -> uint4 {
        const uint32_t row = (uint32_t)(wm0 + 16 * i + lr);
        const int t = wn0 + 32 * jp + piece;
        uint4 h = make_uint4(0u, 0u, 0u, 0u);
        if (decltype(whole)::value || (rows16 && t >= lo && t + 8 <= nt)) {
            h = bload16_stream(rH, (row * Nr + (uint32_t)(cb + t)) * 2u, 0);
        } else if (row < rows_t) {
            const uint16_t *src = a.h_in + (m0 + row) * (int64_t)Nr + cb + t;
            uint16_t e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) e[k] = t + k >= lo && t + k < nt ? src[k] : (uint16_t)0;
            h = make_uint4(e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16,
                           e[6] | (uint32_t)e[7] << 16);
        }
        swap_rows(h.x, h.z);
        swap_rows(h.y, h.w);
        return h;
    };
    auto store = [&](auto whole, const __amdgpu_buffer_rsrc_t &r, uint16_t *base, int i, int jp, const float (&x)[8]) {
        uint32_t d0 = pack_bf16(x[0], x[1]), d1 = pack_bf16(x[2], x[3]);
        uint32_t s0 = pack_bf16(x[4], x[5]), s1 = pack_bf16(x[6], x[7]);
        swap_rows(d0, s0);
        swap_rows(d1, s1);
        const uint32_t row = (uint32_t)(wm0 + 16 * i + lr);
        const int t = wn0 + 32 * jp + piece;
        if (decltype(whole)::value || (rows16 && t >= lo && t + 8 <= nt)) {
            bstore16<kStore>(r, (row * Nr + (uint32_t)(cb + t)) * 2u, make_uint4(d0, d1, s0, s1));
        } else if (row < rows_t) {
            uint16_t *dst = base + (m0 + row) * (int64_t)Nr + cb + t;
            const uint32_t w[4] = {d0, d1, s0, s1};
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (t + k >= lo && t + k < nt) dst[k] = (uint16_t)(w[k >> 1] >> (16 * (k & 1)));
        }
    };

    // slice through LDS: token rows of a.D runs of `span` columns, one per residue
    const int D = (int)a.D;
    const int span = ADD && a.unperm ? (int)pp_slice_span(D, BN) : BN, tb = ADD && a.unperm ? cb / D : 0;
    constexpr int kRound = 16 * (BM / C::WM);              // tokens per block row of all waves
    const int pitch = ADD ? (a.unperm ? (int)pp_slice_pitch(D, BN) : BN + 4) : 0;   // floats
    int at[ADD ? SN : 1][4];
    if constexpr (ADD) {
#pragma unroll
        for (int j = 0; j < SN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = wn0 + 16 * j + 4 * lg + v, c = cb + t;
                at[j][v] = a.unperm ? c % D * span + c / D - tb : t;
            }
    }
    auto slice_at = [&](int i, int j, int v) -> float {
        const uint32_t row = (uint32_t)(wm0 + 16 * i + lr);
        const int t = wn0 + 16 * j + 4 * lg + v, c = cb + t;
        if (row >= rows_t || t < lo || t >= nt) return 0.f;
        const int64_t col = a.unperm ? (int64_t)(c % D) * a.bn + c / D : (int64_t)n0 + t;
        return a.part[((int64_t)a.slice0 * a.M + m0 + row) * a.Nout + col];
    };
    // block rows staged at a time; rows of so many residues that not even one
    // fits are read in place
    const int rounds = ADD ? (int)((int64_t)(C::kLds / 4) / ((int64_t)kRound * pitch)) : SM;

    // two instances, so that the tiles inside a padded block (most of them)
    // carry nothing of the piecemeal form
    auto rows = [&](auto whole) {
#pragma unroll
    for (int i = 0; i < SM; ++i) {
        const float *row_slice = nullptr;
        if constexpr (ADD) {
            if (rounds > 0 && i % rounds == 0) {
                // stage block rows i .. i + rounds - 1 of every wave row
                if (i > 0) __syncthreads();
                const __amdgpu_buffer_rsrc_t rS =
                    buffer_rsrc(a.part + ((int64_t)a.slice0 * a.M + m0) * a.Nout, rows_t * (uint32_t)a.Nout * 4u);
                const int nr = SM - i < rounds ? SM - i : rounds;
                for (int k = 0; k < pitch / 64; ++k) {     // 64-float loads of a token row
                    const int q = 64 * k + lane;
                    uint32_t col;
                    if (a.unperm) {
                        const int r = q / span < D ? q / span : 0;
                        int t = tb + q % span;
                        t = t < (int)a.bn ? t : (int)a.bn - 1;   // places past a residue's columns are not read
                        col = (uint32_t)(r * (int)a.bn + t);
                    } else {
                        col = (uint32_t)(n0 + (q < BN ? q : 0));
                    }
                    for (int er = wave; er < kRound * nr; er += kPPWaves) {
                        // staged row er: wave row (er % kRound) / 16, block row i + er / kRound
                        const uint32_t row = (uint32_t)(er % kRound / 16 * C::WM + 16 * (i + er / kRound) + er % 16);
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(
                            rS, (__attribute__((address_space(3))) void *)(smem + (er * pitch + 64 * k) * 4), 4,
                            (int)((row * (uint32_t)a.Nout + col) * 4u), 0, 0, 0);
                    }
                }
                wait_vm<0>();
                __syncthreads();
            }
            if (rounds > 0) row_slice = reinterpret_cast<const float *>(smem) + ((i % rounds) * kRound + wm0 / C::WM * 16 + lr) * pitch;
        }
        uint4 h[SN / 2];
        if (grad) {
#pragma unroll
            for (int jp = 0; jp < SN / 2; ++jp) h[jp] = load_h(whole, i, jp);
        }
#pragma unroll
        for (int jp = 0; jp < SN / 2; ++jp) {
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int j = 2 * jp + (e >> 2), v = e & 3;
                x[e] = acc[i][j][v];
                if constexpr (ADD) {
                    if (rounds > 0) x[e] += row_slice[at[j][v]];
                    else x[e] += slice_at(i, j, v);
                }
            }
            if (grad) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] *= gelu_grad(unpack_bf16(word_of(h[jp], e >> 1), e & 1));
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] += bias[2 * jp + (e >> 2)][e & 3];
                if (act) {
                    if (keep_h) store(whole, rH, a.h_out, i, jp, x);
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = gelu(x[e]);
                }
            }
            store(whole, rO, a.out, i, jp, x);
        }
    }
    };
    if (!PAD || (rows16 && lo == 0 && nt == BN)) rows(std::true_type{});
    else if constexpr (PAD) rows(std::false_type{});
}

template <int BM, int BN, int WGM, int WGN, bool W_T, int FORM>
__global__ void __launch_bounds__(kPPThreads, 1) dyad_gemm_pp(GemmArgs a) {
    using C = PPCfg<BM, BN, WGM, WGN, W_T>;
    using SA = typename C::A;
    using SB = typename C::B;
    constexpr bool kRes = FORM == kPPRes, kOne = FORM == kPPPairOne;
    constexpr bool kPair = FORM == kPPPair || FORM == kPPPadPair || kRes || kOne;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[C::kLds];
    lds_u8 *lds = (lds_u8 *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // tiles in runs of group_m token panels, panels fastest: the workgroups
    // that run together on an XCD share both input rows and weights
    const int item = xcd_tile(blockIdx.x, a.tiles_total);
    const int tiles_m = a.tiles_total / a.tiles_n, run = a.group_m * a.tiles_n;
    const int first = item / run * a.group_m;
    const int gm = tiles_m - first < a.group_m ? tiles_m - first : a.group_m;
    const int64_t m0 = (int64_t)(first + item % run % gm) * BM;
    const int n0 = item % run / gm * BN;
    const int bk = (int)a.bk, bn = (int)a.bn, Kin = (int)a.Kin;
    const int g = n0 / bn, jb = n0 - g * bn;
    const int ks = bk / kStageK;
    // residue-major form: tile index -> block g, columns t0.. of every residue, residue r fastest
    const int D = (int)a.D;
    const int r = kRes ? n0 / BN % D : 0;
    const int t0 = kRes ? (jb / BN) / D * BN : 0;

    const int64_t rows_left = a.M - m0;
    const uint32_t a_bytes = (uint32_t)((uint64_t)(rows_left < BM ? rows_left : BM) * (uint64_t)Kin * 2u);
    const uint32_t w_bytes = (uint32_t)(a.D * a.bn * a.bk * 2);
    const __amdgpu_buffer_rsrc_t rA1 = buffer_rsrc(a.in + m0 * a.Kin, a_bytes);
    const __amdgpu_buffer_rsrc_t rA2 = kPair ? buffer_rsrc(a.in2 + m0 * a.Kin, a_bytes) : rA1;
    const __amdgpu_buffer_rsrc_t rW1 = buffer_rsrc(a.W1, w_bytes);
    const __amdgpu_buffer_rsrc_t rW2 = kPair ? buffer_rsrc(a.W2, w_bytes) : rW1;

    uint32_t voA[SA::kPer], voB[SB::kPer], loA[SA::kPer], loB[SB::kPer];
    uint32_t voA2[kRes ? SA::kPer : 1], voB2[kRes ? SB::kPer : 1];
#pragma unroll
    for (int q = 0; q < SA::kPer; ++q) {
        int row, byte;
        const int i = pp_instr(wave, q);
        pp_source<BM, false>(i, lane, row, byte);
        voA[q] = (uint32_t)row * (uint32_t)Kin * 2u + (uint32_t)(g * bk) * 2u + (uint32_t)byte;
        if constexpr (kRes) voA2[q] = (uint32_t)row * (uint32_t)Kin * 2u + (uint32_t)(r * bk) * 2u + (uint32_t)byte;
        if constexpr (kOne) voA[q] -= pp_back<BM, false>(i, lane, 0u);
        loA[q] = 1024u * (uint32_t)i;
    }
#pragma unroll
    for (int q = 0; q < SB::kPer; ++q) {
        int row, byte;
        const int i = pp_instr(wave, q);
        pp_source<BN, W_T>(i, lane, row, byte);
        if constexpr (kRes) {
            const int tg = g * (bn / D) + t0;             // weight row (column) of t = 0 in group r
            if constexpr (W_T) {
                voB[q] = ((uint32_t)(g * bk + row) * (uint32_t)bn + (uint32_t)(r * (bn / D) + t0)) * 2u + (uint32_t)byte;
                voB2[q] = ((uint32_t)(r * bk + row) * (uint32_t)bn + (uint32_t)tg) * 2u + (uint32_t)byte;
            } else {
                voB[q] = (uint32_t)(g * bn + r + D * (t0 + row)) * (uint32_t)bk * 2u + (uint32_t)byte;
                voB2[q] = (uint32_t)(r * bn + tg + row) * (uint32_t)bk * 2u + (uint32_t)byte;
            }
        } else if constexpr (W_T) voB[q] = ((uint32_t)(g * bk + row) * (uint32_t)bn + (uint32_t)jb) * 2u + (uint32_t)byte;
        else voB[q] = (uint32_t)(g * bn + jb + row) * (uint32_t)bk * 2u + (uint32_t)byte;
        if constexpr (kOne) voB[q] -= pp_back<BN, W_T>(i, lane, (uint32_t)bn * 2u);
        loB[q] = (uint32_t)C::kOffB + 1024u * (uint32_t)i;
    }
    const uint32_t stepB = W_T ? (uint32_t)(kStageK * 2) * (uint32_t)bn : (uint32_t)(kStageK * 2);
    const int nk = (ks + 1) / 2;                   // units per component; the last may hold one new step
    const int units = kPair ? 2 * nk : nk;
    // unit d: components alternate in the paired forms
    auto unit_k = [&](int d) { return kPair ? d >> 1 : d; };
    auto both = [&](int d) { return 2 * unit_k(d) + 1 < ks; };
    auto unit_step = [&](int d) { return (uint32_t)(kOne ? 0 : pp_unit_step(unit_k(d), ks)); };
    auto issue_a = [&](int d) {
        const __amdgpu_buffer_rsrc_t rs = kPair && (d & 1) ? rA2 : rA1;
        lds_u8 *slot = lds + d % C::kSlotA * SA::kBytes;
#pragma unroll
        for (int q = 0; q < SA::kPer; ++q) {
            uint32_t vo = voA[q];
            if constexpr (kRes) vo = d & 1 ? voA2[q] : vo;
            dma16(rs, slot + loA[q], vo, unit_step(d) * (uint32_t)(kStageK * 2));
        }
    };
    auto issue_b = [&](int d) {
        const __amdgpu_buffer_rsrc_t rs = kPair && (d & 1) ? rW2 : rW1;
        lds_u8 *slot = lds + d % C::kSlotB * SB::kBytes;
#pragma unroll
        for (int q = 0; q < SB::kPer; ++q) {
            uint32_t vo = voB[q];
            if constexpr (kRes) vo = d & 1 ? voB2[q] : vo;
            dma16(rs, slot + loB[q], vo, unit_step(d) * stepB);
        }
    };
    const int wm0 = (wave / WGN) * C::WM, wn0 = (wave % WGN) * C::WN;
    uint32_t fb[W_T ? C::kSubN : 1];
    const uint32_t base = (uint32_t)(uintptr_t)lds;
    const uint32_t fa = base + pp_frag<BM, false>(wm0, 0, lane);
#pragma unroll
    for (int j = 0; j < (W_T ? C::kSubN : 1); ++j)
        fb[j] = base + (uint32_t)C::kOffB + pp_frag<BN, W_T>(wn0, j, lane);
    auto addr = [&](int d, int h, uint32_t &pa, uint32_t (&pb)[W_T ? C::kSubN : 1]) {
        pa = pp_step<BM, false>(fa + (uint32_t)(d % C::kSlotA * SA::kBytes), h);
#pragma unroll
        for (int j = 0; j < (W_T ? C::kSubN : 1); ++j)
            pb[j] = pp_step<BN, W_T>(fb[j] + (uint32_t)(d % C::kSlotB * SB::kBytes), h);
    };

    f32x4_t acc[C::kSubM][C::kSubN];
#pragma unroll
    for (int i = 0; i < C::kSubM; ++i)
#pragma unroll
        for (int j = 0; j < C::kSubN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    pp_loop<C::kSubM, C::kSubN, W_T, 4 * SB::kPitch, SA::kPer, SB::kPer, C::kSlotA, C::kSlotB>(
        units, wave, acc, issue_a, issue_b, addr, both);
    const int no = kRes ? r * (int)(a.Nout / a.D) + g * (bn / D) + t0 : n0;
    pp_epilogue<C, BM, BN, FORM == kPPSlice, FORM == kPPAdd || FORM == kPPPadAdd,
                FORM == kPPPadAdd || FORM == kPPPadPair, kRes>(a, smem, acc, m0, no, g, jb, rows_left, lane, wave, wm0,
                                                               wn0, g * bn + r + D * t0);
}

template <int BM, int BN, int WGM, int WGN, bool W_T, int FORM>
hipError_t launch_pp_tile(GemmArgs a, hipStream_t s) {
    const int64_t tiles_m = (a.M + BM - 1) / BM, tiles_n = a.Nout / BN;
    if (!pp_fits(BM, a.Kin, a.Nout, a.D * a.bn * a.bk) || tiles_m * tiles_n >= ((int64_t)1 << 31))
        return hipErrorNotSupported;
    if ((a.bk < kPPK) != (FORM == kPPPairOne)) return hipErrorNotSupported;
    if (FORM == kPPRes && (a.bn % a.D != 0 || a.bn / a.D % BN != 0)) return hipErrorNotSupported;
    a.tiles_n = (int)tiles_n;
    a.tiles_total = (int)(tiles_m * tiles_n);
    a.splits = 1;
    // About 32 workgroups run together on an XCD: group_m token panels of 32 /
    // group_m column tiles.  Column tiles of one output block read the same
    // input block; with blocks of two to four tiles 8 panels share more.
    const int64_t per_block = a.bn / BN;
    a.group_m = per_block >= 2 && per_block < 8 ? 8 : 4;
    dyad_gemm_pp<BM, BN, WGM, WGN, W_T, FORM><<<a.tiles_total, kPPThreads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace dyad
