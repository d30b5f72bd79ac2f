// The pipelined multiply loop shared by the large matrix-core kernels: an
// eight-wave workgroup multiplies a BM x BN tile out of LDS rings that
// global-to-LDS loads fill, with no staging registers in between.
//
// Units.  The reduction runs in units of 64 indices (two MFMA steps) of one
// operand pair.  A side whose reduction index is contiguous in memory (rows of
// input or untransposed weights) is staged as N rows of 128 bytes, their eight
// 16-byte chunks XORed by (row >> 1) & 7; a side whose reduction index is the
// row (weights read transposed) is staged in its natural layout, 64 rows of N
// columns, 32-byte chunks swizzled by tr_swz, and read with ds_read_b64_tr_b16.
// A global-to-LDS load writes 64 x 16 consecutive bytes, so both swizzles are
// applied to the lane's source address.  Rows of 128 bytes are whole cache
// lines: with 64-byte rows (32 indices) half of every line fetched from the L2
// is evicted before its turn (measured on gfx950, all CUs reading a 2.4 MB panel
// column by column: 16 against 35 TB/s).  Each side has a ring of two or three slots, so a load
// has one or two units of matrix work (1 - 2 us) to arrive.
//
// Ping-pong.  Waves w and w + 4 share a SIMD.  The two halves of the workgroup
// run the same loop one phase apart: while one half reads the fragments of an
// MFMA step from LDS and issues loads, the other half multiplies, so LDS
// reads, load issue and waits sit behind the partner's matrix work.  With unit
// d taking phases 4d .. 4d + 3 of half 0 (read, multiply, read, multiply) and
// 4d + 1 .. 4d + 4 of half 1, one barrier between phases:
//   - every wave waits for its own loads of unit d + 1 before the barrier that
//     ends phase 4d + 3, so unit d + 1 is complete before anyone reads it;
//   - loads issued in a wave's first phase of unit d overwrite slots of unit
//     d - 1, whose last reads (half 1, phase 4d - 1) completed before the
//     barrier that ends that phase.
//
// The fragment reads are one block of instructions that ends in its own wait:
// the compiler orders an LDS read behind every global-to-LDS load in flight
// (it cannot tell the slots apart), which would drain the ring each unit.
#pragma once

#include <type_traits>

#include "mfma_common.h"

namespace dyad {

constexpr int kPPWaves = 8, kPPThreads = 64 * kPPWaves;
constexpr int kPPK = 64;   // reduction indices per unit

// One operand side of a unit: N tile rows or columns.  TR: 64 rows (reduction
// indices) of N columns; else N rows of 64 reduction indices.
template <int N, bool TR>
struct PPSide {
    static constexpr int kPitch = TR ? round256(2 * N) : 2 * kPPK;
    static constexpr int kBytes = (TR ? kPPK : N) * kPitch;
    static constexpr int kInstr = kBytes / 1024;        // 1 KB wave loads
    static constexpr int kPer = kInstr / kPPWaves;      // per wave
    static_assert(kBytes % 1024 == 0 && kInstr % kPPWaves == 0, "whole wave loads, the same number for each wave");
};

// Wave load q of wave `wave`.
__host__ __device__ constexpr int pp_instr(int wave, int q) { return wave + kPPWaves * q; }

// Source of lane `lane` of wave load i: tile row (or reduction row with TR)
// and the byte within that row.  (TR rows padded to 256 bytes: lanes in the
// padding load column 0, which nothing reads.)
template <int N, bool TR>
__host__ __device__ __forceinline__ void pp_source(int i, int lane, int &row, int &byte) {
    if constexpr (!TR) {
        row = 8 * i + (lane >> 3);
        byte = ((lane ^ (row >> 1)) & 7) * 16;
    } else {
        constexpr int P = PPSide<N, TR>::kPitch;
        const int at = 1024 * i + 16 * lane;
        row = at / P;
        byte = tr_swz(tr_sw(row), at % P);
        if constexpr (2 * N != P) byte = byte < 2 * N ? byte : 0;
    }
}

// First of the two steps that unit k of a reduction of ks >= 2 steps loads.
// Where ks is odd the last unit holds one new step, its second, behind the step
// before: a unit that began at its only step would load past the block (past the
// tensor for the last one, and a buffer's range check does not see the scalar
// offset).  Units past the last load it again.
__host__ __device__ constexpr int pp_unit_step(int k, int ks) { return 2 * k < ks - 2 ? 2 * k : ks - 2; }

// A reduction of one step has no step before it: the lanes of the second half
// step back by these bytes and load the first's again (pitch: bytes between the
// source rows).  The step to multiply is the second here too.
template <int N, bool TR>
__host__ __device__ constexpr uint32_t pp_back(int i, int lane, uint32_t pitch) {
    if constexpr (!TR) return (uint32_t)(((lane >> 2) ^ i) & 1) * 64u;   // bit 2 of the lane's chunk
    else return 2 * i >= PPSide<N, TR>::kInstr ? (uint32_t)kStageK * pitch : 0u;
}

// LDS byte (within the side) of the lane's fragment s of a wave whose rows or
// columns start at w0, first MFMA step of the unit.  Without TR consecutive
// fragments are 16 rows apart.
template <int N, bool TR>
__device__ __forceinline__ uint32_t pp_frag(int w0, int s, int lane) {
    if constexpr (!TR) {
        const int lr = lane & 15, lc = lane >> 4;
        return (uint32_t)((w0 + 16 * s + lr) * 128 + ((lc ^ (lr >> 1)) & 7) * 16);
    } else {
        const int trow = 8 * (lane >> 4) + ((lane & 15) >> 2), tcol = 4 * (lane & 3);
        return (uint32_t)(trow * PPSide<N, TR>::kPitch + tr_swz(tr_sw(trow), (w0 + 16 * s + tcol) * 2));
    }
}

// The same address for step h (0 or 1) of the unit: the chunk index differs in
// bit 2, or the rows in 32.
template <int N, bool TR>
__device__ __forceinline__ uint32_t pp_step(uint32_t at, int h) {
    if constexpr (!TR) return at ^ (uint32_t)(h * 64);
    else return at + (uint32_t)(h * kStageK * PPSide<N, TR>::kPitch);
}

__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, lds_u8 *dst, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, (int)voff, (int)soff,
                                             0, 0);
}

template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ void pp_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// ---- fragment reads: SM fragments of side A and SN of side B ----------------
#define PP_RA(i, off) "ds_read_b128 %[a" #i "], %[pa] offset:" #off "\n\t"
#define PP_RB(i, off) "ds_read_b128 %[b" #i "], %[pb] offset:" #off "\n\t"
#define PP_TB(i) "ds_read_b64_tr_b16 %[bl" #i "], %[pb" #i "]\n\tds_read_b64_tr_b16 %[bh" #i "], %[pb" #i "] offset:%[sb]\n\t"
#define PP_OA(i) [a##i] "=&v"(a[i])
#define PP_OB(i) [b##i] "=&v"(b[i])
#define PP_OTB(i) [bl##i] "=&v"(bl[i]), [bh##i] "=&v"(bh[i])
#define PP_IB(i) [pb##i] "v"(pb[i])
#define PP_RA2 PP_RA(0, 0) PP_RA(1, 2048)
#define PP_RA4 PP_RA(0, 0) PP_RA(1, 2048) PP_RA(2, 4096) PP_RA(3, 6144)
#define PP_RA8 PP_RA4 PP_RA(4, 8192) PP_RA(5, 10240) PP_RA(6, 12288) PP_RA(7, 14336)
#define PP_RB2 PP_RB(0, 0) PP_RB(1, 2048)
#define PP_RB4 PP_RB2 PP_RB(2, 4096) PP_RB(3, 6144)
#define PP_RB6 PP_RB4 PP_RB(4, 8192) PP_RB(5, 10240)
#define PP_TB2 PP_TB(0) PP_TB(1)
#define PP_TB4 PP_TB2 PP_TB(2) PP_TB(3)
#define PP_TB6 PP_TB4 PP_TB(4) PP_TB(5)
#define PP_OA2 PP_OA(0), PP_OA(1)
#define PP_OA4 PP_OA(0), PP_OA(1), PP_OA(2), PP_OA(3)
#define PP_OA8 PP_OA4, PP_OA(4), PP_OA(5), PP_OA(6), PP_OA(7)
#define PP_OB2 PP_OB(0), PP_OB(1)
#define PP_OB4 PP_OB2, PP_OB(2), PP_OB(3)
#define PP_OB6 PP_OB4, PP_OB(4), PP_OB(5)
#define PP_OTB2 PP_OTB(0), PP_OTB(1)
#define PP_OTB4 PP_OTB2, PP_OTB(2), PP_OTB(3)
#define PP_OTB6 PP_OTB4, PP_OTB(4), PP_OTB(5)
#define PP_IB2 PP_IB(0), PP_IB(1)
#define PP_IB4 PP_IB2, PP_IB(2), PP_IB(3)
#define PP_IB6 PP_IB4, PP_IB(4), PP_IB(5)
#define PP_WAIT "s_waitcnt lgkmcnt(0)"
// B first, then A: the multiplies walk A within one B
#define PP_READ_RR(NA, NB)                                                                                     \
    asm volatile(PP_RB##NB PP_RA##NA PP_WAIT : PP_OA##NA, PP_OB##NB : [pa] "v"(pa), [pb] "v"(pb[0]) : "memory")
#define PP_READ_RT(NA, NB)                                                                                     \
    asm volatile(PP_TB##NB PP_RA##NA PP_WAIT                                                                   \
                 : PP_OA##NA, PP_OTB##NB                                                                       \
                 : [pa] "v"(pa), PP_IB##NB, [sb] "n"(SB)                                                       \
                 : "memory")
#define PP_CASE(NA, NB)                                                                                        \
    if constexpr (SM == NA && SN == NB) {                                                                      \
        if constexpr (!TB) PP_READ_RR(NA, NB);                                                                 \
        else PP_READ_RT(NA, NB);                                                                               \
    }

// pa / pb: LDS addresses of the fragments (side A's and, without TB, side B's
// are 16 rows apart from the first); SB: bytes from a transposed fragment's
// first four rows to its next four.
template <int SM, int SN, bool TB, int SB>
__device__ __forceinline__ void pp_read(uint32_t pa, const uint32_t (&pb)[TB ? SN : 1], bf16x8_t (&a)[SM],
                                        bf16x8_t (&b)[SN]) {
    bf16x4_t bl[SN], bh[SN];
    PP_CASE(8, 4)
    PP_CASE(4, 6)
    PP_CASE(4, 4)
    PP_CASE(4, 2)
    PP_CASE(2, 2)
    static_assert((SM == 8 && SN == 4) || (SM == 4 && (SN == 6 || SN == 4 || SN == 2)) || (SM == 2 && SN == 2),
                  "a fragment read exists");
    if constexpr (TB) {
#pragma unroll
        for (int j = 0; j < SN; ++j) b[j] = __builtin_shufflevector(bl[j], bh[j], 0, 1, 2, 3, 4, 5, 6, 7);
    }
}

// The loop over `units` units (at least one).  issue_a(d) / issue_b(d) start
// the wave's NVA / NVB loads of unit d's sides into slots d % SLOTA and
// d % SLOTB (for d >= units they load a valid unit again: its slot is never
// read); addr(d, h, pa, pb) gives the fragment addresses of step h;
// both(d) says whether unit d has two steps to multiply, or the second alone.
// LDS is free, and no load is in flight, when it returns (after a barrier).
// Side B's fragments are the first MFMA operand, so a lane's four sums lie
// along side B (4 (l / 16) + v) at row l % 16 of side A.
template <int SM, int SN, bool TB, int SB, int NVA, int NVB, int SLOTA, int SLOTB, class IssueA, class IssueB,
          class Addr, class Both>
__device__ __forceinline__ void pp_loop(int units, int wave, f32x4_t (&acc)[SM][SN], IssueA issue_a, IssueB issue_b,
                                        Addr addr, Both both) {
    bf16x8_t a[SM], b[SN];
    uint32_t pa, pb[TB ? SN : 1];
    const bool half = wave >= kPPWaves / 2;
    // loads still allowed in flight when unit d + 1 must have arrived, after
    // unit d's issues (B of unit d + SLOTB - 1, then A of unit d + SLOTA - 1)
    constexpr int kLeft = (SLOTA - 2) * NVA + (SLOTB - 2) * NVB;
    static_assert(SLOTA >= SLOTB && SLOTB >= 2 && SLOTA <= 3, "A runs at least as far ahead as B");
    issue_a(0);
    issue_b(0);
    if constexpr (SLOTB == 3) issue_b(1);
    if constexpr (SLOTA == 3) issue_a(1);
    wait_vm<kLeft>();
    pp_barrier();
    if (half) pp_barrier();
    auto multiply = [&]() {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int j = 0; j < SN; ++j)
#pragma unroll
            for (int i = 0; i < SM; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
    };
    for (int d = 0; d < units; ++d) {
        issue_b(d + SLOTB - 1);
        addr(d, 0, pa, pb);
        pp_read<SM, SN, TB, SB>(pa, pb, a, b);
        pp_barrier();
        if (both(d)) multiply();
        pp_barrier();
        issue_a(d + SLOTA - 1);
        addr(d, 1, pa, pb);
        pp_read<SM, SN, TB, SB>(pa, pb, a, b);
        if (half) wait_vm<kLeft>();
        pp_barrier();
        multiply();
        if (!half) wait_vm<kLeft>();
        pp_barrier();
    }
    if (!half) pp_barrier();
    wait_vm<0>();
    pp_barrier();
}

}  // namespace dyad
