// fp32 passes on the fp32 matrix instructions (v_mfma_f32_16x16x4_f32), for
// widths that n_dyad divides into blocks of a multiple of 4.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s, twice the vector FMA
// rate without packed forms).  A 128 x 128 tile on four waves of 64 x 64 does
// 64 of those instructions (32 cycles each) per 16 reduction indices against
// 8 LDS reads, so operand traffic is small and a plain double-buffered loop
// with two workgroups per CU suffices.  The decomposition is that of the
// general kernels: a tile's columns lie in one class (g1, g2) of output
// columns, which read the same two input slabs; the weight gradient has one
// product per (component, group), split over the tokens.
//
// Operands.  LDS holds both sides reduction-fastest, rows of 32 values (128
// bytes, whole cache lines of the source) with their 16-byte chunks XORed by
// (row >> 1) & 7.  Each lane reads 4 consecutive reduction indices of one row
// with one 16-byte read and feeds element s to MFMA step s; lane group lg
// holds indices 4 lg + s of both sides, which is all the instruction needs.
// A side is loaded by its strides: along the reduction (16 bytes at a time
// where it is contiguous, else one value at a time), or along the row index
// (16 bytes at a time, transposed on the way into LDS).
//
// Measured on gfx950 against the vector kernels (which keep the other shapes),
// 768 -> 3072, n_dyad 4, 4096 tokens, Dyad-IT: forward 259 -> 128 us (75
// TFLOP/s), input gradient 441 -> 137, weight gradient 212 -> 140.
#include <type_traits>

#include "dyad_device.h"
#include "dyad_internal.h"
#include "mfma_common.h"

namespace dyad {
namespace {

constexpr int kFK = 32;          // reduction indices per stage
constexpr int kFThreads = 256;

// One side of one component: element (row, k) at base + row * rs + k * ks
// (in floats).  kind 0: ks == 1, 16-byte loads along k; 1: one value at a
// time, k fastest over the lanes; 2: rs == 1, 16-byte loads along the rows;
// 3: one value at a time, rows fastest over the lanes.
struct FSide {
    const float *base;
    int64_t rs, ks;
};

// A tile's side of N rows, `rows` of them real.  Thread t's piece q sits a
// fixed number of rows or reduction indices after its piece 0, so a stage
// needs one offset per thread and scalar steps.
template <int N, int KIND>
struct FLoader {
    static constexpr int kPer = N * kFK / (4 * kFThreads);   // 16-byte pieces per thread
    float4 r[kPer];

    // Stage of reduction indices k0 .. k0 + 31 below k_end.
    __device__ __forceinline__ void fetch(const FSide &s, int tid, int64_t k0, int64_t k_end, int rows) {
        // range checks below go through kNoLoad; the stage's own offsets stay below 2^31
        const __amdgpu_buffer_rsrc_t b = buffer_rsrc(s.base + k0 * s.ks, 0x7ffffffcu);
        const int left = (int)(k_end - k0 < kFK ? k_end - k0 : kFK);
        const uint32_t rs = (uint32_t)s.rs * 4u, ks = (uint32_t)s.ks * 4u;
        if constexpr (KIND == 0) {
            const int row = tid >> 3, k = (tid & 7) * 4;
            const uint32_t vo = (uint32_t)row * rs + (uint32_t)k * 4u;
#pragma unroll
            for (int q = 0; q < kPer; ++q)
                r[q] = load16(b, row + 32 * q < rows && k < left ? vo : kNoLoad, 32u * q * rs);
        } else if constexpr (KIND == 2) {
            const int row = tid % (N / 4) * 4, k = tid / (N / 4);
            const uint32_t vo = (uint32_t)row * 4u + (uint32_t)k * ks;
            constexpr int kStep = 4 * kFThreads / N;
#pragma unroll
            for (int q = 0; q < kPer; ++q)
                r[q] = load16(b, row < rows && k + kStep * q < left ? vo : kNoLoad, (uint32_t)(kStep * q) * ks);
        } else {
            constexpr bool kf = KIND == 1;
            const int row = kf ? tid / kFK : tid % N, k = kf ? tid % kFK : tid / N;
            const uint32_t vo = (uint32_t)row * rs + (uint32_t)k * ks;
            constexpr int dr = kf ? kFThreads / kFK : 0 , dk = kf ? 0 : kFThreads / N;
            const uint32_t step = (uint32_t)dr * rs + (uint32_t)dk * ks;
            float v[4 * kPer];
#pragma unroll
            for (int n = 0; n < 4 * kPer; ++n)
                v[n] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    b, (int)(row + dr * n < rows && k + dk * n < left ? vo : kNoLoad), (int)(step * (uint32_t)n), 0));
#pragma unroll
            for (int q = 0; q < kPer; ++q) r[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
    }
    static __device__ __forceinline__ float4 load16(__amdgpu_buffer_rsrc_t b, uint32_t vo, uint32_t so) {
        const uint4 v = bload16(b, vo, so);
        return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    }
    static __device__ __forceinline__ int at(int row, int k) {   // float offset in LDS
        return row * kFK + (((k >> 2) ^ (row >> 1)) & 7) * 4 + (k & 3);
    }
    __device__ __forceinline__ void stash(int tid, float *lds) const {
        if constexpr (KIND == 0) {
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int i = tid + q * kFThreads;
                *reinterpret_cast<float4 *>(lds + at(i >> 3, (i & 7) * 4)) = r[q];
            }
        } else if constexpr (KIND == 2) {
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int i = tid + q * kFThreads, row = i % (N / 4) * 4, k = i / (N / 4);
                lds[at(row, k)] = r[q].x;
                lds[at(row + 1, k)] = r[q].y;
                lds[at(row + 2, k)] = r[q].z;
                lds[at(row + 3, k)] = r[q].w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const float v[4] = {r[q].x, r[q].y, r[q].z, r[q].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = tid + (q * 4 + e) * kFThreads;
                    const int row = KIND == 1 ? i / kFK : i % N, k = KIND == 1 ? i % kFK : i / N;
                    lds[at(row, k)] = v[e];
                }
            }
        }
    }
};

// acc[j][i]: a lane's four sums are columns 16 j + 4 (l / 16) + v of side B at
// row 16 i + l % 16 of side A, over reduction indices k_lo .. k_hi - 1.  perm:
// column 4 v + lg stands where 4 lg + v is meant (16-column blocks transposed
// as 4 x 4), so that lanes lg = 0..3 hold consecutive columns.  KA, KB: the
// sides' kinds.  DB: with do_db, dacc[i] also gets row 16 i + l % 16's sum.
template <int BM, int BN, int SM, int SN, int KA, int KB, bool DB>
__device__ __forceinline__ void f32_loop(const FSide &sa, const FSide &sb, int64_t k_lo, int64_t k_hi, int rows_a,
                                         int rows_b, bool perm, bool do_db, float *lds, f32x4_t (&acc)[SN][SM],
                                         f32x4_t (&dacc)[DB ? SM : 1], int wm0, int wn0) {
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    constexpr int kBuf = (BM + BN) * kFK;
    using LA = FLoader<BM, KA>;
    using LB = FLoader<BN, KB>;
    LA la;
    LB lb;
    const int stages = (int)((k_hi - k_lo + kFK - 1) / kFK);
    if (stages <= 0) return;
    auto fetch = [&](int st) {
        const int64_t k0 = k_lo + (int64_t)st * kFK;
        la.fetch(sa, tid, k0, k_hi, rows_a);
        lb.fetch(sb, tid, k0, k_hi, rows_b);
    };
    auto stash = [&](int st) {
        float *buf = lds + (st & 1) * kBuf;
        la.stash(tid, buf);
        lb.stash(tid, buf + BM * kFK);
    };
    const int pr = perm ? (lr & 3) * 4 + (lr >> 2) : lr;
    fetch(0);
    stash(0);
    __syncthreads();
    for (int st = 0; st < stages; ++st) {
        if (st + 1 < stages) fetch(st + 1);
        const float *bufA = lds + (st & 1) * kBuf, *bufB = bufA + BM * kFK;
#pragma unroll
        for (int h = 0; h < kFK / 16; ++h) {
            f32x4_t a[SM], b[SN];
#pragma unroll
            for (int i = 0; i < SM; ++i)
                a[i] = *reinterpret_cast<const f32x4_t *>(bufA + LA::at(wm0 + 16 * i + lr, 16 * h + 4 * lg));
#pragma unroll
            for (int j = 0; j < SN; ++j)
                b[j] = *reinterpret_cast<const f32x4_t *>(bufB + LB::at(wn0 + 16 * j + pr, 16 * h + 4 * lg));
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < SN; ++j)
#pragma unroll
                    for (int i = 0; i < SM; ++i)
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][s], a[i][s], acc[j][i], 0, 0, 0);
            if constexpr (DB) {
                if (do_db) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int i = 0; i < SM; ++i)
                            dacc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, a[i][s], dacc[i], 0, 0, 0);
                }
            }
        }
        if (st + 1 < stages) stash(st + 1);
        __syncthreads();
    }
}

template <int BM, int BN, bool IN_T, bool OUT_T, bool W_T>
__global__ void __launch_bounds__(kFThreads, 2) f32_gemm_kernel(GemmPass p, int col_tiles) {
    constexpr int SM = BM / 32, SN = BN / 32;      // 2 x 2 waves
    __shared__ __attribute__((aligned(16))) float lds[2 * (BM + BN) * kFK];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    // the classes and column tiles of one token panel run next to each other
    const int per_row = (int)(OUT_T ? p.D * p.D : p.D) * col_tiles;
    const int rt = b / per_row, cls = b % per_row / col_tiles, ct = b % col_tiles;
    const int D = (int)p.D;
    // widths divide evenly: under an output transpose the class's columns are
    // the f of block g1 with f % D == g2, D apart
    const int64_t bk = p.bk, bn = p.bn;
    const int g1 = OUT_T ? cls / D : cls, g2 = OUT_T ? cls % D : cls;
    const int64_t lo = g1 * bn;
    const int64_t first = OUT_T ? lo + ((g2 - lo) % D + D) % D : lo;
    const int64_t step = OUT_T ? D : 1;
    const int64_t count = first < lo + bn ? (lo + bn - first + step - 1) / step : 0;
    const int64_t t0 = (int64_t)ct * BN, m0 = (int64_t)rt * BM;
    if (t0 >= count) return;                       // uniform
    const int rows_a = (int)(p.M - m0 < BM ? p.M - m0 : BM), rows_b = (int)(count - t0 < BN ? count - t0 : BN);
    const float *in = static_cast<const float *>(p.in) + m0 * p.Kin;
    const float *W1 = static_cast<const float *>(p.W1), *W2 = static_cast<const float *>(p.W2);
    const int64_t f0 = first + t0 * step, j1 = f0 - lo, j2 = OUT_T ? f0 / D : j1;
    f32x4_t acc[SN][SM], none[1];
#pragma unroll
    for (int j = 0; j < SN; ++j)
#pragma unroll
        for (int i = 0; i < SM; ++i) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int wm0 = (wave >> 1) * (BM / 2), wn0 = (wave & 1) * (BN / 2);
    const bool perm = OUT_T;
    // kinds: weights read transposed run along the columns, D apart in
    // component 1 under an output transpose (whose component 2 columns start
    // anywhere, so they go one at a time too)
    constexpr int kW = !W_T ? 0 : OUT_T ? 3 : 2;
    const FSide w1 = W_T ? FSide{W1 + g1 * bk * bn + j1, step, bn} : FSide{W1 + (g1 * bn + j1) * bk, step * bk, 1};
    const FSide w2 = W_T ? FSide{W2 + g2 * bk * bn + j2, 1, bn} : FSide{W2 + (g2 * bn + j2) * bk, bk, 1};
    f32_loop<BM, BN, SM, SN, 0, kW, false>(FSide{in + g1 * bk, p.Kin, 1}, w1, 0, bk, rows_a, rows_b, perm, false, lds,
                                           acc, none, wm0, wn0);
    f32_loop<BM, BN, SM, SN, IN_T ? 1 : 0, kW, false>(IN_T ? FSide{in + g2, p.Kin, D} : FSide{in + g2 * bk, p.Kin, 1},
                                                      w2, 0, bk, rows_a, rows_b, perm, false, lds, acc, none, wm0, wn0);

    const int lr = lane & 15, lg = lane >> 4;
    float *out = static_cast<float *>(p.out);
    const float *bias = static_cast<const float *>(p.bias), *h_in = static_cast<const float *>(p.h_in);
    float *h_out = static_cast<float *>(p.h_out);
    const bool grad = p.epilogue == kEpiGeluGrad, act = p.epilogue == kEpiBiasGelu;
    const bool vec = step == 1;   // blocks of a multiple of 4 columns
#pragma unroll
    for (int i = 0; i < SM; ++i) {
        const int row = wm0 + 16 * i + lr;
        if (row >= rows_a) continue;
        const int64_t at = (m0 + row) * p.Nout;
#pragma unroll
        for (int j = 0; j < SN; ++j) {
            const int tb = wn0 + 16 * j;
            float x[4];
            bool ok[4];
            int64_t e[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = tb + (perm ? 4 * v + lg : 4 * lg + v);
                ok[v] = t < rows_b;
                e[v] = at + f0 + t * step;
                x[v] = acc[j][i][v];
            }
            if (vec && ok[3]) {
                if (grad) {
                    const float4 hv = *reinterpret_cast<const float4 *>(h_in + e[0]);
                    x[0] *= gelu_grad_f32(hv.x); x[1] *= gelu_grad_f32(hv.y);
                    x[2] *= gelu_grad_f32(hv.z); x[3] *= gelu_grad_f32(hv.w);
                } else {
                    if (bias) {
                        const float4 bv = *reinterpret_cast<const float4 *>(bias + (e[0] - at));
                        x[0] += bv.x; x[1] += bv.y; x[2] += bv.z; x[3] += bv.w;
                    }
                    if (act) {
                        if (h_out) *reinterpret_cast<float4 *>(h_out + e[0]) = make_float4(x[0], x[1], x[2], x[3]);
#pragma unroll
                        for (int v = 0; v < 4; ++v) x[v] = gelu_f32(x[v]);
                    }
                }
                *reinterpret_cast<float4 *>(out + e[0]) = make_float4(x[0], x[1], x[2], x[3]);
                continue;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (!ok[v]) continue;
                if (grad) {
                    x[v] *= gelu_grad_f32(h_in[e[v]]);
                } else {
                    if (bias) x[v] += bias[e[v] - at];
                    if (act) {
                        if (h_out) h_out[e[v]] = x[v];
                        x[v] = gelu_f32(x[v]);
                    }
                }
                out[e[v]] = x[v];
            }
        }
    }
}

template <int BJ, int BK, bool IN_T, bool OUT_T>
__global__ void __launch_bounds__(kFThreads, 2) f32_dw_kernel(DwPass p, int jt_n, int kt_n, int splits, int64_t tps,
                                                              float *part) {
    constexpr int SM = BJ / 32, SN = BK / 32;
    __shared__ __attribute__((aligned(16))) float lds[2 * (BJ + BK) * kFK];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const int D = (int)p.D;
    const int kt = b % kt_n, jt = b / kt_n % jt_n, gc = b / (kt_n * jt_n) % (2 * D), split = b / (kt_n * jt_n * 2 * D);
    const int comp = gc < D ? 1 : 2, g = gc % D;
    const int64_t m_lo = split * tps, m_hi = m_lo + tps < p.M ? m_lo + tps : p.M;
    const int j0 = jt * BJ, k0 = kt * BK;
    const int rows_a = (int)(p.bo - j0 < BJ ? p.bo - j0 : BJ), rows_b = (int)(p.bi - k0 < BK ? p.bi - k0 : BK);
    const float *dZ = static_cast<const float *>(p.dZ), *X = static_cast<const float *>(p.X);
    f32x4_t acc[SN][SM], dacc[SM];
#pragma unroll
    for (int i = 0; i < SM; ++i) {
        dacc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < SN; ++j) acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    const int wm0 = (wave >> 1) * (BJ / 2), wn0 = (wave & 1) * (BK / 2);
    const bool db = p.db && comp == 1 && kt == 0, my_db = db && (wave & 1) == 0;
    const FSide z1{dZ + g * p.bo + j0, 1, p.n_out}, x1{X + g * p.bi + k0, 1, p.n_in};
    if (comp == 1)
        f32_loop<BJ, BK, SM, SN, 2, 2, true>(z1, x1, m_lo, m_hi, rows_a, rows_b, false, my_db, lds, acc, dacc, wm0, wn0);
    else
        f32_loop<BJ, BK, SM, SN, OUT_T ? 3 : 2, IN_T ? 3 : 2, true>(
            OUT_T ? FSide{dZ + (int64_t)j0 * D + g, D, p.n_out} : z1, IN_T ? FSide{X + (int64_t)k0 * D + g, D, p.n_in} : x1,
            m_lo, m_hi, rows_a, rows_b, false, false, lds, acc, dacc, wm0, wn0);

    const int lr = lane & 15, lg = lane >> 4;
    const int64_t per_comp = p.D * p.bo * p.bi;
    float *dst = part ? part + split * 2 * per_comp + (comp - 1) * per_comp
                      : static_cast<float *>(comp == 1 ? p.dW1 : p.dW2);
    float *dst_db = part ? part + splits * 2 * per_comp + split * p.n_out : static_cast<float *>(p.db);
#pragma unroll
    for (int i = 0; i < SM; ++i) {
        const int j = wm0 + 16 * i + lr;
        if (j >= rows_a) continue;
        if (my_db && lg == 0) dst_db[g * p.bo + j0 + j] = dacc[i][0];
        float *row = dst + (g * p.bo + j0 + j) * p.bi + k0;
#pragma unroll
        for (int jj = 0; jj < SN; ++jj) {
            const int k = wn0 + 16 * jj + 4 * lg;
            if (k + 4 <= rows_b) {               // blocks are multiples of 4
                *reinterpret_cast<f32x4_t *>(row + k) = acc[jj][i];
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (k + v < rows_b) row[k + v] = acc[jj][i][v];
            }
        }
    }
}

}  // namespace

// Blocks of a multiple of 4 that n_dyad divides the widths into: rows of
// weights and gradients are then whole 16-byte pieces.
bool f32_mfma_ok(int64_t n_a, int64_t n_b, int64_t D, int64_t ba, int64_t bb) {
    return n_a == D * ba && n_b == D * bb && ba % 4 == 0 && bb % 4 == 0 && D < 32768;
}

hipError_t launch_f32_gemm(const GemmPass &p, hipStream_t s) {
    if (p.dtype != kF32 || p.M == 0 || !f32_mfma_ok(p.Kin, p.Nout, p.D, p.bk, p.bn)) return hipErrorNotSupported;
    // a tile's 32-bit offsets: 128 input rows; 32 transposed weight rows, or 128 rows D blocks apart
    const int64_t lim = (int64_t)1 << 31;
    if (128 * p.Kin * 4 >= lim || 32 * p.bn * 4 >= lim || 128 * p.D * p.bk * 4 >= lim) return hipErrorNotSupported;
    const int64_t classes = p.out_t ? p.D * p.D : p.D;
    const int64_t per_class = p.out_t ? (p.bn + p.D - 1) / p.D : p.bn;
    // 64-column tiles where a class (the columns of one block and residue)
    // pads 128-column ones by more, or where those leave CUs without a tile
    const int64_t t128 = (per_class + 127) / 128, t64 = (per_class + 63) / 64, rt = (p.M + 127) / 128;
    const bool wide = t64 * 64 > t128 * 128 - 64 && classes * t128 * rt >= 256;
    const int64_t col_tiles = wide ? t128 : t64;
    const int64_t blocks = classes * col_tiles * rt;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorNotSupported;
    auto go = [&](auto in_t, auto out_t, auto w_t) {
        constexpr bool I = decltype(in_t)::value, O = decltype(out_t)::value, W = decltype(w_t)::value;
        if (wide) f32_gemm_kernel<128, 128, I, O, W><<<(unsigned)blocks, kFThreads, 0, s>>>(p, (int)col_tiles);
        else f32_gemm_kernel<128, 64, I, O, W><<<(unsigned)blocks, kFThreads, 0, s>>>(p, (int)col_tiles);
        return hipGetLastError();
    };
    auto with = [&](auto w) {
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        return p.in_t ? (p.out_t ? go(yes, yes, w) : go(yes, no, w)) : (p.out_t ? go(no, yes, w) : go(no, no, w));
    };
    return p.w_t ? with(std::true_type{}) : with(std::false_type{});
}

hipError_t launch_f32_dw_tiles(const DwPass &p, int64_t splits, int64_t tps, float *part, hipStream_t s) {
    if (p.dtype != kF32 || !f32_mfma_ok(p.n_in, p.n_out, p.D, p.bi, p.bo)) return hipErrorNotSupported;
    if (32 * (p.n_in > p.n_out ? p.n_in : p.n_out) * 4 >= (int64_t)1 << 31) return hipErrorNotSupported;
    // 128-wide tiles only where they pad nothing more than 64-wide ones
    const int64_t jw = (p.bo + 63) / 64 % 2 == 0 ? 128 : 64;
    const bool wide = (p.bi + 63) / 64 % 2 == 0;
    const int64_t kw = wide ? 128 : 64;
    const int64_t jt = (p.bo + jw - 1) / jw, kt = (p.bi + kw - 1) / kw, blocks = splits * 2 * p.D * jt * kt;
    if (blocks >= ((int64_t)1 << 31)) return hipErrorNotSupported;
    const unsigned n = (unsigned)blocks;
    auto go = [&](auto in_t, auto out_t) {
        constexpr bool I = decltype(in_t)::value, O = decltype(out_t)::value;
        const int j = (int)jt, k = (int)kt, sp = (int)splits;
        if (jw == 128 && wide) f32_dw_kernel<128, 128, I, O><<<n, kFThreads, 0, s>>>(p, j, k, sp, tps, part);
        else if (jw == 128) f32_dw_kernel<128, 64, I, O><<<n, kFThreads, 0, s>>>(p, j, k, sp, tps, part);
        else if (wide) f32_dw_kernel<64, 128, I, O><<<n, kFThreads, 0, s>>>(p, j, k, sp, tps, part);
        else f32_dw_kernel<64, 64, I, O><<<n, kFThreads, 0, s>>>(p, j, k, sp, tps, part);
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (p.in_t) p.out_t ? go(yes, yes) : go(yes, no);
    else p.out_t ? go(no, yes) : go(no, no);
    return hipGetLastError();
}

}  // namespace dyad
