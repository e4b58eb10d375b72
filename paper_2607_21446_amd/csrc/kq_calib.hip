// Layer-wise calibration of the block transform (Sec. 3.3).
//
// One step evaluates, for the activations X [R, d] and weight W [o, d] of a
// layer and the transform T = diag(T_f), T_f = G_1 (x) ... (x) G_5 (Sec. 3.2),
//   L_out = ||Q(X T) Q(W T^-T)^T - X W^T||^2 / (R o)
//   L_A   = ||Q(X T) - X T||^2 / (R d),   L_W = ||Q(W T^-T) - W T^-T||^2 / (o d)
//   L     = L_out + lambda_A L_A + lambda_W L_W
// and its gradient with respect to the 15 LU parameters of every block,
// with a straight-through estimator for Q: the E2M1 rounding passes the
// gradient unchanged, the E8M0 scale (a step function of the block maximum)
// is held fixed, and an element clipped at +-6 * scale passes none.  The
// forward products come from the quantizers and the W4A4 GEMM of the
// library; this file holds the backward pass:
//   * calib_backward_kernel, calib_reference_kernel: bf16 matrix-core products
//     (v_mfma_f32_32x32x16_bf16) in 256 x 256 or 128 x 128 workgroup tiles, 32-deep
//     K stages loaded straight into three LDS buffers, two in flight.  The
//     dequantized MXFP4 operands are exact in bf16; the fp32 residual enters as two
//     bf16 terms (hi = bf16(r), lo = bf16(r - hi), |r - hi - lo| <= 2^-17 |r|; the
//     W4A4 GEMM writes it so), so every product term is exact and sums run in fp32.
//     Operands whose K index is not the contiguous one are read from LDS transposed.
//     The gradient epilogue turns a tile of dL/dQ into its per-block sums
//     sum_rows left^T (P m) at once, so the R x d gradient never reaches memory;
//   * gram_reduce_kernel: fixed-order sum of the per-workgroup block sums and of the
//     quantizer's sums over clipped elements;
//   * lu_grad_kernel: chain rule through T^-T and the Kronecker product to the
//     2 x 2 factors and their (a, b, c), the losses, and the Adam update.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kq_calib.h"
#include "kq_kernels.h"
#include "kq_lds.h"
#include "kroquant.h"

namespace kq {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 32;  // K per LDS stage (bf16 elements)

// ---------------------------------------------------------------- operands
// A GEMM operand, bf16, rows 16-byte aligned, columns a multiple of 8:
//   K-contiguous  [rows][ld]: a tile row's 32 K values of a stage are 64 bytes;
//   K-strided     [K][ld] (TR): stage rows are K, the tile's columns contiguous,
//                 and fragments come by transposing LDS reads
//                 (ds_read_b64_tr_b16), so no transposed copy is made.
// Rows past the matrix load its last row and columns past it its last 8 (their
// products meet zeros of the other operand, or land in rows or columns the
// epilogues never use).
struct Opnd {
    const uint8_t* p;
    int64_t rows, cols, ld;  // ld in bytes
};

// Until only this wave's LOADS loads of a later stage (if there is one) are outstanding.
template <int LOADS>
__device__ __forceinline__ void wait_stage(bool later) {
    static_assert(LOADS == 4 || LOADS == 6, "loads per stage");
    if (!later) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if (LOADS == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
}

typedef __attribute__((address_space(3))) uint8_t lds_byte;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) uint4 lds_uint4;

// One operand's stage in LDS (64 BX bytes) for a tile of BX rows (or columns).
//   K-contiguous: 16-byte chunk c (of 4) of row r at 64 r + 16 (c ^ ((r >> 2) & 3)), so
//     the 16 lanes of a ds_read_b128 phase cover all banks; one load fills 16 rows.
//   K-strided: chunk c (8 columns) of K row r at 2 BX r + 16 (c ^ ((r & 3) << 2)), so the
//     four K rows a 16-lane group of a transposing read takes lie in different banks;
//     one load fills 512 / BX K rows.
// Fragments: lane (h = lane / 32) holds K values 16 h + 8 s .. + 7 of k-step s.
template <int BX, bool TR>
struct OpndStage {
    uint32_t voff[2], row[2], col[2];  // this lane's two chunks of a stage: byte offset; K row and byte column (TR)
    uint32_t frag;                     // this lane's fragment address for tile 0, k-step 0

    __device__ __forceinline__ void setup(const Opnd& m, int64_t x0, int wave, int lane) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (TR) {
                constexpr int RPI = 512 / BX, LPR = 64 / RPI;
                row[i] = RPI * (2 * wave + i) + lane / LPR;
                const int c = (lane % LPR) ^ ((row[i] & 3) << 2);
                col[i] = 2u * (uint32_t)min<int64_t>(8 * c, m.cols - 8 - x0);
                voff[i] = row[i] * (uint32_t)m.ld + col[i];
            } else {
                const int q = lane >> 2, blk = (lane & 3) ^ ((q >> 2) & 3);
                voff[i] = (uint32_t)min<int64_t>(16 * (2 * wave + i) + q, m.rows - 1 - x0) * (uint32_t)m.ld + 16u * blk;
            }
        }
    }
    // base of the tile: K-contiguous, row x0; K-strided, column x0
    static __device__ __forceinline__ const uint8_t* base(const Opnd& m, int64_t x0) {
        return m.p + (TR ? 2 * x0 : x0 * m.ld);
    }
    // K values k .. k + 31 to LDS address dst (of this operand's stage)
    __device__ __forceinline__ void issue(const Opnd& m, const uint8_t* base, int64_t k, uint32_t dst, int wave) const {
        const uint8_t* const b = base + (TR ? k * m.ld : 2 * k);
        if (TR && k + BK > m.rows) {  // a last stage past the last K row
            const uint32_t last = (uint32_t)(m.rows - 1 - k);
#pragma unroll
            for (int i = 0; i < 2; ++i)
                lds_dma16(dst + 1024u * (2 * wave + i), min(row[i], last) * (uint32_t)m.ld + col[i], b);
        } else {
#pragma unroll
            for (int i = 0; i < 2; ++i) lds_dma16(dst + 1024u * (2 * wave + i), voff[i], b);
        }
    }
    // t0: this wave's first 32-wide tile
    __device__ __forceinline__ void frag_setup(int t0, int lane) {
        const int h = lane >> 5, l32 = lane & 31;
        if (TR) {
            const int jr = (lane >> 2) & 3;  // K row within a group of 4
            const int c = 4 * t0 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
            frag = (16 * h + jr) * (2 * BX) + 16 * (c ^ (jr << 2)) + 8 * (lane & 1);
        } else {
            frag = (32 * t0 + l32) * 64 + 16 * ((2 * h) ^ ((l32 >> 2) & 3));
        }
    }
    // fragment of tile t0 + i (t0 a multiple of the wave's tile count), k-step s
    __device__ __forceinline__ bf16x8 read(lds_byte* stage, int i, int s) const {
        if (TR) {
            lds_byte* const p = stage + (frag ^ (64u * i)) + 8 * s * (2 * BX);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4*>(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4*>(p + 4 * (2 * BX)));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            return __builtin_bit_cast(bf16x8, s16x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
        }
        lds_byte* const p = stage + (frag ^ (16u * s)) + 2048 * i;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<lds_uint4*>(p));
    }
};

// Workgroup tile: WM x WN waves of TM x TN tiles of 32 x 32, A in TA bf16 terms.
template <int TA, int WM, int WN, int TM, int TN>
struct CalibTile {
    static constexpr int BM = 32 * WM * TM, BN = 32 * WN * TN, WAVES = WM * WN, THREADS = 64 * WAVES;
    static_assert(BM == 32 * WAVES && BN == 32 * WAVES, "two loads per wave, operand term and stage");
    static constexpr int kStageBytes = 64 * (TA * BM + BN), kStages = 3;
    static constexpr int kLdsBytes = kStages * kStageBytes;
};

// acc = sum over K values k_lo .. k_hi (a multiple of 32 of them) of A[m0 + m][k]
// B[n0 + n][k]; three stage buffers, two in flight.
//
// PING (eight waves, two per SIMD): waves 4-7 run half a stage behind waves 0-3
// (one extra barrier at the start), so that on every SIMD one wave reads its
// fragments and issues loads while the other computes.  Waves 0-3 read stage k
// and issue stage k + 2 in phase 2k and compute it in phase 2k + 1, waves 4-7 one
// phase later.  Stage k + 2 overwrites the buffer of stage k - 1, whose last reads
// returned before the barrier that ends phase 2k - 1; every wave has waited for
// its loads of stage k before that barrier.
template <int TA, bool ATR, bool BTR, int WM, int WN, int TM, int TN, bool PING>
__device__ __forceinline__ void calib_product(const Opnd (&A)[TA], const Opnd& B, uint8_t* lds_generic, int64_t m0,
                                              int64_t n0, int64_t k_lo, int64_t k_hi, f32x16 (&acc)[TM][TN]) {
    typedef CalibTile<TA, WM, WN, TM, TN> T;
    constexpr int kLoads = 2 * (TA + 1);
    lds_byte* const lds = (lds_byte*)lds_generic;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // the lane's addresses are not kept in registers through the epilogue
    const int wm = wave / WN, wn = wave % WN;
    const int nst = (int)((k_hi - k_lo) / BK);
    OpndStage<T::BM, ATR> sa;  // the terms of A have one layout
    OpndStage<T::BN, BTR> sb;
    sa.setup(A[0], m0, wave, lane);
    sb.setup(B, n0, wave, lane);
    sa.frag_setup(wm * TM, lane);
    sb.frag_setup(wn * TN, lane);
    const uint8_t* abase[TA];
#pragma unroll
    for (int x = 0; x < TA; ++x) abase[x] = sa.base(A[x], m0);
    const uint8_t* const bbase = sb.base(B, n0);
    auto issue = [&](int st, int buf) {
        const int64_t k = k_lo + (int64_t)st * BK;
        const uint32_t dst = lds0 + buf * T::kStageBytes;
#pragma unroll
        for (int x = 0; x < TA; ++x) sa.issue(A[x], abase[x], k, dst + x * 64 * T::BM, wave);
        sb.issue(B, bbase, k, dst + TA * 64 * T::BM, wave);
    };
    const bool behind = PING && wave >= T::WAVES / 2;
    auto stage = [&](int st, auto bufc) {
        constexpr int J = decltype(bufc)::value;
        lds_byte* const sbuf = lds + J * T::kStageBytes;
        bf16x8 fa[2][TA][TM], fb[2][TN];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int x = 0; x < TA; ++x)
#pragma unroll
                for (int i = 0; i < TM; ++i) fa[s][x][i] = sa.read(sbuf + x * 64 * T::BM, i, s);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[s][j] = sb.read(sbuf + TA * 64 * T::BM, j, s);
        }
        if (st + 2 < nst) issue(st + 2, (J + 2) % 3);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        auto products = [&]() {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int x = 0; x < TA; ++x)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][x][i], fb[s][j], acc[i][j], 0, 0, 0);
        };
        if (PING) {
            if (behind) wait_stage<kLoads>(st + 2 < nst);
            stage_barrier();
            products();
            if (!behind) wait_stage<kLoads>(st + 2 < nst);
            stage_barrier();
        } else {
            products();
            wait_stage<kLoads>(st + 2 < nst);
            stage_barrier();
        }
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x16{};
    if (nst <= 0) return;
    issue(0, 0);
    if (nst > 1) issue(1, 1);
    wait_stage<kLoads>(nst > 1);
    stage_barrier();
    if (behind) stage_barrier();
    for (int st = 0; st < nst; st += 3) {
        stage(st, std::integral_constant<int, 0>{});
        if (st + 1 < nst) stage(st + 1, std::integral_constant<int, 1>{});
        if (st + 2 < nst) stage(st + 2, std::integral_constant<int, 2>{});
    }
    if (PING && !behind) stage_barrier();
}

// --------------------------------------------------------------- epilogues
// The accumulator of a 32 x 32 MFMA tile holds, in lane l (h = l / 32) and
// register 4q + r, element (row 8q + 4h + r, column l % 32).

// Yneg = -acc (the reference product of the loss).
template <int WM, int WN, int TM, int TN>
__device__ __forceinline__ void store_neg(const f32x16 (&acc)[TM][TN], float* out, int64_t M, int64_t N, int64_t m0,
                                          int64_t n0) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave / WN, wn = wave % WN, h = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = n0 + 32 * (wn * TN + j) + l32;
            if (col >= N) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t row = m0 + 32 * (wm * TM + i) + 8 * (e / 4) + 4 * h + (e % 4);
                if (row < M) out[row * N + col] = -acc[i][j][e];
            }
        }
}

// One side of the backward pass.  The product's tile holds  P = dL_out/dQ * (R o) / 2
// for the quantized operand Q [M, d] (exact up to the split of K, which is linear).
// With y the operand before quantization and m = [|y| <= 6 * scale] the
// straight-through mask, the gradient is
//   dL/dy = c1 * P * m + c2 * (Q - y) * (m - 1),
// c1 = 2 / (R o), c2 = lambda * 2 / (rows d), and the block transforms take the
// per-block sums  S_j = left_j^T dL/dy_j  (left = the operand before the transform).
// The second term's sums come from the quantizer; this epilogue makes the first's,
// times the power of two of c1 (c1_pow2, exact: the sums leave fp32's range no sooner than
// the gradient does).
struct Side {
    Opnd A[2], B;             // the product: residual terms, dequantized operand
    Opnd left;                // [M, d] bf16
    const uint32_t* clipped;  // [ceil(M / 32), d]: bit r of word (g, c) = not m of row 32 g + r
    float* partial;           // [m_tiles * ks, d / 32, 32, 32]
    int64_t K, kchunk;        // K (a multiple of 32) in ks parts of kchunk
    int64_t ks, works;        // works = m_tiles * ks * ntn
    float c1_pow2;
    // FOLD (one m tile, one K part): the side's gradient sums, in place of strip 0 of the quantizer's
    float* sums;              // [strips, d / 32, 32, 32]
    int64_t strips;
    double c1, c2_unit;       // c1 / c1_pow2; c2 = lambda * c2_unit
    const float* lambda;
};

// The Gram sums of a tile: left^T (P m) per 32-column block, on the matrix cores with
// the rows as the K index.  P comes straight from the accumulators as three bf16
// terms (hi + mid + lo, exact): six instructions of 32 cycles per 32 x 32, where fp32
// ones took 16 of 64.  `left` is staged in the free stage buffers (one round of loads
// for the whole tile; loading it, y, codes and scales from the lanes took a chain of
// 16 memory latencies) and read transposed, its K index in the order the
// accumulators have: k-step s, lane half h holds rows 16 s + 4 h + 0..3, 16 s + 8 + 4 h + 0..3.
// 18432 x 3072 x 3072, both sides: 335 us before, of 1250.
//
// FOLD: a few rows and features of very many columns, where partial sums of their own
// would be most of the workspace.
template <int WM, int WN, int TM, int TN, bool FOLD>
__device__ __forceinline__ void gram_tile(f32x16 (&acc)[TM][TN], const Side& s, uint8_t* lds_generic, int64_t slot,
                                          int64_t m0, int64_t n0) {
    constexpr int WAVES = WM * WN, BM = 32 * WM * TM, BN = 32 * WN * TN;
    constexpr int RPI = 512 / BN, LPR = 64 / RPI, LOADS = 2 * BM * BN / 1024 / WAVES;
    lds_byte* const lds = (lds_byte*)lds_generic;
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));  // the lane's addresses are not kept in registers through the product
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wm = wave / WN, wn = wave % WN, h = lane >> 5, l32 = lane & 31;
    const int64_t d = s.left.cols, M = s.left.rows, nb = d / 32;
    {
        const uint8_t* const base = s.left.p + m0 * s.left.ld + 2 * n0;
        const uint32_t last = (uint32_t)min<int64_t>(BM - 1, M - 1 - m0);
        const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const uint32_t row = RPI * (LOADS * wave + i) + lane / LPR;
            const int c = (lane % LPR) ^ ((row & 3) << 2);
            const uint32_t col = 2u * (uint32_t)min<int64_t>(8 * c, d - 8 - n0);
            lds_dma16(lds0 + 1024u * (LOADS * wave + i), min(row, last) * (uint32_t)s.left.ld + col, base);
        }
    }
    // bit r of pass[i][j]: row r of the tile exists and passes the gradient at this lane's column
    uint32_t pass[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int64_t r0 = m0 + 32 * (wm * TM + i);
        const uint32_t rows = r0 >= M ? 0u : M - r0 >= 32 ? ~0u : (1u << (M - r0)) - 1u;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = n0 + 32 * (wn * TN + j) + l32;
            pass[i][j] = rows;
            if (rows && col < d) pass[i][j] = rows & ~s.clipped[(r0 >> 5) * d + col];
        }
    }
    // c1_pow2 goes in before the sums where the product is large, after them where it is not
    // (there it could take terms of a small one below bf16's range)
    float top = 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) top = fmaxf(top, fabsf(acc[i][j][e]));
    const bool large = __builtin_amdgcn_ballot_w64(top >= 0x1p30f) != 0u;
    const float after = large ? 1.0f : s.c1_pow2;
    if (large) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] *= s.c1_pow2;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    stage_barrier();
    f32x16 gram[TN];
    const int jr = (lane >> 2) & 3;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        gram[j] = f32x16{};
        const int c = (4 * (wn * TN + j) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ (jr << 2);
        lds_byte* const lb = lds + (32 * wm * TM + 4 * h + jr) * (2 * BN) + 16 * c + 8 * (lane & 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const uint32_t bits = pass[i][j] >> (4 * h);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                lds_byte* const p = lb + (32 * i + 16 * k) * (2 * BN);
                const s16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4*>(p));
                const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4*>(p + 8 * (2 * BN)));
                typedef short s16x8 __attribute__((ext_vector_type(8)));
                const bf16x8 lf = __builtin_bit_cast(bf16x8, s16x8{lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w});
                bf16x8 g[3];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    // accumulator 8 k + u is row 16 k + 8 (u / 4) + 4 h + u % 4
                    const int bit = 16 * k + 8 * (u / 4) + (u % 4);
                    const uint32_t keep = (uint32_t)((int32_t)(bits << (31 - bit)) >> 31);
                    const float v = __uint_as_float(__float_as_uint(acc[i][j][8 * k + u]) & keep);
                    g[0][u] = (__bf16)v;
                    const float r1 = v - (float)g[0][u];  // exact
                    g[1][u] = (__bf16)r1;
                    g[2][u] = (__bf16)(r1 - (float)g[1][u]);
                }
#pragma unroll
                for (int term = 2; term >= 0; --term)
                    gram[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf, g[term], gram[j], 0, 0, 0);
            }
        }
    }
    __syncthreads();
    float* const sums = reinterpret_cast<float*>(lds_generic);  // [wm][block of the tile][32][32]
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        float* const dst = sums + ((wm * WN + wn) * TN + j) * 1024;
#pragma unroll
        for (int e = 0; e < 16; ++e) dst[(8 * (e / 4) + 4 * h + (e % 4)) * 32 + l32] = gram[j][e] * after;
    }
    __syncthreads();
    // the WM row groups of a block, in order, and one write per block
    for (int k = 4 * t; k < WN * TN * 1024; k += 4 * 64 * WAVES) {
        const int64_t blk = n0 / 32 + k / 1024;
        if (blk >= nb) continue;
        float4 v = *reinterpret_cast<const float4*>(sums + k);
#pragma unroll
        for (int w = 1; w < WM; ++w) {
            const float4 o = *reinterpret_cast<const float4*>(sums + w * (WN * TN * 1024) + k);
            v = make_float4(v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w);
        }
        if (FOLD) {
            float* const at = s.sums + blk * 1024 + k % 1024;
            const double c2 = -(double)*s.lambda * s.c2_unit;
            double x[4] = {s.c1 * v.x, s.c1 * v.y, s.c1 * v.z, s.c1 * v.w};
            for (int64_t c = 0; c < s.strips && c2 != 0.0; ++c) {
                const float4 q = *reinterpret_cast<const float4*>(at + c * nb * 1024);
                x[0] += c2 * q.x;
                x[1] += c2 * q.y;
                x[2] += c2 * q.z;
                x[3] += c2 * q.w;
            }
            *reinterpret_cast<float4*>(at) = make_float4((float)x[0], (float)x[1], (float)x[2], (float)x[3]);
            continue;
        }
        *reinterpret_cast<float4*>(s.partial + (slot * nb + blk) * 1024 + k % 1024) = v;
    }
}

// Workgroup L of the dispatch order runs on XCD L % 8: each XCD takes a
// contiguous range of the work items.
__device__ __forceinline__ int64_t xcd_work(int64_t L, int64_t G) {
    const int64_t q = G >> 3, r = G & 7, x = L & 7;
    return x * q + (x < r ? x : r) + (L >> 3);
}

struct BackwardArgs {
    Side act, wgt;
    int64_t ntn;
};

// Both backward products in one launch: works 0 .. act.works - 1 are the
// activation side P = res . What (K = o, contiguous in res), the rest the weight
// side P = res^T . Ahat (K = rows, strided in both).  A work is (m tile, K part,
// column tile), the column tile fastest: the column tiles of one m tile and K
// part read the same rows of the residual and run on one XCD.
template <int WM, int WN, int TM, int TN, bool PING, bool FOLD>
__global__ __launch_bounds__(64 * WM * WN) void calib_backward_kernel(const BackwardArgs p) {
    typedef CalibTile<2, WM, WN, TM, TN> T;
    static_assert(WM * WN * TN * 4096 <= T::kLdsBytes && 2 * T::BM * T::BN <= T::kLdsBytes,
                  "the block sums and a tile of `left` fit the stage buffers");
    __shared__ __align__(16) uint8_t lds[T::kLdsBytes];
    const bool act = blockIdx.x < p.act.works;
    const Side s = act ? p.act : p.wgt;
    // each XCD takes its share of both sides (their works differ in length)
    const int64_t wk = xcd_work(act ? blockIdx.x : blockIdx.x - p.act.works, s.works);
    const int64_t n0 = (wk % p.ntn) * T::BN, slot = wk / p.ntn, m0 = slot / s.ks * T::BM;
    const int64_t k_lo = (slot % s.ks) * s.kchunk, k_hi = std::min(s.K, k_lo + s.kchunk);
    f32x16 acc[TM][TN];
    if (act) calib_product<2, false, true, WM, WN, TM, TN, PING>(s.A, s.B, lds, m0, n0, k_lo, k_hi, acc);
    else calib_product<2, true, true, WM, WN, TM, TN, PING>(s.A, s.B, lds, m0, n0, k_lo, k_hi, acc);
    gram_tile<WM, WN, TM, TN, FOLD>(acc, s, lds, slot, m0, n0);
}

// Yneg = -(X W^T): both operands K-contiguous, one term.
template <int WM, int WN, int TM, int TN, bool PING>
__global__ __launch_bounds__(64 * WM * WN) void calib_reference_kernel(const Opnd A, const Opnd B, float* out, int64_t K,
                                                                       uint32_t ntn) {
    typedef CalibTile<1, WM, WN, TM, TN> T;
    __shared__ __align__(16) uint8_t lds[T::kLdsBytes];
    // Rows of tiles one after the other; few rows of many columns, columns one after the other, or
    // every XCD reads all of W.  Row after row / column after column, us: 8 x 24 tiles
    // (1024 x 3072 x 1152) 19.8 / 16.2; 8 x 17 (1024 x 2049 x 2304) 25.7 / 27.4; 72 x 96 at d 640 201 / 213.
    const uint32_t wk = (uint32_t)xcd_work(blockIdx.x, gridDim.x), mt = gridDim.x / ntn;
    const bool few_rows = ntn >= 24 && 3 * mt <= ntn;
    const uint32_t fast = few_rows ? mt : ntn, slow_i = wk / fast, fast_i = wk - slow_i * fast;
    const int64_t n0 = int64_t(few_rows ? slow_i : fast_i) * T::BN, m0 = int64_t(few_rows ? fast_i : slow_i) * T::BM;
    f32x16 acc[TM][TN];
    const Opnd a[1] = {A};
    calib_product<1, false, false, WM, WN, TM, TN, PING>(a, B, lds, m0, n0, 0, K, acc);
    store_neg<WM, WN, TM, TN>(acc, out, A.rows, B.rows, m0, n0);
}

// ------------------------------------------------------------ small kernels

// S = c1 / c1_pow2 sum over the slots of partial - c2 sum over the quantizer's strips of dpart,
// summed in fp64 and a fixed order (16 threads per four elements, each every 16th
// term), in place: partial[0][j][e] the nearest fp32, dpart[0][j][e] that of the rest.
struct ReduceSide {
    float* partial;      // [slots, nb, 1024]
    float* dpart;        // [strips, nb, 1024]
    int64_t slots, strips;
    double c1;           // c1 / c1_pow2
    double c2_unit;      // c2 = lambda * c2_unit
};

__global__ __launch_bounds__(256) void gram_reduce_kernel(const ReduceSide s0, const ReduceSide s1, int64_t nb,
                                                          const float* lambdas) {
    __shared__ double red[16][16][4];
    const ReduceSide s = blockIdx.z ? s1 : s0;
    const double c2 = -(double)lambdas[blockIdx.z] * s.c2_unit;
    const int64_t j = blockIdx.x;
    const int e4 = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int64_t e = 64 * blockIdx.y + 4 * e4;
    double v[4] = {0.0, 0.0, 0.0, 0.0}, w[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int64_t c = part; c < s.slots; c += 16) {
        const float4 x = *reinterpret_cast<const float4*>(s.partial + (c * nb + j) * 1024 + e);
        v[0] += x.x;
        v[1] += x.y;
        v[2] += x.z;
        v[3] += x.w;
    }
#pragma unroll 4
    for (int64_t c = part; c < s.strips; c += 16) {
        const float4 x = *reinterpret_cast<const float4*>(s.dpart + (c * nb + j) * 1024 + e);
        w[0] += x.x;
        w[1] += x.y;
        w[2] += x.z;
        w[3] += x.w;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) red[part][e4][i] = s.c1 * v[i] + (c2 != 0.0 ? c2 * w[i] : 0.0);
    __syncthreads();
    if (threadIdx.x < 64) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][threadIdx.x >> 2][threadIdx.x & 3];
        const int64_t at = j * 1024 + 64 * blockIdx.y + threadIdx.x;
        const float hi = (float)t;
        s.partial[at] = hi;
        s.dpart[at] = (float)(t - (double)hi);
    }
}

__device__ __forceinline__ void decode_g(const float* lu, float (&g)[5][4]) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const float pa = lu[3 * k], pb = lu[3 * k + 1], pc = lu[3 * k + 2];
        g[k][0] = pa;
        g[k][1] = pb;
        g[k][2] = pc * pa;
        g[k][3] = __builtin_fmaf(pc, pb, -(1.0f / pa));
    }
}

__device__ __forceinline__ double block_sum256(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}

struct LuGradArgs {
    const float* lu;
    const float *ga, *ga_lo;  // [nb, 32, 32]  dL/dT of every block from the activation side, in two terms
    const float *gw, *gw_lo;  // [nb, 32, 32]  dL/dU, U = T^-T, from the weight side
    int64_t nb, nfac;  // nfac = nb, or 1: the blocks' sums add up
    float* grad;       // [nfac, 15]
    float* lu_out;
    float* adam_m;
    float* adam_v;
    int adam_t;
    float lr;
    // losses (the last workgroup)
    const double* sr;
    int64_t nsr;
    const double* sqa;
    int64_t nsqa;
    const double* sqw;
    int64_t nsqw;
    double n_out, n_a, n_w;  // R o, R d, o d
    const float* lambdas;
    double* losses;
};

// dL/dT_f = GA_f - U GW_f^T U (U = T_f^-T; d(T^-T) = -U dT^T U), then for
// every factor G_k of T_f = G_1 (x) ... (x) G_5:
//   dL/dG_k[u][v] = sum_{p, q: bit_k(p) = u, bit_k(q) = v} dT[p][q] prod_{l != k} G_l[bit_l(p)][bit_l(q)]
// (bit_1 the most significant of the 5-bit index), and for G = [[a, b], [c a, c b - 1/a]]:
//   dL/da = dG00 + c dG10 + dG11 / a^2,  dL/db = dG01 + c dG11,  dL/dc = a dG10 + b dG11.
//
// TWO: the sums come in two terms (else ga and gw are all there is).
template <bool TWO>
__global__ __launch_bounds__(256) void lu_grad_kernel(const LuGradArgs p) {
    __shared__ float sU[32][33];
    __shared__ float sGW[32][33];
    __shared__ float sV[32][33];
    __shared__ double red[20][256];
    __shared__ float gsum[5][4];
    const int64_t f = blockIdx.x;
    const int t = threadIdx.x;
    if (f == p.nfac) {  // the losses, beside the factors' workgroups
        double s = 0.0;
        for (int64_t i = t; i < p.nsr; i += 256) s += p.sr[i];
        const double sr = block_sum256(s, red[0]);
        s = 0.0;
        for (int64_t i = t; i < p.nsqa; i += 256) s += p.sqa[i];
        const double sa = block_sum256(s, red[0]);
        s = 0.0;
        for (int64_t i = t; i < p.nsqw; i += 256) s += p.sqw[i];
        const double sw = block_sum256(s, red[0]);
        if (t == 0) {
            const double lo = sr / p.n_out, la = sa / p.n_a, lw = sw / p.n_w;
            p.losses[0] = lo;
            p.losses[1] = la;
            p.losses[2] = lw;
            p.losses[3] = lo + double(p.lambdas[0]) * la + double(p.lambdas[1]) * lw;
        }
        return;
    }
    float ga[4];
    {
        double a4[4] = {0.0, 0.0, 0.0, 0.0}, w4[4] = {0.0, 0.0, 0.0, 0.0};
        const int64_t j0 = p.nfac == 1 ? 0 : f, j1 = p.nfac == 1 ? p.nb : f + 1;
#pragma unroll 4
        for (int64_t j = j0; j < j1; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t e = j * 1024 + t + 256 * i;
                a4[i] += TWO ? double(p.ga[e]) + double(p.ga_lo[e]) : double(p.ga[e]);
                w4[i] += TWO ? double(p.gw[e]) + double(p.gw_lo[e]) : double(p.gw[e]);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ga[i] = float(a4[i]);
            sGW[(t + 256 * i) / 32][t % 32] = float(w4[i]);
        }
    }
    float g[5][4];
    decode_g(p.lu + f * 15, g);
    // (G^-1)^T = [[-g11, g10], [g01, -g00]]
    float git[5][4];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        git[k][0] = -g[k][3];
        git[k][1] = g[k][2];
        git[k][2] = g[k][1];
        git[k][3] = -g[k][0];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = t + 256 * i, r = e / 32, q = e % 32;
        float u = 1.0f;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int ee = 2 * ((r >> (4 - k)) & 1) + ((q >> (4 - k)) & 1);
            u *= ee == 0 ? git[k][0] : ee == 1 ? git[k][1] : ee == 2 ? git[k][2] : git[k][3];
        }
        sU[r][q] = u;
    }
    __syncthreads();
    // V = GW^T U
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = t + 256 * i, r = e / 32, q = e % 32;
        float s = 0.f;
#pragma unroll 8
        for (int x = 0; x < 32; ++x) s = __builtin_fmaf(sGW[x][r], sU[x][q], s);
        sV[r][q] = s;
    }
    __syncthreads();
    double dg[5][4];
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) dg[k][e] = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = t + 256 * i, r = e / 32, q = e % 32;
        float s = 0.f;
#pragma unroll 8
        for (int x = 0; x < 32; ++x) s = __builtin_fmaf(sU[r][x], sV[x][q], s);
        const float dT = ga[i] - s;
        float ge[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const int ee = 2 * ((r >> (4 - k)) & 1) + ((q >> (4 - k)) & 1);
            ge[k] = ee == 0 ? g[k][0] : ee == 1 ? g[k][1] : ee == 2 ? g[k][2] : g[k][3];
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            double others = dT;
#pragma unroll
            for (int l = 0; l < 5; ++l)
                if (l != k) others *= ge[l];
            const int ee = 2 * ((r >> (4 - k)) & 1) + ((q >> (4 - k)) & 1);
#pragma unroll
            for (int x = 0; x < 4; ++x) dg[k][x] += (x == ee) ? others : 0.0;
        }
    }
    // the 20 sums over the workgroup through LDS, five per wave (a reduction of
    // each with its own barriers took about 1 us apiece)
#pragma unroll
    for (int k = 0; k < 5; ++k)
#pragma unroll
        for (int x = 0; x < 4; ++x) red[4 * k + x][t] = dg[k][x];
    __syncthreads();
    {
        const int w = t >> 6, lane = t & 63;
        double v[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const double* const r = red[5 * w + i];
            v[i] = (r[lane] + r[lane + 64]) + (r[lane + 128] + r[lane + 192]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int i = 0; i < 5; ++i) v[i] += __shfl_xor(v[i], off);
        if (lane == 0)
#pragma unroll
            for (int i = 0; i < 5; ++i) gsum[(5 * w + i) / 4][(5 * w + i) % 4] = float(v[i]);
    }
    __syncthreads();
    if (t < 5) {
        const int k = t;
        const float pa = p.lu[f * 15 + 3 * k], pb = p.lu[f * 15 + 3 * k + 1], pc = p.lu[f * 15 + 3 * k + 2];
        const float d00 = gsum[k][0], d01 = gsum[k][1], d10 = gsum[k][2], d11 = gsum[k][3];
        float gr[3];
        gr[0] = d00 + pc * d10 + d11 / (pa * pa);
        gr[1] = d01 + pc * d11;
        gr[2] = pa * d10 + pb * d11;
        const float par[3] = {pa, pb, pc};
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const int64_t i = f * 15 + 3 * k + x;
            p.grad[i] = gr[x];
            if (p.adam_t > 0) {
                // Adam (Kingma and Ba), beta1 0.9, beta2 0.999, eps 1e-8
                const float m = 0.9f * p.adam_m[i] + 0.1f * gr[x];
                const float v = 0.999f * p.adam_v[i] + 0.001f * gr[x] * gr[x];
                p.adam_m[i] = m;
                p.adam_v[i] = v;
                const float bc1 = 1.0f - powf(0.9f, float(p.adam_t));
                const float bc2 = 1.0f - powf(0.999f, float(p.adam_t));
                p.lu_out[i] = par[x] - p.lr * (m / bc1) / (sqrtf(v / bc2) + 1e-8f);
            }
        }
    }
}

__global__ void init_kernel(float* m, float* v, int64_t n, float* lambdas) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
        m[i] = 0.f;
        v[i] = 0.f;
    }
    if (blockIdx.x == 0 && threadIdx.x < 2) lambdas[threadIdx.x] = 0.f;
}

// lambda_A = L_out / L_A, lambda_W = L_out / L_W at the initial transform (0 if the denominator is 0).
__global__ void set_lambdas_kernel(const double* losses, float* lambdas) {
    if (threadIdx.x == 0) {
        lambdas[0] = losses[1] > 0.0 ? float(losses[0] / losses[1]) : 0.f;
        lambdas[1] = losses[2] > 0.0 ? float(losses[0] / losses[2]) : 0.f;
    }
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }


}  // namespace

// One side of the backward products: mt x ntn tiles of C, K of `stages` 32-deep
// stages in ks parts.
struct SidePlan {
    int64_t mt, ntn, stages, ks;
    double works() const { return double(mt * ntn * ks); }
    // A work's length in stages of a 256 x 256 tile: its K part and its epilogue.  A 128 x
    // 128 workgroup has a quarter of the products, two share a CU, and its stage feeds
    // half the products per byte.
    double length(bool big) const { return (big ? 1.0 : 0.65) * double(cdiv(stages, ks)) + (big ? 12.0 : 5.0); }
};

// Cost of the launch, `act` works first and `wgt` works into the slots as they come
// free: the time of the last one plus the mean load of a slot (idle slots leave the
// others clock and bandwidth).  2048 x 1152 x 1152, step in us: parts 1 and 4 72.4,
// 1 and 1 84.4, 3 and 6 76.8; 4096 x 1152 x 4608: 1 and 2 247, 2 and 5 296, 1 and 1 292.
static double backward_cost(const SidePlan& act, const SidePlan& wgt, bool big) {
    const double S = big ? 256.0 : 512.0, n1 = act.works(), l1 = act.length(big), n2 = wgt.works(), l2 = wgt.length(big);
    const double q = std::floor(n1 / S), busy = n1 - q * S;    // slots that take a last act work
    const double early = q * l1, late = busy > 0 ? early + l1 : early;
    // works that end by t: slots free at `early` and slots free at `late`
    auto done = [&](double t) {
        return (S - busy) * std::floor((t - early) / l2 + 1e-9) + busy * std::max(0.0, std::floor((t - late) / l2 + 1e-9));
    };
    const double k = std::floor(n2 / S);
    double end = std::max(late, early + (k + 2.0) * l2);
    for (const double t : {early + k * l2, early + (k + 1.0) * l2, late + k * l2, late + (k > 0 ? k - 1.0 : 0.0) * l2})
        if (t >= late && t < end && done(t) >= n2) end = t;
    return end + (n1 * l1 + n2 * l2) / S;
}

// The bytes that a workspace may hold at most, so that one sized by an earlier version of the
// library is large enough (buffers of 6.6 R d + 12 R o + 6.6 o d bytes, and partial sums
// of 128-row tiles): what the step itself leaves of them is the budget of its
// partial sums.  kq_calib_step_noalloc takes the sizes for which this is at most
// KQ_CALIB_NOALLOC_MAX_BYTES.
static size_t workspace_budget(int64_t R, int64_t o, int64_t d, int a, int64_t nfac) {
    const int64_t nb = d / 32, ntn = cdiv(d, 256), act_mt = cdiv(R, 128), w_mt = cdiv(o, 128);
    const int64_t Rp = cdiv(R, BK) * BK, op = cdiv(o, BK) * BK, stages = Rp / BK;
    const int64_t act_chunks = std::max<int64_t>(1, std::min(act_mt, cdiv(2048, ntn)));
    int64_t ks = std::max<int64_t>(1, std::min(cdiv(2048, ntn * w_mt), cdiv(stages, 8)));
    ks = std::max<int64_t>(1, cdiv(Rp, cdiv(cdiv(Rp, ks), BK) * BK));
    const int64_t w_chunks = w_mt * ks, b = 32 / a;
    size_t n = 0;
    for (const int64_t bytes :
         {R * d * 4, R * d / 2, R * nb, o * d * 4, o * d / 2, o * nb, R * o * 4, R * op * 2, R * op * 2, o * Rp * 2,
          o * Rp * 2, d * Rp * 2, d * op * 2, nfac * a * a * 4, nfac * b * b * 4, act_chunks * nb * 4096,
          w_chunks * nb * 4096, act_chunks * ntn * 8, w_chunks * ntn * 8, cdiv(Rp, 64) * cdiv(o, 64) * 8, nfac * 4096,
          nfac * 4096, nfac * 60, nfac * 60, nfac * 60, int64_t(8)})
        n += align256(size_t(bytes));
    return n;
}

CalibPlan calib_plan(int64_t R, int64_t o, int64_t d, int a, int64_t nfac) {
    CalibPlan pl;
    pl.R = R;
    pl.o = o;
    pl.d = d;
    pl.nb = d / 32;
    pl.a = a;
    pl.nfac = nfac;
    pl.Rp = cdiv(std::max<int64_t>(R, 1), BK) * BK;
    pl.op = cdiv(o, BK) * BK;
    pl.nsum = std::max<int64_t>(256, cdiv(pl.Rp, 64) * cdiv(pl.op, 64));  // one per workgroup of the GEMM, any tile
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align256(off + bytes);
        return at;
    };
    pl.cA = take(size_t(R) * d / 2);
    pl.sA = take(size_t(R) * (d / 32));
    pl.qA = take(size_t(R) * d * 2);
    pl.mA = take(size_t(cdiv(R, 32)) * d * 4);
    pl.strips_a = calib_quant_strips(R, pl.nb);
    pl.dA = take(size_t(pl.strips_a) * pl.nb * 4096);
    pl.cW = take(size_t(o) * d / 2);
    pl.sW = take(size_t(o) * (d / 32));
    pl.qW = take(size_t(o) * d * 2);
    pl.mW = take(size_t(cdiv(o, 32)) * d * 4);
    pl.strips_w = calib_quant_strips(o, pl.nb);
    pl.dW = take(size_t(pl.strips_w) * pl.nb * 4096);
    pl.rh = take(size_t(pl.Rp) * pl.op * 2);
    pl.rl = take(size_t(pl.Rp) * pl.op * 2);
    pl.nsqa = pl.strips_a * cdiv(pl.nb, 8);
    pl.nsqw = pl.strips_w * cdiv(pl.nb, 8);
    pl.sqa = take(size_t(pl.nsqa) * 8);
    pl.sqw = take(size_t(pl.nsqw) * 8);
    pl.sr = take(size_t(pl.nsum) * 8);
    pl.grad = take(size_t(nfac) * 15 * 4);
    pl.am = take(size_t(nfac) * 15 * 4);
    pl.av = take(size_t(nfac) * 15 * 4);
    pl.lam = take(2 * 4);
    // both sides with 256 x 256 or both with 128 x 128 tiles, whichever is cheaper, with
    // as many K parts as the budget has room for partial sums
    const size_t budget = workspace_budget(R, o, d, a, nfac), slot = size_t(pl.nb) * 4096;
    const int64_t room = budget > off ? int64_t((budget - off) / slot) : 0;
    double best = HUGE_VAL;
    for (const bool big : {true, false}) {
        const int64_t T = big ? 256 : 128, ntn = cdiv(d, T);
        SidePlan act{cdiv(R, T), ntn, pl.op / BK, 1}, wgt{cdiv(o, T), ntn, pl.Rp / BK, 1};
        constexpr int64_t kParts[] = {1, 2, 3, 4, 6, 8};
        for (const int64_t ka : kParts)
            for (const int64_t kw : kParts) {
                // a part has at least four stages
                if ((ka > 1 && 4 * ka > act.stages) || (kw > 1 && 4 * kw > wgt.stages)) continue;
                if ((ka > 1 || kw > 1) && act.mt * ka + wgt.mt * kw > room) continue;
                act.ks = ka;
                wgt.ks = kw;
                const double cost = backward_cost(act, wgt, big);
                if (cost >= best) continue;
                best = cost;
                pl.big = big;
                pl.ntn = ntn;
                pl.act_mt = act.mt;
                pl.act_kchunk = cdiv(act.stages, ka) * BK;
                pl.w_mt = wgt.mt;
                pl.w_kchunk = cdiv(wgt.stages, kw) * BK;
            }
    }
    pl.act_ks = cdiv(pl.op, pl.act_kchunk);
    pl.w_ks = cdiv(pl.Rp, pl.w_kchunk);
    // no room for one partial sum a side (R + o up to about 70): none of its own
    pl.fold = pl.act_mt * pl.act_ks + pl.w_mt * pl.w_ks > room && R <= 128 && o <= 128;
    if (pl.fold) {
        pl.big = false;
        pl.ntn = cdiv(d, 128);
        pl.act_mt = pl.w_mt = pl.act_ks = pl.w_ks = 1;
        pl.act_kchunk = pl.op;
        pl.w_kchunk = pl.Rp;
    } else {
        pl.gpa = take(size_t(pl.act_mt * pl.act_ks) * slot);
        pl.gpw = take(size_t(pl.w_mt * pl.w_ks) * slot);
    }
    // never below kq_calib_step_noalloc's limit where the budget is above it: callers go by this
    pl.total = std::max(off, std::min(budget, size_t(KQ_CALIB_NOALLOC_MAX_BYTES) + 256));
    return pl;
}

hipError_t launch_calib_reference(const uint16_t* X, int64_t R, int64_t d, const uint16_t* W, int64_t o,
                                  float* Yneg, hipStream_t st) {
    if (R == 0 || o == 0) return hipSuccess;
    const Opnd A{reinterpret_cast<const uint8_t*>(X), R, d, d * 2}, B{reinterpret_cast<const uint8_t*>(W), o, d, d * 2};
    // 256 x 256 tiles, unless there are few of them, they need (nearly) as many rounds as 128 x 128
    // ones (two workgroups a CU), or the stores of a short K outweigh its products: there the
    // 128 x 128 workgroups of a CU store and multiply beside each other.  128 x 128 / 256 x 256, us:
    //   100000 x  100 (2, 2 rounds)   d 64: 15.3 / 22.7; 1152: 61 / 73; 3072: 186 / 181
    //   100000 x  257 (5, 4)          d 640: 72 / 91
    //    18432 x 3072 (7, 4)          d 64: 37 / 45; 160: 51.5 / 56.4; 320: 72.7 / 71.7; 640: 113 / 101
    //   100000 x 1152 (14, 8)         d 64: 94 / 108; 160: 167 / 133
    const int64_t r1 = cdiv(cdiv(R, 128) * cdiv(o, 128), 512), t2 = cdiv(R, 256) * cdiv(o, 256), r2 = cdiv(t2, 256);
    if (t2 >= 128 && 3 * r1 > 4 * r2 && d > 64 && (d > 160 || R * o > (int64_t(1) << 26))) {
        const uint32_t ntn = uint32_t(cdiv(o, 256));
        calib_reference_kernel<4, 2, 2, 4, true><<<unsigned(cdiv(R, 256) * ntn), 512, 0, st>>>(A, B, Yneg, d, ntn);
    } else {
        const uint32_t ntn = uint32_t(cdiv(o, 128));
        calib_reference_kernel<2, 2, 2, 2, false><<<unsigned(cdiv(R, 128) * ntn), 256, 0, st>>>(A, B, Yneg, d, ntn);
    }
    return hipGetLastError();
}

hipError_t launch_calib_backward(const CalibPlan& pl, const CalibStepArgs& s, int64_t nsr, hipStream_t st) {
    unsigned char* ws = s.ws;
    const int64_t R = pl.R, o = pl.o, d = pl.d;
    const Opnd rh{ws + pl.rh, pl.Rp, pl.op, pl.op * 2}, rl{ws + pl.rl, pl.Rp, pl.op, pl.op * 2};
    const double c1 = 2.0 / (double(R) * double(o));
    // (at most 1/2: what comes out near FLT_MAX still rounds to a finite bf16)
    const float c1_pow2 = float(std::ldexp(1.0, std::min(std::ilogb(c1), -1)));
    BackwardArgs b{};
    b.ntn = pl.ntn;
    // activation side: P = res . What  (M = R, N = d, K = o)
    b.act = Side{{rh, rl},
                 {ws + pl.qW, o, d, d * 2},
                 {reinterpret_cast<const uint8_t*>(s.X), R, d, d * 2},
                 reinterpret_cast<const uint32_t*>(ws + pl.mA),
                 reinterpret_cast<float*>(ws + pl.gpa),
                 pl.op,
                 pl.act_kchunk,
                 pl.act_ks,
                 pl.act_mt * pl.act_ks * pl.ntn,
                 c1_pow2,
                 reinterpret_cast<float*>(ws + pl.dA),
                 pl.strips_a,
                 c1 / c1_pow2,
                 2.0 / (double(R) * double(d)),
                 s.lambdas};
    // weight side: P = res^T . Ahat  (M = o, N = d, K = R)
    b.wgt = Side{{rh, rl},
                 {ws + pl.qA, R, d, d * 2},
                 {reinterpret_cast<const uint8_t*>(s.W), o, d, d * 2},
                 reinterpret_cast<const uint32_t*>(ws + pl.mW),
                 reinterpret_cast<float*>(ws + pl.gpw),
                 pl.Rp,
                 pl.w_kchunk,
                 pl.w_ks,
                 pl.w_mt * pl.w_ks * pl.ntn,
                 c1_pow2,
                 reinterpret_cast<float*>(ws + pl.dW),
                 pl.strips_w,
                 c1 / c1_pow2,
                 2.0 / (double(o) * double(d)),
                 s.lambdas + 1};
    const unsigned works = unsigned(b.act.works + b.wgt.works);
    if (pl.fold) calib_backward_kernel<2, 2, 2, 2, false, true><<<works, 256, 0, st>>>(b);
    else if (pl.big) calib_backward_kernel<4, 2, 2, 4, true, false><<<works, 512, 0, st>>>(b);
    else calib_backward_kernel<2, 2, 2, 2, false, false><<<works, 256, 0, st>>>(b);
    auto reduce_side = [&](const Side& x) {
        return ReduceSide{x.partial, x.sums, x.works / pl.ntn, x.strips, x.c1, x.c2_unit};
    };
    if (!pl.fold)
        gram_reduce_kernel<<<dim3(unsigned(pl.nb), 16, 2), 256, 0, st>>>(reduce_side(b.act), reduce_side(b.wgt), pl.nb, s.lambdas);
    LuGradArgs la{};
    la.lu = s.lu;
    la.ga = pl.fold ? b.act.sums : b.act.partial;
    la.ga_lo = b.act.sums;
    la.gw = pl.fold ? b.wgt.sums : b.wgt.partial;
    la.gw_lo = b.wgt.sums;
    la.nb = pl.nb;
    la.nfac = pl.nfac;
    la.grad = s.grad;
    la.lu_out = s.lu_out;
    la.adam_m = s.adam_m;
    la.adam_v = s.adam_v;
    la.adam_t = s.adam_t;
    la.lr = s.lr;
    la.sr = reinterpret_cast<double*>(ws + pl.sr);
    la.nsr = nsr;
    la.sqa = reinterpret_cast<double*>(ws + pl.sqa);
    la.nsqa = pl.nsqa;
    la.sqw = reinterpret_cast<double*>(ws + pl.sqw);
    la.nsqw = pl.nsqw;
    la.n_out = double(R) * double(o);
    la.n_a = double(R) * double(d);
    la.n_w = double(o) * double(d);
    la.lambdas = s.lambdas;
    la.losses = s.losses;
    if (pl.fold) lu_grad_kernel<false><<<unsigned(pl.nfac + 1), 256, 0, st>>>(la);
    else lu_grad_kernel<true><<<unsigned(pl.nfac + 1), 256, 0, st>>>(la);
    return hipGetLastError();
}

hipError_t launch_calib_init(float* adam_m, float* adam_v, int64_t n, float* lambdas, hipStream_t st) {
    init_kernel<<<1, 256, 0, st>>>(adam_m, adam_v, n, lambdas);
    return hipGetLastError();
}

hipError_t launch_calib_set_lambdas(const double* losses, float* lambdas, hipStream_t st) {
    set_lambdas_kernel<<<1, 64, 0, st>>>(losses, lambdas);
    return hipGetLastError();
}

}  // namespace kq
