// W4A4 MXFP4 GEMM: the consumer of the quantizer's output (Sec. 3.1 eq. (1),
// Sec. 3.4): C[M, N] (+)= deq(Xq)[M, K] . deq(Wq)[N, K]^T, both operands in
// the MXFP4 layout the quantizer writes -- codes [rows, K/2] (element 2i in
// the low nibble of byte i) and E8M0 scales [rows, K/32] -- so activations
// from kq_quantize* and weights from kq_weight_transform feed it unchanged.
//
// Matrix cores: v_mfma_scale_f32_32x32x64_f8f6f4 with both operands E2M1.  In
// that instruction lane l supplies row (A) or column (B) l % 32 and the 32
// K-values 32 (l / 32) .. 32 (l / 32) + 31 of the 64-wide K step, 16 bytes,
// plus one E8M0 byte for them: exactly one 32-element block and its scale in
// the quantizer's layout, so fragments are plain 16-byte loads and no
// re-layout or pre-shuffle of codes or scales is needed.  Products of E2M1
// values times the two scales are exact in fp32; the sum over K is
// accumulated in fp32 (order not specified).
//
// Kernels: a pipelined one on a 256 x 256 (eight waves) or 128 x 128 (four waves)
// tile of C, for K up to 2^24 (32-bit offsets within a tile), and one whose waves
// split K, on tiles of 32 x 32 to 64 x 64, for few tiles (and any K).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kq_kernels.h"
#include "kq_lds.h"

namespace kq {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16g __attribute__((ext_vector_type(16)));

namespace {

// One lane's share of a K step: the 16 code bytes of one block (as the low
// half of the 8-dword operand; E2M1 uses 4 dwords) and its scale byte.
struct Frag {
    uint4 codes;
    uint32_t scale;
};

__device__ __forceinline__ i32x8 operand(const Frag& f) {
    i32x8 v = {(int)f.codes.x, (int)f.codes.y, (int)f.codes.z, (int)f.codes.w, 0, 0, 0, 0};
    return v;
}

// C, the bias and the 16-bit C are accessed in whole vectors at any alignment of their
// elements (global memory takes such accesses, and the rows of an odd ldc start anywhere).
// With vectors only where all rows were 16-byte aligned and single elements elsewhere,
// us: 4608 x 3001 x 3072 bf16 54.9 with the quantizer, 40.0 now; 4608 x 3004 x 1152 38.8
// and 23.5 (3072 columns: 23.1); 4096 x 3001 x 1152 fp32 37.5 and 26.7.
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32b __attribute__((aligned(2)));
typedef uint32_t u32x2b __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32x4b __attribute__((ext_vector_type(4), aligned(2)));

// Four consecutive fp32 C values of row m from column n.  (One vector access: as
// float4, four members, the compiler shared the last with the other branch.)
__device__ __forceinline__ void store_c4(const GemmParams& g, int64_t m, int64_t n, float4 v) {
    float* const c = g.C + m * g.ldc_out + n;
    if (n + 3 < g.N) {
        *reinterpret_cast<f32x4*>(c) = f32x4{v.x, v.y, v.z, v.w};
    } else {
        c[0] = v.x;
        if (n + 1 < g.N) c[1] = v.y;
        if (n + 2 < g.N) c[2] = v.z;
        if (n + 3 < g.N) c[3] = v.w;
    }
}

// The values they are added to: the bias, C (accumulate) or zeros; zeros past M and N.
__device__ __forceinline__ float4 base_c4(const GemmParams& g, int64_t m, int64_t n) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* const src = g.bias ? g.bias : g.accumulate ? g.C : nullptr;
    if (src && m < g.M && n < g.N) {
        const float* const b = src + m * g.ldc_out + n;
        if (n + 3 < g.N) {
            const f32x4 o = *reinterpret_cast<const f32x4*>(b);
            v = make_float4(o.x, o.y, o.z, o.w);
        } else {
            v.x = b[0];
            if (n + 1 < g.N) v.y = b[1];
            if (n + 2 < g.N) v.z = b[2];
            if (n + 3 < g.N) v.w = b[3];
        }
    }
    return v;
}

// Four consecutive bf16 C values.
__device__ __forceinline__ void store_b4(const GemmParams& g, int64_t m, int64_t n, float4 v) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    const bf16x4 b = {(__bf16)v.x, (__bf16)v.y, (__bf16)v.z, (__bf16)v.w};
    const uint2 w = __builtin_bit_cast(uint2, b);
    uint16_t* const c = g.C16 + m * g.ldc_out + n;
    if (n + 3 < g.N) {
        *reinterpret_cast<u32x2b*>(c) = u32x2b{w.x, w.y};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < g.N) c[e] = (uint16_t)((e < 2 ? w.x : w.y) >> (16 * (e & 1)));
    }
}

// Four consecutive values of the residual as two bf16 terms (zero past M and N, up to
// rows_pad and ldr); their squares are added to sq.
__device__ __forceinline__ void store_r4(const GemmParams& g, int64_t m, int64_t n, float4 v, double& sq) {
    const bool in = m < g.M;
    const float f[4] = {in && n < g.N ? v.x : 0.f, in && n + 1 < g.N ? v.y : 0.f, in && n + 2 < g.N ? v.z : 0.f,
                        in && n + 3 < g.N ? v.w : 0.f};
    uint32_t hi[2], lo[2];
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const bf16x2 h2 = {(__bf16)f[e], (__bf16)f[e + 1]};
        const bf16x2 l2 = {(__bf16)(f[e] - (float)h2[0]), (__bf16)(f[e + 1] - (float)h2[1])};
        hi[e / 2] = __builtin_bit_cast(uint32_t, h2);
        lo[e / 2] = __builtin_bit_cast(uint32_t, l2);
        sq += (double)f[e] * (double)f[e] + (double)f[e + 1] * (double)f[e + 1];
    }
    *reinterpret_cast<uint2*>(g.rh + m * g.ldr + n) = make_uint2(hi[0], hi[1]);
    *reinterpret_cast<uint2*>(g.rl + m * g.ldr + n) = make_uint2(lo[0], lo[1]);
}

// The workgroup's sum of sq to its place (red: one entry per wave).
template <int WAVES>
__device__ __forceinline__ void block_squares(double sq, double* red, const GemmParams& g) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = red[0];
#pragma unroll
        for (int i = 1; i < WAVES; ++i) tot += red[i];
        g.sq_part[blockIdx.x] = tot;
    }
}

}  // namespace

// ------------------------------------------------------------------ pipelined kernels
// K advances 128 (four 32-blocks) per stage.  Codes and scales go from global
// memory straight into LDS (global_load_lds: lane l's 16 bytes land at the
// wave-uniform LDS address + 16 l), three stages ahead, so there is no register
// staging and no ds_write (scale rows that no such load can take: see DMA_SCALES).
constexpr int kStages = 4;  // LDS stage buffers: one in use, three in flight

// Until at most 4 * later code loads of this wave are outstanding.
__device__ __forceinline__ void wait_stage(int later) {
    if (later >= 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// LDS slot of block b of tile row q: 4 q + (b ^ ((q >> 2) & 3)).  A DMA
// instruction fills 64 consecutive slots (16 rows), so lane l reads row
// 16 i + l / 4, block (l % 4) ^ (((l / 4) >> 2) & 3): each instruction reads
// 16 contiguous 64-byte row segments, and a fragment read (32 rows, one
// block) spreads over all LDS banks.
__device__ __forceinline__ int pipe_slot(int q, int b) { return 4 * q + (b ^ ((q >> 2) & 3)); }

// Workgroup tile of BN (N) x BM (M): WN x WM waves of TN x TM instruction tiles
// of 32 x 32.  Every wave issues four code loads (16 rows x 64 bytes each) per
// stage and one scale load (64 rows x 16 bytes) per four stages.
template <int WN, int WM, int TN, int TM>
struct Tile {
    static constexpr int BN = 32 * WN * TN, BM = 32 * WM * TM, ROWS = BN + BM, WAVES = WN * WM;
    static_assert(ROWS == 64 * WAVES, "four code loads and one scale load per wave");
    // rows 0 .. BN-1 are W rows, BN .. ROWS-1 X rows, in every array
    struct Lds {
        uint4 codes[kStages][4 * ROWS];  // slot pipe_slot(row, block of the stage)
        uint4 scales[2][ROWS];           // [chunk parity][row]: the 16 scales of four stages
    };
};

// The 16 (or the last nvalid) scale bytes at p, any alignment.  Fewer than 16 come as
// up to four loads of 8, 4, 2 and 1 bytes that are all in flight before the first is
// waited for.  Byte by byte each load was waited for by itself, up to 15 memory latencies
// in a row; calls of K 320, 480, 1120 and 2240 took 3, 4, 0.6 and 1.3 % longer so.
__device__ __forceinline__ uint4 load_scales16(const uint8_t* p, int nvalid) {
    typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(1)));
    typedef uint32_t u32x2u __attribute__((ext_vector_type(2), aligned(1)));
    typedef uint32_t u32u __attribute__((aligned(1)));
    typedef uint16_t u16u __attribute__((aligned(1)));
    if (nvalid >= 16) {
        const u32x4u v = *reinterpret_cast<const u32x4u*>(p);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    u32x2u e = {0u, 0u};
    uint32_t q = 0u, d = 0u, b = 0u;
    if (nvalid & 8) e = *reinterpret_cast<const u32x2u*>(p);
    if (nvalid & 4) q = *reinterpret_cast<const u32u*>(p + (nvalid & 8));
    if (nvalid & 2) d = *reinterpret_cast<const u16u*>(p + (nvalid & 12));
    if (nvalid & 1) b = p[nvalid & 14];
    // the dword that the last 3 bytes begin
    const uint32_t tail = d | (b << (8 * (nvalid & 2)));
    uint32_t w[4] = {e.x, e.y, 0u, 0u};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i == (nvalid & 8) / 4) w[i] |= q;
        if (i == (nvalid & 12) / 4) w[i] |= tail;
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// C tile [nb0, nb0 + BN) x [mb0, mb0 + BM).  Rows past N or M read row N-1 or
// M-1 (their products land in C rows or columns that are never stored).
//
// PING (eight waves, two per SIMD): waves 4-7 run half a stage behind waves
// 0-3, held apart by one extra barrier at the start, so that on every SIMD one
// wave reads its fragments from LDS and issues loads while the other runs its
// matrix-core instructions; with both in step the LDS reads (about 770 cycles a
// stage at 128 bytes a cycle) and the matrix cores (1024 cycles) add up.
// In phase 2k waves 0-3 read stage k and issue stage k + 3, and compute it in
// phase 2k + 1; waves 4-7 do so in phases 2k + 1 and 2k + 2.  Stage k + 3
// overwrites the buffer of stage k - 1, last read in phase 2k - 1, whose reads
// have returned before that phase's barrier.  Every wave has waited for its
// loads of stage k before the barrier that ends phase 2k - 1.
//
// Per stage (K 12288 less K 3072, 216 tiles, C stores left out): 0.91 us, of which
// 0.59 is what the matrix cores take at the clock they hold; 0.75 without the
// loads, 0.69 without the matrix instructions.  Both groups in step, with three
// buffers: 1.15 us.
//
// DMA_SCALES: a scale row has a multiple of 4 bytes, at least 16, and starts
// at a multiple of 4: the 16 scales of four stages come by a DMA load per row.
// The last such load of the last row would pass the end of the array, so it
// ends there instead and is read at an offset.  Otherwise each thread loads
// its row's 16 bytes into registers (byte-exact) and parks them in LDS two
// stages later; the compiler waits for them with vmcnt(0), which drains the stages in
// flight once per four stages (the other path never does).
template <int WN, int WM, int TN, int TM, bool PING, bool DMA_SCALES>
__device__ __forceinline__ void gemm_tile(const GemmParams& g, typename Tile<WN, WM, TN, TM>::Lds& lds, int64_t nb0,
                                          int64_t mb0, f32x16g (&acc)[TN][TM]) {
    typedef Tile<WN, WM, TN, TM> T;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r = lane & 31, h = lane >> 5, wn = wave / WM, wm = wave % WM;
    const int64_t row_bytes = g.K / 2, nkb = g.K / 32;
    const int nst = (int)((nkb + 3) / 4), tb = (int)(nkb & 3);  // tb: blocks of a partial last stage
    const int nch = (int)((nkb + 15) / 16);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&lds;
    constexpr uint32_t kStageBytes = 64u * T::ROWS;
    constexpr uint32_t kScales0 = kStages * kStageBytes, kChunkBytes = 16u * T::ROWS;

    // this wave's code rows 64 wave .. 64 wave + 63 (all W or all X), its scale rows the same
    const bool isw = 64 * wave < T::BN;
    const int rel0 = 64 * wave - (isw ? 0 : T::BN);
    const int64_t row0 = (isw ? nb0 : mb0) + rel0, rows = isw ? g.N : g.M;
    const int last = (int)min<int64_t>(63, max<int64_t>(0, rows - 1 - row0));  // last row of the 64 to read
    const int64_t rowc = min(row0, rows - 1);
    const uint8_t* const cbase = (isw ? g.b_codes : g.a_codes) + rowc * row_bytes;
    const uint8_t* const sbase = (isw ? g.b_scales : g.a_scales) + rowc * nkb;
    const int q = lane >> 2, blk = (lane & 3) ^ ((q >> 2) & 3);
    uint32_t voff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) voff[i] = (uint32_t)min(16 * i + q, last) * (uint32_t)row_bytes + 16u * blk;
    const uint32_t soff = (uint32_t)min(lane, last) * (uint32_t)nkb;
    const uint32_t dst0 = lds0 + 4096u * wave, sdst0 = lds0 + kScales0 + 1024u * wave;

    auto issue_codes = [&](int st, int buf) {
        const uint8_t* const base = cbase + 64 * (int64_t)st;
        // blocks past K (a partial last stage) read its last block; they are masked below
        const uint32_t back = (tb && st == nst - 1 && blk >= tb) ? 16u * (blk - tb + 1) : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) lds_dma16(dst0 + buf * kStageBytes + 1024u * i, voff[i] - back, base);
    };
    // distance by which the last chunk's load of the matrix's last row ends early
    // (the chunk's offset is added first: a row's own offset may be smaller than it)
    const uint32_t early = DMA_SCALES ? (uint32_t)(-nkb & 15) : 0u;
    auto issue_scales = [&](int ch) {
        const bool back = early && ch == nch - 1 && row0 + min(lane, last) >= rows - 1;
        lds_dma16(sdst0 + (ch & 1) * kChunkBytes, soff + 16u * ch - (back ? early : 0u), sbase);
    };
    uint4 parked = make_uint4(0u, 0u, 0u, 0u);
    auto fetch_scales = [&](int ch) {
        parked = load_scales16(sbase + soff + 16 * (int64_t)ch, (int)min<int64_t>(16, nkb - 16 * (int64_t)ch));
    };
    auto park_scales = [&](int ch) { lds.scales[ch & 1][threadIdx.x] = parked; };

    // fragment and scale addresses of this lane
    const uint32_t psel = h ? 0x0c0c0301u : 0x0c0c0200u;
    const int wrow = wn * 32 * TN + r, xrow = T::BN + wm * 32 * TM + r;
    const uint4* const sc0 = lds.scales[0];
    uint32_t late = 0;  // bit i (W) or 8 + j (X): this lane's row is the matrix's last
    if (DMA_SCALES && early) {
#pragma unroll
        for (int i = 0; i < TN; ++i) late |= (nb0 + wrow + 32 * i >= g.N - 1 ? 1u : 0u) << i;
#pragma unroll
        for (int j = 0; j < TM; ++j) late |= (mb0 + xrow - T::BN + 32 * j >= g.M - 1 ? 1u : 0u) << (8 + j);
    }
    struct Frags {
        uint4 w[2][TN], x[2][TM];
        uint32_t sw[TN], sx[TM];
    };
    auto read_frags = [&](int st, int buf, int j4, Frags& f) {
        const uint4* const cb = lds.codes[buf];
        const int ch = st >> 2;
        const uint32_t* const sp = reinterpret_cast<const uint32_t*>(sc0 + (ch & 1) * T::ROWS) + j4;
        if (DMA_SCALES && early && ch == nch - 1) {
            const uint32_t e = early / 4;
#pragma unroll
            for (int i = 0; i < TN; ++i) f.sw[i] = sp[4 * (wrow + 32 * i) + ((late >> i) & 1u) * e];
#pragma unroll
            for (int j = 0; j < TM; ++j) f.sx[j] = sp[4 * (xrow + 32 * j) + ((late >> (8 + j)) & 1u) * e];
        } else {
#pragma unroll
            for (int i = 0; i < TN; ++i) f.sw[i] = sp[4 * (wrow + 32 * i)];
#pragma unroll
            for (int j = 0; j < TM; ++j) f.sx[j] = sp[4 * (xrow + 32 * j)];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int i = 0; i < TN; ++i) f.w[s][i] = cb[pipe_slot(wrow + 32 * i, 2 * s + h)];
#pragma unroll
            for (int j = 0; j < TM; ++j) f.x[s][j] = cb[pipe_slot(xrow + 32 * j, 2 * s + h)];
        }
    };
    // scales to the byte order of the instruction's selectors; blocks past K: zero codes, scale 1
    auto finish_frags = [&](int st, Frags& f) {
#pragma unroll
        for (int i = 0; i < TN; ++i) f.sw[i] = __builtin_amdgcn_perm(0u, f.sw[i], psel);
#pragma unroll
        for (int j = 0; j < TM; ++j) f.sx[j] = __builtin_amdgcn_perm(0u, f.sx[j], psel);
        if (tb && st == nst - 1) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bool past = 2 * s + h >= tb;
                const uint32_t keep = past ? 0u : ~0u;
                const uint32_t one = past ? 127u << (8 * s) : 0u, smask = past ? ~(255u << (8 * s)) : ~0u;
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    f.w[s][i] = make_uint4(f.w[s][i].x & keep, f.w[s][i].y & keep, f.w[s][i].z & keep, f.w[s][i].w & keep);
                    f.sw[i] = (f.sw[i] & smask) | one;
                }
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    f.x[s][j] = make_uint4(f.x[s][j].x & keep, f.x[s][j].y & keep, f.x[s][j].z & keep, f.x[s][j].w & keep);
                    f.sx[j] = (f.sx[j] & smask) | one;
                }
            }
        }
    };
    auto products = [&](const Frags& f) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(Frag{f.w[0][i], 0u}),
                                                                             operand(Frag{f.x[0][j], 0u}), acc[i][j], 4, 4,
                                                                             0, (int)f.sw[i], 0, (int)f.sx[j]);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(Frag{f.w[1][i], 0u}),
                                                                             operand(Frag{f.x[1][j], 0u}), acc[i][j], 4, 4,
                                                                             1, (int)f.sw[i], 1, (int)f.sx[j]);
    };

#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = f32x16g{};
    if (DMA_SCALES) issue_scales(0);
    else fetch_scales(0);
#pragma unroll
    for (int s = 0; s < kStages - 1; ++s)
        if (s < nst) issue_codes(s, s);
    if (!DMA_SCALES) {
        park_scales(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    const bool behind = PING && wave >= T::WAVES / 2;

    // stage st in buffer J = st % 4
    auto stage = [&](int st, auto Jc) {
        constexpr int J = decltype(Jc)::value;
        Frags f;
        read_frags(st, J, J, f);
        if (DMA_SCALES) {
            if (J == 0 && (st >> 2) + 1 < nch) issue_scales((st >> 2) + 1);
        } else {
            if (J == 2 && (st >> 2) + 1 < nch) park_scales((st >> 2) + 1);
            if (J == 0 && (st >> 2) + 1 < nch) fetch_scales((st >> 2) + 1);
        }
        if (st + 3 < nst) issue_codes(st + 3, (J + 3) & 3);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        finish_frags(st, f);
        if (PING) {
            if (behind) wait_stage(nst - 2 - st);
            stage_barrier();
            products(f);
            if (!behind) wait_stage(nst - 2 - st);
            stage_barrier();
        } else {
            products(f);
            wait_stage(nst - 2 - st);
            stage_barrier();
        }
    };
    wait_stage(nst - 1);
    stage_barrier();
    if (behind) stage_barrier();
    for (int st = 0; st < nst; st += 4) {
        stage(st, std::integral_constant<int, 0>{});
        if (st + 1 < nst) stage(st + 1, std::integral_constant<int, 1>{});
        if (st + 2 < nst) stage(st + 2, std::integral_constant<int, 2>{});
        if (st + 3 < nst) stage(st + 3, std::integral_constant<int, 3>{});
    }
    if (PING && !behind) stage_barrier();
}

// The tile's accumulators, acc[i][j][4q + e] = C[mb0 + 32 (wm TM + j) + r][nb0 +
// 32 (wn TN + i) + 8 q + 4 h + e], to C through LDS, so that C (and the bias) is
// accessed along its rows, 512 bytes at a time, and not in 8- or 16-byte pieces
// of 32 rows (4608 x 12288 x 3072, bf16 / fp32: 141 / 155 us so, 119 / 131 along rows).
// Rows in LDS are 16 bytes apart from a multiple of 512 (256), so that the 16 rows of a
// write phase cover all banks.  When a tile of fp32 does not fit, it goes in NP passes of
// TN / NP of every wave's column tiles.
//
// OUT 0: fp32 (bias, accumulate); 1: bf16; 2: the residual v = bias + product as its
// two bf16 terms hi = bf16(v), lo = bf16(v - hi), zero in the padding columns and
// rows up to ldr and rows_pad, and the workgroup's sum of v^2 (fp64).
//
// BASE (the bias or C is added): all loads of a pass are issued before its stores (a
// wait for a load waits for every store issued before it too).
// 4096 x 5600 x 2240 and 18432 x 3072 x 3072 onto C, us: 104 and 220 with the loads
// among the stores, 88 and 188 so.
template <int WN, int WM, int TN, int TM, int OUT, bool BASE>
__device__ __forceinline__ void store_tile(const GemmParams& g, uint8_t* lds, int64_t nb0, int64_t mb0,
                                           const f32x16g (&acc)[TN][TM]) {
    typedef Tile<WN, WM, TN, TM> T;
    constexpr bool BF16 = OUT == 1;
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int NP = (T::BM * (T::BN * ES + 16) <= (int)sizeof(typename T::Lds)) ? 1 : 2;
    constexpr int TP = TN / NP;                    // column tiles per wave and pass
    constexpr int RB = T::BN / NP * ES, RS = RB + 16;  // data and stride of a row in bytes
    static_assert(T::BM * RS <= (int)sizeof(typename T::Lds), "a pass fits LDS");
    constexpr int CPR = RB / 16, EPC = 16 / ES;    // 16-byte chunks per row, elements per chunk
    constexpr int STEP = 64 * T::WAVES / CPR;      // rows that the workgroup covers at a time
    constexpr int CH = T::BM / STEP;               // chunks per thread and pass
    static_assert(64 * T::WAVES % CPR == 0, "a thread keeps its column");
    const int t = threadIdx.x;
    const int wave = t >> 6, lane = t & 63;
    const int r = lane & 31, h = lane >> 5, wn = wave / WM, wm = wave % WM;
    const int last = (int)min<int64_t>(T::BM, g.M - mb0) - 1;  // the tile's last row of C
    // A thread takes one chunk of columns of every STEP-th row: whether the chunk is whole,
    // cut by N or past it is decided once a pass.  Decided for every chunk, in nested
    // branches, and so: 1000 x 1152 x 1152 onto C 12.3 and 8.8 us, fp32 8.6 and 7.8, bf16 7.3
    // and 7.0; 4096 x 5600 x 2240 onto C 76 and 67; 18432 x 3072 x 3072 onto C 169 and 151.
    const int trow = t / CPR, cl = t % CPR * EPC, seg = cl / (32 * TP);
    float4 base[BASE ? CH : 1];
    double sq = 0.0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        // column of C of this thread's chunk: the pass holds TP tiles of each of the WN waves' column ranges
        const int64_t n = nb0 + seg * 32 * TN + 32 * p * TP + (cl - seg * 32 * TP);
        const bool whole = n + EPC <= g.N;
        if (p > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                uint8_t* const dst = lds + (32 * (wm * TM + j) + r) * RS + (32 * (wn * TP + i) + 4 * h) * ES;
                const f32x16g& c = acc[p * TP + i][j];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (BF16) {
                        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
                        const bf16x4 v = {(__bf16)c[4 * q], (__bf16)c[4 * q + 1], (__bf16)c[4 * q + 2], (__bf16)c[4 * q + 3]};
                        *reinterpret_cast<uint2*>(dst + 16 * q) = __builtin_bit_cast(uint2, v);
                    } else {
                        *reinterpret_cast<float4*>(dst + 32 * q) =
                            make_float4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
                    }
                }
            }
        __builtin_amdgcn_sched_barrier(0);  // the pass's accumulators are free for what is loaded
        if (BASE) {
            // rows past M load this thread's first row again (or the tile's first); not used
            const float* const src = (g.bias ? g.bias : g.C) + mb0 * g.ldc_out + n;
            const float* const first = src + (trow <= last ? trow : 0) * g.ldc_out;
#pragma unroll
            for (int k = 0; k < CH; ++k) base[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (whole) {
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    const float* const b = trow + k * STEP <= last ? first + k * STEP * g.ldc_out : first;
                    const f32x4 o = *reinterpret_cast<const f32x4*>(b);
                    base[k] = make_float4(o.x, o.y, o.z, o.w);
                }
            } else if (n < g.N) {
                const int left = (int)(g.N - 1 - n);  // 0 to 2; columns past N load the last one again
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    const float* const b = trow + k * STEP <= last ? first + k * STEP * g.ldc_out : first;
                    base[k] = make_float4(b[0], b[min(1, left)], b[left], 0.f);
                }
            }
        }
        __syncthreads();
        const uint8_t* const from = lds + trow * RS + 16 * (t % CPR);
        auto value = [&](int k) {
            float4 f = *reinterpret_cast<const float4*>(from + k * STEP * RS);
            if (BASE) f = make_float4(base[k].x + f.x, base[k].y + f.y, base[k].z + f.z, base[k].w + f.w);
            return f;
        };
        const int64_t at = (mb0 + trow) * g.ldc_out + n;
        if (OUT == 2) {
            if (n < g.ldr) {
#pragma unroll
                for (int k = 0; k < CH; ++k)
                    if (mb0 + trow + k * STEP < g.rows_pad) store_r4(g, mb0 + trow + k * STEP, n, value(k), sq);
            }
        } else if (whole) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                if (trow + k * STEP > last) break;
                if (BF16) {
                    const uint4 v = *reinterpret_cast<const uint4*>(from + k * STEP * RS);
                    *reinterpret_cast<u32x4b*>(g.C16 + at + k * STEP * g.ldc_out) = u32x4b{v.x, v.y, v.z, v.w};
                } else {
                    const float4 f = value(k);
                    *reinterpret_cast<f32x4*>(g.C + at + k * STEP * g.ldc_out) = f32x4{f.x, f.y, f.z, f.w};
                }
            }
        } else if (n < g.N) {
            const int left = (int)(g.N - 1 - n);
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                if (trow + k * STEP > last) break;
                if (BF16) {  // 1 to 7 values, as four, two and one
                    const uint4 v = *reinterpret_cast<const uint4*>(from + k * STEP * RS);
                    uint16_t* const c = g.C16 + at + k * STEP * g.ldc_out;
                    const int n = left + 1;
                    if (n & 4) *reinterpret_cast<u32x2b*>(c) = u32x2b{v.x, v.y};
                    if (n & 2) *reinterpret_cast<u32b*>(c + (n & 4)) = n & 4 ? v.z : v.x;
                    if (n & 1) c[n & 6] = (uint16_t)(n & 4 ? (n & 2 ? v.w : v.z) : (n & 2 ? v.y : v.x));
                } else {
                    const float4 f = value(k);
                    float* const c = g.C + at + k * STEP * g.ldc_out;
                    c[0] = f.x;
                    if (left >= 1) c[1] = f.y;
                    if (left >= 2) c[2] = f.z;
                }
            }
        }
    }
    if (OUT == 2) {
        __syncthreads();
        block_squares<T::WAVES>(sq, reinterpret_cast<double*>(lds), g);
    }
}

// Tile of workgroup blockIdx.x of gx x gy tiles.  Workgroups
// are dealt to the 8 XCDs round-robin by linear id, so XCD k runs ids
// k, k + 8, ...; those get consecutive logical ids (a bijection for any
// count), and logical ids walk the tiles in groups of 4 M rows (N fastest
// within a group, M fastest within a column), so each XCD's L2 sees a compact
// block of about 4 x (T / 32) tiles instead of every M row.
__device__ __forceinline__ void xcd_tile(int64_t gx, int64_t gy, int64_t& tn, int64_t& tm) {
    const int64_t T = gx * gy;
    const int64_t i = blockIdx.x;
    const int64_t k = i % 8, j = i / 8;
    const int64_t L = k * (T / 8) + (k < T % 8 ? k : T % 8) + j;
    constexpr int64_t GM = 4;
    const int64_t gsize = GM * gx;
    const int64_t first_m = (L / gsize) * GM;
    const int64_t gm = gy - first_m < GM ? gy - first_m : GM;
    tm = first_m + (L % gsize) % gm;
    tn = (L % gsize) / gm;
}

// Few tiles: W waves share one tile of 32 TM (M) x 32 TN (N), each taking every W-th
// 128-wide chunk of K with fragments straight from global memory (D chunks in flight),
// and their sums meet in LDS in wave order.  With fewer tiles than CUs the pipelined
// kernels walk K alone, a memory latency or more per few stages; here K is as wide as
// the workgroup.
template <int TN, int TM, int W, int D>
__global__ __launch_bounds__(64 * W) void mxfp4_gemm_split_kernel(const GemmParams g, int64_t gx, int64_t gy) {
    constexpr int BN = 32 * TN, BM = 32 * TM, RS = BN + 4;  // LDS row in floats
    __shared__ float sums[W * BM * RS];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int r = lane & 31, h = lane >> 5;
    int64_t tn, tm;
    xcd_tile(gx, gy, tn, tm);
    const int64_t nb0 = tn * BN, mb0 = tm * BM, nkb = g.K / 32, row_bytes = g.K / 2;
    const int nch = (int)((nkb + 3) / 4), tb = (int)(nkb & 3);
    // rows past N or M read the last row (their sums are never stored)
    const uint8_t *cw[TN], *cx[TM], *sw[TN], *sx[TM];
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const int64_t n = min(nb0 + 32 * i + r, g.N - 1);
        cw[i] = g.b_codes + n * row_bytes;
        sw[i] = g.b_scales + n * nkb;
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int64_t m = min(mb0 + 32 * j + r, g.M - 1);
        cx[j] = g.a_codes + m * row_bytes;
        sx[j] = g.a_scales + m * nkb;
    }
    struct Chunk {
        uint4 w[2][TN], x[2][TM];
        uint32_t sw[TN], sx[TM];
    };
    auto scales4 = [&](const uint8_t* p, int valid) {
        typedef uint32_t u32u __attribute__((aligned(1)));
        if (valid >= 4) return *reinterpret_cast<const u32u*>(p);
        uint32_t v = p[0];
        if (valid > 1) v |= (uint32_t)p[1] << 8;
        if (valid > 2) v |= (uint32_t)p[2] << 16;
        return v;
    };
    auto load = [&](int c, Chunk& f) {
        const int valid = (tb && c == nch - 1) ? tb : 4;  // blocks of the chunk; those past K read its last block
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int64_t at = 16 * (4 * (int64_t)c + min(2 * s + h, valid - 1));
#pragma unroll
            for (int i = 0; i < TN; ++i) f.w[s][i] = *reinterpret_cast<const uint4*>(cw[i] + at);
#pragma unroll
            for (int j = 0; j < TM; ++j) f.x[s][j] = *reinterpret_cast<const uint4*>(cx[j] + at);
        }
#pragma unroll
        for (int i = 0; i < TN; ++i) f.sw[i] = scales4(sw[i] + 4 * (int64_t)c, valid);
#pragma unroll
        for (int j = 0; j < TM; ++j) f.sx[j] = scales4(sx[j] + 4 * (int64_t)c, valid);
    };
    const uint32_t psel = h ? 0x0c0c0301u : 0x0c0c0200u;
    f32x16g acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = f32x16g{};
    auto multiply = [&](int c, Chunk& f) {
#pragma unroll
        for (int i = 0; i < TN; ++i) f.sw[i] = __builtin_amdgcn_perm(0u, f.sw[i], psel);
#pragma unroll
        for (int j = 0; j < TM; ++j) f.sx[j] = __builtin_amdgcn_perm(0u, f.sx[j], psel);
        if (tb && c == nch - 1) {  // blocks past K: zero codes, scale 1
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bool past = 2 * s + h >= tb;
                const uint32_t keep = past ? 0u : ~0u, one = past ? 127u << (8 * s) : 0u, sm = past ? ~(255u << (8 * s)) : ~0u;
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    f.w[s][i] = make_uint4(f.w[s][i].x & keep, f.w[s][i].y & keep, f.w[s][i].z & keep, f.w[s][i].w & keep);
                    f.sw[i] = (f.sw[i] & sm) | one;
                }
#pragma unroll
                for (int j = 0; j < TM; ++j) f.sx[j] = (f.sx[j] & sm) | one;
            }
        }
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(Frag{f.w[0][i], 0u}),
                                                                             operand(Frag{f.x[0][j], 0u}), acc[i][j], 4, 4,
                                                                             0, (int)f.sw[i], 0, (int)f.sx[j]);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(operand(Frag{f.w[1][i], 0u}),
                                                                             operand(Frag{f.x[1][j], 0u}), acc[i][j], 4, 4,
                                                                             1, (int)f.sw[i], 1, (int)f.sx[j]);
    };
    Chunk f[D];
#pragma unroll
    for (int u = 0; u < D; ++u)
        if (wave + u * W < nch) load(wave + u * W, f[u]);
    for (int c = wave; c < nch; c += D * W) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int cu = c + u * W;
            if (cu < nch) {
                multiply(cu, f[u]);
                if (cu + D * W < nch) load(cu + D * W, f[u]);
            }
        }
    }
    // acc[i][j][4q + e] = (row 32 j + r, column 32 i + 8 q + 4 h + e)
    const int active = min(W, nch);
    if (wave < active) {
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(sums + (wave * BM + 32 * j + r) * RS + 32 * i + 8 * q + 4 * h) =
                        make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    }
    __syncthreads();
    const int64_t mend = g.rh ? g.rows_pad : g.M, nend = g.rh ? g.ldr : g.N;
    double sq = 0.0;
    for (int k = t; k < BM * BN / 4; k += 64 * W) {
        const int row = k / (BN / 4), col = 4 * (k % (BN / 4));
        const int64_t m = mb0 + row, n = nb0 + col;
        if (m >= mend || n >= nend) continue;
        const bool based = g.bias || g.accumulate;
        const float4 b = based ? base_c4(g, m, n) : make_float4(0.f, 0.f, 0.f, 0.f);
        float4 v = *reinterpret_cast<const float4*>(sums + row * RS + col);
        for (int w = 1; w < active; ++w) {
            const float4 o = *reinterpret_cast<const float4*>(sums + (w * BM + row) * RS + col);
            v = make_float4(v.x + o.x, v.y + o.y, v.z + o.z, v.w + o.w);
        }
        if (based) v = make_float4(b.x + v.x, b.y + v.y, b.z + v.z, b.w + v.w);
        if (g.C16) store_b4(g, m, n, v);
        else if (g.rh) store_r4(g, m, n, v, sq);
        else store_c4(g, m, n, v);
    }
    if (g.rh) {
        __shared__ double red[W];
        block_squares<W>(sq, red, g);
    }
}

// OUT, BASE: as store_tile (one kernel each: every epilogue in one is 78 KB of code).
template <int WN, int WM, int TN, int TM, bool PING, bool DMA_SCALES, int OUT, bool BASE>
__global__ __launch_bounds__(64 * WN * WM) void mxfp4_gemm_pipe_kernel(const GemmParams g, int64_t gx, int64_t gy) {
    typedef Tile<WN, WM, TN, TM> T;
    __shared__ typename T::Lds lds;
    int64_t tn, tm;
    xcd_tile(gx, gy, tn, tm);
    f32x16g acc[TN][TM];
    gemm_tile<WN, WM, TN, TM, PING, DMA_SCALES>(g, lds, tn * T::BN, tm * T::BM, acc);
    uint8_t* const stage = reinterpret_cast<uint8_t*>(&lds);
    store_tile<WN, WM, TN, TM, OUT, BASE>(g, stage, tn * T::BN, tm * T::BM, acc);
}

// The pipelined kernels index a tile's 256 rows with 32-bit byte offsets.
constexpr int64_t kPipeMaxK = int64_t(1) << 24;

// Tile of a call.  Measured, us (bf16 C, K 512 / 1152 / 3072 / 9600):
//   32 x 32 split (8 waves)     128 x  512: 3.4 / 3.8 /  7.0 / 11.0; 128 x 128 4.7 / 6.7 / 11.9 / 30.3
//   32 (M) x 64 (N) split       256 x 1152: 3.9 / 4.4 /  9.2 / 15.3; 32 x 32 3.9 / 4.5 / 10.9 / 19.0
//   64 x 64 split               512 x 2048: 5.0 / 6.0 / 12.2 / 24.9; 128 x 128 5.0 / 6.9 / 12.0 / 30.7
//   128 x 128 pipelined         512 x 4096: 5.4 / 7.4 / 12.9 / 32.0; 64 x 64 8.6 / 10.6 / 22.8 / 48.2
//                              4096 x 2048: 8.4 / 12.1 / 23.9 / 62.5; 256 x 256 11.2 / 15.1 / 25.8 / 63.8
//   256 x 256 pipelined        3000 x 3000: 11.1 / 15.5 / 25.8 / 63.9; 128 x 128 10.8 / 16.1 / 30.8 / 83.7
// So the smallest split tile that still gives a CU no more than one workgroup, and
// past 256 tiles of 64 x 64 the pipelined tile that needs fewer rounds (two 128 x
// 128 workgroups share a CU and take as long as one of 256 x 256).  But:
//
// K <= 1536: stores (and C, where it is added to) take as long as the products, and of two
// workgroups on a CU one stores while the other multiplies.  There 128 x 128 unless
// it needs twice the rounds.  128 x 128 over 256 x 256, in time, 39 sizes with more rounds but
// less than twice: K 1152 0.72 - 0.97, 1536 0.75 - 1.01, 1920 0.77 - 1.09, 2240 0.83 - 1.16
// (onto C 0.72 - 0.95, 0.75 - 0.96, 0.78 - 0.98, 0.83 - 1.04); with twice the rounds 0.83 - 1.10 at
// 1152, 0.86 - 1.14 at 1536.  For the residual, which moves 8 bytes an element and has the
// most work besides, at any number of rounds: the calibration step by 256 x 256 and 128 x
// 128 tiles, us: 9216 x 512 x 2048 158, 147; 6000 x 1024 x 2900 223, 204; 4096 x 1152 x 4608
// 271, 259; 18432 x 1152 x 3072 626, 614; 8192 x 1536 x 3072 387, 381; 18432 x 3072 x 3072 1295, 1300.
// K <= 128, a single stage: 128 x 128 always (0.79 - 1.03).
//
// N <= 32 with more than 256 tiles of 32 x 32 (C is four times narrower than a 128 x 128
// tile): 32 x 32 tiles of two waves, many on a CU.  Not the residual, whose sums of
// squares have room for one a tile of 64 x 64.  128 x 128 and so, us, K 64 / 480 / 1152 /
// 3072: 18432 x 32 4.2 / 5.5 / 6.8 / 12.2 and 3.8 / 4.3 / 5.7 / 15.6; 70000 x 8 onto C
// 11.1 / 14.5 / 20.3 / 33.9 and 6.7 / 8.0 / 13.5 / 33.7.
enum class GemmTile { Thin32, Split32, Split32x64, Split64, Pipe128, Pipe256 };

static GemmTile gemm_tile_of(const GemmParams& g) {
    auto tiles = [&](int64_t tm, int64_t tn) { return ((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn); };
    if (tiles(32, 32) <= 256) return GemmTile::Split32;
    if (g.N <= 32 && g.K <= 1152 && !g.rh) return GemmTile::Thin32;
    if (tiles(32, 64) <= 256) return GemmTile::Split32x64;
    if (tiles(64, 64) <= 256 || g.K > kPipeMaxK) return GemmTile::Split64;
    const int64_t rounds128 = (tiles(128, 128) + 511) / 512, rounds256 = (tiles(256, 256) + 255) / 256;
    if (g.K <= 1536 && (g.rh || rounds128 < 2 * rounds256)) return GemmTile::Pipe128;
    return g.K <= 128 || rounds128 <= rounds256 ? GemmTile::Pipe128 : GemmTile::Pipe256;
}

int64_t mxfp4_gemm_workgroups(const GemmParams& g) {
    auto tiles = [&](int64_t tm, int64_t tn) { return ((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn); };
    switch (gemm_tile_of(g)) {
        case GemmTile::Thin32:
        case GemmTile::Split32: return tiles(32, 32);
        case GemmTile::Split32x64: return tiles(32, 64);
        case GemmTile::Split64: return tiles(64, 64);
        case GemmTile::Pipe128: return tiles(128, 128);
        default: return tiles(256, 256);
    }
}

template <int TN, int TM, int W, int D>
static void launch_split(const GemmParams& g, hipStream_t st) {
    const int64_t gx = (g.N + 32 * TN - 1) / (32 * TN), gy = (g.M + 32 * TM - 1) / (32 * TM);
    hipLaunchKernelGGL((mxfp4_gemm_split_kernel<TN, TM, W, D>), dim3((unsigned)(gx * gy)), dim3(64 * W), 0, st, g, gx, gy);
}

template <int WN, int WM, int TN, int TM, bool PING, bool DMA_SCALES>
static void launch_pipe_out(const GemmParams& g, hipStream_t st) {
    typedef Tile<WN, WM, TN, TM> T;
    const int64_t gx = (g.N + T::BN - 1) / T::BN, gy = (g.M + T::BM - 1) / T::BM;
    const dim3 grid((unsigned)(gx * gy)), b(64 * T::WAVES);
#define KQ_PIPE(OUT, BASE) \
    hipLaunchKernelGGL((mxfp4_gemm_pipe_kernel<WN, WM, TN, TM, PING, DMA_SCALES, OUT, BASE>), grid, b, 0, st, g, gx, gy)
    if (g.C16) KQ_PIPE(1, false);
    else if (g.rh) KQ_PIPE(2, true);
    else if (g.bias || g.accumulate) KQ_PIPE(0, true);
    else KQ_PIPE(0, false);
#undef KQ_PIPE
}

template <int WN, int WM, int TN, int TM, bool PING>
static void launch_pipe(const GemmParams& g, hipStream_t st) {
    const int64_t nkb = g.K / 32;
    if (nkb % 4 == 0 && nkb >= 16 && g.scales_aligned) launch_pipe_out<WN, WM, TN, TM, PING, true>(g, st);
    else launch_pipe_out<WN, WM, TN, TM, PING, false>(g, st);
}

hipError_t launch_mxfp4_gemm(const GemmParams& g, hipStream_t st) {
    switch (gemm_tile_of(g)) {
        case GemmTile::Thin32: launch_split<1, 1, 2, 4>(g, st); break;
        case GemmTile::Split32: launch_split<1, 1, 8, 4>(g, st); break;
        case GemmTile::Split32x64: launch_split<2, 1, 8, 3>(g, st); break;
        case GemmTile::Split64: launch_split<2, 2, 8, 2>(g, st); break;
        case GemmTile::Pipe128: launch_pipe<2, 2, 2, 2, false>(g, st); break;
        case GemmTile::Pipe256: launch_pipe<2, 4, 4, 2, true>(g, st); break;
    }
    return hipGetLastError();
}

}  // namespace kq
