// Dense layers of the DNN chemistry integrator on gfx950 matrix cores.
//
// C[M][N] = act(A[M][K] . B[N][K]^T + bias[N]), A = activations (one row per
// cell), B = weights (out x in, row-major), bf16 inputs, fp32 accumulation
// with v_mfma_f32_16x16x32_bf16, GELU epilogue, bf16 output.
// Block tile 128 x 160 with four wave64s in a 2 x 2 arrangement, each wave
// owning a 64 x 80 sub-tile (4 x 5 MFMA tiles); operands are staged through
// LDS 64 deep in K by loads that write LDS directly, one or three stages ahead
// of the MFMAs.  The MFMAs take the weight fragment as their first operand, so
// that each lane ends with four consecutive
// outputs of one row, converted with one packed bf16 conversion pair: the GELU
// epilogues (inference, with GELU from an LDS table, and the training forward and
// backward) stage them per wave in LDS and write 16-byte row pieces.  Tiles sharing
// the same rows of A are mapped to the same XCD so the A
// panel is fetched into that XCD's L2 once.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "df_fp8.h"
#include "df_internal.h"
#include "df_phi_table.h"

namespace df {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int BM = kGemmBM, BN = kGemmBN, BK = kGemmBK;
constexpr int kThreads = 256;
constexpr int WM = 64, WN = 80;          // per-wave sub-tile
constexpr int TM = WM / 16, TN = WN / 16;  // MFMA tiles per wave

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// GELU(x) = x Phi(x) of the inference and training epilogues without branches: Phi(x) = erfc(-x/sqrt 2) / 2,
// with erfc(a) for a >= 0 from the Chebyshev fit erfcc of Press et al., Numerical Recipes
// (Sec. 6.2), erfc(a) = t exp(-a^2 + P(t)), t = 1 / (1 + a/2), fractional error below 1.2e-7
// for every a >= 0; for x >= 0, Phi = 1 - erfc(x/sqrt 2) / 2.  Its error is far below the bf16
// rounding that follows.  NaN stays NaN; GELU(+inf) = +inf, GELU(-inf) = NaN as x Phi(x) gives.
__device__ __forceinline__ float phi_erfc(float x) {
    const float z = x * 0.70710678118654752f;
    const float a = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(1.0f + 0.5f * a);
    float q = 0.17087277f;
    q = fmaf(q, t, -0.82215223f);
    q = fmaf(q, t, 1.48851587f);
    q = fmaf(q, t, -1.13520398f);
    q = fmaf(q, t, 0.27886807f);
    q = fmaf(q, t, -0.18628806f);
    q = fmaf(q, t, 0.09678418f);
    q = fmaf(q, t, 0.37409196f);
    q = fmaf(q, t, 1.00002368f);
    q = fmaf(q, t, -1.26551223f);
    const float h = 0.5f * t * __expf(fmaf(-a, a, q));  // erfc(a) / 2
    return (z >= 0.0f) ? 1.0f - h : h;
}
__device__ __forceinline__ float gelu_erfc(float x) { return x * phi_erfc(x); }

// four floats to bf16 with two packed conversions (v_cvt_pk_bf16_f32): round to nearest even and
// NaN kept, except that fp32 subnormal inputs (|x| < 2^-126) are rounded toward zero, at most one
// bf16 subnormal unit (2^-133) from the nearest-even result
__device__ __forceinline__ bf16x4 to_bf16x4(floatx4 v) { return __builtin_convertvector(v, bf16x4); }

// d GELU / dx = Phi(x) + x phi(x), Phi as in gelu_erfc (no branches)
__device__ __forceinline__ float gelu_grad(float x) {
    return fmaf(x * 0.39894228040143268f, __expf(-0.5f * x * x), phi_erfc(x));
}

// GELU of the inference epilogues, GELU(x) = x Phi(x), with Phi from the table of one cubic per
// interval of 12/256 on [-6, 6] (kPhiTable, from erfc in double), which the block keeps in LDS.
// Interpolation error 1.5e-9; the position s = x 256/12 is rounded relative to x, so with the
// float32 evaluation the result is within about 1e-7 of x Phi(x), as close as gelu_erfc, so that
// the bf16 rounding that follows differs from that of the exact value as rarely.  Beyond the table
// Phi is 0 (x < -6 - 12/256, where the exact value is below 7e-10) or 1 (x >= 6).  NaN stays NaN;
// GELU(+inf) = +inf and GELU(-inf) = NaN, as x Phi(x) gives.  About 11 VALU instructions and one
// 16-byte LDS read per value, against about 28 instruction slots for gelu_erfc (reciprocal and
// exponential at a quarter of the rate).
constexpr int kPhiLdsFloats = 4 * kPhiEntries;  // 4,128 bytes of LDS per block

__device__ __forceinline__ float gelu_tab(float x, const float *__restrict__ tab) {
    constexpr float kScale = float(kPhiIntervals) / 12.0f, kHalf = 0.5f * float(kPhiIntervals);
    // position in intervals from 0, clamped to the table: entry 0 (zeros) below -6, entries
    // 1 .. kPhiIntervals the cubics, entry kPhiIntervals + 1 from 6 on; fmaxf maps NaN to entry 0
    const float s = fminf(fmaxf(x * kScale, -kHalf - 1.0f), kHalf);
    const int k = int(floorf(s)) + int(kHalf) + 1;  // 0 .. kPhiIntervals + 1
    const float u = __builtin_amdgcn_fractf(s);
    const floatx4 c = *reinterpret_cast<const floatx4 *>(tab + 4 * k);
    return x * fmaf(fmaf(fmaf(c[3], u, c[2]), u, c[1]), u, c[0]);
}

// copies the table into the block's LDS copy in 16-byte pieces; a barrier must follow before the
// first gelu_tab
template <int NT = kThreads>
__device__ __forceinline__ void copy_phi_table(float *__restrict__ lds, int t) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(kPhiTable);
    u32x4 *dst = reinterpret_cast<u32x4 *>(lds);
    for (int i = t; i < kPhiLdsFloats / 4; i += NT) dst[i] = src[i];
}

// Output staging of the inference epilogues: a wave writes rows of 160 output bytes (80 bf16 or
// 160 FP8 values) into its own LDS region, stride 176 bytes, and then stores them as 16-byte
// pieces, consecutive lanes along a row.  In the MFMA layout a store covers 16 rows x 32 bytes
// (bf16) or 16 bytes (FP8); a store-only probe of the first layer's tiles measured that 1.7 times
// slower than row pieces (65,536 x 1600 bf16: 55.4 against 32.5 us, a plain stream 32.5 us).
constexpr int kStgRowB = 160, kStgStrideB = kStgRowB + 16;

// the wave's own LDS region: its LDS operations execute in order, so reads after writes see them
// and later writes follow earlier reads; the fences keep the compiler from moving LDS accesses
// across
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ROWS staged rows to dst (the first row's first byte, 16-byte aligned), ld_bytes apart
template <int ROWS>
__device__ __forceinline__ void stage_flush(const uint8_t *stg, uint8_t *dst, int64_t ld_bytes, int lane) {
    constexpr int kPer = kStgRowB / 16, kPieces = ROWS * kPer;
    static_assert(kPieces % 64 == 0, "whole waves of pieces");
    wave_lds_fence();
#pragma unroll
    for (int p0 = 0; p0 < kPieces; p0 += 64) {
        const int c = p0 + lane, r = c / kPer, ch = c % kPer;
        const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + r * kStgStrideB + ch * 16);
        *reinterpret_cast<u32x4 *>(dst + r * ld_bytes + ch * 16) = v;
    }
    wave_lds_fence();
}

// Epilogues: inference (bias, GELU); training forward (bias, GELU, and the pre-activation
// stored to P with C's layout); training backward (the product times GELU'(P), no bias).
enum { kEpiGelu = 0, kEpiGeluSave = 2, kEpiGeluGrad = 3 };

// Operand stages in LDS: 128 bytes of the reduction per row (64 bf16 or 128 FP8 values), the rows of
// A, then the BN rows of B.  A stage is filled by loads that write LDS directly (16 bytes a
// lane: lane l of an instruction writes the 16 bytes at base + 16 l), so no register holds it and several
// stages are in flight.  The rows are unpadded for that; instead chunk c of row r lies at chunk
// c ^ (r % 8), which the loading lane arranges by its global address, so that the 8 lanes of a
// fragment read that take the same chunk of 8 rows touch all the banks.
constexpr int kStRowB = 128, kABytes = BM * kStRowB, kStageB = kABytes + BN * kStRowB;

typedef __attribute__((address_space(3))) void lds_void;

// buffer descriptor of `bytes` bytes from p (the same in every lane): the loads then need one 32-bit lane offset,
// and the rest of the address stays in scalar registers
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}

// 8 NI rows of a stage, 8 rows per instruction: this lane's 16 bytes of the first instruction lie at off + base,
// `step` is the bytes of 8 rows
template <int NI>
__device__ __forceinline__ void dma_rows(__amdgpu_buffer_rsrc_t src, int off, int base, int step, uint8_t *dst) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void *)(dst + i * 1024), 16, off, base + i * step, 0, 0);
}

// All but the last N vector loads of this wave have landed, then the same for the block (and every wave has read
// its last fragments of the stage before).  Only the stage loads are issued in a stage loop, so N
// counts whole stages.
template <int N>
__device__ __forceinline__ void stage_barrier() {
    asm volatile("" ::: "memory");
    // vmcnt(N) lgkmcnt(0), known to the compiler's own wait counting
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4) << 14 | 0x0070);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The stage loop (NST = 2 or 4, or 1 for a single stage): NST - 1 stages are loaded ahead; a stage's buffer is refilled after the barrier that follows
// its last read.  Separate arrays, a loop unrolled over them and loads without a branch let the
// compiler see that a read of one stage does not wait for the loads of another: a load
// beyond the last stage, or of a lane beyond K, is out of the descriptor's range and reads no memory (what
// it leaves in LDS is not read).
constexpr int kNoRow = 0x7ff00000;  // lane offset beyond every descriptor's range

template <int NST, int L, class Load, class Mma>
__device__ __forceinline__ void stage_loop(int S, uint8_t *b0, uint8_t *b1, uint8_t *b2, uint8_t *b3, Load load, Mma mma) {
    load(0, b0);
    if constexpr (NST == 1) {
        stage_barrier<0>();
        mma(0, b0);
        stage_barrier<0>();
        return;
    }
    if constexpr (NST > 2) {
        load(1, b1);
        load(2, b2);
    }
    auto step = [&](int s, uint8_t *cur, uint8_t *nxt) {
        stage_barrier<(NST > 2 ? NST - 2 : 0) * L>();
        load(s + NST - 1, nxt);
        mma(s, cur);
    };
    int s = 0;
    for (; s + NST <= S; s += NST) {
        step(s, b0, NST > 2 ? b3 : b1);
        step(s + 1, b1, b0);
        if constexpr (NST > 2) {
            step(s + 2, b2, b1);
            step(s + 3, b3, b2);
        }
    }
    if (s < S) step(s, b0, NST > 2 ? b3 : b1);
    if (NST > 2 && s + 1 < S) step(s + 1, b1, b0);
    if (NST > 2 && s + 2 < S) step(s + 2, b2, b1);
    stage_barrier<0>();  // every load has landed and every wave has read its last fragments
}

// What bounds it: with one block per CU a 64-deep stage takes about 0.9 us however the loads are hidden (18
// fragment reads and 40 MFMAs of 16 cycles per wave between barriers); two blocks overlap.  Staged through registers, with padded rows and two
// barriers per stage, 65,536 rows took 216 us (1600 -> 800) and 87 us (800 -> 400); with direct LDS loads and
// one barrier 188 us (890 TFLOP/s) and 79 us.  256-row tiles (waves of 128 x 80, one block per CU, three
// stages) took 275 us: one wave per SIMD hides too little, and the accumulators moved between register files.
// NST: stages in LDS (1 for K <= 64).
template <int EPI, int NST>
__global__ __launch_bounds__(kThreads, NST == 4 ? 1 : NST == 2 ? 2 : 3) void gemm_kernel(const bf16_t *__restrict__ A, int lda,
                                                       const bf16_t *__restrict__ B, int ldb,
                                                       const float *__restrict__ bias, bf16_t *__restrict__ C,
                                                       int ldc, int K, int n_tiles_n,
                                                       bf16_t *__restrict__ P) {
    constexpr int kNa = BM / 32, kNb = BN / 32;  // load instructions of a wave per stage (8 rows each)
    // the operand stages; after the stage loop the epilogues stage their outputs in the first
    __shared__ __attribute__((aligned(1024))) uint8_t St0[kStageB];
    __shared__ __attribute__((aligned(1024))) uint8_t St1[NST > 1 ? kStageB : 16];
    __shared__ __attribute__((aligned(1024))) uint8_t St2[NST > 2 ? kStageB : 16];
    __shared__ __attribute__((aligned(1024))) uint8_t St3[NST > 2 ? kStageB : 16];
    __shared__ __attribute__((aligned(16))) float Ptab[EPI == kEpiGelu ? kPhiLdsFloats : 4];

    // XCD-aware tile order: workgroups are dispatched round-robin over the 8 XCDs, so
    // block b runs on XCD b % 8; give each XCD a contiguous range of logical tiles.
    const int nb = gridDim.x, b = blockIdx.x;
    const int logical = (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
    const int tile_m = logical / n_tiles_n, tile_n = logical % n_tiles_n;
    const int64_t row0 = int64_t(tile_m) * BM;
    const int col0 = tile_n * BN;

    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = w >> 1, wn = w & 1;

    // wave w fills rows 32 w .. of A and 40 w .. of B (8 rows per instruction)
    const int lr = lane >> 3, lc = (lane & 7) ^ lr;  // row of 8, and the chunk that belongs at chunk lane % 8
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int ra = 8 * kNa * wu, rb = 8 * kNb * wu;
    const int sta = 16 * lda, stb = 16 * ldb;  // bytes of 8 rows
    const __amdgpu_buffer_rsrc_t ba = buffer_of(A + (row0 + ra) * lda, kNa * sta),
                                 bb = buffer_of(B + int64_t(col0 + rb) * ldb, kNb * stb);
    const int oa = lr * 2 * lda + lc * 16, ob = lr * 2 * ldb + lc * 16;
    auto load = [&](int s, uint8_t *st) {
        const bool in = lc * 8 < K - 64 * s;  // the last stage may hold 32 inputs: its other chunks are not read
        dma_rows<kNa>(ba, in ? oa : kNoRow, 128 * s, sta, st + ra * kStRowB);
        dma_rows<kNb>(bb, in ? ob : kNoRow, 128 * s, stb, st + kABytes + rb * kStRowB);
    };

    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // MFMA 16x16x32 operands: lane l supplies row (l % 16) of the A tile and column (l % 16) of
    // the B tile, with 8 consecutive k values (one chunk) starting at 8 * (l / 16)
    const int fr = lane & 15, fg = lane >> 4;
    const int fa = (wm * WM + fr) * kStRowB, fb = kABytes + (wn * WN + fr) * kStRowB;
    // one stage in STEPS 32-deep MFMA steps, in k order
    auto mma = [&](const uint8_t *st, auto STEPS) {
#pragma unroll
        for (int kk = 0; kk < decltype(STEPS)::value; ++kk) {
            const int c = ((4 * kk + fg) ^ (fr & 7)) * 16;
            bf16x8 af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) af[i] = *reinterpret_cast<const bf16x8 *>(st + fa + i * 16 * kStRowB + c);
#pragma unroll
            for (int j = 0; j < TN; ++j) bfr[j] = *reinterpret_cast<const bf16x8 *>(st + fb + j * 16 * kStRowB + c);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
    };
    if (EPI == kEpiGelu) copy_phi_table(Ptab, t);  // visible after the stage loop's barriers
    stage_loop<NST, kNa + kNb>((K + 63) / 64, St0, St1, St2, St3, load, [&](int s, const uint8_t *st) {
        if (K - 64 * s >= 64)
            mma(st, std::integral_constant<int, 2>{});
        else
            mma(st, std::integral_constant<int, 1>{});
    });
    // epilogue: with the weights as the first MFMA operand, lane l holds row (l % 16) and the four
    // columns 4 * (l / 16) + r of each 16 x 16 tile
    // staged through the operand buffers, in two halves of 32 rows per wave; the training
    // forward stages its pre-activations (P) first and then its outputs
    static_assert(WN * 2 == kStgRowB, "staging");
    uint8_t *const stg = St0 + w * (32 * kStgStrideB);
    const int64_t ldb_c = 2 * int64_t(ldc);
    const int64_t off0 = (row0 + wm * WM) * ldb_c + 2 * (col0 + wn * WN);
    const int fc = (lane >> 4) * 4;  // the lane's first column in a 16 x 16 tile
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        floatx4 v[TN][2];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const floatx4 bc = (EPI == kEpiGeluGrad)
                                   ? floatx4{0.f, 0.f, 0.f, 0.f}
                                   : *reinterpret_cast<const floatx4 *>(bias + col0 + wn * WN + j * 16 + fc);
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) v[j][ii] = acc[2 * hf + ii][j] + bc;
        }
        if constexpr (EPI == kEpiGeluSave) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int ii = 0; ii < 2; ++ii)
                    *reinterpret_cast<bf16x4 *>(stg + (ii * 16 + fr) * kStgStrideB + 2 * (j * 16 + fc)) =
                        to_bf16x4(v[j][ii]);
            stage_flush<32>(stg, reinterpret_cast<uint8_t *>(P) + off0 + hf * 32 * ldb_c, ldb_c, lane);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                floatx4 x = v[j][ii];
                if constexpr (EPI == kEpiGelu) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = gelu_tab(x[r], Ptab);
                } else if constexpr (EPI == kEpiGeluSave) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] = gelu_erfc(x[r]);
                } else {
                    const int64_t row = row0 + wm * WM + (2 * hf + ii) * 16 + fr;
                    const bf16x4 pv =
                        *reinterpret_cast<const bf16x4 *>(P + row * ldc + col0 + wn * WN + j * 16 + fc);
#pragma unroll
                    for (int r = 0; r < 4; ++r) x[r] *= gelu_grad(float(pv[r]));
                }
                *reinterpret_cast<bf16x4 *>(stg + (ii * 16 + fr) * kStgStrideB + 2 * (j * 16 + fc)) =
                    to_bf16x4(x);
            }
        stage_flush<32>(stg, reinterpret_cast<uint8_t *>(C) + off0 + hf * 32 * ldb_c, ldb_c, lane);
    }
}

// A value the E4M3FN conversion takes as is: |x| <= 448 unchanged; 448 < |x| <= 464 rounds to
// 448 (ties to even) and is passed as 448; a value that would round beyond 448, an infinity or a
// NaN becomes NaN, the format's only non-finite value, so that it propagates to the cell's
// status as in the bf16 path.  The block scale keeps every finite scaled value within 448; the
// other cases arise only when the block's maximum itself is not finite.
__device__ __forceinline__ float fp8_in_range(float x) {
    // without branches: clamp to [-448, 448] (leaves |x| <= 448 and -0 as they are), then NaN
    // where |x| > 464 or x is NaN (the comparison is false for NaN)
    const float c = __builtin_amdgcn_fmed3f(x, -448.0f, 448.0f);
    return (fabsf(x) <= 464.0f) ? c : __builtin_nanf("");
}

// E4M3FN bytes of four floats (round to nearest even)
__device__ __forceinline__ uint32_t to_fp8x4(float a, float b, float c, float d) {
    a = fp8_in_range(a);
    b = fp8_in_range(b);
    c = fp8_in_range(c);
    d = fp8_in_range(d);
    int v = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);  // bytes 0, 1
    v = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, v, true);       // bytes 2, 3
    return uint32_t(v);
}

// E4M3FN bytes of four values of a block with largest magnitude m and scale factor sc.  With a finite m the
// scale keeps every scaled value within 448 (a NaN value stays NaN through the conversion), so the
// range rule has nothing to do.
__device__ __forceinline__ uint32_t fp8_word(floatx4 f, float m, float sc) {
    if (m <= 3.40282347e38f) {
        const int v = __builtin_amdgcn_cvt_pk_fp8_f32(f[0] * sc, f[1] * sc, 0, false);
        return uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(f[2] * sc, f[3] * sc, v, true));
    }
    return to_fp8x4(f[0] * sc, f[1] * sc, f[2] * sc, f[3] * sc);
}

// FP8 output of a layer whose result feeds an FP8 layer, for a wave that owns whole 32-column
// blocks: v0 and v1 are the GELU outputs of the 16 x 16 tiles 2q and 2q + 1 of a 16-row tile
// (lane l: row l % 16, columns 4 (l / 16) + r of each), so a block's 32 values of a row lie with
// the four lanes l % 16 + 16 g'.  Each value is rounded to bf16 first (the hidden activations are
// bf16 values in every precision), the block's largest magnitude is combined over the four lanes
// (NaN ignored), and the values are quantised with the block's scale: the lane's E4M3FN bytes of
// Q[row][c0 .. c0 + 32) as two words (bytes 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3), and the
// E8M0 scale byte to S[row][c0 / 32].
__device__ __forceinline__ void quant_fp8_block(floatx4 v0, floatx4 v1, uint8_t *__restrict__ S, int64_t row,
                                                int sst, int c0, int g, uint32_t &w0, uint32_t &w1) {
    const bf16x4 h0 = to_bf16x4(v0), h1 = to_bf16x4(v1);
    float f[8];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        f[r] = float(h0[r]);
        f[4 + r] = float(h1[r]);
    }
    float m = 0.0f;
#pragma unroll
    for (int r = 0; r < 8; ++r) m = fmaxf(m, fabsf(f[r]));
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    const int e = fp8_scale_exp(m);
    const float sc = ldexpf(1.0f, -e);
    w0 = fp8_word(floatx4{f[0], f[1], f[2], f[3]}, m, sc);
    w1 = fp8_word(floatx4{f[4], f[5], f[6], f[7]}, m, sc);
    if (g == 0) S[row * sst + c0 / kFp8Block] = uint8_t(127 + e);
}

// Inference layer with a shallow reduction (K = KD <= 64, the first hidden layer: the network's
// inputs padded to 32 or 64): no K loop to pipeline, so the time is the GELU epilogue and the
// stores of the M x N outputs.  Each block keeps one 160-column weight panel in registers as MFMA
// fragments and walks down the row tiles tile_m = g, g + G, ... (G = gridDim.x / n_tiles_n),
// loading each tile's activation fragments straight from global memory (16 rows x 64 contiguous
// bytes per load) one tile ahead, so that the loads of the next tile are in flight during the
// epilogue of the current one; LDS holds only the GELU table (one barrier, at the start).  Same tile shape, operand order and
// epilogue (bias, GELU, bf16) as gemm_kernel; with Q8 the output is the FP8 copy the next layer
// reads (quant_fp8_block), and the four waves take 32 rows x 160 columns each so that every
// wave owns whole 32-column blocks.  Each wave writes its outputs (160 bytes per row either way)
// to its own LDS region first and then to memory as 16-byte pieces, consecutive lanes along a
// row: the MFMA layout would give 16 rows x 32 bytes (bf16) or 16 bytes (FP8) per store, which
// measured about 1.7 times slower than row pieces for these outputs.  In the FP8 copy the bias
// row is read from LDS in the epilogue: held in registers (40 of them next to a 160-column weight
// panel) it left none for the staging at KD = 64, which then spilled and ran 14 % slower.
template <int KD, bool Q8>
__global__ __launch_bounds__(kThreads, 2) void gemm_shallow_kernel(const bf16_t *__restrict__ A, int lda,
                                                                const bf16_t *__restrict__ B, int ldb,
                                                                const float *__restrict__ bias,
                                                                bf16_t *__restrict__ C, int ldc,
                                                                uint8_t *__restrict__ S, int sst, int n_tiles_m,
                                                                int n_tiles_n) {
    constexpr int KS = KD / 32;  // 32-deep MFMA steps
    constexpr int WMq = Q8 ? 32 : WM, WNq = Q8 ? 160 : WN, TMq = WMq / 16, TNq = WNq / 16;
    const int tile_n = int(blockIdx.x) % n_tiles_n, g0 = int(blockIdx.x) / n_tiles_n;
    const int G = int(gridDim.x) / n_tiles_n;
    const int col0 = tile_n * BN;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = Q8 ? w : w >> 1, wn = Q8 ? 0 : w & 1;
    const int fr = lane & 15, fg = lane >> 4, fk = fg * 8;
    __shared__ __attribute__((aligned(16))) float Ptab[kPhiLdsFloats];
    copy_phi_table(Ptab, t);
    // the wave's staging rows (160 bytes of outputs each)
    static_assert((Q8 ? WNq : 2 * WNq) == kStgRowB, "staging layout");
    __shared__ __attribute__((aligned(16))) uint8_t Stage[4 * WMq * kStgStrideB];
    __shared__ __attribute__((aligned(16))) float Bias[Q8 ? BN : 4];
    if (Q8 && t < BN / 4)
        reinterpret_cast<floatx4 *>(Bias)[t] = reinterpret_cast<const floatx4 *>(bias + col0)[t];
    uint8_t *stg = Stage + w * (WMq * kStgStrideB);
    uint8_t *const Cb = reinterpret_cast<uint8_t *>(C);
    const int col0b = Q8 ? col0 : 2 * (col0 + wn * WNq);  // byte column of the wave's sub-tile
    const int64_t ldcb = Q8 ? ldc : 2 * int64_t(ldc);

    bf16x8 bfr[KS][TNq];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < TNq; ++j)
            bfr[s][j] = *reinterpret_cast<const bf16x8 *>(B + int64_t(col0 + wn * WNq + j * 16 + fr) * ldb + s * 32 + fk);
    floatx4 bc[Q8 ? 1 : TNq];  // the bf16 path holds its 80-column bias slice in registers
    if constexpr (!Q8) {
#pragma unroll
        for (int j = 0; j < TNq; ++j)
            bc[j] = *reinterpret_cast<const floatx4 *>(bias + col0 + wn * WNq + j * 16 + fg * 4);
    }

    auto load_a = [&](int tm, bf16x8 (&af)[KS][TMq]) {
        const int64_t r0 = int64_t(tm) * BM + wm * WMq + fr;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < TMq; ++i)
                af[s][i] = *reinterpret_cast<const bf16x8 *>(A + (r0 + i * 16) * lda + s * 32 + fk);
    };
    bf16x8 an[KS][TMq];
    if (g0 < n_tiles_m) load_a(g0, an);
    __syncthreads();  // the table is in LDS
    for (int tm = g0; tm < n_tiles_m; tm += G) {
        bf16x8 af[KS][TMq];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int i = 0; i < TMq; ++i) af[s][i] = an[s][i];
        if (tm + G < n_tiles_m) load_a(tm + G, an);
        floatx4 acc[TMq][TNq];
#pragma unroll
        for (int i = 0; i < TMq; ++i)
#pragma unroll
            for (int j = 0; j < TNq; ++j) {
                acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[s][j], af[s][i], acc[i][j], 0, 0, 0);
            }
        const int64_t rowt = int64_t(tm) * BM + wm * WMq;  // first row of the wave's sub-tile
        if constexpr (Q8) {
#pragma unroll
            for (int i = 0; i < TMq; ++i)
#pragma unroll
                for (int q = 0; q < TNq / 2; ++q) {
                    const floatx4 *bl = reinterpret_cast<const floatx4 *>(Bias + 32 * q + fg * 4);
                    floatx4 v0 = acc[i][2 * q] + bl[0], v1 = acc[i][2 * q + 1] + bl[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        v0[r] = gelu_tab(v0[r], Ptab);
                        v1[r] = gelu_tab(v1[r], Ptab);
                    }
                    uint32_t w0, w1;
                    quant_fp8_block(v0, v1, S, rowt + i * 16 + fr, sst, col0 + 32 * q, fg, w0, w1);
                    uint8_t *p = stg + (i * 16 + fr) * kStgStrideB + 32 * q + 4 * fg;
                    *reinterpret_cast<uint32_t *>(p) = w0;
                    *reinterpret_cast<uint32_t *>(p + 16) = w1;
                }
        } else {
#pragma unroll
            for (int j = 0; j < TNq; ++j) {
#pragma unroll
                for (int i = 0; i < TMq; ++i) {
                    floatx4 v = acc[i][j] + bc[j];
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = gelu_tab(v[r], Ptab);
                    *reinterpret_cast<bf16x4 *>(stg + (i * 16 + fr) * kStgStrideB + 2 * (j * 16 + fg * 4)) =
                        to_bf16x4(v);
                }
            }
        }
        stage_flush<WMq>(stg, Cb + rowt * ldcb + col0b, ldcb, lane);
    }
}

// FP8 layer on the block-scaled matrix cores: the tiling and staging of gemm_kernel (128 x 160 block tile,
// 2 x 2 waves of 64 x 80) with 128-deep stages of E4M3FN bytes; 65,536 rows, 3200 -> 1600 (FP8 output) and
// 1600 -> 800: 570 and 174 us staged through registers with 144-byte LDS rows (a third of the LDS time was bank
// conflicts) and waves of 32 x 160 for the FP8 output, 441 and 149 us so.  In a 16x16x128 product with
// 8-bit operands, lane l supplies row l % 16 of its operand at the stage's inputs 16 g .. 16 g + 15
// (bytes 0-15) and 64 + 16 g .. 64 + 16 g + 15 (bytes 16-31), g = l / 16, and the E8M0 scale of
// the inputs 32 g .. 32 g + 31 of that row: its two halves lie with lanes g' = 2 (g % 2) and
// 2 (g % 2) + 1 (measured on gfx950 with one-hot data and per-lane scales).  So each lane reads
// the two 16-byte pieces of its row at 16 g and 64 + 16 g, and passes the scale of activation
// block g of the stage (the weight row's scale, 127 + wexp, is the same for all blocks).  Inputs
// at or beyond K (the last stage of a K that is not a multiple of 128) are zeros with scale 2^0.
typedef int i32x8 __attribute__((ext_vector_type(8)));
constexpr int KD8 = 128;  // stage depth

template <bool Q8, int NST>
__global__ __launch_bounds__(kThreads, NST == 2 ? 2 : 1) void gemm_fp8_kernel(const uint8_t *__restrict__ A8, int lda,
                                                           const uint8_t *__restrict__ SA, int sst,
                                                           const uint8_t *__restrict__ W8, int ldb,
                                                           const int32_t *__restrict__ wexp,
                                                           const float *__restrict__ bias, bf16_t *__restrict__ C,
                                                           int ldc, uint8_t *__restrict__ SC, int sstc, int K,
                                                           int n_tiles_n) {
    constexpr int kNa = BM / 32, kNb = BN / 32;  // load instructions of a wave per stage (8 rows each)
    // the operand stages, each followed by the four block scales of its A rows as a word per row; after the
    // stage loop the epilogue stages its outputs in the first
    constexpr int kScOff = kStageB, kSt = kStageB + 4 * BM;
    __shared__ __attribute__((aligned(1024))) uint8_t St0[kSt];
    __shared__ __attribute__((aligned(1024))) uint8_t St1[kSt];
    __shared__ __attribute__((aligned(1024))) uint8_t St2[NST > 2 ? kSt : 16];
    __shared__ __attribute__((aligned(1024))) uint8_t St3[NST > 2 ? kSt : 16];
    __shared__ __attribute__((aligned(16))) float Ptab[kPhiLdsFloats];

    const int nb = gridDim.x, b = blockIdx.x;
    const int logical = (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
    const int tile_m = logical / n_tiles_n, tile_n = logical % n_tiles_n;
    const int64_t row0 = int64_t(tile_m) * BM;
    const int col0 = tile_n * BN;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int wm = w >> 1, wn = w & 1;
    const int fr = lane & 15, fg = lane >> 4;

    // loads as in gemm_kernel, and one of 64 rows' scales; the last stage of a K that is not a multiple of 128
    // gets zeros from ordinary LDS stores at its inputs beyond K
    const int lr = lane >> 3, lc = (lane & 7) ^ lr, wu = __builtin_amdgcn_readfirstlane(w);
    const int ra = 8 * kNa * wu, rb = 8 * kNb * wu;
    const int ws = 64 * (wu % 2);  // the rows whose scales this wave loads
    const int sta = 8 * lda, stb = 8 * ldb;  // bytes of 8 rows
    const __amdgpu_buffer_rsrc_t ba = buffer_of(A8 + (row0 + ra) * lda, kNa * sta),
                                 bb = buffer_of(W8 + int64_t(col0 + rb) * ldb, kNb * stb),
                                 bs = buffer_of(SA + (row0 + ws) * sst, 64 * sst);
    const int oa = lr * lda + lc * 16, ob = lr * ldb + lc * 16, os = lane * sst;
    auto load = [&](int s, uint8_t *st) {
        uint8_t *pa = st + ra * kStRowB, *pb = st + kABytes + rb * kStRowB;
        const bool in = lc * 16 < K - KD8 * s;
        dma_rows<kNa>(ba, in ? oa : kNoRow, KD8 * s, sta, pa);
        dma_rows<kNb>(bb, in ? ob : kNoRow, KD8 * s, stb, pb);
        if (K - KD8 * s > 0 && !in) {
            const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int i = 0; i < kNa; ++i) *reinterpret_cast<u32x4 *>(pa + i * 1024 + lane * 16) = z;
#pragma unroll
            for (int i = 0; i < kNb; ++i) *reinterpret_cast<u32x4 *>(pb + i * 1024 + lane * 16) = z;
        }
        // (a word is 4-byte aligned, sst % 16 = 0, and inside the row's sst bytes)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(bs, (lds_void *)(st + kScOff + 4 * ws), 4,
                                                 KD8 * s < K ? os : kNoRow, 4 * s, 0, 0);
    };

    int sw[TN];  // E8M0 scale of the weight row each lane supplies
#pragma unroll
    for (int j = 0; j < TN; ++j) sw[j] = 127 + wexp[col0 + wn * WN + j * 16 + fr];
    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int fa = (wm * WM + fr) * kStRowB, fb = kABytes + (wn * WN + fr) * kStRowB;
    const int c0 = (fg ^ (fr & 7)) * 16, c1 = ((4 + fg) ^ (fr & 7)) * 16;
    copy_phi_table(Ptab, t);  // visible after the stage loop's barriers
    stage_loop<NST, kNa + kNb + 1>((K + KD8 - 1) / KD8, St0, St1, St2, St3, load, [&](int s, const uint8_t *st) {
        auto frag = [&](const uint8_t *row) {
            const u32x4 lo = *reinterpret_cast<const u32x4 *>(row + c0);
            const u32x4 hi = *reinterpret_cast<const u32x4 *>(row + c1);
            return i32x8{int(lo[0]), int(lo[1]), int(lo[2]), int(lo[3]), int(hi[0]), int(hi[1]), int(hi[2]), int(hi[3])};
        };
        // this lane's block of a row's scale word, 2^0 where the block is at or beyond K
        const bool in = s * KD8 + fg * kFp8Block < K;
        const uint32_t mask = in ? 0xffu : 0u, fill = in ? 0u : 127u;
        // the activation fragments (fewer than the weight ones) held, the weight fragments a few at a time
        i32x8 af[TM];
        int sa[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            af[i] = frag(st + fa + i * 16 * kStRowB);
            const uint32_t v = *reinterpret_cast<const uint32_t *>(st + kScOff + 4 * (wm * WM + i * 16 + fr));
            sa[i] = int(((v >> (8 * fg)) & mask) | fill);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            // keeps the scheduler from moving all the weight fragments up, which spills
            if (j % 2 == 0) __builtin_amdgcn_sched_barrier(0);
            const i32x8 wf = frag(st + fb + j * 16 * kStRowB);
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wf, af[i], acc[i][j], 0, 0, 0, sw[j], 0, sa[i]);
        }
    });

    if constexpr (Q8) {
        // A wave's 80 columns are two 32-column blocks and half of the block that it shares with the other wave
        // of its rows (the last half of wave 0's, the first of wave 1's columns): the two exchange
        // that block's row maxima through LDS.  The FP8 rows (160 bytes of both waves) are staged by row.
        static_assert(kStgRowB == 2 * WN, "staging");
        float *const Mx = reinterpret_cast<float *>(St1);  // [2][BM]
        uint8_t *const stg = St0 + wm * (WM * kStgStrideB);
        float mx[TM][TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const floatx4 bc = *reinterpret_cast<const floatx4 *>(bias + col0 + wn * WN + j * 16 + fg * 4);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                floatx4 v = acc[i][j] + bc;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = gelu_tab(v[r], Ptab);
                const bf16x4 h = to_bf16x4(v);
                float m = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[i][j][r] = float(h[r]);
                    m = fmaxf(m, fabsf(acc[i][j][r]));
                }
                m = fmaxf(m, __shfl_xor(m, 16));
                mx[i][j] = fmaxf(m, __shfl_xor(m, 32));
            }
        }
        if (fg == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WM + i * 16 + fr;
                if (wn)
                    Mx[BM + row] = mx[i][0];
                else
                    Mx[row] = mx[i][TN - 1];
            }
        }
        __syncthreads();
        // columns of 16-column tile j of this wave within the panel: block (5 wn + j) / 2
        auto finish = [&](auto WN_) {
            constexpr int kW = decltype(WN_)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WM + i * 16 + fr;
                const float other = Mx[(1 - kW) * BM + row];
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int c16 = TN * kW + j;  // in 16s, from the panel's first column
                    const int jp = j + (c16 % 2 ? -1 : 1);
                    float m = fmaxf(mx[i][j], other);
                    if (jp >= 0 && jp < TN) m = fmaxf(mx[i][j], mx[i][jp]);
                    const int e = fp8_scale_exp(m);
                    *reinterpret_cast<uint32_t *>(stg + (i * 16 + fr) * kStgStrideB + c16 * 16 + 4 * fg) =
                        fp8_word(acc[i][j], m, ldexpf(1.0f, -e));
                    // the block's scale, from the wave that holds its first half
                    if (c16 % 2 == 0 && fg == 0)
                        SC[(row0 + row) * sstc + (col0 + c16 * 16) / kFp8Block] = uint8_t(127 + e);
                }
            }
        };
        if (wn)
            finish(std::integral_constant<int, 1>{});
        else
            finish(std::integral_constant<int, 0>{});
        __syncthreads();
        // half of the rows for each of the two waves
        stage_flush<WM / 2>(stg + wn * (WM / 2 * kStgStrideB),
                            reinterpret_cast<uint8_t *>(C) + (row0 + wm * WM + wn * (WM / 2)) * int64_t(ldc) + col0,
                            ldc, lane);
    } else {
        uint8_t *const stg = St0 + w * (32 * kStgStrideB);
        const int64_t ldb_c = 2 * int64_t(ldc);
        uint8_t *const dst = reinterpret_cast<uint8_t *>(C) + (row0 + wm * WM) * ldb_c + 2 * (col0 + wn * WN);
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const floatx4 bc = *reinterpret_cast<const floatx4 *>(bias + col0 + wn * WN + j * 16 + fg * 4);
#pragma unroll
                for (int ii = 0; ii < 2; ++ii) {
                    floatx4 v = acc[2 * hf + ii][j] + bc;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = gelu_tab(v[r], Ptab);
                    *reinterpret_cast<bf16x4 *>(stg + (ii * 16 + fr) * kStgStrideB + 2 * (j * 16 + fg * 4)) =
                        to_bf16x4(v);
                }
            }
            stage_flush<32>(stg, dst + hf * 32 * ldb_c, ldb_c, lane);
        }
    }
}

// Layers of few rows.  A grid of 128 x 160 tiles is then a few blocks, each bound by the latency of its
// serial stages (a global load, two barriers and the LDS round trip per 32 or 64 inputs), and most of
// its rows may be padding.  Here every wave owns one small tile, 16 RT rows x 16 CT columns, over the
// whole reduction, and loads its operand fragments straight from global memory, D 32-deep steps ahead in a
// second set of registers: no barrier in the loop, and only the row tiles in use.  The MFMAs,
// their operand order and the ascending K order are those of the tiled kernels, so are the epilogues, so
// every output has the same bits.
template <int EPI, bool Q8, int RT, int CT, int D>
__global__ __launch_bounds__(64) void gemm_rows_kernel(const bf16_t *__restrict__ A, int lda,
                                                            const bf16_t *__restrict__ B, int ldb,
                                                            const float *__restrict__ bias, bf16_t *__restrict__ C,
                                                            int ldc, uint8_t *__restrict__ S, int sst, int K,
                                                            int n_tiles_n, bf16_t *__restrict__ P) {
    static_assert(!Q8 || (CT == 2 && EPI == kEpiGelu), "whole 32-column blocks");
    __shared__ __attribute__((aligned(16))) float Ptab[EPI == kEpiGelu ? kPhiLdsFloats : 4];
    const int lane = threadIdx.x, fr = lane & 15, fg = lane >> 4;
    const int tile_m = int(blockIdx.x) / n_tiles_n, tile_n = int(blockIdx.x) % n_tiles_n;
    const int64_t row0 = int64_t(tile_m) * (16 * RT);
    const int col0 = tile_n * (16 * CT);
    const bf16_t *ap = A + (row0 + fr) * lda + fg * 8, *bp = B + int64_t(col0 + fr) * ldb + fg * 8;
    const int steps = K / 32;
    bf16x8 a[2][D][RT], b[2][D][CT];
    floatx4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int s0, bf16x8 (&af)[D][RT], bf16x8 (&bf)[D][CT]) {
        if (s0 >= steps) return;
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = 32 * min(s0 + u, steps - 1);  // past the end: the last step again, not used
#pragma unroll
            for (int i = 0; i < RT; ++i) af[u][i] = *reinterpret_cast<const bf16x8 *>(ap + int64_t(16 * i) * lda + k);
#pragma unroll
            for (int j = 0; j < CT; ++j) bf[u][j] = *reinterpret_cast<const bf16x8 *>(bp + int64_t(16 * j) * ldb + k);
        }
    };
    auto mma = [&](int s0, bf16x8 (&af)[D][RT], bf16x8 (&bf)[D][CT]) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (s0 + u >= steps) break;
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < CT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[u][j], af[u][i], acc[i][j], 0, 0, 0);
        }
    };
    load(0, a[0], b[0]);
    if (EPI == kEpiGelu) {
        copy_phi_table<64>(Ptab, lane);
        __syncthreads();
    }
    for (int s0 = 0; s0 < steps; s0 += 2 * D) {
        load(s0 + D, a[1], b[1]);
        mma(s0, a[0], b[0]);
        load(s0 + 2 * D, a[0], b[0]);
        mma(s0 + D, a[1], b[1]);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int64_t row = row0 + i * 16 + fr;
        floatx4 v[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = col0 + j * 16 + fg * 4;
            const int64_t off = row * ldc + col;
            v[j] = acc[i][j] + (EPI == kEpiGeluGrad ? floatx4{0.f, 0.f, 0.f, 0.f}
                                                    : *reinterpret_cast<const floatx4 *>(bias + col));
            if constexpr (EPI == kEpiGeluSave) *reinterpret_cast<bf16x4 *>(P + off) = to_bf16x4(v[j]);
            bf16x4 pv = {};
            if constexpr (EPI == kEpiGeluGrad) pv = *reinterpret_cast<const bf16x4 *>(P + off);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (EPI == kEpiGelu) v[j][r] = gelu_tab(v[j][r], Ptab);
                if constexpr (EPI == kEpiGeluSave) v[j][r] = gelu_erfc(v[j][r]);
                if constexpr (EPI == kEpiGeluGrad) v[j][r] *= gelu_grad(float(pv[r]));
            }
            if constexpr (!Q8) *reinterpret_cast<bf16x4 *>(C + off) = to_bf16x4(v[j]);
        }
        if constexpr (Q8) {
            uint32_t w0, w1;
            quant_fp8_block(v[0], v[1], S, row, sst, col0, fg, w0, w1);
            uint8_t *q = reinterpret_cast<uint8_t *>(C) + row * ldc + col0 + 4 * fg;
            *reinterpret_cast<uint32_t *>(q) = w0;
            *reinterpret_cast<uint32_t *>(q + 16) = w1;
        }
    }
}

// the same for an FP8 layer: 128-deep steps, operands and scales as in gemm_fp8_kernel
template <bool Q8, int RT, int D>
__global__ __launch_bounds__(64) void gemm_fp8_rows_kernel(const uint8_t *__restrict__ A8, int lda,
                                                                const uint8_t *__restrict__ SA, int sst,
                                                                const uint8_t *__restrict__ W8, int ldb,
                                                                const int32_t *__restrict__ wexp,
                                                                const float *__restrict__ bias,
                                                                bf16_t *__restrict__ C, int ldc,
                                                                uint8_t *__restrict__ SC, int sstc, int K,
                                                                int n_tiles_n) {
    constexpr int CT = 2;
    __shared__ __attribute__((aligned(16))) float Ptab[kPhiLdsFloats];
    const int lane = threadIdx.x, fr = lane & 15, fg = lane >> 4;
    const int tile_m = int(blockIdx.x) / n_tiles_n, tile_n = int(blockIdx.x) % n_tiles_n;
    const int64_t row0 = int64_t(tile_m) * (16 * RT);
    const int col0 = tile_n * (16 * CT);
    const uint8_t *ap = A8 + (row0 + fr) * lda, *bp = W8 + int64_t(col0 + fr) * ldb;
    const uint8_t *sp = SA + (row0 + fr) * sst;
    const int steps = (K + KD8 - 1) / KD8;
    i32x8 a[2][D][RT], b[2][D][CT];
    int sa[2][D][RT], sw[CT];
    floatx4 acc[RT][CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) sw[j] = 127 + wexp[col0 + j * 16 + fr];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // 32 bytes of a row at k0 + 16 fg and k0 + 64 + 16 fg; zeros at or beyond K
    auto frag = [&](const uint8_t *row, int k0) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        const int k = k0 + fg * 16;
        const u32x4 lo = (k < K) ? *reinterpret_cast<const u32x4 *>(row + k) : z;
        const u32x4 hi = (k + 64 < K) ? *reinterpret_cast<const u32x4 *>(row + k + 64) : z;
        return i32x8{int(lo[0]), int(lo[1]), int(lo[2]), int(lo[3]), int(hi[0]), int(hi[1]), int(hi[2]), int(hi[3])};
    };
    auto load = [&](int s0, i32x8 (&af)[D][RT], int (&sf)[D][RT], i32x8 (&bf)[D][CT]) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k0 = KD8 * (s0 + u);
            if (k0 >= K) break;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                af[u][i] = frag(ap + int64_t(16 * i) * lda, k0);
                const int q = k0 / kFp8Block + fg;
                sf[u][i] = (q * kFp8Block < K) ? int(sp[int64_t(16 * i) * sst + q]) : 127;
            }
#pragma unroll
            for (int j = 0; j < CT; ++j) bf[u][j] = frag(bp + int64_t(16 * j) * ldb, k0);
        }
    };
    auto mma = [&](int s0, i32x8 (&af)[D][RT], int (&sf)[D][RT], i32x8 (&bf)[D][CT]) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (s0 + u >= steps) break;
#pragma unroll
            for (int j = 0; j < CT; ++j)
#pragma unroll
                for (int i = 0; i < RT; ++i)
                    acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(bf[u][j], af[u][i], acc[i][j], 0, 0, 0,
                                                                                 sw[j], 0, sf[u][i]);
        }
    };
    load(0, a[0], sa[0], b[0]);
    copy_phi_table<64>(Ptab, lane);
    __syncthreads();
    for (int s0 = 0; s0 < steps; s0 += 2 * D) {
        load(s0 + D, a[1], sa[1], b[1]);
        mma(s0, a[0], sa[0], b[0]);
        load(s0 + 2 * D, a[0], sa[0], b[0]);
        mma(s0 + D, a[1], sa[1], b[1]);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int64_t row = row0 + i * 16 + fr;
        floatx4 v[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = col0 + j * 16 + fg * 4;
            v[j] = acc[i][j] + *reinterpret_cast<const floatx4 *>(bias + col);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[j][r] = gelu_tab(v[j][r], Ptab);
            if constexpr (!Q8) *reinterpret_cast<bf16x4 *>(C + row * ldc + col) = to_bf16x4(v[j]);
        }
        if constexpr (Q8) {
            uint32_t w0, w1;
            quant_fp8_block(v[0], v[1], SC, row, sstc, col0, fg, w0, w1);
            uint8_t *q = reinterpret_cast<uint8_t *>(C) + row * ldc + col0 + 4 * fg;
            *reinterpret_cast<uint32_t *>(q) = w0;
            *reinterpret_cast<uint32_t *>(q + 16) = w1;
        }
    }
}

// Rows and columns, in 16s, of a wave's tile for `rows` rows of an N x K layer; 0 = the tiled kernels.  A
// wave's tile re-reads its operands (no sharing between waves), so the rows kernel's time grows with waves x K
// once the CUs are full, while a tiled launch of less than a wave of blocks takes the same time
// for any row count.  Measured, rows kernel / tiled kernel in us, N x K, rows:
//   16-wide tile, 800 x 1600: 1 row 6.9 / 27, 128 rows 10.2 / 27; 400 x 800: 128 rows 4.3 / 19
//   32-wide, 800 x 1600: 512 rows (400 waves) 16.5 / 27.5, 1,000 (800) 26.8 / 27.6, 2,048 (1,600) 44 / 28
//   32-wide, 400 x 800:  2,048 rows (832) 12.3 / 22.9, 4,096 (1,664) 21.0 / 23.2, 8,192 38 / 24
//   32-wide, 1600 x 800 (backward): 1,024 rows (1,600) 18.2 / 25.9, 2,048 (3,200) 33 / 26
//   32-wide, 1600 x 32:  512 rows (800) 5.8 / 7.6, 1,000 (1,600) 7.7 / 7.7, 2,048 11.5 / 9.0
//   32-wide, FP8, 800 x 1600: 1 row 9.9 / 27, 1,000 rows 15.3 / 26.4, 2,048 (1,600) 21.6 / 26.7, 4,096 39 / 29
//   32-wide, FP8, 1600 x 3200: 1,000 rows (1,600) 48.5 / 46.3
int rows_tile(int64_t rows, int N, int K, bool fp8_in, bool fp8_out) {
    if (!fp8_in && !fp8_out && (rows + 15) / 16 * (N / 16) <= 800) return 1;
    const int64_t waves = (rows + 31) / 32 * (N / 32);
    return (waves <= 1600 && waves * K <= (fp8_in ? 2700000 : 1300000)) ? 2 : 0;
}

// Q8: only the 32-wide tile; training epilogues too (their row counts are whole multiples of 128)
template <int EPI, bool Q8>
void launch_rows(int tile, const bf16_t *A, int lda, const bf16_t *B, int ldb, const float *bias, bf16_t *C, int ldc,
                 uint8_t *S, int sst, int64_t rows, int N, int K, bf16_t *P, hipStream_t stream) {
    if constexpr (EPI == kEpiGelu && !Q8) {
        if (tile == 1) {
            const int tn = N / 16;
            hipLaunchKernelGGL((gemm_rows_kernel<EPI, false, 1, 1, 13>), dim3(unsigned((rows + 15) / 16 * tn)), dim3(64),
                               0, stream, A, lda, B, ldb, bias, C, ldc, S, sst, K, tn, P);
            return;
        }
    }
    const int tn = N / 32;
    hipLaunchKernelGGL((gemm_rows_kernel<EPI, Q8, 2, 2, 5>), dim3(unsigned((rows + 31) / 32 * tn)),
                       dim3(64), 0, stream, A, lda, B, ldb, bias, C, ldc, S, sst, K, tn, P);
}

// Four stages in LDS and one block per CU for grids of at most one block per CU, where only the stages in flight
// hide the loads; otherwise two stages and two blocks per CU, which hide each other's loads and
// epilogues.  N x K, rows (tiles), two / four stages in us: 800 x 1600, 4,096 (160) 26.0 / 24.2;
// 1600 x 3200, 2,048 (160) 45 / 40; 400 x 800, 8,192 (192) 17.8 / 17.1; beyond 256 tiles the four-stage
// form would take two rounds.
bool deep_stages(int64_t tiles) { return tiles <= 256; }

// the shallow-reduction layer (K = 32 or 64, shapes checked by the caller): about two blocks per
// CU, each on one 160-column panel and every G-th row tile; S != nullptr: FP8 output (C holds the
// E4M3FN bytes with row stride ldc, S the block scales with row stride sst)
df_status launch_shallow(const bf16_t *A, int lda, const bf16_t *B, int ldb, const float *bias, bf16_t *C, int ldc,
                         uint8_t *S, int sst, int64_t M, int N, int K, hipStream_t stream) {
    const int64_t tm = M / BM;
    const int tn = N / BN;
    if (tm > 0x7fffffff) return fail(DF_E_UNSUPPORTED, "gemm: too many row tiles");
    // the outputs are written as 16-byte row pieces
    if ((reinterpret_cast<uintptr_t>(C) & 15) || (S ? ldc % 16 : ldc % 8))
        return fail(DF_E_INVALID, "gemm: the output rows must be 16-byte aligned");
    const int G = int(std::max<int64_t>(1, std::min<int64_t>(tm, std::max(1, 512 / tn))));
    const dim3 g = dim3(unsigned(int64_t(G) * tn)), b = dim3(kThreads);
#define DF_SHALLOW(KD, Q)                                                                                        \
    hipLaunchKernelGGL((gemm_shallow_kernel<KD, Q>), g, b, 0, stream, A, lda, B, ldb, bias, C, ldc, S, sst, int(tm), \
                       tn)
    if (K == 32) {
        if (S)
            DF_SHALLOW(32, true);
        else
            DF_SHALLOW(32, false);
    } else {
        if (S)
            DF_SHALLOW(64, true);
        else
            DF_SHALLOW(64, false);
    }
#undef DF_SHALLOW
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
    return DF_OK;
}

}  // namespace

df_status launch_gemm_bf16(const bf16_t *A, int lda, const bf16_t *B, int ldb, const float *bias, bf16_t *C, int ldc,
                           int64_t M, int64_t rows, int N, int K, hipStream_t stream) {
    return launch_gemm_bf16_epi(A, lda, B, ldb, bias, C, ldc, M, rows, N, K, GemmEpi::gelu, nullptr, stream);
}

df_status launch_gemm_bf16_epi(const bf16_t *A, int lda, const bf16_t *B, int ldb, const float *bias, bf16_t *C,
                               int ldc, int64_t M, int64_t rows, int N, int K, GemmEpi epi, bf16_t *P,
                               hipStream_t stream) {
    if (rows < 0 || rows > M || M % BM || N % BN || K % BK || K <= 0 || lda % 8 || ldb % 8)
        return fail(DF_E_INVALID, "gemm: shapes must be multiples of the tile sizes");
    // the outputs are written as 16-byte row pieces
    if ((reinterpret_cast<uintptr_t>(C) & 15) || ldc % 8 ||
        (epi == GemmEpi::gelu_save && (reinterpret_cast<uintptr_t>(P) & 15)))
        return fail(DF_E_INVALID, "gemm: the output rows must be 16-byte aligned");
    if ((epi == GemmEpi::gelu_save || epi == GemmEpi::gelu_grad) && !P)
        return fail(DF_E_INVALID, "gemm: the epilogue needs the pre-activation array");
    if (M == 0) return DF_OK;
    const int64_t tiles = (M / BM) * (N / BN);
    if (tiles > 0x7fffffff) return fail(DF_E_UNSUPPORTED, "gemm: too many tiles");
    if (const int tile = rows_tile(rows, N, K, false, false)) {
        if (rows == 0) return DF_OK;
        if (epi == GemmEpi::gelu)
            launch_rows<kEpiGelu, false>(tile, A, lda, B, ldb, bias, C, ldc, nullptr, 0, rows, N, K, nullptr, stream);
        else if (epi == GemmEpi::gelu_save)
            launch_rows<kEpiGeluSave, false>(tile, A, lda, B, ldb, bias, C, ldc, nullptr, 0, rows, N, K, P, stream);
        else
            launch_rows<kEpiGeluGrad, false>(tile, A, lda, B, ldb, bias, C, ldc, nullptr, 0, rows, N, K, P, stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(DF_E_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
        return DF_OK;
    }
    if (epi == GemmEpi::gelu && (K == 32 || K == 64))
        return launch_shallow(A, lda, B, ldb, bias, C, ldc, nullptr, 0, M, N, K, stream);
    const dim3 g = dim3(unsigned(tiles)), b = dim3(kThreads);
#define DF_GEMM(E, NST) \
    hipLaunchKernelGGL((gemm_kernel<E, NST>), g, b, 0, stream, A, lda, B, ldb, bias, C, ldc, K, N / BN, P)
    const bool deep = deep_stages(tiles);
    switch (epi) {
        case GemmEpi::gelu:
            if (deep)
                DF_GEMM(kEpiGelu, 4);
            else
                DF_GEMM(kEpiGelu, 2);
            break;
        case GemmEpi::gelu_save:
            if (K <= 64)
                DF_GEMM(kEpiGeluSave, 1);
            else if (deep)
                DF_GEMM(kEpiGeluSave, 4);
            else
                DF_GEMM(kEpiGeluSave, 2);
            break;
        case GemmEpi::gelu_grad:
            if (deep)
                DF_GEMM(kEpiGeluGrad, 4);
            else
                DF_GEMM(kEpiGeluGrad, 2);
            break;
    }
#undef DF_GEMM
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
    return DF_OK;
}

df_status launch_gemm_bf16_fp8out(const bf16_t *A, int lda, const bf16_t *B, int ldb, const float *bias, uint8_t *Q,
                                  int ldq, uint8_t *S, int sst, int64_t M, int64_t rows, int N, int K,
                                  hipStream_t stream) {
    if (rows < 0 || rows > M || M % BM || N % BN || lda % 8 || ldb % 8 || ldq % 16 || sst % 16 || sst < N / kFp8Block || !Q || !S)
        return fail(DF_E_INVALID, "gemm: shapes must be multiples of the tile sizes");
    if (K != 32 && K != 64) return fail(DF_E_UNSUPPORTED, "gemm with FP8 output: only a reduction depth of 32 or 64");
    if (M == 0) return DF_OK;
    if (rows > 0 && rows_tile(rows, N, K, false, true)) {
        launch_rows<kEpiGelu, true>(2, A, lda, B, ldb, bias, reinterpret_cast<bf16_t *>(Q), ldq, S, sst, rows, N, K, nullptr,
                                    stream);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(DF_E_HIP, std::string("gemm launch: ") + hipGetErrorString(e));
        return DF_OK;
    }
    return launch_shallow(A, lda, B, ldb, bias, reinterpret_cast<bf16_t *>(Q), ldq, S, sst, M, N, K, stream);
}

df_status launch_gemm_fp8(const uint8_t *A8, int lda, const uint8_t *S, int sst, const uint8_t *W8, int ldb,
                          const int32_t *wexp, const float *bias, bf16_t *C, int ldc, uint8_t *SC, int sstc,
                          int64_t M, int64_t rows, int N, int K, hipStream_t stream) {
    if (rows < 0 || rows > M || M % BM || N % BN || K % kFp8Block || K <= 0 || lda % 16 || ldb % 16 || sst % 16 || lda < K || ldb < K ||
        sst < K / kFp8Block || (SC && (ldc % 16 || sstc % 16 || sstc < N / kFp8Block)))
        return fail(DF_E_INVALID, "gemm fp8: shapes must be multiples of the tile sizes (rows of 16 bytes)");
    if (!A8 || !S || !W8 || !wexp) return fail(DF_E_INVALID, "gemm fp8: null activation, scale, weight or exponent array");
    if (reinterpret_cast<uintptr_t>(S) & 3) return fail(DF_E_INVALID, "gemm fp8: the scale array must be 4-byte aligned");
    if ((reinterpret_cast<uintptr_t>(C) & 15) || ldc % 8)  // outputs written as 16-byte row pieces
        return fail(DF_E_INVALID, "gemm fp8: the output rows must be 16-byte aligned");
    if (M == 0) return DF_OK;
    const int64_t tiles = (M / BM) * (N / BN);
    if (tiles > 0x7fffffff) return fail(DF_E_UNSUPPORTED, "gemm fp8: too many tiles");
    if (rows > 0 && rows_tile(rows, N, K, true, SC != nullptr)) {
        const int tn = N / 32;
        const dim3 g = dim3(unsigned((rows + 31) / 32 * tn)), b = dim3(64);
        if (SC)
            hipLaunchKernelGGL((gemm_fp8_rows_kernel<true, 2, 2>), g, b, 0, stream, A8, lda, S, sst, W8, ldb, wexp,
                               bias, C, ldc, SC, sstc, K, tn);
        else
            hipLaunchKernelGGL((gemm_fp8_rows_kernel<false, 2, 2>), g, b, 0, stream, A8, lda, S, sst, W8, ldb,
                               wexp, bias, C, ldc, SC, sstc, K, tn);
    } else {
        const dim3 g = dim3(unsigned(tiles)), b = dim3(kThreads);
#define DF_GEMM8(Q, W)                                                                                              \
    hipLaunchKernelGGL((gemm_fp8_kernel<Q, W>), g, b, 0, stream, A8, lda, S, sst, W8, ldb, wexp, bias, C, ldc, SC, sstc, \
                       K, N / BN)
        if (SC && !deep_stages(tiles))
            DF_GEMM8(true, 2);
        else if (SC)
            DF_GEMM8(true, 4);
        else if (!deep_stages(tiles))
            DF_GEMM8(false, 2);
        else
            DF_GEMM8(false, 4);
#undef DF_GEMM8
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("gemm fp8 launch: ") + hipGetErrorString(e));
    return DF_OK;
}

}  // namespace df
