// DNN form of the chemistry step (the paper's DNNInferencer::inference in three
// stages, Sec. "Description of the new classes"; network structure from Sec.
// "Chemistry Integration"):
//   1. pre   : x = (T, p, BoxCox(Y)), training-range test, z-score, bf16
//   2. layers: hidden layers as bf16 MFMA GEMMs with GELU (df_mlp.hip), output
//              layer on the matrix cores inside the post kernel; with FP8 precision the
//              layers between two hidden layers run on block-scaled E4M3FN operands (df_fp8.h)
//   3. post  : inverse normalisation and Box-Cox, optional renormalisation of Y,
//              T from enthalpy conservation at fixed p (FP64 Newton), rr
// Cells outside the training range are compacted into an index list and
// advanced by the integrator kernel in the same stream (status DNN_FALLBACK).
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <type_traits>

#include "df_fp8.h"
#include "df_internal.h"

namespace df {
namespace {

constexpr int kPreThreads = 256;

__device__ __forceinline__ bf16_t f2bf(float x) {
    unsigned u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return bf16_t((u >> 16) | ((u & 0x007fffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);
    return bf16_t(u >> 16);
}

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(unsigned(h) << 16); }

__device__ __forceinline__ double boxcox(double Y, double lam) { return (pow(fmax(Y, 0.0), lam) - 1.0) / lam; }

// x^n for 1 <= n by repeated squaring (the inverse Box-Cox power when 1/lambda is an integer)
__device__ __forceinline__ double ipow(double x, int n) {
    double r = 1.0;
    while (n) {
        if (n & 1) r *= x;
        x *= x;
        n >>= 1;
    }
    return r;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Normalised network inputs and flags: 1 = network, 0 = fallback (out of training range),
// 2 = non-finite input.  Cell i's row of in_pad bf16 inputs (zero beyond the K + 2 features, and
// for the padding rows i >= n) is written as 16-byte pieces.  The first block also clears the fallback
// counter, which the output kernel (a later launch) advances.
// The time is the FP64 power of each feature (some 200 instructions), so a block of 256 threads takes 32
// cells and spreads their features over its 8 half-waves, cells along the lanes: with one thread per
// cell and its features in sequence, 9 species, 1 / 65,536 cells took 9.8 / 15.0 us and 53 species,
// 65,536 cells 60 us (1,024 waves, one per SIMD); spread 4.2 / 9.5 us and 37 us.
constexpr int kPreCells = 32;

template <int K>
__global__ __launch_bounds__(kPreThreads) void pre_kernel(DnnDevParams prm, int64_t first, int64_t n, int64_t n_pad, int64_t ld,
                                                          const double *__restrict__ p, const double *__restrict__ T,
                                                          const double *__restrict__ Y, bf16_t *__restrict__ xb,
                                                          int in_pad, int8_t *__restrict__ flag,
                                                          int32_t *__restrict__ count,
                                                          int32_t *__restrict__ status, double *__restrict__ rr,
                                                          int fallback) {
    constexpr int NI = K + 2, NQ = (NI + 7) / 8, LDX = 8 * NQ + 8;  // features, 16-byte pieces holding them
    __shared__ __attribute__((aligned(16))) bf16_t xs[kPreCells * LDX];
    __shared__ int bad[kPreCells];  // bit 0: out of range, bit 1: not finite
    const int t = threadIdx.x, c = t % kPreCells, f0 = t / kPreCells;
    const int64_t i0 = first + int64_t(blockIdx.x) * kPreCells, i = i0 + c;
    if (i0 == 0 && t == 0) *count = 0;
    if (t < kPreCells) bad[t] = 0;
    for (int e = t; e < kPreCells * LDX / 8; e += kPreThreads)
        reinterpret_cast<u32x4 *>(xs)[e] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    if (i < n) {
        int b = 0;
#pragma unroll
        for (int f = f0; f < NI; f += kPreThreads / kPreCells) {
            double x;
            if (f < 2) {
                x = f == 0 ? T[i] : p[i];
                if (!(isfinite(x) && x > 0.0)) b |= 2;
            } else {
                const double y = Y[(f - 2) * ld + i];
                if (!isfinite(y)) b |= 2;
                x = boxcox(y, prm.lambda);
            }
            if (!(x >= prm.lo[f] && x <= prm.hi[f])) b |= 1;
            xs[c * LDX + f] = f2bf(float((x - prm.mu_in[f]) / prm.sig_in[f]));
        }
        if (b) atomicOr(&bad[c], b);
    }
    __syncthreads();
    // the rows, zero where the network does not run
    for (int e = t; e < kPreCells * (in_pad / 8); e += kPreThreads) {
        const int r = e / (in_pad / 8), q = e % (in_pad / 8);
        if (i0 + r >= n_pad) break;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (q < NQ && !bad[r]) v = *reinterpret_cast<const u32x4 *>(xs + r * LDX + 8 * q);
        *reinterpret_cast<u32x4 *>(xb + (i0 + r) * in_pad + 8 * q) = v;
    }
    if (i >= n) return;
    const int f = (bad[c] & 2) ? 2 : (bad[c] ? 0 : 1);
    if (f0 == 0) flag[i] = int8_t(f);
    if (f != 1 && !(f == 0 && fallback)) {
        // non-finite input, or out of range with the fallback switched off: state left as is
        if (status && f0 == 0) status[i] = (f == 2) ? DF_CELL_NONFINITE : DF_CELL_DNN_FALLBACK;
        if (rr)
            for (int k = f0; k < K; k += kPreThreads / kPreCells) rr[k * ld + i] = 0.0;
    }
}

// output layer + stage 3, 16 cells per block of four waves.  The output layer u = W h (bf16
// operands, fp32 sums) runs on the matrix cores as 16 x 16 x 32 MFMAs with the weight rows (zero
// beyond the K outputs) as the first operand, so that lane l ends with outputs 4 (l / 16) + r of
// cell l % 16.  The activation rows are read as 16-byte fragments, 16 rows x 64 contiguous bytes per
// load.  With at most 16 outputs (one output tile) the four waves split the reduction, wave w
// taking the 32-deep steps w, w + 4, ..., and their partial sums meet in LDS and are added in wave
// order; with more outputs wave w takes output tile w.
// Stage 3 in FP64 is what takes the time (a power per species, and a Newton iteration that needs every
// species' enthalpy), so its species are spread over the lanes too: the powers one per thread with the
// cells along the lanes, the sums over the species as 16 lanes per cell.  With one lane per cell it was
// one long chain per lane: 9 species, 1 / 1,000 / 65,536 cells 13.9 / 20.4 / 35 us, 53 species, 65,536 cells
// 172 us; spread 5.5 / 6.8 / 32 us and 147 us.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kPostThreads = 256, kPostCells = 16;

// sum over the 16 lanes of a DPP row (the same bits in every lane)
__device__ __forceinline__ double row_add(double x) {
    auto step = [](double v, auto ctrl) {
        const long long b = __double_as_longlong(v);
        const unsigned l = unsigned(__builtin_amdgcn_mov_dpp(int(b), decltype(ctrl)::value, 0xf, 0xf, true));
        const unsigned h = unsigned(__builtin_amdgcn_mov_dpp(int(b >> 32), decltype(ctrl)::value, 0xf, 0xf, true));
        return v + __longlong_as_double((long long)((unsigned long long)h << 32 | l));
    };
    x = step(x, std::integral_constant<int, 0xb1>{});   // quad_perm [1, 0, 3, 2]
    x = step(x, std::integral_constant<int, 0x4e>{});   // quad_perm [2, 3, 0, 1]
    x = step(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
    return step(x, std::integral_constant<int, 0x140>{});  // row_mirror
}

template <int K>
__global__ __launch_bounds__(kPostThreads) void post_kernel(DnnDevParams prm, MechDev m, int64_t first, int64_t n, int64_t ld,
                                                            double dt, const bf16_t *__restrict__ h, int h_ld,
                                                            const bf16_t *__restrict__ W, const float *__restrict__ b,
                                                            int k_in, const int8_t *__restrict__ flag,
                                                            const double *__restrict__ p, double *__restrict__ T,
                                                            double *__restrict__ Y, double *__restrict__ rr,
                                                            int32_t *__restrict__ status, int renormalise,
                                                            int32_t *__restrict__ idx, int32_t *__restrict__ count,
                                                            int fallback) {
    constexpr int NT = (K + 15) / 16;  // 16-output tiles
    static_assert(NT <= 4, "an output tile per wave");
    constexpr bool kSplit = NT == 1;
    constexpr int NP = 16 * NT + 1;    // LDS row stride (odd: conflict-free reads)
    constexpr int SP = NT;             // species per lane of stage 3
    __shared__ float su[kSplit ? 4 : 1][kPostCells * NP];
    __shared__ double s0[kPostCells * NP], s1[kPostCells * NP];
    const int lane = int(threadIdx.x) & 63, wv = int(threadIdx.x) >> 6;
    const int fr = lane & 15, fg = lane >> 4;
    const int64_t cell0 = first + int64_t(blockIdx.x) * kPostCells;
    if (kSplit || wv < NT) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        const bf16x8 zero = {};
        const int o = (kSplit ? 0 : wv * 16) + fr;
        const int64_t c = cell0 + fr;
        const bf16_t *wr = W + int64_t(o) * k_in + fg * 8, *hr = h + c * h_ld + fg * 8;
#pragma unroll 8
        for (int k0 = kSplit ? 32 * wv : 0; k0 < k_in; k0 += kSplit ? 128 : 32) {
            const bf16x8 wf = (o < K) ? *reinterpret_cast<const bf16x8 *>(wr + k0) : zero;
            const bf16x8 hf = (c < n) ? *reinterpret_cast<const bf16x8 *>(hr + k0) : zero;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, hf, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            su[kSplit ? wv : 0][fr * NP + (kSplit ? 0 : wv * 16) + fg * 4 + r] = acc[r];
    }
    __syncthreads();
    // ---- stage 3, FP64.  One species (or NT) of one cell per thread, cells along the lanes
    const int ca = int(threadIdx.x) % kPostCells, ka = int(threadIdx.x) / kPostCells;
    const int64_t ia = cell0 + ca;
    const int fa = ia < n ? int(flag[ia]) : 2;
    // the fallback list for the integrator's launch (its order does not change any cell's result)
    if (ka == 0 && fa == 0 && fallback) idx[atomicAdd(count, 1)] = int32_t(ia);
    // 1/lambda as an exact small integer (lambda = 0.1 gives 10): the power by squaring
    const int n_inv = (prm.inv_lambda == rint(prm.inv_lambda) && prm.inv_lambda >= 1.0 && prm.inv_lambda <= 64.0)
                          ? int(prm.inv_lambda)
                          : 0;
#pragma unroll
    for (int q = 0; q < SP; ++q) {
        const int k = ka + 16 * q;
        double y0 = 0.0, yn = 0.0;
        if (k < K && fa == 1) {
            float u = su[0][ca * NP + k];
            if (kSplit) {
#pragma unroll
                for (int w = 1; w < 4; ++w) u += su[w][ca * NP + k];
            }
            y0 = Y[k * ld + ia];
            const double z1 = boxcox(y0, prm.lambda) + (double(u + b[k]) * prm.sig_out[k] + prm.mu_out[k]);
            // the base clamped at 0 from below; a NaN (a non-finite network output) stays NaN, so
            // that the cell's temperature recovery fails and it is flagged non-finite
            const double b1 = 1.0 + prm.lambda * z1;
            const double base = (b1 < 0.0) ? 0.0 : b1;
            yn = n_inv ? ipow(base, n_inv) : pow(base, prm.inv_lambda);
        }
        s0[ca * NP + k] = y0;
        s1[ca * NP + k] = yn;
    }
    __syncthreads();
    // sixteen lanes per cell: the sums over the species, and T from h(T, Yn) = h0 by Newton with
    // dh/dT = cp
    const int cb = wv * 4 + fg;
    const int64_t ib = cell0 + cb;
    const bool run = ib < n && flag[ib] == 1;
    double cf[SP][10], Yn[SP];
    double sYW = 0.0, h0 = 0.0, sum = 0.0;
    const double T0 = run ? T[ib] : 1.0, iT0 = 1.0 / T0;
#pragma unroll
    for (int q = 0; q < SP; ++q) {
        const int k = fr + 16 * q;
        const double *r = m.sp + (k < K ? k : 0) * kSpTab;
        const double iW = k < K ? r[1] : 0.0;
#pragma unroll
        for (int e = 0; e < 5; ++e) cf[q][e] = r[2 + e] * iW;       // cp/R over 1, T .. T^4
#pragma unroll
        for (int e = 0; e < 4; ++e) cf[q][5 + e] = r[9 + e] * iW;   // h/(R T) over T .. T^4
        cf[q][9] = r[7] * iW;                                       // and 1/T
        const double y0 = s0[cb * NP + k];
        Yn[q] = s1[cb * NP + k];
        sYW += y0 * iW;
        h0 += y0 * (cf[q][0] + T0 * (cf[q][5] + T0 * (cf[q][6] + T0 * (cf[q][7] + T0 * cf[q][8]))) + cf[q][9] * iT0);
        sum += Yn[q];
    }
    sYW = row_add(sYW);
    h0 = row_add(h0) * T0;
    sum = row_add(sum);
    if (renormalise && sum > 0.0) {
        const double is = 1.0 / sum;
#pragma unroll
        for (int q = 0; q < SP; ++q) Yn[q] *= is;
    }
    double Tn = T0;
    bool conv = false, go = run;
    for (int it = 0; it < 20 && __ballot(go) != 0ull; ++it) {
        double hm = 0.0, cp = 0.0;
        const double iTn = 1.0 / Tn;
#pragma unroll
        for (int q = 0; q < SP; ++q) {
            const double *a = cf[q];
            cp += Yn[q] * (a[0] + Tn * (a[1] + Tn * (a[2] + Tn * (a[3] + Tn * a[4]))));
            hm += Yn[q] * (a[0] + Tn * (a[5] + Tn * (a[6] + Tn * (a[7] + Tn * a[8]))) + a[9] * iTn);
        }
        const double dT = (row_add(hm) * Tn - h0) / row_add(cp);
        if (go) {
            Tn -= dT;
            conv = isfinite(Tn) && fabs(dT) <= 1e-9;
            go = isfinite(Tn) && !conv;
        }
    }
    if (run) {
        const double rdt = rr ? p[ib] / (sYW * kR * T0) / dt : 0.0;
#pragma unroll
        for (int q = 0; q < SP; ++q) {
            const int k = fr + 16 * q;
            s0[cb * NP + k] = rdt * (Yn[q] - s0[cb * NP + k]);
            s1[cb * NP + k] = Yn[q];
        }
        if (fr == 0) {
            T[ib] = Tn;
            if (status) status[ib] = conv ? DF_CELL_OK : DF_CELL_NONFINITE;
        }
    }
    __syncthreads();
    if (fa != 1) return;
#pragma unroll
    for (int q = 0; q < SP; ++q) {
        const int k = ka + 16 * q;
        if (k >= K) continue;
        Y[k * ld + ia] = s1[ca * NP + k];
        if (rr) rr[k * ld + ia] = s0[ca * NP + k];
    }
}

int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

struct WsLayout {
    int64_t n_pad;
    size_t o_x, o_a, o_b, o_flag, o_idx, o_cnt, total;
    int wa, wb;  // widths of the two activation buffers
};

WsLayout workspace_layout(const df_dnn *d, int64_t n) {
    WsLayout w{};
    w.n_pad = round_up(std::max<int64_t>(n, 1), kGemmBM);
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const int nh = int(d->layers.size()) - 1;
    w.wa = w.wb = 0;
    for (int l = 0; l < nh; ++l) {
        if (l % 2 == 0)
            w.wa = std::max(w.wa, d->layers[l].n_pad);
        else
            w.wb = std::max(w.wb, d->layers[l].n_pad);
    }
    size_t o = 0;
    w.o_x = o;
    o = al(o + size_t(w.n_pad) * d->layers[0].k_pad * 2);
    w.o_a = o;
    o = al(o + size_t(w.n_pad) * w.wa * 2);
    w.o_b = o;
    o = al(o + size_t(w.n_pad) * w.wb * 2);
    w.o_flag = o;
    o = al(o + size_t(w.n_pad));
    w.o_idx = o;
    o = al(o + size_t(w.n_pad) * 4);
    w.o_cnt = o;
    o = al(o + 4);
    w.total = o;
    return w;
}

// Device blob of a network: per layer the bf16 weights [n_pad][k_pad] and fp32 biases [n_pad],
// the normalisation parameters, then per layer between two hidden layers the E4M3FN weights
// [n_pad][k_pad] and their row exponents [n_pad] (int32).  Offsets follow from the widths alone.
struct BlobLayout {
    std::vector<size_t> W, b, w8, e8;
    size_t prm = 0, total = 0;
};

BlobLayout blob_layout(const std::vector<DnnLayer> &layers, int n_in) {
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const int L = int(layers.size());
    BlobLayout bl;
    bl.W.assign(L, 0);
    bl.b.assign(L, 0);
    bl.w8.assign(L, 0);
    bl.e8.assign(L, 0);
    size_t o = 0;
    for (int l = 0; l < L; ++l) {
        bl.W[l] = o;
        o = al(o + size_t(layers[l].n_pad) * layers[l].k_pad * 2);
        bl.b[l] = o;
        o = al(o + size_t(layers[l].n_pad) * 4);
    }
    bl.prm = o;
    o = al(o + size_t(6) * n_in * 8);
    for (int l = 1; l + 1 < L; ++l) {
        bl.w8[l] = o;
        o = al(o + size_t(layers[l].n_pad) * layers[l].k_pad);
        bl.e8[l] = o;
        o = al(o + size_t(layers[l].n_pad) * 4);
    }
    bl.total = o;
    return bl;
}

// E4M3FN byte of v, |v| <= 448: round to nearest, ties to even; a non-finite v gives the
// format's NaN (the format has no infinity), so that it propagates as in the bf16 path
uint8_t e4m3_byte(float v) {
    const uint8_t sgn = std::signbit(v) ? 0x80 : 0x00;
    if (!std::isfinite(v)) return uint8_t(sgn | 0x7f);
    const float a = std::fabs(v);
    if (!(a > 0.0f)) return sgn;
    int k = 0;
    (void)std::frexp(a, &k);               // a = f 2^k, f in [0.5, 1): floor(log2 a) = k - 1
    int E = std::max(k - 1, -6);           // below 2^-6 the spacing stays 2^-9
    int m = int(std::nearbyint(std::ldexp(a, 3 - E)));  // a / 2^(E-3), exact before rounding
    if (E == -6 && m < 8) return uint8_t(sgn | m);     // subnormal
    if (m == 16) {
        m = 8;
        ++E;
    }
    return uint8_t(sgn | ((E + 7) << 3) | (m - 8));
}

// The input and output kernels take up to 16 threads per cell, and a launch holds fewer than 2^32: cells from `first`
// on in launches of at most kLaunchCells.
constexpr int64_t kLaunchCells = int64_t(1) << 27;
static_assert(kPostThreads / kPostCells <= 16 && kPreThreads / kPreCells <= 16, "threads per cell");
int64_t launch_cells(int64_t first, int64_t n) { return std::min(kLaunchCells, n - first); }

template <int K>
df_status launch_dnn_k(const df_dnn *d, const df_mech *m, int64_t n, int64_t ld, double dt, const double *p,
                       double *T, double *Y, double *rr, int32_t *status, void *ws, const df_dnn_opts &o,
                       const df_chem_opts &fo, hipStream_t s) {
    const WsLayout w = workspace_layout(d, n);
    auto *base = static_cast<unsigned char *>(ws);
    auto *xb = reinterpret_cast<bf16_t *>(base + w.o_x);
    auto *ba = reinterpret_cast<bf16_t *>(base + w.o_a);
    auto *bb = reinterpret_cast<bf16_t *>(base + w.o_b);
    auto *flag = reinterpret_cast<int8_t *>(base + w.o_flag);
    auto *idx = reinterpret_cast<int32_t *>(base + w.o_idx);
    auto *cnt = reinterpret_cast<int32_t *>(base + w.o_cnt);
    const int in_pad = d->layers[0].k_pad;
    for (int64_t first = 0; first < w.n_pad; first += kLaunchCells)
        hipLaunchKernelGGL(pre_kernel<K>, dim3(unsigned((launch_cells(first, w.n_pad) + kPreCells - 1) / kPreCells)),
                           dim3(kPreThreads), 0, s, d->prm, first, n, w.n_pad, ld, p, T, Y, xb, in_pad, flag, cnt, status,
                           rr, o.fallback);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("dnn pre launch: ") + hipGetErrorString(e));
    // hidden layers
    const bf16_t *in = xb;
    int in_ld = in_pad;
    const int nh = int(d->layers.size()) - 1;
    const bool fp8 = (o.precision == 1);
    const BlobLayout bl = fp8 ? blob_layout(d->layers, d->prm.n_in) : BlobLayout{};
    auto *blob = static_cast<unsigned char *>(d->dev_blob);
    // FP8 input of the current layer (E4M3FN bytes and block scales), when its producer wrote one
    const uint8_t *a8 = nullptr, *a8s = nullptr;
    int a8_sst = 0;
    for (int l = 0; l < nh; ++l) {
        const DnnLayer &L = d->layers[l];
        bf16_t *out = (l % 2 == 0) ? ba : bb;
        const int out_ld = (l % 2 == 0) ? w.wa : w.wb;
        // layers 1..nh-1 (between two hidden layers) in FP8: each reads the E4M3FN copy of its
        // input (bytes and block scales), written by the layer before it (the first layer, whose
        // K is 32 or 64 for every compiled species count, or an FP8 layer).  An FP8 copy fills
        // the layer's activation buffer as bytes [n_pad][out_ld] followed by the scales
        // [n_pad][sst].
        const bool q_next = fp8 && l + 1 < nh;
        auto *o8 = reinterpret_cast<uint8_t *>(out);
        uint8_t *o8s = o8 + size_t(w.n_pad) * out_ld;
        const int o8_sst = fp8_scale_stride(out_ld);
        df_status st;
        bool wrote8 = false;
        if (fp8 && l >= 1) {
            if (!a8) return fail(DF_E_UNSUPPORTED, "dnn step: FP8 needs a first layer with 32 or 64 padded inputs");
            st = launch_gemm_fp8(a8, in_ld, a8s, a8_sst, blob + bl.w8[l], L.k_pad,
                                 reinterpret_cast<const int32_t *>(blob + bl.e8[l]), L.b, out, out_ld,
                                 q_next ? o8s : nullptr, o8_sst, w.n_pad, n, L.n_pad, L.k_pad, s);
            wrote8 = q_next;
        } else if (q_next) {
            st = launch_gemm_bf16_fp8out(in, in_ld, L.W, L.k_pad, L.b, o8, out_ld, o8s, o8_sst, w.n_pad, n,
                                         L.n_pad, L.k_pad, s);
            wrote8 = true;
        } else {
            st = launch_gemm_bf16(in, in_ld, L.W, L.k_pad, L.b, out, out_ld, w.n_pad, n, L.n_pad, L.k_pad, s);
        }
        if (st != DF_OK) return st;
        a8 = wrote8 ? o8 : nullptr;
        a8s = wrote8 ? o8s : nullptr;
        a8_sst = o8_sst;
        in = out;
        in_ld = out_ld;
    }
    const DnnLayer &Lo = d->layers.back();
    for (int64_t first = 0; first < n; first += kLaunchCells)
        hipLaunchKernelGGL(post_kernel<K>, dim3(unsigned((launch_cells(first, n) + kPostCells - 1) / kPostCells)),
                           dim3(kPostThreads), 0, s, d->prm, m->dev, first, n, ld, dt, in, in_ld, Lo.W, Lo.b, Lo.k_pad,
                           flag, p, T, Y, rr, status, o.renormalise, idx, cnt, o.fallback);
    e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("dnn post launch: ") + hipGetErrorString(e));
    if (o.fallback) {
        const StepArgs a{n, ld, dt, nullptr, p, T, Y, nullptr, rr, status, nullptr, kernel_opts(fo),
                         DF_CELL_DNN_FALLBACK};
        return launch_chem_step(m->dev, a, fo.mapping, idx, cnt, s);
    }
    return DF_OK;
}

template <class T>
bool rd(std::ifstream &f, T *v, size_t n) {
    f.read(reinterpret_cast<char *>(v), std::streamsize(sizeof(T) * n));
    return bool(f);
}

}  // namespace
}  // namespace df

using namespace df;

extern "C" {

df_status df_dnn_load(const char *path, const df_mech *mech, int32_t device, df_dnn **out) {
    clear_error();
    if (!path || !mech || !out) return fail(DF_E_INVALID, "df_dnn_load: null path, mechanism or out");
    *out = nullptr;
    std::ifstream f(path, std::ios::binary);
    if (!f) return fail(DF_E_IO, std::string("cannot open DNN file ") + path);
    char magic[8];
    int32_t L = 0, K = 0, reserved = 0;
    if (!rd(f, magic, 8) || std::memcmp(magic, "DFDNN01", 7) != 0 || !rd(f, &L, 1) || L < 2 || L > 15)
        return fail(DF_E_FORMAT, std::string(path) + ": not a DFDNN01 file with 2..15 layers");
    std::vector<int32_t> dims(L + 1);
    double lam = 0, dtt = 0;
    if (!rd(f, dims.data(), dims.size()) || !rd(f, &K, 1) || !rd(f, &reserved, 1) || !rd(f, &lam, 1) ||
        !rd(f, &dtt, 1))
        return fail(DF_E_FORMAT, std::string(path) + ": truncated header");
    if (K != mech->host.K || dims[0] != K + 2 || dims[L] != K)
        return fail(DF_E_INVALID, "df_dnn_load: network widths do not match the mechanism's species count");
    for (int l = 0; l <= L; ++l)
        if (dims[l] < 1 || dims[l] > 65536) return fail(DF_E_FORMAT, "df_dnn_load: bad layer width");
    if (!(lam > 0) || !(dtt > 0)) return fail(DF_E_FORMAT, "df_dnn_load: lambda and dt_train must be > 0");
    const int ni = K + 2;
    std::vector<double> prm_h(size_t(6) * ni, 0.0);  // mu_in, sig_in, mu_out, sig_out, lo, hi
    for (int a = 0; a < 6; ++a) {
        const int cnt = (a == 2 || a == 3) ? K : ni;
        if (!rd(f, &prm_h[size_t(a) * ni], cnt)) return fail(DF_E_FORMAT, "df_dnn_load: truncated parameters");
    }
    for (int c = 0; c < ni; ++c)
        if (!(prm_h[size_t(ni) + c] > 0)) return fail(DF_E_FORMAT, "df_dnn_load: sig_in must be > 0");
    auto *d = new df_dnn;
    d->device = device;
    d->K = K;
    d->L = L;
    d->dims.assign(dims.begin(), dims.end());
    d->lambda = lam;
    d->dt_train = dtt;
    // padded device layout
    std::vector<std::vector<bf16_t>> Wh(L);
    std::vector<std::vector<float>> bh(L);
    int prev_pad = int(round_up(dims[0], kGemmBK));
    d->layers.resize(L);
    for (int l = 0; l < L; ++l) {
        DnnLayer &Ly = d->layers[l];
        Ly.n_in = dims[l];
        Ly.n_out = dims[l + 1];
        Ly.k_pad = prev_pad;
        Ly.n_pad = (l < L - 1) ? int(round_up(dims[l + 1], kGemmBN)) : dims[l + 1];
        std::vector<bf16_t> w(size_t(Ly.n_out) * Ly.n_in);
        std::vector<float> b(Ly.n_out);
        if (!rd(f, w.data(), w.size()) || !rd(f, b.data(), b.size())) {
            delete d;
            return fail(DF_E_FORMAT, std::string(path) + ": truncated weights");
        }
        Wh[l].assign(size_t(Ly.n_pad) * Ly.k_pad, 0);
        bh[l].assign(Ly.n_pad, 0.0f);
        for (int o = 0; o < Ly.n_out; ++o) {
            std::memcpy(&Wh[l][size_t(o) * Ly.k_pad], &w[size_t(o) * Ly.n_in], sizeof(bf16_t) * Ly.n_in);
            bh[l][o] = b[o];
        }
        prev_pad = Ly.n_pad;
    }
    // one device allocation
    const BlobLayout bl = blob_layout(d->layers, ni);
    const std::vector<size_t> &offW = bl.W, &offb = bl.b;
    const size_t offP = bl.prm, o = bl.total;
    int prev = 0;
    if (hipGetDevice(&prev) != hipSuccess || hipSetDevice(device) != hipSuccess) {
        delete d;
        return fail(DF_E_HIP, "df_dnn_load: cannot select device");
    }
    void *blob = nullptr;
    hipError_t e = hipMalloc(&blob, o);
    if (e == hipSuccess) {
        std::vector<unsigned char> h(o, 0);
        for (int l = 0; l < L; ++l) {
            std::memcpy(h.data() + offW[l], Wh[l].data(), Wh[l].size() * 2);
            std::memcpy(h.data() + offb[l], bh[l].data(), bh[l].size() * 4);
        }
        std::memcpy(h.data() + offP, prm_h.data(), prm_h.size() * 8);
        // E4M3FN copies of the weights between two hidden layers, one power-of-two scale per row
        for (int l = 1; l + 1 < L; ++l) {
            const DnnLayer &Ly = d->layers[l];
            auto *e8 = reinterpret_cast<int32_t *>(h.data() + bl.e8[l]);
            for (int r = 0; r < Ly.n_pad; ++r) {
                const bf16_t *wr = &Wh[l][size_t(r) * Ly.k_pad];
                auto bf = [](bf16_t x) {
                    uint32_t u = uint32_t(x) << 16;
                    float f;
                    std::memcpy(&f, &u, 4);
                    return f;
                };
                float wmax = 0.0f;
                for (int c = 0; c < Ly.k_pad; ++c) wmax = std::max(wmax, std::fabs(bf(wr[c])));
                const int e = fp8_scale_exp(wmax);
                e8[r] = e;
                uint8_t *q = h.data() + bl.w8[l] + size_t(r) * Ly.k_pad;
                for (int c = 0; c < Ly.k_pad; ++c) q[c] = e4m3_byte(std::ldexp(bf(wr[c]), -e));
            }
        }
        e = hipMemcpy(blob, h.data(), o, hipMemcpyHostToDevice);
    }
    (void)hipSetDevice(prev);
    if (e != hipSuccess) {
        if (blob) (void)hipFree(blob);
        delete d;
        return fail(DF_E_HIP, std::string("df_dnn_load: ") + hipGetErrorString(e));
    }
    d->dev_blob = blob;
    auto *base = static_cast<unsigned char *>(blob);
    for (int l = 0; l < L; ++l) {
        d->layers[l].W = reinterpret_cast<bf16_t *>(base + offW[l]);
        d->layers[l].b = reinterpret_cast<float *>(base + offb[l]);
    }
    const double *P = reinterpret_cast<const double *>(base + offP);
    d->prm = DnnDevParams{K, ni, lam, 1.0 / lam, P, P + ni, P + 2 * ni, P + 3 * ni, P + 4 * ni, P + 5 * ni};
    *out = d;
    return DF_OK;
}

void df_dnn_free(df_dnn *d) {
    if (!d) return;
    int prev = 0;
    if (hipGetDevice(&prev) == hipSuccess && hipSetDevice(d->device) == hipSuccess) {
        (void)hipFree(d->dev_blob);
        (void)hipSetDevice(prev);
    }
    delete d;
}

df_status df_dnn_info(const df_dnn *d, int32_t *n_layers, int32_t *dims, double *lambda, double *dt_train) {
    clear_error();
    if (!d) return fail(DF_E_INVALID, "df_dnn_info: null handle");
    if (n_layers) *n_layers = d->L;
    if (dims)
        for (int l = 0; l <= d->L; ++l) dims[l] = d->dims[l];
    if (lambda) *lambda = d->lambda;
    if (dt_train) *dt_train = d->dt_train;
    return DF_OK;
}

df_status df_dnn_workspace_size(const df_dnn *d, int64_t n_cells, size_t *bytes) {
    clear_error();
    if (!d || !bytes || n_cells < 0) return fail(DF_E_INVALID, "df_dnn_workspace_size: bad arguments");
    *bytes = workspace_layout(d, n_cells).total;
    return DF_OK;
}

#define DF_DNN_SPECIES_LIST(X) X(2) X(4) X(9) X(53)

df_status df_dnn_step(const df_dnn *d, const df_mech *m, int64_t n, int64_t ld, double dt, const double *p, double *T,
                      double *Y, double *rr, int32_t *status, void *ws, size_t ws_bytes, const df_dnn_opts *opts,
                      const df_chem_opts *fallback_opts, void *hip_stream) {
    clear_error();
    if (!d || !m) return fail(DF_E_INVALID, "df_dnn_step: null DNN or mechanism handle");
    if (d->K != m->host.K || d->device != m->device)
        return fail(DF_E_INVALID, "df_dnn_step: DNN and mechanism differ in species count or device");
    if (n < 0 || ld < n) return fail(DF_E_INVALID, "df_dnn_step: need 0 <= n_cells <= ld");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(DF_E_INVALID, "df_dnn_step: dt must be finite and > 0");
    if (std::fabs(dt - d->dt_train) > 1e-12 * d->dt_train)
        return fail(DF_E_UNSUPPORTED, "df_dnn_step: dt differs from the time step the network was trained for");
    if (n > 0 && (!p || !T || !Y)) return fail(DF_E_INVALID, "df_dnn_step: null p, T or Y");
    if (n > 0x7fffffff) return fail(DF_E_UNSUPPORTED, "df_dnn_step: more than 2^31-1 cells");
    df_dnn_opts o;
    df_dnn_default_opts(&o);
    if (opts) o = *opts;
    if ((o.renormalise != 0 && o.renormalise != 1) || (o.fallback != 0 && o.fallback != 1) ||
        (o.precision != 0 && o.precision != 1) || o.reserved1)
        return fail(DF_E_INVALID, "df_dnn_opts: renormalise, fallback and precision must be 0 or 1, reserved 0");
    df_chem_opts fo;
    df_chem_default_opts(&fo);
    if (fallback_opts) fo = *fallback_opts;
    df_status st = validate_chem_opts(fo);
    if (st != DF_OK) return st;
    if (n == 0) return DF_OK;
    const size_t need = workspace_layout(d, n).total;
    if (!ws || ws_bytes < need)
        return fail(DF_E_INVALID, "df_dnn_step: workspace missing or smaller than df_dnn_workspace_size");
    if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return fail(DF_E_INVALID, "df_dnn_step: workspace not 256-byte aligned");
    int prev = 0;
    if (hipGetDevice(&prev) != hipSuccess) return fail(DF_E_HIP, "df_dnn_step: hipGetDevice failed");
    if (prev != d->device && hipSetDevice(d->device) != hipSuccess)
        return fail(DF_E_HIP, "df_dnn_step: cannot select the device");
    auto s = static_cast<hipStream_t>(hip_stream);
    switch (d->K) {
#define DF_CASE(k)                                                                \
    case k:                                                                       \
        st = launch_dnn_k<k>(d, m, n, ld, dt, p, T, Y, rr, status, ws, o, fo, s); \
        break;
        DF_DNN_SPECIES_LIST(DF_CASE)
#undef DF_CASE
        default:
            st = fail(DF_E_UNSUPPORTED, "df_dnn_step: no compiled kernels for " + std::to_string(d->K) + " species");
    }
    if (prev != d->device) (void)hipSetDevice(prev);
    return st;
}

}  // extern "C"
