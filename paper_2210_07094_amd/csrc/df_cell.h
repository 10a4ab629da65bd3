// One wavefront per cell for small mechanisms: lane exchanges, elementary functions, and the rate and
// Jacobian phases that the integrator (df_chem_cell.hip) and the reverse sweep of its
// adjoint (df_adjoint_cell.hip) share.  The lane layout is described in df_chem_cell.hip.
#pragma once

#include <type_traits>

#include "df_internal.h"
#include "df_kinetics.h"

namespace df {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

// Order LDS accesses of the wave's lanes: one wave's LDS requests are served in order, so only the
// compiler must not move memory operations across this point.
__device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int lo32(double x) { return int(__double_as_longlong(x)); }
__device__ __forceinline__ int hi32(double x) { return int(__double_as_longlong(x) >> 32); }
__device__ __forceinline__ double mk64(int lo, int hi) {
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const int l = lo32(x), h = hi32(x);
    return mk64(__builtin_amdgcn_mov_dpp(l, CTRL, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(h, CTRL, 0xf, 0xf, true));
}
constexpr int kXor1 = 0xb1, kXor2 = 0x4e, kHalfMirror = 0x141, kMirror = 0x140, kQuad0 = 0x00;

// sum over the lanes of a quad, and over the 16 lanes of a row (the same bits in every lane)
__device__ __forceinline__ double quad_sum(double x) {
    x += dpp<kXor1>(x);
    return x + dpp<kXor2>(x);
}
__device__ __forceinline__ double row_sum(double x) {
    x = quad_sum(x);
    x += dpp<kHalfMirror>(x);
    return x + dpp<kMirror>(x);
}
__device__ __forceinline__ int row_max(int x) {
    x = max(x, __builtin_amdgcn_update_dpp(0, x, kXor1, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, kXor2, 0xf, 0xf, false));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, kHalfMirror, 0xf, 0xf, false));
    return max(x, __builtin_amdgcn_update_dpp(0, x, kMirror, 0xf, 0xf, false));
}

// the two halves of the wave (lane l and l ^ 32): a = the lower half's value, b = the upper's
__device__ __forceinline__ void halves(double x, double &a, double &b) {
    const auto l = __builtin_amdgcn_permlane32_swap(unsigned(lo32(x)), unsigned(lo32(x)), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(unsigned(hi32(x)), unsigned(hi32(x)), false, false);
    a = mk64(int(l[0]), int(h[0]));
    b = mk64(int(l[1]), int(h[1]));
}
// rows 0/1 and 2/3 of a half: a = the even row's value, b = the odd row's
__device__ __forceinline__ void rows(double x, double &a, double &b) {
    const auto l = __builtin_amdgcn_permlane16_swap(unsigned(lo32(x)), unsigned(lo32(x)), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(unsigned(hi32(x)), unsigned(hi32(x)), false, false);
    a = mk64(int(l[0]), int(h[0]));
    b = mk64(int(l[1]), int(h[1]));
}
__device__ __forceinline__ double half_sum(double x) {
    double a, b;
    halves(x, a, b);
    return a + b;
}
// sum over the four copies of a row
__device__ __forceinline__ double copies_sum(double x) {
    double a, b;
    halves(x, a, b);
    rows(a + b, a, b);
    return a + b;
}
// the value that copy G of the row holds, in all four
template <int G>
__device__ __forceinline__ double copy_of(double x) {
    double a, b;
    halves(x, a, b);
    rows((G & 2) ? b : a, a, b);
    return (G & 1) ? b : a;
}
__device__ __forceinline__ double lane_value(double x, int lane) {
    return mk64(__builtin_amdgcn_readlane(lo32(x), lane), __builtin_amdgcn_readlane(hi32(x), lane));
}
__device__ __forceinline__ double from_lane(int addr, double x) {  // addr = 4 * lane, per lane
    return mk64(__builtin_amdgcn_ds_bpermute(addr, lo32(x)), __builtin_amdgcn_ds_bpermute(addr, hi32(x)));
}

// 1/b for normal finite b: the hardware estimate and one third-order step, r + r (e + e^2) with
// e = 1 - b r (the estimate's e is below 2^-20, so e^3 is below the last bit).
__device__ __forceinline__ double frcp3(double b) {
    const double r = __builtin_amdgcn_rcp(b);
    const double e = fma(-b, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// Coefficients of the logarithm and the exponential, held in scalar registers: the kernel sets them
// once and hides their values, so that the compiler neither rebuilds a literal at each use nor
// copies it into a vector register (their signs are flipped: a negated addend keeps the
// three-operand form of the multiply-add).  Both polynomials interpolate at Chebyshev points.
struct Coef {
    double l[8];   // -(atanh(s)/s - 1)/s^2 over s^2 in [0, 0.0295], interpolation error 5e-19
    double e[10];  // -(e^r - 1 - r)/r^2 over |r| <= 0.3466, interpolation error 1.3e-17 of e^r
    double log2e, ln2h, ln2l, sqh;
    __device__ __forceinline__ void set() {
        constexpr double L[8] = {0.3333333333333333,  0.2000000000000044,  0.14285714285401616, 0.11111111195900235,
                                 0.09090897815442377, 0.07693120102906739, 0.06634379834280306, 0.06543383504974087};
        constexpr double E[10] = {0.5000000000000001,     0.16666666666666669,    0.04166666666662413,
                                  0.008333333333330062,   0.0013888888917213717,  0.00019841269863053618,
                                  2.4801521295954376e-05, 2.7557268459997064e-06, 2.7620088445409746e-07,
                                  2.510038549551032e-08};
        for (int i = 0; i < 8; ++i) {
            l[i] = -L[i];
            asm("" : "+s"(l[i]));
        }
        for (int i = 0; i < 10; ++i) {
            e[i] = -E[i];
            asm("" : "+s"(e[i]));
        }
        log2e = 1.44269504088896340736;
        ln2h = -kLn2Hi;
        ln2l = -kLn2Lo;
        sqh = 0.70710678118654752440;
        asm("" : "+s"(log2e));
        asm("" : "+s"(ln2h));
        asm("" : "+s"(ln2l));
        asm("" : "+s"(sqh));
    }
};

// e^x: n = rint(x / ln 2), r = x - n ln 2 in two parts, e^r = 1 + (r + r^2 P(r)), scaled by 2^n.
// Overflow gives +inf, underflow 0 or a denormal, NaN stays NaN.  |x| below 1e44: beyond, the rounding of n ln 2 leaves
// an r whose polynomial overflows (the coefficient rows are kept at 1e30 when they are packed).
__device__ __forceinline__ double dexp(const Coef &c, double x) {
    const double n = __builtin_rint(x * c.log2e);
    const double r = fma(n, c.ln2l, fma(n, c.ln2h, x));
    double q = fma(r, -c.e[9], -c.e[8]);
#pragma unroll
    for (int i = 7; i >= 0; --i) q = fma(q, r, -c.e[i]);
    return ldexp(1.0 + fma(q, r * r, r), int(n));
}

// ln x for positive finite x: x = 2^e m with m in [1/sqrt 2, sqrt 2), ln m = 2 atanh(s),
// s = (m - 1)/(m + 1).  Anything else gives NaN.
__device__ __forceinline__ double dlogp(const Coef &c, double x) {
    int e;
    double m = frexp(x, &e);
    const bool lo = m < c.sqh;
    m = lo ? m + m : m;
    e = lo ? e - 1 : e;
    const double b = m + 1.0, a = m - 1.0;
    const double ib = frcp3(b);
    const double s0 = a * ib;
    const double s = fma(ib, fma(-b, s0, a), s0);
    const double z = s * s;
    double q = fma(z, -c.l[7], -c.l[6]);
#pragma unroll
    for (int i = 5; i >= 0; --i) q = fma(q, z, -c.l[i]);
    const double t = s + s;
    const double lm = fma(t * z, q, t);
    const double de = double(e);
    const double r = fma(-de, c.ln2h, fma(-de, c.ln2l, lm));
    return x > 0.0 ? r : __builtin_nan("");
}

// The cell of a one-wave block in a launch of n such blocks: eight neighbouring cells (64 bytes of each
// cell-minor array) go to blocks eight apart, which run on the same XCD.
__device__ __forceinline__ int64_t cell_of_block(int64_t n) {
    const int64_t b = blockIdx.x;
    return b < n / 64 * 64 ? b / 64 * 64 + b % 8 * 8 + b / 8 % 8 : b;
}

// the mechanism as these kernels read it
struct CellMech {
    const double *xd;   // per-lane rows
    const int *xi;
    const double *eff;  // [M][K + 4]
    int M, troe, both;
};

template <int K, int EL>
struct CellWave {
    static constexpr int N = K + 1;
    static constexpr int NC = (N + 2 + 3) / 4;  // record columns (T, species, q, density) per lane
    static constexpr int NI = (N + 3) / 4;      // matrix columns per lane
    static constexpr int MR = 4 * EL;           // reaction records (a row of zeros beyond M)
    static constexpr int RS = 17;               // record stride: columns 0..15 and a scratch column
    static_assert(N + 2 <= 16, "the record's columns and the rows fit 16 lanes");

    // LDS, in doubles
    static constexpr int oY = 0;                // stage state
    static constexpr int oV = oY + 16;          // right-hand side in pivot order; slot 16 takes idle rows
    static constexpr int oC = oV + 18;          // concentrations (slot 0 = 1)
    static constexpr int oCp = oC + 16;         // cp_k of the rows
    static constexpr int oQ = oCp + 16;         // q_j, then q_j dH_j/(R T)
    static constexpr int oRec = oQ + 64;
    static constexpr int oEff = oRec + MR * RS; // third-body efficiencies of the reactions
    static constexpr int kEnd = oEff + 32 * K;

    // the lane's rows of the mechanism, loaded once per wave
    struct Row {
        double e[7], dh[6], iW, W, a[5], wq, cnt, sg, eeff[3], w[K], lc[EL], nu[EL], icol[NI];
        int sl[3], li[EL], ec[3], em[3], src, flags, cw;
    };
    // flags: 1 = third-body reaction, 2 = falloff reaction, 4 = quad of a falloff reaction,
    // 8 = entry of a species that is on both sides, product side (added to the reactant side's)

    __device__ __forceinline__ static void load_row(const CellMech &m, int lane, Row &o) {
        const double *d = m.xd + lane;
        const int *q = m.xi + lane;
        int f = 0;
        auto D = [&]() { return d[64 * f++]; };
#pragma unroll
        for (int i = 0; i < 7; ++i) o.e[i] = D();
#pragma unroll
        for (int i = 0; i < 6; ++i) o.dh[i] = D();
        o.iW = D();
        o.W = D();
#pragma unroll
        for (int i = 0; i < 5; ++i) o.a[i] = D();
        o.wq = D();
        o.cnt = D();
        o.sg = D();
#pragma unroll
        for (int i = 0; i < 3; ++i) o.eeff[i] = D();
#pragma unroll
        for (int i = 0; i < K; ++i) o.w[i] = D();
#pragma unroll
        for (int i = 0; i < NI; ++i) o.icol[i] = D();
#pragma unroll
        for (int i = 0; i < EL; ++i) o.lc[i] = D();
#pragma unroll
        for (int i = 0; i < EL; ++i) o.nu[i] = D();
        o.cw = (lane & 15) ? (lane & 15) : 15;  // row 0 has no concentration; slot 0 stays 1
        f = 0;
        auto I = [&]() { return q[64 * f++]; };
#pragma unroll
        for (int i = 0; i < 3; ++i) o.sl[i] = I();
#pragma unroll
        for (int i = 0; i < 3; ++i) o.ec[i] = I();
#pragma unroll
        for (int i = 0; i < 3; ++i) o.em[i] = I();
        o.src = I();
        o.flags = I();
#pragma unroll
        for (int i = 0; i < EL; ++i) o.li[i] = I();
    }

    // the LDS of a wave at its start: zeros, and the efficiencies of the reactions
    __device__ __forceinline__ static void load_eff(const CellMech &m, int lane, double *sh) {
        constexpr int kPer = (32 * K + 63) / 64;
        double ef[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            const int i = 64 * e + lane, j = i / K;
            ef[e] = (j < m.M) ? m.eff[j * (K + 4) + i % K] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < (oEff + 63) / 64; ++e)
            if (64 * e + lane < oEff) sh[64 * e + lane] = 0.0;
#pragma unroll
        for (int e = 0; e < kPer; ++e)
            if (64 * e + lane < 32 * K) sh[oEff + 64 * e + lane] = ef[e];
    }

    // what the rates share with the caller
    struct Rates {
        double T, iT, Wbar, irho, c6, Mc, kk, c0, c1, c2, P, X, dl, gM, cpR;
        // adjoint only: 1 - d ln k/d ln A of falloff reactions, and what its second derivatives need
        double h, E, arg, lx, lc, dlr;
    };

    // per-cell constants
    struct Cell {
        double p, ip, c6p, lc6p;  // p, 1/p, 1e-6 p/R and its logarithm
    };

    // rate constants and signed one-way rates X of the lane's reaction side at state y (row yr in
    // the lane, all rows through LDS); MODE 1 and 2 also their logarithmic T-derivative and dk/d[M],
    // 2 the adjoint's members
    template <int MODE>
    __device__ __forceinline__ static void rates(const CellMech &mg, const Coef &kc, const Row &o, const Cell &c, double *sh, int lane,
                                                 int r, double yr, Rates &s) {
        constexpr bool JAC = MODE > 0;
        lds_order();
        sh[oY + r] = yr;
        lds_order();
        double y[N];
#pragma unroll
        for (int k = 0; k < N; ++k) y[k] = sh[oY + k];
        s.T = y[0];
        double m0 = 0.0, m1 = 0.0;
#pragma unroll
        for (int k = 0; k < K; k += 2) m0 = fma(y[1 + k], o.w[k], m0);
#pragma unroll
        for (int k = 1; k < K; k += 2) m1 = fma(y[1 + k], o.w[k], m1);
        const double m = m0 + m1, sYW = lane_value(m, 63);
        s.iT = frcp3(s.T);
        s.Wbar = frcp3(sYW);
        s.c6 = c.c6p * s.iT * s.Wbar;
        s.irho = (kR * c.ip) * s.T * sYW;
        const double lx = dlogp(kc, lane == 0 ? s.T : m);
        const double lT = lane_value(lx, 0);
        lds_order();
        sh[oC + o.cw] = s.c6 * yr * o.iW;
        lds_order();
        s.c0 = sh[oC + o.sl[0]];
        s.c1 = sh[oC + o.sl[1]];
        s.c2 = sh[oC + o.sl[2]];
        s.cpR = fma(s.T, fma(s.T, fma(s.T, fma(s.T, o.a[4], o.a[3]), o.a[2]), o.a[1]), o.a[0]);
        double arg = fma(s.T, fma(s.T, fma(s.T, fma(s.T, o.e[6], o.e[5]), o.e[4]), o.e[3]), o.e[0]);
        arg = fma(o.e[2], s.iT, arg);
        arg = fma(o.e[1], lT, arg);
        const double E = dexp(kc, arg);
        s.Mc = m * s.c6;
        s.dl = 0.0;
        s.gM = 0.0;
        if (JAC)
            s.dl = fma(fma(-o.e[2], s.iT, o.e[1]), s.iT,
                       fma(s.T, fma(s.T, fma(4.0 * s.T, o.e[6], 3.0 * o.e[5]), 2.0 * o.e[4]), o.e[3]));
        s.h = 0.0;
        if (MODE == 2) {
            s.E = E;
            s.arg = arg;
            s.lx = lx;
            s.lc = c.lc6p - lT - lane_value(lx, 63);
            s.dlr = s.dl;
        }
        double k = E;
        if (mg.troe) {
            // Lindemann form times the Troe broadening factor F, in the four lanes of the reaction's
            // quad: lane 0 holds k0/k_inf, lanes 1..3 the terms of F_cent
            const double wE = o.wq * E;
            const double Fc = quad_sum(wE);
            const double lFc = dlogp(kc, Fc) * kInvLn10;
            const double lPr = (dpp<kQuad0>(arg) + lx + (c.lc6p - lT - lane_value(lx, 63))) * kInvLn10;
            const double k0 = dpp<kQuad0>(E);
            const double Pr = k0 * s.Mc;
            const double cc = fma(-0.67, lFc, -0.4);
            const double nn = fma(-1.27, lFc, 0.75);
            const double x = lPr + cc;
            const double den = fma(-0.14, x, nn);
            double iden, f1, q1;  // f1 = x/den, q1 = 1/(1 + f1^2)
            if (JAC) {
                iden = frcp3(den);
                f1 = x * iden;
                q1 = frcp3(fma(f1, f1, 1.0));
            } else {
                const double d2 = den * den;
                q1 = d2 * frcp3(fma(x, x, d2));
            }
            const double F = dexp(kc, kLn10 * (lFc * q1));
            const double iPr1 = frcp3(1.0 + Pr);
            const bool quad = o.flags & 4;
            const double fac = quad ? Pr * iPr1 * F : 1.0;
            k = E * from_lane(o.src, fac);
            if (JAC) {
                const double gq = 2.0 * f1 * q1 * q1;
                const double g2 = lFc * gq * (iden * iden);
                const double dlF_dlPr = -g2 * nn;
                const double dlF_dlFc = fma(-g2, fma(1.27, x, -0.67 * nn), q1);
                const double dFc = quad_sum(wE * s.dl);
                const double h = iPr1 + dlF_dlPr;
                const double dlp = h * dpp<kQuad0>(s.dl) + dlF_dlFc * fdiv(dFc, Fc);
                s.gM = from_lane(o.src, quad ? F * k0 * iPr1 * h : 0.0);
                s.dl += from_lane(o.src, quad ? dlp : 0.0);
                s.gM *= E * o.sg;
                if (MODE == 2) s.h = from_lane(o.src, quad ? h : 0.0);
            }
        }
        s.kk = k * o.sg;
        s.P = s.c0 * s.c1 * s.c2;
        s.X = s.kk * s.P;
    }

    // component r of f(y)
    __device__ __forceinline__ static double rhs(const CellMech &mg, const Coef &kc, const Row &o, const Cell &c, double *sh, int lane,
                                                 int r, double yr) {
        Rates s;
        rates<0>(mg, kc, o, c, sh, lane, r, yr, s);
        const double dH = fma(s.T, fma(s.T, fma(s.T, fma(s.T, o.dh[4], o.dh[3]), o.dh[2]), o.dh[1]),
                              fma(o.dh[5], s.iT, o.dh[0]));
        const double cps = row_sum(yr * o.iW * s.cpR);
        const double icp = frcp3(cps);
        const double co = 1e6 * s.irho * ((r == 0) ? -s.T * icp : o.W);
        const double q = half_sum(s.X) * ((o.flags & 1) ? s.Mc : 1.0);
        sh[oQ + lane] = q * dH;  // dH = 1 in the lower half
        lds_order();
        double b0 = 0.0, b1 = 0.0;
#pragma unroll
        for (int e = 0; e < EL; e += 2) {
            b0 = fma(o.lc[e], sh[oQ + o.li[e]], b0);
            b1 = fma(o.lc[e + 1], sh[oQ + o.li[e + 1]], b1);
        }
        return co * copies_sum(b0 + b1);
    }

    // each reaction's record: column 0 its T-derivative dq, 1 + l the derivative with respect to the
    // concentration of species l, N its rate q; G = d q / d [M], Mq = [M] for third-body rows, else 1
    __device__ __forceinline__ static void records(const CellMech &mg, const Row &o, const Rates &s, double *sh,
                                                   int lane, double G, double Mq, double q, double dq) {
        const double km = Mq * s.kk;
        const double P0 = km * (s.c1 * s.c2), P1 = km * (s.c0 * s.c2), P2 = km * (s.c0 * s.c1);
        const int j = lane & 31;
        double *rc = sh + oRec + (j < mg.M ? j : 0) * RS;  // lanes beyond M write the scratch column only
        if ((o.flags & 3) && lane < 32) {
            const double *ef = sh + oEff + j * K;
#pragma unroll
            for (int l = 0; l < K; ++l) rc[1 + l] = G * ef[l];
        }
        lds_order();
        // entry e: the species of slot e, whose derivative counts once for each of the side's slots it fills
        const double v[3] = {o.em[0] * P0, o.em[1] * P1, o.em[2] * P2};
        if (!mg.both) {
#pragma unroll
            for (int e = 0; e < 3; ++e) rc[o.ec[e]] = fma(G, o.eeff[e], v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (!(o.flags & (8 << e))) rc[o.ec[e]] = fma(G, o.eeff[e], v[e]);
            lds_order();
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (o.flags & (8 << e)) rc[o.ec[e]] += v[e];
        }
        if (lane < mg.M) {
            rc[N] = q;
            rc[0] = dq;
        }
    }

    // f_r, and J in the 2D layout: J[i] = entry (r, 4 i + g)
    __device__ __forceinline__ static double jacobian(const CellMech &mg, const Coef &kc, const Row &o, const Cell &c, double *sh,
                                                      int lane, int r, int g, double yr, double (&J)[NI]) {
        Rates s;
        rates<1>(mg, kc, o, c, sh, lane, r, yr, s);
        const double dH = fma(s.T, fma(s.T, fma(s.T, fma(s.T, o.dh[4], o.dh[3]), o.dh[2]), o.dh[1]),
                              fma(o.dh[5], s.iT, o.dh[0]));
        const bool tb = o.flags & 1;
        const double Mq = tb ? s.Mc : 1.0;
        const double X = half_sum(s.X);
        const double G = half_sum(tb ? s.X : s.gM * s.P);  // d q / d [M]
        const double S = fma(G, s.Mc, Mq * half_sum(s.X * o.cnt));
        const double dq = Mq * half_sum(s.X * s.dl);
        records(mg, o, s, sh, lane, G, Mq, Mq * X, dq);
        if (lane < mg.M) sh[oRec + lane * RS + N + 1] = S;
        if (lane >= 32) sh[oQ + lane] = dH;
        sh[oCp + r] = s.cpR * kR * o.iW;  // cp_r in J/kg/K (row 0: 0)
        lds_order();
        // records^T (16 columns x reactions) times (reactions x 16 rows)
        d4 D = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            const double A = sh[oRec + (4 * e + g) * RS + r];
            const double dh = sh[oQ + 32 + 4 * e + g];
            D = __builtin_amdgcn_mfma_f64_16x16x4f64(A, (r == 0) ? dh : o.nu[e], D, 0, 0, 0);
        }
        double cpc[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) cpc[i] = sh[oCp + 4 * i + g];
        const double wd = copy_of<N % 4>(D[N / 4]);
        const double sq = copy_of<(N + 1) % 4>(D[(N + 1) / 4]);
        const double yiw = yr * o.iW;
        const double cps = row_sum(yiw * s.cpR);
        const double dcpR = fma(s.T, fma(s.T, fma(4.0 * s.T, o.a[4], 3.0 * o.a[3]), 2.0 * o.a[2]), o.a[1]);
        const double dcp = kR * row_sum(yiw * dcpR);
        const double icp = frcp3(kR * cps);
        const double Wm = (r == 0) ? kR * s.T : o.W;
        const double co = 1e6 * Wm * s.irho;
        const double f = co * wd;  // row 0: sum_k h_k f_k
        const double cf = row_sum(s.cpR * kR * o.iW * f);
        const double fT = -f * icp;
        const double dif = co * (wd - sq);
        const double gk = dif * s.Wbar;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            double v = fma(Wm, D[i], gk) * o.icol[i];
            double dc = cpc[i];
            double ex = 0.0;
            if (i == 0) {
                v = (g == 0) ? fma(dif, s.iT, co * D[0]) : v;
                dc = (g == 0) ? dcp : dc;
                ex = (g == 0) ? cf : 0.0;
            }
            const double v0 = -(fma(fT, dc, v) + ex) * icp;
            v = (r == 0) ? v0 : v;
            J[i] = (4 * i + g < N) ? v : 0.0;
        }
        return (r == 0) ? fT : f;
    }

    // In-place Gauss-Jordan inverse of a (2D layout) with partial pivoting: at step k the pivot is the
    // unused row of largest |a_ik|, by a 32-bit key as in the 16-lane kernel (exponent and 16 mantissa
    // bits, ties to the lowest row).  Rows are not moved while eliminating: with p_k the pivot row of
    // step k, entry (p_k, j) ends as entry (k, p_j) of the inverse.  A pivot row is divided by its pivot
    // only at the end (steps act on it as on its multiple), so that a step changes every row but its own
    // pivot's in the same way.  On return lane (r, g) holds row r of the inverse, column p_(4 i + g) in a[i];
    // prow = p_r; slot is the step at which row r was the pivot (16 for idle rows): the place of
    // row r's right-hand side.
    __device__ __forceinline__ static void invert(double (&a)[NI], int r, int g, int &prow, int &slot) {
        int low = (r < N) ? 15 - r : -17;  // the key's low bits; -1 - k once row r was the pivot of step k
        double sc = 0.0;                   // 1/pivot of row r
        auto step = [&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int ik = k / 4, gk = k % 4;
            const double cv = from_lane(4 * r + 64 * gk, a[ik]);
            const double inv = frcp3(cv);
            const int key = row_max((hi32(cv) & 0x7ffffff0) | low);
            const int pk = min(15 - (__builtin_amdgcn_readfirstlane(key) & 15), N - 1);
            const int addr = 4 * pk + 64 * g;
            double pr[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) pr[i] = from_lane(addr, a[i]);
            const bool piv = (r == pk);
            const double cm = cv * -lane_value(inv, pk);
            const double m = piv ? 0.0 : cm;
#pragma unroll
            for (int i = 0; i < NI; ++i) a[i] = fma(m, pr[i], a[i]);
            a[ik] = (g == gk) ? (piv ? 1.0 : m) : a[ik];
            sc = piv ? inv : sc;
            low = piv ? -1 - k : low;
        };
        each(step, std::integral_constant<int, 0>{});
        slot = ~low;
        const int lane0 = 64 * g;
        prow = __builtin_amdgcn_ds_permute(lane0 + 4 * ((r < N) ? slot : r), r);
        const int addr = 4 * prow + 64 * g;
#pragma unroll
        for (int i = 0; i < NI; ++i) a[i] = from_lane(addr, a[i] * sc);
    }
    template <class F, int k>
    __device__ __forceinline__ static void each(F &f, std::integral_constant<int, k> c) {
        f(c);
        if constexpr (k + 1 < N) each(f, std::integral_constant<int, k + 1>{});
    }
};

}  // namespace
}  // namespace df
