// Reverse sweep of the discrete adjoint on gfx950 with one wavefront per cell, for the mechanisms of
// the one-wave-per-cell integrator (the lane layout is described in df_chem_cell.hip) whose rows' lists of
// slot derivatives fit 32 entries.  The sweep
// itself, and the formulas it reverses, are those of df_adjoint.hip:
//   ubar_i = b_i lam, ybar = lam;  for i = 5 .. 0:  rbar_i = W^-T ubar_i,
//     v = J(Y_i)^T rbar_i (i >= 1), ybar += v, ubar_j += a_ij v + (c_ij/h) rbar_i (j < i);
//   lam = ybar + sum_i grad_y <rbar_i, J(y) u_i> + J(y)^T rbar_0
// What bounds it is the number of instructions a wave issues, so the two kinds of products are laid
// out for that:
//   * J(Y_i)^T rbar_i is a reverse pass over the rates of the stage state (vjp): the adjoint weights of
//     the production rates meet the reactions through the slots, each reaction lane writes the
//     derivatives of its side, and the row lanes gather them from lists.
//   * The six second-order products share the point y, so they are contracted over the stages before
//     they reach the reactions: with om^i the production-rate weights of rbar_i, dc^i the direction u_i in
//     concentrations, a reaction needs only A = sum_i nu.dom^i, B = sum_i Q^i dT_i and
//     C_l = sum_i Q^i dc^i_l (Q^i = nu.om^i), and then the gradient of A q + B q_T + sum_l C_l q_l: one pass
//     in derivative arithmetic along (B, C), the direction being the lane's own.  The species level of the six
//     directions runs one direction per lane, its two products with the concentration Jacobian
//     (all six directions at once) on the FP64 matrix cores.
// Measured on MI355X (4,096 cells, 240 sub-steps on average, 707 at most): 93 ms with eight lanes per cell
// (whose reaction loops ran 24 reactions one after the other per lane), 14.7 ms here, 37k cycles per
// sub-step for its 6,000 instructions.  One wave per SIMD with 448 registers: at two waves (256 registers,
// 628 bytes of scratch per lane) it takes 16.3 ms.  Cells in index order instead of longest first:
// 22.9 ms (two waves).
#include <cmath>

#include "df_cell.h"

namespace df {
namespace {

struct SweepArgs {
    int64_t n, ld;
    const double *p;
    const double *tape;
    int32_t cap;
    const double *Tb, *Yb;
    double *T0b, *Y0b, *thc, *wth;
    const int *src;
    const double *sp;   // species rows
    const double *ad;   // slot lists
    const int *ai;
    int32_t *order;  // cells, most sub-steps first; null: by index
    int64_t first;   // the launch's first place in that order
};

// The cells by decreasing number of sub-steps (the sweep's chains; a late start of a long one would set
// the launch's time), a counting sort on the count in one block: its time (some microseconds per ten
// thousand cells) is small against the sweep's.  Cells without a tape come last.
constexpr int kSortThreads = 1024, kSortBuckets = 4096;

__global__ __launch_bounds__(kSortThreads) void sweep_order(const int32_t *__restrict__ cnt, int n,
                                                            int32_t *__restrict__ order) {
    constexpr int R = kSortBuckets / kSortThreads;
    __shared__ int32_t loc[kSortBuckets], sum[kSortThreads];
    const int t = threadIdx.x;
    for (int b = t; b < kSortBuckets; b += kSortThreads) loc[b] = 0;
    __syncthreads();
    auto bucket = [&](int i) {
        const int c = cnt[i];
        return kSortBuckets - 1 - (c < 0 ? 0 : (c < kSortBuckets ? c : kSortBuckets - 1));
    };
    for (int i = t; i < n; i += kSortThreads) atomicAdd(&loc[bucket(i)], 1);
    __syncthreads();
    int32_t run = 0, c[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        c[q] = loc[t * R + q];
        run += c[q];
    }
    sum[t] = run;
    __syncthreads();
    for (int off = 1; off < kSortThreads; off <<= 1) {
        const int32_t add = (t >= off) ? sum[t - off] : 0;
        __syncthreads();
        sum[t] += add;
        __syncthreads();
    }
    int32_t base = sum[t] - run;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        loc[t * R + q] = base;
        base += c[q];
    }
    __syncthreads();
    for (int i = t; i < n; i += kSortThreads) order[atomicAdd(&loc[bucket(i)], 1)] = i;
}

constexpr int kLS = 8;  // slot-list entries per lane

template <int K, int EL>
struct Sweep : CellWave<K, EL> {
    using C = CellWave<K, EL>;
    using typename C::Cell;
    using typename C::Rates;
    using typename C::Row;
    static constexpr int N = C::N, NI = C::NI;
    static constexpr int kDirS = 17;  // stride of the direction arrays (row 6 stays zero)

    // LDS after the integrator's, in doubles
    static constexpr int oOm = C::kEnd;            // production-rate weights of the rows (row 0 zero)
    static constexpr int oS = oOm + 16;            // slot derivatives, then d q/d [M], then T-derivatives
    static constexpr int oU = oS + 256;            // stage vectors u_i
    static constexpr int oR = oU + 7 * kDirS;      // rbar_i
    static constexpr int oWt = oR + 7 * kDirS;     // weights om^i
    static constexpr int oDc = oWt + 96;           // directions dc^i
    static constexpr int oSp = oDc + 96;           // per row: c, R cp/R, R T h/(R T), R dcp/R/dT, wd, W
    static constexpr int oX = oSp + 96;            // per direction: dlnfy, dT
    static constexpr int oG = oX + 32;             // a gradient on its way to the rows
    static constexpr int kSize = oG + 16;

    struct Lists {
        double a6, c[kLS];
        int i[kLS];
    };

    // thermodynamics of the row's species and the mixture
    struct Mix {
        double kcp, hw, icp, dcp, fy, yiw, dcr;
    };
    __device__ __forceinline__ static Mix mixture(const Row &o, double a6, const Rates &s, double yr) {
        Mix m;
        const double hRT = fma(a6, s.iT, fma(s.T, fma(s.T, fma(s.T, fma(s.T, 0.2 * o.a[4], 0.25 * o.a[3]),
                                                               (1.0 / 3) * o.a[2]), 0.5 * o.a[1]), o.a[0]));
        m.hw = kR * s.T * hRT;
        m.kcp = kR * s.cpR;
        m.dcr = kR * fma(s.T, fma(s.T, fma(4.0 * s.T, o.a[4], 3.0 * o.a[3]), 2.0 * o.a[2]), o.a[1]);
        m.yiw = yr * o.iW;
        m.icp = frcp3(row_sum(m.yiw * m.kcp));
        m.dcp = row_sum(m.yiw * m.dcr);
        m.fy = 1e6 * s.irho;
        return m;
    }
    // the row's sum over its list of slot derivatives
    __device__ __forceinline__ static double gather(const Lists &l, const double *sh) {
        double b0 = 0.0, b1 = 0.0;
#pragma unroll
        for (int e = 0; e < kLS; e += 2) {
            b0 = fma(l.c[e], sh[oS + l.i[e]], b0);
            b1 = fma(l.c[e + 1], sh[oS + l.i[e + 1]], b1);
        }
        return copies_sum(b0 + b1);
    }
    // the lane's side of sum_k nu_k w_k of its reaction, both sides added
    __device__ __forceinline__ static double through(const Row &o, const double *w) {
        return half_sum(-o.sg * (w[o.sl[0]] + w[o.sl[1]] + w[o.sl[2]]));
    }

    // row r of J(Y)^T lam at the state Y (row yr), and th += lam . df/dlnA of the lane's reaction
    __device__ __forceinline__ static double vjp(const CellMech &mg, const Coef &kc, const Row &o, const Lists &l,
                                                 const Cell &c, double *sh, int lane, int r, double yr, double lam,
                                                 double &th) {
        Rates s;
        C::template rates<2>(mg, kc, o, c, sh, lane, r, yr, s);
        const Mix m = mixture(o, l.a6, s, yr);
        const double lT = lane_value(lam, 0);
        const double om = m.fy * fma(-lT * m.icp, m.hw, lam * o.W);
        lds_order();
        sh[oOm + r] = om;
        lds_order();
        const double Qb = through(o, sh + oOm);
        const bool tb = o.flags & 1;
        const double Mq = tb ? s.Mc : 1.0;
        const double q = Mq * half_sum(s.X);
        th = fma(Qb * q, 1.0 - s.h, th);
        const double a = Qb * Mq * s.kk;
        const double G = Qb * half_sum(tb ? s.X : s.gM * s.P);
        const double Tv = Qb * Mq * half_sum(s.X * s.dl);
        lds_order();
        sh[oS + lane] = a * (s.c1 * s.c2);
        sh[oS + 64 + lane] = a * (s.c0 * s.c2);
        sh[oS + 128 + lane] = a * (s.c0 * s.c1);
        sh[oS + 192 + lane] = (lane < 32) ? G : Tv;
        sh[C::oQ + lane] = q;
        lds_order();
        double b0 = 0.0, b1 = 0.0;
#pragma unroll
        for (int e = 0; e < EL; e += 2) {
            b0 = fma(o.lc[e], sh[C::oQ + o.li[e]], b0);
            b1 = fma(o.lc[e + 1], sh[C::oQ + o.li[e + 1]], b1);
        }
        const double wd = copies_sum(b0 + b1);
        const double cb = gather(l, sh);
        const double Z = row_sum(fma(om, wd, -cb * (s.c6 * m.yiw)));
        const double fT = -m.fy * row_sum(m.hw * wd) * m.icp;
        const double FC = m.fy * row_sum(m.kcp * wd);
        const double t = lT * m.icp * fT;
        const double g0 = fma(s.iT, Z, cb) - lT * m.icp * FC - t * m.dcp;
        const double gk = o.iW * (fma(s.c6, cb, s.Wbar * Z) - t * m.kcp);
        return (r == 0) ? g0 : gk;
    }

    // Falloff reactions, in the quad lanes: h = d ln k/d ln [M] and the T-derivative L of ln (phi F), and
    // their derivatives along dT = B, d[M] = CM (the lane's reaction's)
    __device__ __forceinline__ static void troe_dual(const Coef &kc, const Row &o, const Rates &s, double ddlr, double B,
                                                     double CM, double &dh, double &dL) {
        const double wE = o.wq * s.E;
        const double dwE = wE * s.dlr * B;
        const double Fc = quad_sum(wE), iFc = frcp3(Fc);
        const double dFc = quad_sum(dwE);
        const double F1 = quad_sum(wE * s.dlr);  // dF_cent/dT
        const double dF1 = quad_sum(fma(dwE, s.dlr, wE * ddlr * B));
        const double dl0 = dpp<kQuad0>(s.dlr), ddl0 = dpp<kQuad0>(ddlr) * B;
        const double iM = frcp3(s.Mc);
        const double lFc = dlogp(kc, Fc) * kInvLn10, dlFc = dFc * iFc * kInvLn10;
        const double lPr = (dpp<kQuad0>(s.arg) + s.lx + s.lc) * kInvLn10;
        const double dlnPr = fma(dl0, B, CM * iM), dlPr = dlnPr * kInvLn10;
        const double nn = fma(-1.27, lFc, 0.75), dnn = -1.27 * dlFc;
        const double x = lPr + fma(-0.67, lFc, -0.4), dx = fma(-0.67, dlFc, dlPr);
        const double iden = frcp3(fma(-0.14, x, nn)), diden = -iden * iden * fma(-0.14, dx, dnn);
        const double f1 = x * iden, df1 = fma(dx, iden, x * diden);
        const double q1 = frcp3(fma(f1, f1, 1.0)), dq1 = -2.0 * q1 * q1 * f1 * df1;
        const double gq = 2.0 * f1 * q1 * q1, dgq = 2.0 * q1 * fma(q1, df1, 2.0 * f1 * dq1);
        const double i2 = iden * iden, di2 = 2.0 * iden * diden;
        const double t = lFc * gq * i2;
        const double dt = fma(fma(dlFc, gq, lFc * dgq), i2, lFc * gq * di2);
        const double w = fma(1.27, x, -0.67 * nn), dw = fma(1.27, dx, -0.67 * dnn);
        const double lF = fma(-t, w, q1), dlF = dq1 - fma(dt, w, t * dw);  // d lg F/d lg F_cent
        const double Pr = dpp<kQuad0>(s.E) * s.Mc;
        const double iPr1 = frcp3(1.0 + Pr), diPr1 = -iPr1 * iPr1 * Pr * dlnPr;
        const double h = fma(-t, nn, iPr1);
        dh = diPr1 - fma(dt, nn, t * dnn);
        const double sF = F1 * iFc, dsF = fma(-sF, dFc, dF1) * iFc;
        dL = fma(dh, dl0, h * ddl0) + fma(dlF, sF, lF * dsF);
    }

    // row r of sum_i grad_y <rbar_i, J(y) u_i> + J(y)^T rbar_0 at the sub-step's start state, and the
    // lane's reaction's part of its ln A derivative
    __device__ __forceinline__ static double second(const CellMech &mg, const Coef &kc, const Row &o, const Lists &l,
                                                    const Cell &c, double *sh, int lane, int r, int g, double yr,
                                                    double &th) {
        Rates s;
        C::template rates<2>(mg, kc, o, c, sh, lane, r, yr, s);
        const Mix m = mixture(o, l.a6, s, yr);
        const double d2 = kR * row_sum(m.yiw * fma(s.T, fma(12.0 * s.T, o.a[4], 6.0 * o.a[3]), 2.0 * o.a[2]));
        const bool tb = o.flags & 1;
        const double Mq = tb ? s.Mc : 1.0;
        const double XT = half_sum(s.X), S1 = half_sum(s.X * s.dl);
        const double q = Mq * XT;
        C::records(mg, o, s, sh, lane, half_sum(tb ? s.X : s.gM * s.P), Mq, q, Mq * S1);
        lds_order();
        // concentration-space Jacobian of the production rates (columns: T, species, the rates): D holds
        // (row r, column 4 i + g), E (row 4 i + g, column r)
        d4 D = {0.0, 0.0, 0.0, 0.0}, E = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < EL; ++e) {
            const double A = sh[C::oRec + (4 * e + g) * C::RS + r];
            D = __builtin_amdgcn_mfma_f64_16x16x4f64(A, o.nu[e], D, 0, 0, 0);
            E = __builtin_amdgcn_mfma_f64_16x16x4f64(o.nu[e], A, E, 0, 0, 0);
        }
        const double wd = copy_of<N % 4>(D[N / 4]);
        const double cr = s.c6 * m.yiw;
        sh[oSp + r] = cr;
        sh[oSp + 16 + r] = m.kcp;
        sh[oSp + 32 + r] = m.hw;
        sh[oSp + 48 + r] = m.dcr;
        sh[oSp + 64 + r] = wd;
        lds_order();
        const double H = m.fy * row_sum(m.hw * wd), FC = m.fy * row_sum(m.kcp * wd), FD = m.fy * row_sum(m.dcr * wd);
        const double fT = -H * m.icp;

        // one direction per lane: direction r (zero from 6 on), species rows 4 s + g
        const int di = r < 6 ? r : 6;
        double u[NI], kcp[NI], hw[NI], dcr[NI], cs[NI], wds[NI], om[NI], dom[NI], dc[NI];
        double rb[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int k = 4 * i + g;
            u[i] = sh[oU + di * kDirS + k];
            rb[i] = sh[oR + di * kDirS + k];
            cs[i] = sh[oSp + k];
            kcp[i] = sh[oSp + 16 + k];
            hw[i] = sh[oSp + 32 + k];
            dcr[i] = sh[oSp + 48 + k];
            wds[i] = sh[oSp + 64 + k];
        }
        const double dT = copy_of<0>(u[0]), lT = copy_of<0>(rb[0]);
        double e0 = 0.0, e1 = 0.0, e2 = 0.0;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const double x = u[i] * o.icol[i];
            e0 += x;
            e1 = fma(x, kcp[i], e1);
            e2 = fma(x, dcr[i], e2);
        }
        const double dS = copies_sum(e0);
        const double sig = fma(dT, s.iT, s.Wbar * dS);  // d ln fy = - d ln rho
        const double dcp = fma(m.dcp, dT, copies_sum(e1));
        const double ddcp = fma(d2, dT, copies_sum(e2));
        const double li = lT * m.icp;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            om[i] = m.fy * fma(-li, hw[i], rb[i] * sh[oSp + 80 + 4 * i + g]);
            dom[i] = fma(sig, om[i], -li * m.fy * fma(-hw[i] * m.icp, dcp, kcp[i] * dT));
            dc[i] = fma(s.c6 * o.icol[i], u[i], -cs[i] * sig);
        }
        // all directions at once: derivative of the production rates, and the concentration adjoints (row
        // 0: the T adjoint, row N: <rbar_i, f>)
        d4 V = {0.0, 0.0, 0.0, 0.0}, B4 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const double x = (i == 0 && g == 0) ? u[0] : dc[i];
            V = __builtin_amdgcn_mfma_f64_16x16x4f64(D[i], x, V, 0, 0, 0);
            B4 = __builtin_amdgcn_mfma_f64_16x16x4f64(E[i], om[i], B4, 0, 0, 0);
        }
        const double Tb = copy_of<0>(B4[0]), Lv = copy_of<N % 4>(B4[N / 4]);
        double f0 = 0.0, f1 = 0.0, f2 = 0.0, f3 = 0.0, f4 = 0.0;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            f0 = fma(B4[i], cs[i], f0);
            f1 = fma(B4[i], dc[i], f1);
            f2 = fma(dom[i], wds[i], fma(om[i], V[i], f2));
            f3 = fma(kcp[i], V[i], f3);
            f4 = fma(hw[i], V[i], f4);
        }
        const double CB = copies_sum(f0), dCB = copies_sum(f1), dL = copies_sum(f2);
        const double dFC = fma(sig, FC, fma(m.fy, copies_sum(f3), FD * dT));
        const double dH = fma(FC, dT, fma(sig, H, m.fy * copies_sum(f4)));
        const double dfT = -m.icp * fma(fT, dcp, dH);
        const double one = (r == 0) ? 1.0 : 0.0;  // the first-order product of stage 0
        const double LC = Lv - CB, dLC = dL - dCB;
        const double ic2 = m.icp * m.icp;
        const double lf = li * fT;
        double GT = s.iT * fma(-s.iT * dT, LC, dLC) - lT * fma(m.icp, dFC, -ic2 * dcp * FC) -
                    lT * (m.icp * fma(dfT, m.dcp, fT * ddcp) - fT * ic2 * dcp * m.dcp);
        GT = fma(one, fma(s.iT, LC, Tb) - li * FC - lf * m.dcp, GT);
        const double A1 = row_sum(fma(one * s.Wbar, LC, s.Wbar * fma(-s.Wbar * dS, LC, dLC)));
        const double A2 = row_sum(fma(one, lf, lT * fma(dfT, m.icp, -fT * ic2 * dcp)));
        const double A3 = row_sum(lf * dT);
        GT = row_sum(GT);
        const double sg1 = one - sig;
        lds_order();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int k = 4 * i + g;
            sh[oG + k] = row_sum(sg1 * B4[i]);
            sh[oOm + k] = row_sum(dom[i]);
            if (r < 6) {
                sh[oWt + r * 16 + k] = om[i];
                sh[oDc + r * 16 + k] = dc[i];
            }
        }
        sh[oX + r] = sig;
        sh[oX + 16 + r] = dT;
        lds_order();

        // the lane's reaction: weights A, B, C contracted over the directions
        const double A = through(o, sh + oOm);
        double B = 0.0, C0 = 0.0, C1 = 0.0, C2 = 0.0, Cs = 0.0, Q0 = 0.0, v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = 0.0;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const double Qi = through(o, sh + oWt + 16 * i);
            if (i == 0) Q0 = Qi;
            const double *d = sh + oDc + 16 * i;
            B = fma(Qi, sh[oX + 16 + i], B);
            Cs = fma(Qi, sh[oX + i], Cs);
            C0 = fma(Qi, d[o.sl[0]], C0);
            C1 = fma(Qi, d[o.sl[1]], C1);
            C2 = fma(Qi, d[o.sl[2]], C2);
#pragma unroll
            for (int k = 0; k < K; ++k) v[k] = fma(Qi, sh[oU + i * kDirS + 1 + k], v[k]);
        }
        double CM = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) CM = fma(o.w[k], v[k], CM);
        CM = fma(s.c6, CM, -s.Mc * Cs);  // sum_i Q^i d[M]^i
        // second T-derivative of the row's exponent
        const double ddlr = fma(fma(2.0 * o.e[2], s.iT, -o.e[1]), s.iT * s.iT,
                                fma(s.T, fma(12.0 * s.T, o.e[6], 6.0 * o.e[5]), 2.0 * o.e[4]));
        double dh = 0.0, Ddl = ddlr * B, gl = 0.0, Dgl = 0.0;
        if (mg.troe) {
            const bool fall = o.flags & 2, quad = o.flags & 4;
            // a quad takes B and [M]'s direction from its reaction's lane
            const double Bq = from_lane(o.src, B), Mq4 = from_lane(o.src, CM);
            double qh, qL;
            troe_dual(kc, o, s, ddlr, Bq, Mq4, qh, qL);
            // other lanes read their own, which is zero
            const double rh = from_lane(o.src, quad ? qh : 0.0), rL = from_lane(o.src, quad ? qL : 0.0);
            dh = fall ? rh : 0.0;
            Ddl += fall ? rL : 0.0;
            const double iM = fall ? frcp3(s.Mc) : 0.0;
            gl = s.h * iM;
            Dgl = fma(-gl, CM, dh) * iM;
        }
        const double P0 = s.c1 * s.c2, P1 = s.c0 * s.c2, P2 = s.c0 * s.c1;
        const double D0 = fma(C1, s.c2, s.c1 * C2), D1 = fma(C0, s.c2, s.c0 * C2), D2 = fma(C0, s.c1, s.c0 * C1);
        const double Dk = fma(s.dl, B, gl * CM);  // d ln k
        const double DX = fma(s.X, Dk, s.kk * fma(C0, P0, fma(C1, P1, C2 * P2)));
        const double DM = tb ? CM : 0.0;
        const double Phi = fma(A, q, fma(DM, XT, Mq * half_sum(DX)));
        th += fma(Q0 * q + Phi, 1.0 - s.h, -q * dh);
        const double AX = fma(A, s.X, DX);
        const double G = half_sum(tb ? AX : fma(AX, gl, s.X * Dgl));
        const double Tv = fma(fma(A, Mq, DM), S1, Mq * half_sum(fma(DX, s.dl, s.X * Ddl)));
        const double a = s.kk * fma(Mq, Dk, fma(A, Mq, DM)), b = s.kk * Mq;
        sh[oS + lane] = fma(a, P0, b * D0);
        sh[oS + 64 + lane] = fma(a, P1, b * D1);
        sh[oS + 128 + lane] = fma(a, P2, b * D2);
        sh[oS + 192 + lane] = (lane < 32) ? G : Tv;
        lds_order();
        const double cb = gather(l, sh);
        const double CH = row_sum(cb * cr);
        const double g0 = GT + fma(-s.iT, CH, cb);
        const double gk = o.iW * (fma(s.c6, sh[oG + r] + cb, A1 - s.Wbar * CH) - fma(A2, m.kcp, A3 * m.dcr));
        return (r == 0) ? g0 : gk;
    }
};

template <int K, int EL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 1))) void sweep_kernel(CellMech mg, SweepArgs a) {
    using C = CellWave<K, EL>;
    using S = Sweep<K, EL>;
    constexpr int N = C::N, NI = C::NI;
    extern __shared__ double sh[];
    const int lane = threadIdx.x, r = lane & 15, g = lane >> 4;
    const int64_t slot = a.first + blockIdx.x, i = a.order ? int64_t(a.order[slot]) : slot;
    for (int e = C::kEnd + lane; e < S::kSize; e += 64) sh[e] = 0.0;
    typename C::Row o;
    C::load_row(mg, lane, o);
    C::load_eff(mg, lane, sh);
    typename S::Lists l;
#pragma unroll
    for (int e = 0; e < kLS; ++e) {
        l.c[e] = a.ad[64 * e + lane];
        l.i[e] = a.ai[64 * e + lane];
    }
    l.a6 = (r >= 1 && r <= K) ? a.sp[(r - 1) * kSpTab + 7] : 0.0;
    Coef kc;
    kc.set();
    sh[S::oSp + 80 + r] = o.W;
    lds_order();
    if (lane == 0) sh[C::oC] = 1.0;
    lds_order();
    const Tape tp(K, a.n, a.cap);
    const int32_t cnt = __builtin_amdgcn_readfirstlane(tp.count(a.tape)[i]);
    const double *T = a.tape + i;
    typename C::Cell c;
    c.p = a.p[i];
    c.ip = frcp(c.p);
    c.c6p = c.p * (1e-6 / kR);
    c.lc6p = dlogp(kc, c.c6p);
    double lam = 0.0, th = 0.0;
    if (r == 0) lam = a.Tb[i];
    if (r >= 1 && r <= K) lam = a.Yb[int64_t(r - 1) * a.ld + i];
    // the sub-step's record: W^-T in the 2D layout, y, and stage vectors g and g + 4 of the row
    double wn[NI], yn = 0.0, un = 0.0, vn = 0.0, hn = 1.0;
    auto load = [&](int64_t s) {
#pragma unroll
        for (int j = 0; j < NI; ++j) wn[j] = (r < N && 4 * j + g < N) ? T[tp.w(s, (4 * j + g) * N + r)] : 0.0;
        if (r < N) {
            yn = T[tp.y(s, r)];
            un = T[tp.u(s, g * N + r)];
            if (g < 2) vn = T[tp.u(s, (g + 4) * N + r)];
        }
        hn = T[tp.h(s)];
    };
    if (cnt > 0) load(cnt - 1);
    for (int64_t s = int64_t(cnt) - 1; s >= 0; --s) {
        double w[NI], ub[6], u[5];
#pragma unroll
        for (int j = 0; j < NI; ++j) w[j] = wn[j];
        const double yr = yn, ih = frcp(hn);
        lds_order();
        sh[S::oU + g * S::kDirS + r] = un;
        if (g < 2) sh[S::oU + (g + 4) * S::kDirS + r] = vn;
        lds_order();
        if (s > 0) load(s - 1);  // in flight while this sub-step runs
#pragma unroll
        for (int j = 0; j < 5; ++j) u[j] = sh[S::oU + j * S::kDirS + r];
#pragma unroll
        for (int j = 0; j < 6; ++j) ub[j] = (j < 5 ? Rodas4::a[5][j] : 1.0) * lam;
        double yb = lam;
#pragma unroll
        for (int si = 5; si >= 0; --si) {
            // rbar = W^-T ubar_i
            lds_order();
            sh[S::oG + r] = ub[si];
            lds_order();
            double rb = 0.0;
#pragma unroll
            for (int j = 0; j < NI; ++j) rb = fma(w[j], sh[S::oG + 4 * j + g], rb);
            rb = copies_sum(rb);
            sh[S::oR + si * S::kDirS + r] = rb;
            if (si > 0) {
                double ys = yr;
#pragma unroll
                for (int j = 0; j < si; ++j) ys = fma(Rodas4::a[si][j], u[j], ys);
                const double v = S::vjp(mg, kc, o, l, c, sh, lane, r, ys, rb, th);
                yb += v;
#pragma unroll
                for (int j = 0; j < si; ++j)
                    ub[j] = fma(Rodas4::a[si][j], v, fma(Rodas4::c[si][j] * ih, rb, ub[j]));
            }
        }
        lam = yb + S::second(mg, kc, o, l, c, sh, lane, r, g, yr, th);
    }
    const bool ok = cnt > 0;
    if (lane == 0) a.T0b[i] = ok ? lam : 0.0;
    if (lane >= 1 && lane <= K) a.Y0b[int64_t(lane - 1) * a.ld + i] = ok ? lam : 0.0;
    if (lane < mg.M) {
        const double v = ok ? th : 0.0;
        a.wth[int64_t(lane) * a.n + i] = v;
        if (a.thc) a.thc[int64_t(a.src[lane]) * a.ld + i] = v;
    }
}

template <int K, int EL>
df_status launch_k(const MechDev &m, SweepArgs a, hipStream_t s) {
    const Tape tp(K, a.n, a.cap);
    if (a.order)
        hipLaunchKernelGGL(sweep_order, dim3(1), dim3(kSortThreads), 0, s, tp.count(a.tape), int(a.n), a.order);
    const CellMech cm{m.xd, m.xi, m.ceff, m.M, m.xtroe, m.xboth};
    const size_t lds = size_t(Sweep<K, EL>::kSize) * sizeof(double);
    for (; a.first < a.n; a.first += max_blocks(64)) {
        const int64_t blocks = a.n - a.first < max_blocks(64) ? a.n - a.first : max_blocks(64);
        hipLaunchKernelGGL((sweep_kernel<K, EL>), dim3(unsigned(blocks)), dim3(64), lds, s, cm, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(DF_E_HIP, std::string("df_chem_adjoint launch: ") + hipGetErrorString(e));
    }
    return DF_OK;
}

}  // namespace

// (the adjoint takes at most 24 reactions, which six list entries per lane cover)
bool sweep_cell_supported(const MechDev &m) { return m.xel == 6 && m.xad && chem_cell_supported(m); }

df_status launch_sweep_cell(const MechDev &m, int64_t n, int64_t ld, const double *p, const double *tape, int32_t cap,
                            const double *Tb, const double *Yb, double *T0b, double *Y0b, double *thc, double *wth,
                            int32_t *order, hipStream_t s) {
    const SweepArgs a{n, ld, p, tape, cap, Tb, Yb, T0b, Y0b, thc, wth, m.src, m.sp, m.xad, m.xai, order, 0};
#define DF_CASE(k)                                   \
    case k:                                          \
        return launch_k<k, 6>(m, a, s);
    switch (m.K) {
        DF_CHEM_SPECIES_LIST(DF_CASE)
        default:
            break;
    }
#undef DF_CASE
    return fail(DF_E_UNSUPPORTED, "df_chem_adjoint: no one-wave-per-cell sweep for this mechanism");
}

}  // namespace df
