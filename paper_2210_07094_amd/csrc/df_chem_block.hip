// Detailed-chemistry step with one block of eight wavefronts per cell, for hydrocarbon-size mechanisms:
// FP64 throughout.  The reactor, the RODAS4 method, its error norm and its controller are those of the
// other kernels.
//
// What bounds it: a stiff cell is one chain of a few thousand dependent sub-steps, and the longest chain of a
// launch its time.  On one wave (df_chem_wave.hip) a sub-step of the 53-species mechanism took 415,000
// cycles, nearly all of it waiting for one wave's table loads, LDS reads and serial steps: 153,000 in the
// Jacobian, 62,000 in the factorisation, the rest in five right-hand sides and six triangular solves.  Eight
// waves take 147,000 with a CU to themselves (Jacobian 36,000, inverse 50,000, right-hand sides 40,000,
// solves 6,000) and 180,000 to 230,000 beside a second cell:
//  * one reaction per thread, its coefficients in registers for the whole launch.  The falloff and
//    third-body reactions are dealt out eight to a wave, so that eight lanes can share each one's sum over
//    the species (the sum stays inside the wave: no barrier);
//  * production rates: eight lanes per species walk its list, kept in LDS with the thermo rows;
//  * Jacobian: the sparse entries' rounds and the species rows are dealt out to the waves;
//  * W = I/(g h) - J with row r in lane r and seven neighbouring columns per wave is inverted in place by
//    Gauss-Jordan with partial pivoting (rows stay in their lanes).  A wave takes the steps of its own seven
//    columns by itself, then the others follow from LDS: eight barriers, where a barrier per step (the next
//    pivot's wave going ahead) measured 62,000 cycles;
//  * each solve is then a product: seven columns per wave, the eight partial sums meet in LDS.
// Both sides: 500 cells of the hydrocarbon field: 350 ms on one wave each, 128 ms here; 32,768 cells,
// 100 ns, where every CU is full either way: 2,800 and 2,523 ms.
// The state, the norms and the step control are computed by every wave from the same numbers, so all waves
// take the same branches with the same bits.
#include <algorithm>
#include <cmath>

#include "df_cell.h"
#include "df_internal.h"
#include "df_kinetics.h"

namespace df {
namespace {

constexpr int kBW = 8, kBT = 64 * kBW;      // waves and threads of a block
constexpr int kTb = 8 * kBW;                // falloff and third-body reactions: eight per wave
constexpr int kPlain = 56 * kBW;            // plain reactions: the other lanes

// the tableau indexed by a stage that is not a compile-time constant
struct Tableau {
    double v[6][5];
};
constexpr Tableau tableau(const double (&t)[6][5]) {
    Tableau r{};
    for (int s = 0; s < 6; ++s)
        for (int j = 0; j < 5; ++j) r.v[s][j] = t[s][j];
    return r;
}
__constant__ const Tableau kTabA = tableau(Rodas4::a), kTabC = tableau(Rodas4::c);

__device__ __forceinline__ double wsum(double v) { return copies_sum(row_sum(v)); }
// sum over the eight lanes of a group
__device__ __forceinline__ double oct_sum(double v) {
    v = quad_sum(v);
    return v + dpp<kHalfMirror>(v);
}
// a table pointer that the compiler knows nothing about: its loads stay where they are written, instead of
// being hoisted out of the sub-step loop into registers that then spill
template <class T>
__device__ __forceinline__ const T *fresh(const T *p) {
    asm volatile("" : "+s"(p));
    return p;
}
// packed table entries: index | (coefficient + 8) << 20
__device__ __forceinline__ int ent_idx(int v) { return v & 0xfffff; }
__device__ __forceinline__ int ent_nu(int v) { return (v >> 20) - 8; }
constexpr int kPad = 8 << 20;

template <int K>
struct Block {
    static constexpr int N = K + 1, LDJ = N + 1;  // row stride of the staged Jacobian (doubles)
    static constexpr int NI = (N + kBW - 1) / kBW;  // matrix columns per wave
    static constexpr int NE = (K + 7) / 8;          // species per lane of a third-body sum
    static_assert(N <= 64 && 8 * K <= kBT, "a row per lane and eight lanes per species");

    // LDS (doubles): J [N LDJ]; q, S, dq/dT, G [M] each; D [(wsr + wsp) M]; concentrations [64]; per
    // species production rate, sum_m c_m dq/dc_m and dq/dT [64] each; partial sums [8][64]; pivot
    // columns [2][NI][64], pivot reciprocals [64]; the species' thermo rows [kTh][64]; then ints: the species lists
    // [wnl], the rows' dense terms [wnd] and their offsets [64], pivot rows [64], a panel's pivots [2][8]
    static constexpr int kTh = 14;
    struct Lds {
        double *J, *q, *S, *dT, *G, *D, *c, *wd, *sq, *dt, *part, *mv, *piv, *th;
        int *list, *dense, *drow, *perm, *pv;
    };
    static size_t lds_bytes(const MechDev &m) {
        return 8 * (size_t(N) * LDJ + size_t(4 + m.wsr + m.wsp) * m.M + 64 * 4 + 64 * kBW + 128 * NI + 64 + 64 * kTh) +
               4 * (size_t(m.wnl) + size_t(m.wnd) + 128 + 16);
    }
    __device__ static Lds layout(double *b, const MechDev &m) {
        Lds L;
        const int M = m.M;
        L.J = b;
        L.q = L.J + N * LDJ;
        L.S = L.q + M;
        L.dT = L.S + M;
        L.G = L.dT + M;
        L.D = L.G + M;
        L.c = L.D + (m.wsr + m.wsp) * M;
        L.wd = L.c + 64;
        L.sq = L.wd + 64;
        L.dt = L.sq + 64;
        L.part = L.dt + 64;
        L.mv = L.part + 64 * kBW;
        L.piv = L.mv + 128 * NI;
        L.th = L.piv + 64;
        L.list = reinterpret_cast<int *>(L.th + 64 * kTh);
        L.dense = L.list + m.wnl;
        L.drow = L.dense + m.wnd;
        L.perm = L.drow + 64;
        L.pv = L.perm + 64;
        return L;
    }

    // what a thread keeps of the mechanism
    struct Own {
        double a[10];      // ln k_f and ln k_r rows of its reaction
        double ef[NE];     // its share of the efficiencies of third-body reaction 8 w + lane / 8
        int jd, type;      // its reaction (-1: none) and type
        int sl0, sl1;      // its six slots, six bits each
        int l0, l1;        // its species' list
        bool tb;           // third-body reaction 8 w + lane / 8 exists
        Coef kc;
    };
    __device__ static void own(const MechDev &m, Own &o, int w, int lane) {
        const int M = m.M, nt = m.wtb;
        const int jt = 8 * w + lane, jp = nt + 56 * w + lane - 8;
        o.jd = lane < 8 ? (jt < nt ? jt : -1) : (jp < M ? jp : -1);
        const int j = o.jd < 0 ? 0 : o.jd;
#pragma unroll
        for (int f = 0; f < 10; ++f) o.a[f] = m.wcr[f * M + j];
        o.type = o.jd < 0 ? 0 : m.wci[j];
        int s[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) s[f] = m.wci[(1 + f) * M + j];
        o.sl0 = s[0] | s[1] << 6 | s[2] << 12;
        o.sl1 = s[3] | s[4] << 6 | s[5] << 12;
        const int jg = 8 * w + lane / 8;
        o.tb = jg < nt;
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int k = lane % 8 + 8 * i;
            o.ef[i] = (o.tb && k < K) ? m.weff[k * M + jg] : 0.0;
        }
        const int k = threadIdx.x / 8;
        o.l0 = k < K ? m.wlo[k] : 0;
        o.l1 = k < K ? m.wlo[k + 1] : 0;
        o.kc.set();
    }

    // thermo of the lane's species (lane 1 + k holds species k) and the mixture
    struct Mix {
        double T, iT, lT, T2, T3, T4;
        double rho, Wbar, cp;
        double W, iW, cpR, hRT, Yk;
    };
    __device__ static void state(const MechDev &m, const Lds &L, const Coef &kc, double p, double y, int lane, Mix &s) {
        const bool spl = lane >= 1 && lane <= K;
        s.T = lane_value(y, 0);
        s.iT = 1.0 / s.T;
        s.lT = dlogp(kc, s.T);
        s.T2 = s.T * s.T;
        s.T3 = s.T2 * s.T;
        s.T4 = s.T2 * s.T2;
        // the thermo rows' fields: 0 W, 1 1/W, 2..6 a1..a5, 7 a6, 8..11 those of H, 12.. see jacobian
        const double *r = L.th + lane;
        const double T = s.T;
        s.W = r[0];
        s.iW = r[64];
        s.cpR = r[64 * 2] + T * (r[64 * 3] + T * (r[64 * 4] + T * (r[64 * 5] + T * r[64 * 6])));
        s.hRT = r[64 * 2] + T * (r[64 * 8] + T * (r[64 * 9] + T * (r[64 * 10] + T * r[64 * 11]))) + r[64 * 7] * s.iT;
        s.Yk = spl ? y : 0.0;
        const double sYW = wsum(s.Yk * s.iW);
        const double cpm = wsum(s.Yk * s.cpR * s.iW);
        s.Wbar = 1.0 / sYW;
        s.rho = p * s.Wbar * s.iT * (1.0 / kR);
        s.cp = cpm * kR;
        // every wave writes the same concentrations (slot 0 = 1), so it may read them without a barrier; the last
        // readers of the old ones are a barrier behind
        L.c[lane] = (lane == 0) ? 1.0 : 1e-6 * s.rho * s.Yk * s.iW;
        lds_order();
    }

    // this thread's reaction at the concentrations in LDS; with DER the derivatives, all to LDS
    template <bool DER>
    __device__ static void rates(const MechDev &m, const Lds &L, const Own &o, const Mix &s, int lane) {
        const int M = m.M;
        // the falloff coefficients, on their way while the sums below run
        const int type = o.type;
        const double *cr = fresh(m.wcr) + (o.jd < 0 ? 0 : o.jd);
        double fo[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        if (type == 2) {
#pragma unroll
            for (int f = 0; f < 7; ++f) fo[f] = cr[(16 + f) * M];
        }
        // third-body concentrations sum_k eff_k c_k, eight lanes each; lane l < 8 takes group l's
        double Mc = 0.0;
        if (__ballot(o.tb) != 0ull) {
            double p0 = 0.0, p1 = 0.0;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int k = lane % 8 + 8 * i;
                const double ck = L.c[k < K ? 1 + k : 0];
                if (i % 2)
                    p1 = fma(o.ef[i], ck, p1);
                else
                    p0 = fma(o.ef[i], ck, p0);
            }
            Mc = from_lane(4 * (8 * (lane & 7)), oct_sum(p0 + p1));
        }
        if (o.jd < 0) return;
        double lf = fma(o.a[1], s.lT, fma(o.a[2], s.iT, o.a[0]));
        double lr = fma(o.a[4], s.lT, fma(o.a[5], s.iT, o.a[3]));
        lr = fma(o.a[6], s.T, lr);
        lr = fma(o.a[7], s.T2, lr);
        lr = fma(o.a[8], s.T3, lr);
        lr = fma(o.a[9], s.T4, lr);
        double phi = 1.0, dphiM = 0.0, dlphi = 0.0;
        if (type == 2) {
            // Lindemann form times the Troe broadening factor F (ln F folded into both
            // exponentials), phi = Pr/(1 + Pr)
            const double c16 = fo[0], c17 = fo[1], c18 = fo[2], al = fo[3], c20 = fo[4], c21 = fo[5], c22 = fo[6];
            const double e3 = dexp(o.kc, c20 * s.T), e1 = dexp(o.kc, c21 * s.T), e2 = dexp(o.kc, c22 * s.iT);
            const double ek0 = dexp(o.kc, fma(c17, s.lT, fma(c18, s.iT, c16)));  // k0 / k_inf
            const double Fc = fma(1.0 - al, e3, fma(al, e1, e2));
            const double Pr = ek0 * Mc;
            const double lFc = dlogp(o.kc, Fc) * kInvLn10;
            const double lPr = dlogp(o.kc, Pr) * kInvLn10;
            const double cc = -0.4 - 0.67 * lFc;
            const double nn = 0.75 - 1.27 * lFc;
            const double x = lPr + cc;
            const double iden = frcp(nn - 0.14 * x);
            const double f1 = x * iden;
            const double q1 = frcp(1.0 + f1 * f1);
            const double lF = lFc * q1;
            const double iPr1 = frcp(1.0 + Pr);
            lf = fma(kLn10, lF, lf);
            lr = fma(kLn10, lF, lr);
            phi = Pr * iPr1;
            if (DER) {
                const double gq = 2.0 * f1 * q1 * q1;
                const double dlF_dlPr = -lFc * gq * nn * iden * iden;
                const double dlF_dlFc = q1 - lFc * gq * (1.27 * x - 0.67 * nn) * iden * iden;
                const double dFc = (1.0 - al) * c20 * e3 + al * c21 * e1 - c22 * s.iT * s.iT * e2;
                const double dlnPr = (c17 - c18 * s.iT) * s.iT;
                dlphi = (iPr1 + dlF_dlPr) * dlnPr + dlF_dlFc * fdiv(dFc, Fc);
                dphiM = ek0 * iPr1 * (iPr1 + dlF_dlPr);
            }
        }
        const double Ef = dexp(o.kc, lf), Er = dexp(o.kc, lr);
        const double kf = Ef * phi, kr = Er * phi;
        const double c0 = L.c[o.sl0 & 63], c1 = L.c[o.sl0 >> 6 & 63], c2 = L.c[o.sl0 >> 12];
        const double d0 = L.c[o.sl1 & 63], d1 = L.c[o.sl1 >> 6 & 63], d2 = L.c[o.sl1 >> 12];
        const double Pf = c0 * c1 * c2, Pb = d0 * d1 * d2;
        const double fwd = kf * Pf, rev = kr * Pb, X = fwd - rev;
        const double Mq = (type == 1) ? Mc : 1.0;
        L.q[o.jd] = Mq * X;
        if (DER) {
            const double dlf = (o.a[1] - o.a[2] * s.iT) * s.iT + dlphi;
            const double dlr = (o.a[4] - o.a[5] * s.iT) * s.iT +
                               fma(s.T, fma(s.T, fma(4.0 * o.a[9], s.T, 3.0 * o.a[8]), 2.0 * o.a[7]), o.a[6]) + dlphi;
            const double G = (type == 1) ? X : ((type == 2) ? (Ef * dphiM) * Pf - (Er * dphiM) * Pb : 0.0);
            L.dT[o.jd] = Mq * (fwd * dlf - rev * dlr);
            L.G[o.jd] = G;
            L.S[o.jd] = Mq * (cr[23 * M] * fwd - cr[24 * M] * rev) + (type != 0 ? Mc * G : 0.0);
            const double kfM = Mq * kf, krM = Mq * kr;
            const double D[6] = {kfM * c1 * c2,  kfM * c0 * c2,  kfM * c0 * c1,
                                 -krM * d1 * d2, -krM * d0 * d2, -krM * d0 * d1};
            // the slot derivatives of the slots in use
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < m.wsr) L.D[i * M + o.jd] = D[i];
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < m.wsp) L.D[(m.wsr + i) * M + o.jd] = D[3 + i];
        }
    }

    // component `lane` of f(y), in every wave
    __device__ static double rhs(const MechDev &m, const Lds &L, const Own &o, double p, double y, int lane) {
        Mix s;
        state(m, L, o.kc, p, y, lane, s);
        rates<false>(m, L, o, s, lane);
        __syncthreads();
        double wd = 0.0;
        for (int e = o.l0 + lane % 8; e < o.l1; e += 8) wd = fma(double(ent_nu(L.list[e])), L.q[ent_idx(L.list[e])], wd);
        wd = oct_sum(wd);
        if (lane % 8 == 0 && int(threadIdx.x) / 8 < K) L.wd[threadIdx.x / 8] = wd;
        __syncthreads();
        const bool spl = lane >= 1 && lane <= K;
        wd = spl ? L.wd[lane - 1] : 0.0;
        const double hs = wsum(s.hRT * wd);
        if (lane == 0) return -hs * (1e6 * kR) * s.T / (s.rho * s.cp);
        return (1e6 / s.rho) * s.W * wd;
    }

    // the columns of W = ig I - J of wave w (column NI w + i in a[i], row r in lane r), and f(y).  ig is known
    // only after f(y), so the diagonal is added by the caller
    __device__ static double jacobian(const MechDev &m, const Lds &L, const Own &o, double p, double y, int w, int lane,
                                      double (&a)[NI]) {
        const int M = m.M, t = threadIdx.x;
        Mix s;
        state(m, L, o.kc, p, y, lane, s);
        for (int e = t; e < N * LDJ; e += kBT) L.J[e] = 0.0;
        rates<true>(m, L, o, s, lane);
        __syncthreads();
        // per species: production rate, sum_m c_m dq/dc_m and dq/dT at fixed c
        {
            double wd = 0.0, sq = 0.0, dt = 0.0;
            for (int e = o.l0 + lane % 8; e < o.l1; e += 8) {
                const int v = L.list[e], j = ent_idx(v);
                const double nu = double(ent_nu(v));
                wd = fma(nu, L.q[j], wd);
                sq = fma(nu, L.S[j], sq);
                dt = fma(nu, L.dT[j], dt);
            }
            wd = oct_sum(wd);
            sq = oct_sum(sq);
            dt = oct_sum(dt);
            if (lane % 8 == 0 && t / 8 < K) {
                L.wd[t / 8] = wd;
                L.sq[t / 8] = sq;
                L.dt[t / 8] = dt;
            }
        }
        // concentration-space derivatives A_kl = sum_j nu_kj dq_j/dc_l: whole entries per lane, rounds of
        // 64 entries per wave
        const int *well = fresh(m.well), *wrb = fresh(m.wrb), *wrc = fresh(m.wrc), *wtk = fresh(m.wtk);
        for (int r = w; r < m.wnr; r += kBW) {
            const int e1 = r * 64 + lane;
            const int *ep = well + wrb[r] + lane;
            const int cm = wrc[r];
            double acc = 0.0;
            int e0 = 0;
            for (; e0 + 8 <= cm; e0 += 8) {
                int v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = ep[(e0 + i) * 64];
#pragma unroll
                for (int i = 0; i < 8; ++i) acc = fma(double(ent_nu(v[i])), L.D[ent_idx(v[i])], acc);
            }
            for (; e0 < cm; e0 += 2) {  // most lists hold one to three entries
                const int v0 = ep[e0 * 64], v1 = (e0 + 1 < cm) ? ep[(e0 + 1) * 64] : kPad;
                acc = fma(double(ent_nu(v0)), L.D[ent_idx(v0)], acc);
                acc = fma(double(ent_nu(v1)), L.D[ent_idx(v1)], acc);
            }
            if (e1 < m.wnt) L.J[wtk[e1]] = acc;
        }
        __syncthreads();
        const bool spl = lane >= 1 && lane <= K;
        const double wd = spl ? L.wd[lane - 1] : 0.0, sq = spl ? L.sq[lane - 1] : 0.0, dt = spl ? L.dt[lane - 1] : 0.0;
        const double T = s.T;
        const double coef = (1e6 / s.rho) * s.W;
        const double gk = coef * s.Wbar * (wd - sq);
        const double fk = spl ? coef * wd : 0.0;
        const double hm = spl ? s.hRT * kR * T * s.iW : 0.0;   // J/kg
        const double cpm = spl ? s.cpR * kR * s.iW : 0.0;      // J/kg/K
        const double *r = L.th + lane;
        const double dcpR = r[64 * 3] + T * (2.0 * r[64 * 4] + T * (r[64 * 12] + T * r[64 * 13]));
        const double dcpdT = wsum(spl ? s.Yk * dcpR * kR * s.iW : 0.0);
        const double icp = 1.0 / s.cp;
        const double fT = -wsum(hm * fk) * icp;
        const double cf = wsum(cpm * fk);
        // Species rows, row 1 + k by wave k % 8: the dense third-body terms (dq/dc_l gains eff_l G), then the
        // map to (T, Y) with dc_m/dY_l = 1e-6 rho delta_ml / W_m - c_m Wbar / W_l and
        // dc_m/dT = -c_m / T; lane l holds column 1 + l.  The wave's share of sum_k h_k J_kl beside it
        const double iWl = (lane < K) ? L.th[64 + 1 + lane] : 0.0;
        const double *effl = fresh(m.ceff) + ((lane < K) ? lane : 0);
        double hJ = 0.0;
        for (int k = w; k < K; k += kBW) {
            const int b0 = __builtin_amdgcn_readfirstlane(L.drow[k]), b1 = __builtin_amdgcn_readfirstlane(L.drow[k + 1]);
            const double Wk = lane_value(s.W, 1 + k);
            double *Jr = L.J + (1 + k) * LDJ + 1 + (lane < K ? lane : 0);
            double v = *Jr;
            for (int e0 = b0; e0 < b1; e0 += 4) {
                int x[4];
                double ef[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) x[i] = (e0 + i < b1) ? L.dense[e0 + i] : kPad;
#pragma unroll
                for (int i = 0; i < 4; ++i) ef[i] = effl[size_t(ent_idx(x[i])) * (K + 4)];
#pragma unroll
                for (int i = 0; i < 4; ++i) v = fma(double(ent_nu(x[i])) * L.G[ent_idx(x[i])], ef[i], v);
            }
            v = (Wk * v + lane_value(gk, 1 + k)) * iWl;
            if (lane < K) *Jr = v;
            hJ = fma(lane_value(hm, 1 + k), v, hJ);
        }
        L.part[w * 64 + (lane < K ? 1 + lane : (lane == K ? 0 : lane))] = (lane < K) ? hJ : 0.0;
        const double J0 = coef * (dt + (wd - sq) * s.iT);  // the temperature column
        const double hJ0 = wsum(spl ? hm * J0 : 0.0);
        __syncthreads();
        // temperature row (lane c: column c), f_T = -sum_k h_k f_k / cp
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < kBW; ++i) acc += L.part[i * 64 + lane];
        const double tr = (lane == 0) ? -(hJ0 + cf + fT * dcpdT) * icp : -(acc + fT * cpm) * icp;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int c = NI * w + i;
            double v = 0.0;
            if (c < N && lane < N) v = (c == 0) ? J0 : L.J[lane * LDJ + c];
            const double v0 = lane_value(tr, c);
            a[i] = (c < N && lane < N) ? -(lane == 0 ? v0 : v) : 0.0;
        }
        return (lane == 0) ? fT : fk;
    }

    // one step's update of column a: the other rows lose their multiple of row p (mcol: minus their entry of the
    // pivot column over the pivot, 0 in row p).  Row p itself would be divided by its pivot; that is left to the
    // end, where every row r is multiplied by the reciprocal in piv[r]
    __device__ __forceinline__ static double gj(double a, double mcol, int p) { return fma(mcol, lane_value(a, p), a); }

    // W^-1 in place: on return a[i] in lane r is the coefficient, in the unknown that row r was the pivot of
    // (pos), of the right-hand side's component pr[i].  Wave P takes the NI steps of its own columns by itself and
    // publishes each step's column and pivot row; after a barrier the other waves follow, wave P + 1 first of
    // all in time, since its panel is next
    __device__ static void invert(const Lds &L, int w, int lane, double (&a)[NI], int &pos, int (&pr)[NI]) {
        bool used = lane >= N;
        pos = -1;
#pragma unroll 1
        for (int P = 0; P * NI < N; ++P) {
            double *mv = L.mv + (P & 1) * (64 * NI);
            int *pv = L.pv + (P & 1) * 8;
            if (w == P) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int k = NI * P + i;
                    if (k >= N) break;
                    // the largest magnitude of the rows left (as the upper words order them, to 2^-20), ties to the
                    // lowest lane
                    const int key = used ? -1 : (hi32(a[i]) & 0x7fffffff);
                    int mx = row_max(key);
                    mx = max(max(__builtin_amdgcn_readlane(mx, 0), __builtin_amdgcn_readlane(mx, 16)),
                             max(__builtin_amdgcn_readlane(mx, 32), __builtin_amdgcn_readlane(mx, 48)));
                    const int p = __ffsll(static_cast<long long>(__ballot(!used && key == mx))) - 1;
                    const double inv = frcp3(lane_value(a[i], p));
                    const bool me = lane == p;
                    const double mc = me ? 0.0 : -a[i] * inv;
#pragma unroll
                    for (int c = 0; c < NI; ++c)
                        if (c != i) a[c] = gj(a[c], mc, p);
                    a[i] = me ? 1.0 : mc;
                    used = used || me;
                    pos = me ? k : pos;
                    mv[64 * i + lane] = mc;
                    if (lane == 0) {
                        pv[i] = p;
                        L.perm[k] = p;
                        L.piv[p] = inv;
                    }
                }
            }
            __syncthreads();
            if (w != P) {
                double mc[NI];
                int p[NI];
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    mc[i] = mv[64 * i + lane];
                    p[i] = pv[i];
                }
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int k = NI * P + i;
                    if (k >= N) break;
                    const int pi = __builtin_amdgcn_readfirstlane(p[i]);
                    const bool me = lane == pi;
                    used = used || me;
                    pos = me ? k : pos;
#pragma unroll
                    for (int c = 0; c < NI; ++c) a[c] = gj(a[c], mc[i], pi);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int c = NI * w + i;
            pr[i] = __builtin_amdgcn_readfirstlane(c < N ? L.perm[c] : 0);
        }
        const double sc = lane < N ? L.piv[lane] : 0.0;
#pragma unroll
        for (int i = 0; i < NI; ++i) a[i] *= sc;
    }

    // x = W^-1 b, b and x by component in lane order, in every wave
    __device__ static double solve(const Lds &L, const double (&a)[NI], int pos, const int (&pr)[NI], int w, int lane,
                                   double b) {
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const double v = lane_value(b, pr[i]);  // columns beyond N are zero
            if (i % 2)
                s1 = fma(a[i], v, s1);
            else
                s0 = fma(a[i], v, s0);
        }
        if (pos >= 0) L.part[w * 64 + pos] = s0 + s1;
        __syncthreads();
        double x = 0.0;
#pragma unroll
        for (int i = 0; i < kBW; ++i) x += lane < N ? L.part[i * 64 + lane] : 0.0;
        return x;
    }
};

template <int K>
__global__ __launch_bounds__(kBT, 4) void chem_block_kernel(MechDev m, StepArgs ar,
                                                            const int32_t *__restrict__ cidx,
                                                            const int32_t *__restrict__ dcount) {
    using B = Block<K>;
    constexpr int N = K + 1, NI = B::NI;
    extern __shared__ double lds[];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int64_t limit = dcount ? int64_t(*dcount) : ar.n;
    if (int64_t(blockIdx.x) >= limit) return;
    const typename B::Lds L = B::layout(lds, m);
    const Opts &op = ar.o;
    typename B::Own own;
    B::own(m, own, w, lane);
    for (int e = threadIdx.x; e < m.wnl; e += kBT) L.list[e] = m.wlp[e];
    for (int e = threadIdx.x; e < m.wnd; e += kBT) L.dense[e] = m.wdp[e];
    if (threadIdx.x <= K) L.drow[threadIdx.x] = m.wdo[threadIdx.x];
    for (int f = w; f < B::kTh; f += kBW) {
        constexpr int kField[14] = {0, 1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 17, 18};
        int g = 0;
#pragma unroll
        for (int q = 0; q < B::kTh; ++q) g = (f == q) ? kField[q] : g;
        L.th[64 * f + lane] = m.sp[(lane >= 1 && lane <= K ? lane - 1 : 0) * kSpTab + g];
    }
    const double sc_abs = (lane == 0) ? op.atol_T : op.atol_Y;
    const bool act = lane < N, spl = lane >= 1 && lane <= K;

    for (int64_t slot = blockIdx.x; slot < limit; slot += gridDim.x) {
        const int64_t i = cidx ? int64_t(cidx[slot]) : slot;
        __syncthreads();  // the list is in LDS; every wave has left the cell before
        const double p = ar.p[i];
        const double dtc = ar.dts ? ar.dts[i] : ar.dt;
        const double y0 = (lane == 0) ? ar.T[i] : (spl ? ar.Y[(lane - 1) * ar.ld + i] : 0.0);
        const bool okl = isfinite(y0) && (lane != 0 || y0 > 0.0);
        const bool ok = __ballot(!okl) == 0ull && isfinite(p) && p > 0.0 && isfinite(dtc) && dtc > 0.0;
        if (!ok) {
            if (w == 0) {
                if (lane == 0) {
                    if (ar.status) ar.status[i] = DF_CELL_NONFINITE;
                    if (ar.nsteps) {
                        ar.nsteps[i] = 0;
                        ar.nsteps[ar.n + i] = 0;
                    }
                }
                if (ar.rr && spl) ar.rr[(lane - 1) * ar.ld + i] = 0.0;
            }
            continue;
        }
        const double h_in = ar.h_io ? ar.h_io[i] : 0.0;
        bool fresh = !(h_in > 0.0);
        double h = fresh ? 0.0 : fmin(h_in, dtc);
        if (!fresh && !(h >= op.h_min)) h = op.h_min;
        double t = 0.0, h_final = 0.0;
        int acc = 0, rej = 0, st = DF_CELL_OK;
        bool prev_rej = false;
        double y = y0;
        __syncthreads();  // every wave has read the cell's input

        while (true) {
            if (acc + rej >= op.max_steps) {
                st = DF_CELL_MAX_STEPS;
                break;
            }
            double a[NI];
            const double f0 = B::jacobian(m, L, own, p, y, w, lane, a);
            if (fresh) {
                // initial sub-step from the weighted norms of y0 and f(y0)
                const double sc = sc_abs + op.rtol * fabs(y);
                const double ny = sqrt(wsum(act ? (y / sc) * (y / sc) : 0.0) / N);
                const double nf = sqrt(wsum(act ? (f0 / sc) * (f0 / sc) : 0.0) / N);
                h = (nf > 0.0) ? fmin(0.01 * ny / nf, dtc) : dtc;
                if (!(h >= op.h_min)) h = op.h_min;
                fresh = false;
            }
            const bool last = (t + h >= dtc);
            const double ht = last ? dtc - t : h;
            const double ig = 1.0 / (Rodas4::g * ht);
#pragma unroll
            for (int q = 0; q < NI; ++q) a[q] = (lane == NI * w + q && act) ? ig + a[q] : a[q];
            int pos, pr[NI];
            B::invert(L, w, lane, a, pos, pr);
            const double ih = 1.0 / ht;
            // one copy of the stage's code (five would not fit the instruction cache): the tableau's zeros stand
            // in for the stages to come
            double u[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, ys = y, u5 = 0.0;
#pragma unroll 1
            for (int s = 0; s < 6; ++s) {
                double v = f0;
                if (s > 0) {
                    double x = y;
#pragma unroll
                    for (int j = 0; j < 5; ++j) x = fma(kTabA.v[s][j], u[j], x);
                    ys = x;
                    v = B::rhs(m, L, own, p, ys, lane);
                    double c = 0.0;
#pragma unroll
                    for (int j = 0; j < 5; ++j) c = fma(kTabC.v[s][j], u[j], c);
                    v = fma(c, ih, v);
                }
                u5 = B::solve(L, a, pos, pr, w, lane, act ? v : 0.0);
#pragma unroll
                for (int j = 0; j < 5; ++j) u[j] = (s == j) ? u5 : u[j];
            }
            // y_new = (stage-6 state) + u5 ; error = u5
            const double yn = ys + u5;
            const double sc = sc_abs + op.rtol * fmax(fabs(y), fabs(yn));
            const double rr = u5 / sc;
            const double err = sqrt(wsum(act ? rr * rr : 0.0) / N);
            const double fmx = prev_rej ? 1.0 : 6.0;
            double fac;
            if (!isfinite(err))
                fac = 0.2;
            else if (err == 0.0)
                fac = fmx;
            else
                fac = fmin(fmx, fmax(0.2, 0.9 * pow(err, -0.25)));
            if (isfinite(err) && err <= 1.0) {
                ++acc;
                y = yn;
                h_final = h;
                prev_rej = false;
                if (last) break;
                t += ht;
                h = ht * fac;
            } else {
                ++rej;
                prev_rej = true;
                h = ht * fac;
                if (h < op.h_min) {
                    st = DF_CELL_H_UNDERFLOW;
                    break;
                }
            }
        }
        if (w != 0) continue;
        // results; rr = rho0 (Y - Y0) / dt with rho0 the density of the input state
        if (ar.rr) {
            const double T0 = lane_value(y0, 0);
            const double sYW = wsum(spl ? y0 * m.sp[(lane - 1) * kSpTab + 1] : 0.0);
            const double rdt = (p / (sYW * kR * T0)) / dtc;
            if (spl) ar.rr[(lane - 1) * ar.ld + i] = rdt * (y - y0);
        }
        if (lane == 0) ar.T[i] = y;
        if (spl) ar.Y[(lane - 1) * ar.ld + i] = y;
        if (lane == 0) {
            if (ar.h_io) ar.h_io[i] = (st == DF_CELL_OK) ? h_final : h;
            if (ar.status) ar.status[i] = (st == DF_CELL_OK) ? ar.status_ok : st;
            if (ar.nsteps) {
                ar.nsteps[i] = acc;
                ar.nsteps[ar.n + i] = rej;
            }
        }
    }
}

}  // namespace

// 53 species, reactions that fit the threads (one each), and two blocks' LDS per CU
bool chem_block_supported(const MechDev &m) {
    return m.K == 53 && m.wtb <= kTb && m.M - m.wtb <= kPlain && Block<53>::lds_bytes(m) <= 80 * 1024;
}

df_status launch_chem_block(const MechDev &m, const StepArgs &a, const int32_t *cidx, const int32_t *dcount,
                            hipStream_t stream) {
    if (a.n == 0) return DF_OK;
    if (a.tape) return fail(DF_E_UNSUPPORTED, "df_chem_step: the one-block-per-cell kernel records no tape");
    const size_t lds = Block<53>::lds_bytes(m);
    auto kernel = chem_block_kernel<53>;
    if (lds > 65536 &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            int(lds)) != hipSuccess)
        return fail(DF_E_HIP, "df_chem_step: cannot raise the LDS limit of the one-block-per-cell kernel");
    // a device-side count (the fallback cells of a DNN step, usually few): an empty list then costs at most
    // 2,048 blocks instead of one per cell
    const int64_t blocks = std::min(a.n, dcount ? 2048 : max_blocks(kBT));
    hipLaunchKernelGGL(kernel, dim3(unsigned(blocks)), dim3(kBT), lds, stream, m, a, cidx, dcount);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("chem_step block launch: ") + hipGetErrorString(e));
    return DF_OK;
}

}  // namespace df
