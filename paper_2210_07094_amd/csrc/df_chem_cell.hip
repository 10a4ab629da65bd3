// Detailed-chemistry step on gfx950 with one wavefront per cell, for mechanisms whose rates fit one
// wave: at most 13 species, 32 reactions, and a group of four spare lanes per falloff reaction
// (pack_cell_tables decides; larger mechanisms of the same species counts take the 16-lane kernel).
//
// Same integration as the other kernels (constant-pressure reactor, RODAS4, identical step-size
// controller).  What bounds it: a stiff cell's sub-steps run one after the other, and a lone wave
// issues one instruction every four to five cycles, so an attempt costs its instruction count, not
// its arithmetic.  The layout gives every lane the same short stream and shares it 64 ways:
//   * rates: one exponential per lane covers everything: lane j < 32 the forward constant of
//     reaction j, lane 32 + j the reverse one (ln k_f and ln k_f - ln K_c are dot products over
//     (1, ln T, 1/T, T .. T^4)), and four spare lanes per falloff reaction its k_0/k_inf and the
//     three Troe exponentials; each lane also forms its reaction's [M] from its own row, and one
//     logarithm stream gives ln T, ln sum Y/W (lane 63) and every ln [M].  The rows stay in registers.
//   * row lanes: lane l holds row r = l % 16 of every vector (T, Y_1 .. Y_K), four copies; sums
//     over lists of reactions and over matrix columns are split over the four copies g = l / 16
//     and added with lane swaps;
//   * Jacobian: each reaction lane writes the derivatives of its rate of progress with respect to
//     the concentrations, T, and density to an LDS record; the records times the stoichiometric
//     matrix is a product on the FP64 matrix cores (row 0 holds the reaction enthalpies, which gives
//     the temperature row), whose result layout leaves row r, columns 4 i + g in lane (r, g);
//   * linear algebra: W = I/(gamma h) - J stays in that layout and is inverted in place
//     (Gauss-Jordan with partial pivoting, three columns per lane, pivot rows fetched by lane
//     permutation), so a stage solve is three products and two lane swaps per lane.
// Measured on MI355X: an attempt of a lone wave takes 18.4k cycles (47k with 16 lanes per cell, whose wave
// issues 9,000 instructions for four cells), of which right-hand sides 9k, Jacobian 4.3k, inverse 4.4k;
// with two waves per SIMD a SIMD finishes one every 12 to 15k cycles, its vector unit busy 85 % of the
// time with 2,400 vector instructions (1,400 of them FP64) per attempt.  Whole calls, 16 lanes -> this
// kernel: 21 ignition cells 3.02 -> 1.35 ms, 1,001 cells 3.43 -> 1.51 ms, 65,536-cell hot-kernel field
// 5.1-5.4 -> 2.5-2.9 ms, developed flame 0.526 -> 0.461 ms, 262,144-cell mixing layer 31 -> 23 ms.
// Every scalar that steers control flow is the same in all 64 lanes (butterfly sums), so a wave
// never diverges.
#include <cmath>

#include "df_cell.h"

namespace df {
namespace {

// The queue of the cell order.  An atomic on one address from all eight XCDs costs about 12 ns, one after
// the other (65,536 short cells spent 340 us in them), so the order is dealt out to kCellQueues groups of
// blocks, slot x of group s being order[s + 8 x]: neighbouring blocks run on different XCDs, so a
// group's counter stays in one XCD's L2.  A group's units are its first quarter (the stiffest cells), and
// in any case the first four per wave, one cell each, then four cells each.  The front waves take
// units from the start, the others from the end: the first unit of each wave is fixed, the others are
// claimed; a claim on top of h front and t back units is valid while h + t is below the number of units,
// so every unit is taken once.  A wave whose group is empty goes on with the next group's units.
struct Queue {
    unsigned long long *ctr;  // of the group
    int64_t n, one, units;    // cells, single-cell units, all units of the group
    int s, fw, bw;            // group, its front and back waves

    __device__ __forceinline__ void group(unsigned long long *base, int64_t cells, int grp, int waves) {
        s = grp;
        ctr = base + 16 * s;
        n = (cells - s + kCellQueues - 1) / kCellQueues;
        const int blocks = (int(gridDim.x) - s + kCellQueues - 1) / kCellQueues;
        fw = blocks * (waves < 4 ? waves : 4);
        bw = blocks * waves - fw;
        const int64_t w = int64_t(fw + bw) * 4;
        one = n / 4 > w ? n / 4 : w;
        one = one < n ? one : n;
        units = one + (n - one + 3) / 4;
    }
};
// group slots [first, first + cells)
struct Span {
    int64_t first;
    int cells;
};
__device__ __forceinline__ Span unit_span(const Queue &q, int64_t u) {
    if (u < q.one) return {u, 1};
    const int64_t f = q.one + (u - q.one) * 4;
    return {f, int(f + 4 < q.n ? 4 : q.n - f)};
}
__device__ __forceinline__ unsigned long long claim(const Queue &q, bool front, int lane) {
    unsigned long long old = 0;
    if (lane == 0) old = atomicAdd(q.ctr, front ? 1ull : (1ull << 32));
    return old;
}
// the unit of a claim (cells = 0: the group is empty)
__device__ __forceinline__ Span claimed(const Queue &q, unsigned long long old, bool front) {
    const int64_t h = q.fw + int64_t(unsigned(__builtin_amdgcn_readfirstlane(int(old))));
    const int64_t t = q.bw + int64_t(unsigned(__builtin_amdgcn_readfirstlane(int(old >> 32))));
    if (h + t >= q.units) return {0, 0};
    return unit_span(q, front ? h : q.units - 1 - t);
}

constexpr int kQueueWaves = 8;  // per block of the queue: two per SIMD

// TAPE: every accepted sub-step is recorded for the adjoint (with the queue, except the length of the last
// one the tape can hold: the order lies there).
template <int K, int EL, bool TAPE>
__global__ __launch_bounds__(64 * kQueueWaves) void chem_cell_kernel(CellMech mg, StepArgs a, CellQueue q) {
    using C = CellWave<K, EL>;
    constexpr int N = C::N, NI = C::NI;
    extern __shared__ double lds[];
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), waves = int(blockDim.x) >> 6;
    double *const sh = lds + wave * C::kEnd;
    const int64_t limit = q.dcount ? int64_t(*q.dcount) : a.n;
    const bool queue = q.ctr != nullptr;
    // the second wave of each SIMD works from the cold end of the order, so that the stiffest
    // cells do not share a SIMD with one another
    const bool front = wave < 4;
    Queue u;
    Span span = {TAPE ? cell_of_block(a.n) : int64_t(blockIdx.x) * waves + wave, 1};
    if (queue) {
        u.group(q.ctr, limit, int(blockIdx.x) % kCellQueues, waves);
        const int64_t k = int64_t(blockIdx.x) / kCellQueues * (front ? (waves < 4 ? waves : 4) : waves - 4) +
                          (front ? wave : wave - 4);
        const int64_t x = front ? k : u.units - 1 - k;
        span = (x < u.units && x >= (front ? 0 : u.fw)) ? unit_span(u, x) : Span{0, 0};
    } else if (span.first >= limit) {
        return;
    }
    for (int i = lane; i < C::oEff; i += 64) sh[i] = 0.0;
    for (int i = lane; i < 32 * K; i += 64) {
        const int j = i / K;
        sh[C::oEff + i] = (j < mg.M) ? mg.eff[j * (K + 4) + i % K] : 0.0;
    }
    typename C::Row o;
    C::load_row(mg, lane, o);
    Coef kc;
    kc.set();
    lds_order();
    if (lane == 0) sh[C::oC] = 1.0;
    lds_order();
    const Opts &op = a.o;
    const double atol = (r == 0) ? op.atol_T : op.atol_Y;
    const int32_t *order = queue ? q.order : q.cidx;
    double *const yp = (r == 0) ? a.T : a.Y + int64_t(r <= K ? r - 1 : 0) * a.ld;  // the lane's row
    double *const rrp = a.rr ? a.rr + int64_t(r >= 1 && r <= K ? r - 1 : 0) * a.ld : nullptr;
    // cell indices of a span, one per lane, and one cell's state
    auto indices = [&](const Span &v) {
        if (queue) return lane < v.cells ? order[u.s + kCellQueues * (v.first + lane)] : 0;
        return order ? order[v.first] : 0;
    };
    int64_t i = 0;
    double yn = 0.0, pn = 0.0, dtn = 0.0;
    auto fetch = [&](const Span &v, int32_t idx, int cell) {
        i = order ? int64_t(__builtin_amdgcn_readlane(idx, cell)) : v.first;
        if (r < N) yn = yp[i];
        pn = a.p[i];
        dtn = a.dts ? a.dts[i] : a.dt;
    };
    // the next span after a unit that claimed nothing ahead; false at the end
    int left = kCellQueues - 1;  // groups not tried yet
    auto next = [&]() {
        if (!queue) {
            span.first += int64_t(gridDim.x) * waves;
            return span.first < limit;
        }
        for (;;) {
            span = claimed(u, claim(u, front, lane), front);
            if (span.cells > 0) return true;
            for (;;) {  // look before claiming: an empty group's counter is only read
                if (left-- == 0) return false;
                u.group(q.ctr, limit, (u.s + 1) % kCellQueues, waves);
                const unsigned long long c = __hip_atomic_load(u.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (int64_t(c & 0xffffffffull) + int64_t(c >> 32) + u.fw + u.bw < u.units) break;
            }
        }
    };
    if (span.cells == 0 && !next()) return;
    int32_t idx = indices(span);
    fetch(span, idx, 0);
    for (;;) {
        // a unit of several (short) cells: the next claim is in flight while they run, and each cell's
        // state while the one before it runs; a single cell may be a long one, and claims nothing ahead
        const int cells = span.cells;
        const bool ahead = cells > 1;
        const unsigned long long old = ahead ? claim(u, front, lane) : 0;
        Span span2 = {0, 0};
        int32_t idx2 = 0;
        for (int cell = 0; cell < cells; ++cell) {
            const int64_t ic = i;
            typename C::Cell c;
            double yr = yn;
            c.p = pn;
            const double dtc = dtn;
            if (ahead && cell == cells - 2) {
                span2 = claimed(u, old, front);
                idx2 = indices(span2);
            }
            if (cell + 1 < cells)
                fetch(span, idx, cell + 1);
            else if (span2.cells > 0)
                fetch(span2, idx2, 0);
            // non-finite rows, T <= 0, p or dt unusable: left untouched
            const bool bad = !isfinite(yr) || (r == 0 && !(yr > 0.0)) || !isfinite(c.p) || !(c.p > 0.0) ||
                             !isfinite(dtc) || !(dtc > 0.0);
            if (__builtin_amdgcn_ballot_w64(bad) != 0ull) {
                if (lane == 0) {
                    if (a.status) a.status[ic] = DF_CELL_NONFINITE;
                    if (a.nsteps) {
                        a.nsteps[ic] = 0;
                        a.nsteps[a.n + ic] = 0;
                    }
                    if (TAPE) Tape(K, a.n, a.tape_cap).count(a.tape)[ic] = -1;
                }
                if (a.rr && lane >= 1 && lane <= K) rrp[ic] = 0.0;
                continue;
            }
            c.ip = frcp(c.p);
            c.c6p = c.p * (1e-6 / kR);
            c.lc6p = dlogp(kc, c.c6p);
            const double y0 = yr;
            double rho0 = 0.0;
            if (a.rr) {  // input density over dt, for rr
                const double sYW = row_sum((r == 0) ? 0.0 : yr * o.iW);
                rho0 = fdiv(c.p, sYW * kR * lane_value(yr, 0) * dtc);
            }
            const double h_in = a.h_io ? a.h_io[ic] : 0.0;
            bool fresh = !(h_in > 0.0);
            double h = fresh ? 0.0 : fmin(h_in, dtc);
            if (!fresh && !(h >= op.h_min)) h = op.h_min;
            double t = 0.0, h_final = 0.0;
            int acc = 0, rej = 0;
            bool prev_rej = false;
            int st;
            for (;;) {
                if (acc + rej >= op.max_steps) {
                    st = DF_CELL_MAX_STEPS;
                    break;
                }
                double w[NI];
                const double f0 = C::jacobian(mg, kc, o, c, sh, lane, r, g, yr, w);
                if (fresh) {
                    // initial sub-step from the weighted norms of y0 and f(y0)
                    const double isc = frcp(atol + op.rtol * fabs(yr));
                    const double qy = (r < N) ? yr * isc : 0.0, qf = (r < N) ? f0 * isc : 0.0;
                    const double ny = lane_value(row_sum(qy * qy), 0), nf = lane_value(row_sum(qf * qf), 0);
                    h = (nf > 0.0) ? fmin(0.01 * sqrt(ny / nf), dtc) : dtc;
                    if (!(h >= op.h_min)) h = op.h_min;
                    fresh = false;
                }
                const bool last = (t + h >= dtc);
                const double ht = last ? dtc - t : h;
                const double ih = frcp(ht), ig = ih * (1.0 / Rodas4::g);
#pragma unroll
                for (int j = 0; j < NI; ++j) w[j] = ((4 * j + g == r && r < N) ? ig : 0.0) - w[j];
                int prow, vs;
                C::invert(w, r, g, prow, vs);
                // own components: stage vectors u_s[r]
                double u[6], ysr = yr;
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    double fs = f0;
                    if (s > 0) {
                        ysr = yr;
#pragma unroll
                        for (int j = 0; j < s; ++j) ysr = fma(Rodas4::a[s][j], u[j], ysr);
                        fs = C::rhs(mg, kc, o, c, sh, lane, r, ysr);
                    }
                    double cu = 0.0;
#pragma unroll
                    for (int j = 0; j < s; ++j) cu = fma(Rodas4::c[s][j], u[j], cu);
                    lds_order();
                    sh[C::oV + vs] = fma(cu, ih, fs);
                    lds_order();
                    double us = 0.0;
#pragma unroll
                    for (int j = 0; j < NI; ++j) us = fma(w[j], sh[C::oV + 4 * j + g], us);
                    u[s] = copies_sum(us);
                }
                // y_new = (stage-6 state) + u6 ; error = u6
                const double ynr = ysr + u[5];
                const double sc = atol + op.rtol * fmax(fabs(yr), fabs(ynr));
                const double er = (r < N) ? fdiv(u[5], sc) : 0.0;
                const double err = lane_value(sqrt(row_sum(er * er) * (1.0 / N)), 0);
                const double fmx = prev_rej ? 1.0 : 6.0;
                double fac;
                if (!isfinite(err))
                    fac = 0.2;
                else if (err == 0.0)
                    fac = fmx;
                else
                    fac = fmin(fmx, fmax(0.2, 0.9 / sqrt(sqrt(err))));  // 0.9 err^(-1/4)
                if (isfinite(err) && err <= 1.0) {
                    if (TAPE) {
                        int pc[NI];
#pragma unroll
                        for (int j = 0; j < NI; ++j) pc[j] = __builtin_amdgcn_ds_bpermute(4 * (4 * j + g), prow);
                        if (acc < a.tape_cap && r < N) {
                            // the accepted sub-step for the adjoint
                            const Tape tp(K, a.n, a.tape_cap);
                            const int64_t s = acc;
#pragma unroll
                            for (int j = 0; j < NI; ++j)
                                if (4 * j + g < N) a.tape[tp.w(s, r * N + pc[j]) + ic] = w[j];
                            if (g == 0) {
                                a.tape[tp.y(s, r) + ic] = yr;
                                if (r == 0 && !(queue && s == a.tape_cap - 1)) a.tape[tp.h(s) + ic] = ht;
#pragma unroll
                                for (int si = 0; si < 6; ++si) a.tape[tp.u(s, si * N + r) + ic] = u[si];
                            }
                        }
                    }
                    ++acc;
                    yr = (r < N) ? ynr : 0.0;
                    h_final = h;
                    prev_rej = false;
                    if (last) {
                        st = DF_CELL_OK;
                        break;
                    }
                    t += ht;
                    h = ht * fac;
                    // a long chain issues before the SIMD's other wave
                    if (acc == 16) __builtin_amdgcn_s_setprio(1);
                    if (acc == 128) __builtin_amdgcn_s_setprio(2);
                    if (acc == 384) __builtin_amdgcn_s_setprio(3);
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
            __builtin_amdgcn_s_setprio(0);
            if (TAPE) {
                // a cell whose accepted sub-steps did not all fit keeps its result but has no tape
                if (st == DF_CELL_OK && acc > a.tape_cap) st = DF_CELL_TAPE_FULL;
                if (lane == 0) Tape(K, a.n, a.tape_cap).count(a.tape)[ic] = (st == DF_CELL_OK) ? acc : -1;
            }
            if (lane < N) yp[ic] = yr;
            if (lane == 0) {
                if (a.h_io) a.h_io[ic] = (st == DF_CELL_OK) ? h_final : h;
                if (a.status) a.status[ic] = (st == DF_CELL_OK) ? a.status_ok : st;
                if (a.nsteps) {
                    a.nsteps[ic] = acc;
                    a.nsteps[a.n + ic] = rej;
                }
            } else if (lane <= K && a.rr) {
                rrp[ic] = rho0 * (yr - y0);
            }
        }
        if (span2.cells > 0) {
            span = span2;
            idx = idx2;
            continue;
        }
        if (!next()) return;
        idx = indices(span);
        fetch(span, idx, 0);
    }
}

template <int K, int EL>
df_status launch_k(const MechDev &m, const StepArgs &a, const CellQueue &q, hipStream_t stream) {
    // the queue runs a persistent grid, one block of two waves per SIMD and compute unit, with as
    // many front waves as there are SIMDs; a device-side count a grid of single waves that stride over
    // it; otherwise one cell per block, so that the hardware balances the cells
    int dev = 0, cus = 0, waves = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return fail(DF_E_HIP, "chem_step: cannot read the device's compute units");
    int64_t blocks = a.n;
    if (q.ctr) {
        waves = a.n <= int64_t(cus) * 4 ? 1 : kQueueWaves;
        blocks = waves == 1 ? a.n : cus;
    } else if (q.dcount) {
        blocks = blocks < int64_t(cus) * 8 ? blocks : int64_t(cus) * 8;
    }
    blocks = blocks < max_blocks(64) ? blocks : max_blocks(64);  // (beyond, the blocks stride)
    const size_t lds = size_t(waves) * CellWave<K, EL>::kEnd * sizeof(double);
    const CellMech cm{m.xd, m.xi, m.ceff, m.M, m.xtroe, m.xboth};
    if (a.tape)
        hipLaunchKernelGGL((chem_cell_kernel<K, EL, true>), dim3(unsigned(blocks)), dim3(64 * waves), lds, stream, cm, a,
                           q);
    else
        hipLaunchKernelGGL((chem_cell_kernel<K, EL, false>), dim3(unsigned(blocks)), dim3(64 * waves), lds, stream, cm, a,
                           q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(DF_E_HIP, std::string("chem_step launch: ") + hipGetErrorString(e));
    return DF_OK;
}

}  // namespace

bool chem_cell_supported(const MechDev &m) { return m.xel != 0; }

df_status launch_chem_cell(const MechDev &m, const StepArgs &a, const CellQueue &q, hipStream_t stream) {
    if (a.n == 0) return DF_OK;
#define DF_CASE(k)                                            \
    case k:                                                   \
        if (m.xel == 6) return launch_k<k, 6>(m, a, q, stream); \
        if (m.xel == 8) return launch_k<k, 8>(m, a, q, stream); \
        break;
    switch (m.K) {
        DF_CHEM_SPECIES_LIST(DF_CASE)
        default:
            break;
    }
#undef DF_CASE
    return fail(DF_E_UNSUPPORTED, "chem_step: no one-wave-per-cell kernel for this mechanism");
}

}  // namespace df
