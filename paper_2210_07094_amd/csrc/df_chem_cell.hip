// Detailed-chemistry step on gfx950 with one wavefront per cell, for mechanisms whose rates fit one
// wave: at most 31 reactions (lane 63 forms sum Y/W), and a group of four spare lanes per falloff reaction
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
// Measured on MI355X: an attempt of a lone wave takes 17k cycles (47k with 16 lanes per cell, whose wave issues
// 9,000 instructions for four cells); with two waves per SIMD a SIMD finishes one every 12k, its vector unit busy
// 84 % of the time with 2,190 vector instructions per attempt (79 % and 2,430 per one-sub-step cell, its start and end
// included).  Whole calls with a workspace, 16 lanes -> this kernel: 21 ignition cells 2.98 -> 1.21 ms, 1,001 cells
// 3.40 -> 1.37 ms, 32,768 cells 19.5 -> 17.1 ms (the 16-lane queue 17.9), 65,536-cell hot-kernel field 4.97 -> 2.58 ms,
// 65,536-cell developed flame 0.526 -> 0.405 ms, 65,536-cell mixing layer 27.6 -> 10.6 ms.
// Every scalar that steers control flow is the same in all 64 lanes (butterfly sums), so a wave
// never diverges.
#include <cmath>

#include "df_cell.h"

namespace df {
namespace {

// The queue of the cell order.  An atomic on one address from all eight XCDs costs about 12 ns, one after
// the other (65,536 short cells spent 340 us in them), so the order is dealt out to kCellQueues groups of
// blocks, cell x of group s being order[s + 8 x]: neighbouring blocks run on different XCDs, so a
// group's counter stays in one XCD's L2.  The front waves take cells from the start, the others from the
// end: the first cell of each wave is fixed, the others are claimed; a claim on top of h front and t back
// cells is valid while h + t is below the number of cells, so every cell is taken once.  A wave whose
// group is empty goes on with the next group's cells.
struct Queue {
    unsigned long long *ctr;  // of the group
    int n, s, fw, bw;         // cells, group, its front and back waves

    __device__ __forceinline__ void group(unsigned long long *base, int64_t cells, int grp, int waves) {
        s = grp;
        ctr = base + 16 * s;
        n = int((cells - s + kCellQueues - 1) / kCellQueues);
        const int blocks = (int(gridDim.x) - s + kCellQueues - 1) / kCellQueues;
        fw = blocks * (waves < 4 ? waves : 4);
        bw = blocks * waves - fw;
    }
    // the group's cell of a claim whose counter read `old` (-1: none left)
    __device__ __forceinline__ int claimed(unsigned long long old, bool front) const {
        const int64_t h = fw + int64_t(unsigned(__builtin_amdgcn_readfirstlane(int(old))));
        const int64_t t = bw + int64_t(unsigned(__builtin_amdgcn_readfirstlane(int(old >> 32))));
        return h + t >= n ? -1 : int(front ? h : n - 1 - t);
    }
};

constexpr int kQueueWaves = 8;  // per block of the queue: two per SIMD

// TAPE: every accepted sub-step is recorded for the adjoint (with the queue, except the length of the last
// one the tape can hold: the order lies there).
template <int K, int EL, bool TAPE>
__global__ __launch_bounds__(64 * kQueueWaves) void chem_cell_kernel(CellMech mg, StepArgs a, CellQueue q) {
    using C = CellWave<K, EL>;
    constexpr int N = C::N, NI = C::NI;
    extern __shared__ double lds[];
    __shared__ int taken;
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), waves = int(blockDim.x) >> 6;
    double *const sh = lds + wave * C::kEnd;
    const int64_t limit = q.dcount ? int64_t(*q.dcount) : a.n;
    const bool queue = q.ctr != nullptr;
    // the second wave of each SIMD works from the cold end of the order, so that the stiffest
    // cells do not share a SIMD with one another
    const bool front = wave < 4;
    Queue grp;
    // Without a queue: one cell per one-wave block, or (several waves) a block takes one cell of each run of gridDim.x
    // cells, another place in each run, so that a hot column of a field meets every block, and its waves
    // share them out through a counter in LDS.  One wave per cell for any number of cells, whose start (its rows of
    // the mechanism) a one-sub-step cell pays a sixth of its time for: flame of 8,000 cells 75 us, 65,536 cells
    // 522 us, this way 58 and 387 us (16 lanes 65 and 476); hot-kernel field of 65,536 cells 5.4 and 3.5 ms (10.3).
    const bool local = !queue && waves > 1;
    int64_t at = TAPE ? cell_of_block(a.n) : int64_t(blockIdx.x);  // place of the wave's cell
    auto local_place = [&]() {
        int x = 0;
        if (lane == 0) x = atomicAdd(&taken, 1);
        x = __builtin_amdgcn_readfirstlane(x);
        const unsigned grid = gridDim.x;
        const int64_t place = int64_t(x) * grid + (blockIdx.x + unsigned(x) * 37u) % grid;
        return place < limit ? place : int64_t(-1);
    };
    if (queue) {
        grp.group(q.ctr, limit, int(blockIdx.x) % kCellQueues, waves);
        const int k = int(blockIdx.x) / kCellQueues * (front ? (waves < 4 ? waves : 4) : waves - 4) +
                      (front ? wave : wave - 4);
        const int x = front ? k : grp.n - 1 - k;
        at = (x < grp.n && x >= (front ? 0 : grp.fw)) ? grp.s + int64_t(kCellQueues) * x : -1;
    } else if (local) {
        if (threadIdx.x == 0) taken = 0;
        __syncthreads();
        if ((at = local_place()) < 0) return;
    } else if (at >= limit) {
        return;
    }
    // (every load of the wave's start is in flight before the first is waited for)
    typename C::Row o;
    C::load_row(mg, lane, o);
    C::load_eff(mg, lane, sh);
    Coef kc;
    kc.set();
    lds_order();
    if (lane == 0) sh[C::oC] = 1.0;
    lds_order();
    // The arguments, read from the kernel's argument segment where they are used: held in registers, they would push
    // what every attempt needs out of them, some of it to scratch memory, which an empty launch pays for too (the
    // fallback of a DNN step on one cell: 0.7 of its 34 us).
    typedef const __attribute__((address_space(4))) StepArgs *ArgPtr;
    const auto seg = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
    auto args = [&]() {
        auto p = ArgPtr(seg + (sizeof(CellMech) + alignof(StepArgs) - 1) / alignof(StepArgs) * alignof(StepArgs));
        asm volatile("" : "+s"(p));
        return p;
    };
    auto atol = [&](ArgPtr b) { return (r == 0) ? b->o.atol_T : b->o.atol_Y; };
    const int32_t *order = queue ? q.order : q.cidx;
    // the lane's row of T and Y, or of rr, at a cell
    const unsigned row = r >= 1 && r <= K ? r - 1 : 0;
    auto row_of = [&](ArgPtr b, int64_t cell) { return r == 0 ? b->T + cell : b->Y + (row * b->ld + cell); };
    auto rr_of = [&](ArgPtr b, int64_t cell) { return b->rr + (row * b->ld + cell); };
    // A place's cell and the cell's state.  (Loads by an index that the compiler takes for different in each lane:
    // a scalar load would be waited for by the next LDS access.)
    auto vector_zero = []() {
        int z = 0;
        asm("" : "+v"(z));
        return z;
    };
    auto cell_at = [&](int64_t place) { return order ? order[place + vector_zero()] : int32_t(place); };
    int64_t i = 0;
    double yn = 0.0, pn = 0.0, dtn = 0.0;
    auto fetch = [&](int32_t cell) {
        const auto b = args();
        i = int64_t(__builtin_amdgcn_readfirstlane(cell));
        if (r < N) yn = *row_of(b, i);
        const int64_t iv = i + vector_zero();
        pn = b->p[iv];
        dtn = b->dts ? b->dts[iv] : b->dt;
    };
    auto claim = [&]() {
        unsigned long long old = 0;
        if (lane == 0) old = atomicAdd(grp.ctr, front ? 1ull : (1ull << 32));
        return old;
    };
    auto place_of = [&](int x) { return x < 0 ? int64_t(-1) : grp.s + int64_t(kCellQueues) * x; };
    // the next place when nothing was claimed ahead (empty: that was tried, and there is none, in this group of
    // a queue); -1 at the end
    int left = kCellQueues - 1;  // groups not tried yet
    auto next = [&](bool empty) {
        if (!queue) return local && !empty ? local_place() : int64_t(-1);
        for (;;) {
            const int64_t place = empty ? -1 : place_of(grp.claimed(claim(), front));
            if (place >= 0) return place;
            empty = false;
            for (;;) {  // look before claiming: an empty group's counter is only read
                if (left-- == 0) return int64_t(-1);
                grp.group(q.ctr, limit, (grp.s + 1) % kCellQueues, waves);
                const unsigned long long c = __hip_atomic_load(grp.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const int64_t taken_front = unsigned(__builtin_amdgcn_readfirstlane(int(c)));
                const int64_t taken_back = unsigned(__builtin_amdgcn_readfirstlane(int(c >> 32)));
                if (taken_front + taken_back + grp.fw + grp.bw < grp.n) break;
            }
        }
    };
    if (at < 0 && (at = next(false)) < 0) return;
    fetch(cell_at(at));
    for (;;) {
        // The cell that follows is claimed when an attempt starts that would end this one, and its index and
        // state are loaded while that attempt's stages run; a chain that goes on holds no other cell back.  With a
        // claim after each single cell, and four cells per claim in the order's colder part, small flames waited for
        // them (24,000 cells 212 us, now 171; 16 lanes 202) and uniformly stiff fields for the last units (32,768
        // ignition cells 22.4 ms, now 17.1).
        enum { kNone, kClaimed, kIndexed, kLoaded, kEmpty };
        int ahead = kNone;
        unsigned long long old = 0;
        int32_t following = 0;
        {
            const int64_t ic = i;
            const auto b = args();
            typename C::Cell c;
            double yr = yn;
            c.p = pn;
            const double dtc = dtn;
            // non-finite rows, T <= 0, p or dt unusable: left untouched
            const bool bad = !isfinite(yr) || (r == 0 && !(yr > 0.0)) || !isfinite(c.p) || !(c.p > 0.0) ||
                             !isfinite(dtc) || !(dtc > 0.0);
            if (__builtin_amdgcn_ballot_w64(bad) != 0ull) {
                if (lane == 0) {
                    if (b->status) b->status[ic] = DF_CELL_NONFINITE;
                    if (b->nsteps) {
                        b->nsteps[ic] = 0;
                        b->nsteps[b->n + ic] = 0;
                    }
                    if (TAPE) Tape(K, b->n, b->tape_cap).count(b->tape)[ic] = -1;
                }
                if (b->rr && lane >= 1 && lane <= K) *rr_of(b, ic) = double(vector_zero());
                if ((at = next(false)) < 0) return;
                fetch(cell_at(at));
                continue;
            }
            c.ip = frcp(c.p);
            c.c6p = c.p * (1e-6 / kR);
            c.lc6p = dlogp(kc, c.c6p);
            const double y0 = yr;
            const double h_in = b->h_io ? b->h_io[ic] : 0.0;
            bool fresh = !(h_in > 0.0);
            double h = fresh ? 0.0 : fmin(h_in, dtc);
            if (!fresh && !(h >= b->o.h_min)) h = b->o.h_min;
            double t = 0.0;
            int acc = 0, rej = 0;
            bool prev_rej = false;
            int st;
            for (;;) {
                const auto e = args();
                if (acc + rej >= e->o.max_steps) {
                    st = DF_CELL_MAX_STEPS;
                    break;
                }
                double w[NI];
                const double f0 = C::jacobian(mg, kc, o, c, sh, lane, r, g, yr, w);
                if (fresh) {
                    // initial sub-step from the weighted norms of y0 and f(y0)
                    const double isc = frcp(atol(e) + e->o.rtol * fabs(yr));
                    const double qy = (r < N) ? yr * isc : 0.0, qf = (r < N) ? f0 * isc : 0.0;
                    const double ny = lane_value(row_sum(qy * qy), 0), nf = lane_value(row_sum(qf * qf), 0);
                    h = (nf > 0.0) ? fmin(0.01 * sqrt(ny / nf), dtc) : dtc;
                    if (!(h >= e->o.h_min)) h = e->o.h_min;
                    fresh = false;
                }
                const bool last = (t + h >= dtc);
                const double ht = last ? dtc - t : h;
                if (last && ahead == kNone) {
                    if (queue) old = claim();
                    ahead = kClaimed;
                }
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
                    if (s == 2 && ahead == kClaimed) {
                        at = queue ? place_of(grp.claimed(old, front)) : next(false);
                        if (at >= 0) following = cell_at(at);
                        ahead = at >= 0 ? kIndexed : kEmpty;
                    }
                    if (s == 4 && ahead == kIndexed) {
                        fetch(following);
                        ahead = kLoaded;
                    }
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
                const double sc = atol(e) + e->o.rtol * fmax(fabs(yr), fabs(ynr));
                const double er = (r < N) ? u[5] * frcp3(sc) : 0.0;
                const double e2 = lane_value(row_sum(er * er) * (1.0 / N), 0);  // squared norm
                const double fmx = prev_rej ? 1.0 : 6.0;
                // 0.9 err^(-1/4) = 0.9 e2^(-1/8) from three reciprocal square root estimates and a Newton step,
                // within [0.2, fmx] (reached below 1e-12)
                double fac = 0.2;
                if (isfinite(e2)) {
                    const double x = fmax(e2, 1e-12);
                    const double v = __builtin_amdgcn_rsq(__builtin_amdgcn_rsq(__builtin_amdgcn_rsq(x)));
                    const double v2 = v * v, v4 = v2 * v2;
                    fac = fmin(fmx, fmax(0.2, 0.9 * fma(v, fma(-0.125 * x * v4, v4, 0.125), v)));
                }
                if (isfinite(e2) && e2 <= 1.0) {
                    if (TAPE) {
                        int pc[NI];
#pragma unroll
                        for (int j = 0; j < NI; ++j) pc[j] = __builtin_amdgcn_ds_bpermute(4 * (4 * j + g), prow);
                        if (acc < e->tape_cap && r < N) {
                            // the accepted sub-step for the adjoint
                            const Tape tp(K, e->n, e->tape_cap);
                            const int64_t s = acc;
#pragma unroll
                            for (int j = 0; j < NI; ++j)
                                if (4 * j + g < N) e->tape[tp.w(s, r * N + pc[j]) + ic] = w[j];
                            if (g == 0) {
                                e->tape[tp.y(s, r) + ic] = yr;
                                if (r == 0 && !(queue && s == e->tape_cap - 1)) e->tape[tp.h(s) + ic] = ht;
#pragma unroll
                                for (int si = 0; si < 6; ++si) e->tape[tp.u(s, si * N + r) + ic] = u[si];
                            }
                        }
                    }
                    ++acc;
                    yr = (r < N) ? ynr : 0.0;
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
                    if (h < e->o.h_min) {
                        st = DF_CELL_H_UNDERFLOW;
                        break;
                    }
                }
            }
            __builtin_amdgcn_s_setprio(0);
            const auto e = args();
            if (TAPE) {
                // a cell whose accepted sub-steps did not all fit keeps its result but has no tape
                if (st == DF_CELL_OK && acc > e->tape_cap) st = DF_CELL_TAPE_FULL;
                if (lane == 0) Tape(K, e->n, e->tape_cap).count(e->tape)[ic] = (st == DF_CELL_OK) ? acc : -1;
            }
            if (lane < N) *row_of(e, ic) = yr;
            if (e->rr) {  // rr = rho0 (Y - Y0) / dt with the input state's density rho0
                const double sYW = row_sum((r == 0) ? 0.0 : y0 * o.iW);
                const double rho0 = fdiv(1e6 * c.c6p, sYW * lane_value(y0, 0) * dtc);
                if (lane >= 1 && lane <= K) *rr_of(e, ic) = rho0 * (yr - y0);
            }
            if (lane == 0) {
                if (e->h_io) e->h_io[ic] = h;  // (an accepted sub-step that ended the cell left it as it was)
                if (e->status) e->status[ic] = (st == DF_CELL_OK) ? e->status_ok : st;
                if (e->nsteps) {
                    e->nsteps[ic] = acc;
                    e->nsteps[e->n + ic] = rej;
                }
            }
        }
        if (ahead == kLoaded) continue;
        if ((at = next(ahead == kEmpty)) < 0) return;
        fetch(cell_at(at));
    }
}

template <int K, int EL>
df_status launch_k(const MechDev &m, const StepArgs &a, const CellQueue &q, hipStream_t stream) {
    // the queue, and calls without an order of more cells than waves fit at once, run a persistent grid, one
    // block of two waves per SIMD and compute unit (the queue with as many front waves as there are SIMDs);
    // otherwise one cell per wave
    int dev = 0, cus = 0, waves = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return fail(DF_E_HIP, "chem_step: cannot read the device's compute units");
    if (a.n > int64_t(cus) * (q.ctr ? 4 : kQueueWaves)) waves = kQueueWaves;
    const int64_t blocks = waves == 1 ? a.n : cus;
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

bool chem_cell_supported(const MechDev &m) {
    bool compiled = false;
#define DF_CASE(k) compiled = compiled || m.K == k;
    DF_CHEM_SPECIES_LIST(DF_CASE)
#undef DF_CASE
    return compiled && m.xel != 0;
}

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
