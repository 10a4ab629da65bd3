// Host stand-in for <hip/hip_runtime.h>: lets the integrator kernel sources compile as plain C++
// and run on the CPU, so that they can be checked under AddressSanitizer and
// UndefinedBehaviorSanitizer against the oracle.  Test infrastructure: the GPU library never
// includes it.
//
// What is emulated, and how:
//  * a launch runs one block at a time; each thread of the block is a fiber (ucontext) on one OS
//    thread, so a block's LDS (__shared__ arrays and the dynamic area) is shared by its threads
//    and the run is deterministic;
//  * __syncthreads, the wave barrier and every cross-lane operation (lane reads and permutations,
//    the DPP row permutations the kernels use, ballot, matrix products) are meeting points of a
//    wave: each fiber writes its operand and yields; once every live fiber of its wave has arrived
//    (one round of the scheduler), each reads its source lanes.  Meetings alternate between two
//    buffers, so a fiber that has moved on to the next meeting does not overwrite operands others
//    still read.  The scheduler checks that all live fibers of a wave arrive at the same meeting
//    (same count, same kind) and aborts with a message otherwise: a cross-lane operation in
//    divergent control flow shows up that way;
//  * the waves of a block run a few meetings at a time in an order drawn from EMU_SEED, and wait
//    for each other at __syncthreads only, so that a barrier that is missing between waves
//    gives other results with another seed;
//  * a lane that has returned is inactive for ballot;
//  * the hardware reciprocal and reciprocal square root are the exact ones (the kernels refine them);
//  * device memory is host memory.
#pragma once

#include <math.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#if defined(__SANITIZE_ADDRESS__)
#include <sanitizer/common_interface_defs.h>
#define EMU_ASAN 1
#endif

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) alignas(n)

using std::isfinite;
using std::isnan;
using std::max;
using std::min;

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
struct emu_uint3 {
    unsigned x, y, z;
};
inline emu_uint3 threadIdx, blockIdx;
inline dim3 blockDim, gridDim;

typedef int hipError_t;
typedef void *hipStream_t;
constexpr hipError_t hipSuccess = 0;
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize };
inline const char *hipGetErrorString(hipError_t) { return "emulated"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipMalloc(void **p, size_t n) {
    *p = std::calloc(n ? n : 1, 1);
    return *p ? hipSuccess : 2;
}
inline hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 2;  // compute units
    return hipSuccess;
}

namespace emu {

constexpr size_t kStack = size_t(1) << 18;  // bytes of stack per emulated thread

enum Kind { kSync = 1, kExchange = 2, kBallot = 3, kWave = 4 };

struct Fiber {
    ucontext_t ctx;
    std::vector<char> stack;
    bool done = false;
    long count = 0;  // meetings passed
    int kind = 0;    // kind of the meeting it waits at
};

struct Sched {
    ucontext_t main;
    std::vector<Fiber> f;
    int cur = -1;
    uint64_t buf[2][1024];
    long tag[2][1024];  // the meeting that the operand belongs to
    void (*entry)(void *) = nullptr;
    void *arg = nullptr;
#ifdef EMU_ASAN
    const void *main_bottom = nullptr;
    size_t main_size = 0;
#endif
};

inline Sched *S = nullptr;

// the order of the waves
inline uint32_t draw() {
    static uint64_t x = [] {
        const char *e = std::getenv("EMU_SEED");
        return uint64_t(e ? std::atoll(e) : 0) * 2 + 1;
    }();
    x = x * 6364136223846793005ull + 1442695040888963407ull;
    return uint32_t(x >> 40);
}
inline std::vector<unsigned char> dyn_lds_area;

template <class T>
T *dyn_lds() {
    return reinterpret_cast<T *>(dyn_lds_area.data());
}

// from a fiber back to the scheduler
inline void yield_to_main() {
    Fiber &me = S->f[S->cur];
#ifdef EMU_ASAN
    __sanitizer_start_switch_fiber(nullptr, S->main_bottom, S->main_size);
#endif
    swapcontext(&me.ctx, &S->main);
#ifdef EMU_ASAN
    __sanitizer_finish_switch_fiber(nullptr, nullptr, nullptr);
#endif
}

inline void fiber_entry() {
#ifdef EMU_ASAN
    __sanitizer_finish_switch_fiber(nullptr, &S->main_bottom, &S->main_size);
#endif
    S->entry(S->arg);
    S->f[S->cur].done = true;
    yield_to_main();  // never resumed
}

// wait at a meeting of the given kind; returns the buffer the meeting's operands went to
inline int meet(int kind) {
    Fiber &me = S->f[S->cur];
    const int p = int(me.count & 1);
    me.kind = kind;
    yield_to_main();
    ++me.count;
    return p;
}

inline uint64_t exchange(uint64_t v, int src) {
    const int p = int(S->f[S->cur].count & 1);
    S->buf[p][threadIdx.x] = v;
    meet(kExchange);
    return S->buf[p][src];
}

// every lane's operand of a meeting: element l is lane l's of this wave
inline const uint64_t *exchange_all(uint64_t v) {
    const int p = int(S->f[S->cur].count & 1);
    S->buf[p][threadIdx.x] = v;
    S->tag[p][threadIdx.x] = S->f[S->cur].count;
    meet(kExchange);
    return S->buf[p] + (threadIdx.x & ~63u);
}
// whether lane l of this wave was at the meeting that this fiber has just left (it may have returned since)
inline bool attended(int l) {
    const long c = S->f[S->cur].count - 1;
    return S->tag[c & 1][(threadIdx.x & ~63u) + l] == c;
}

template <class F, class... A>
void launch(F kernel, dim3 grid, dim3 block, size_t shmem, A... args) {
    if (grid.y != 1 || grid.z != 1 || block.y != 1 || block.z != 1 || block.x > 1024) {
        std::fprintf(stderr, "emulated launch: only 1-D grids of at most 1024 threads\n");
        std::abort();
    }
    if (dyn_lds_area.size() < shmem) dyn_lds_area.assign(shmem, 0);
    auto call = [&] { kernel(args...); };
    using Call = decltype(call);
    Sched sched;
    Sched *prev = S;
    S = &sched;
    sched.entry = [](void *c) { (*static_cast<Call *>(c))(); };
    sched.arg = &call;
    blockDim = block;
    gridDim = grid;
    for (unsigned bx = 0; bx < grid.x; ++bx) {
        blockIdx = emu_uint3{bx, 0, 0};
        sched.f.assign(block.x, Fiber{});
        std::memset(sched.tag, 0xff, sizeof(sched.tag));
        for (unsigned t = 0; t < block.x; ++t) {
            Fiber &fb = sched.f[t];
            fb.stack.assign(kStack, 0);
            getcontext(&fb.ctx);
            fb.ctx.uc_stack.ss_sp = fb.stack.data();
            fb.ctx.uc_stack.ss_size = kStack;
            fb.ctx.uc_link = nullptr;
            makecontext(&fb.ctx, fiber_entry, 0);
        }
        const unsigned waves = (block.x + 63) / 64;
        struct Wave {
            int live;
            bool waits;  // at __syncthreads
        };
        std::vector<Wave> w(waves);
        for (unsigned v = 0; v < waves; ++v) w[v] = Wave{int(block.x - 64 * v < 64 ? block.x - 64 * v : 64), false};
        for (unsigned live = waves; live > 0;) {
            unsigned ready = 0;
            for (unsigned v = 0; v < waves; ++v) ready += w[v].live > 0 && !w[v].waits;
            if (ready == 0)  // every wave that is left has arrived
                for (unsigned v = 0; v < waves; ++v) w[v].waits = false;
            unsigned v = draw() % waves;
            while (w[v].live == 0 || w[v].waits) v = (v + 1) % waves;
            for (int rounds = int(draw() % 8) + 1; rounds > 0 && w[v].live > 0 && !w[v].waits; --rounds) {
                long count = -1;
                int kind = 0;
                for (unsigned t = 64 * v; t < 64 * v + 64 && t < block.x; ++t) {
                    Fiber &fb = sched.f[t];
                    if (fb.done) continue;
                    sched.cur = int(t);
                    threadIdx = emu_uint3{t, 0, 0};
#ifdef EMU_ASAN
                    const void *bottom = nullptr;
                    __sanitizer_start_switch_fiber(nullptr, fb.stack.data(), kStack);
#endif
                    swapcontext(&sched.main, &fb.ctx);
#ifdef EMU_ASAN
                    __sanitizer_finish_switch_fiber(nullptr, &bottom, nullptr);
#endif
                    if (fb.done) {
                        if (--w[v].live == 0) --live;
                        continue;
                    }
                    if (count < 0) {
                        count = fb.count;
                        kind = fb.kind;
                    } else if (fb.count != count || fb.kind != kind) {
                        std::fprintf(stderr,
                                     "emulated block %u: thread %u waits at meeting %ld (kind %d), others at %ld "
                                     "(kind %d): a cross-lane operation or barrier in divergent control flow\n",
                                     bx, t, fb.count, fb.kind, count, kind);
                        std::abort();
                    }
                }
                w[v].waits = count >= 0 && kind == kSync;
            }
        }
    }
    S = prev;
}

}  // namespace emu

#define hipLaunchKernelGGL(kernel, grid, block, shmem, stream, ...) \
    ::emu::launch(kernel, dim3(grid), dim3(block), size_t(shmem), __VA_ARGS__)

inline void __syncthreads() { (void)emu::meet(emu::kSync); }
inline void __builtin_amdgcn_wave_barrier() { (void)emu::meet(emu::kWave); }
#define __builtin_amdgcn_fence(...) ((void)0)
inline void __builtin_amdgcn_s_setprio(int) {}

inline int emu_lane(int v, int l) {  // lane l's value, within the wave
    return int(uint32_t(emu::exchange(uint64_t(uint32_t(v)), int(threadIdx.x & ~63u) + (l & 63))));
}
inline int __builtin_amdgcn_readlane(int v, int l) { return emu_lane(v, l); }
inline int __builtin_amdgcn_readfirstlane(int v) {
    const uint64_t *all = emu::exchange_all(uint64_t(uint32_t(v)));
    int l = 0;
    while (!emu::attended(l)) ++l;
    return int(uint32_t(all[l]));
}
inline int __builtin_amdgcn_ds_bpermute(int addr, int v) { return emu_lane(v, addr >> 2); }
// the value of the (last) lane that sends to this one, 0 without one
inline int __builtin_amdgcn_ds_permute(int addr, int v) {
    const uint64_t *all = emu::exchange_all(uint64_t(uint32_t(v)) << 8 | uint64_t((addr >> 2) & 63));
    int r = 0;
    for (int l = 0; l < 64; ++l)
        if (int(all[l] & 63) == int(threadIdx.x & 63u)) r = int(uint32_t(all[l] >> 8));
    return r;
}
struct emu_pair {
    unsigned v[2];
    unsigned operator[](int i) const { return v[i]; }
};
// the second half (odd rows) of a and the first half (even rows) of b change places
inline emu_pair emu_swap(unsigned a, unsigned b, int width) {
    const int l = int(threadIdx.x & 63u);
    const uint64_t *all = emu::exchange_all(uint64_t(a) << 32 | b);
    return (l & width) ? emu_pair{unsigned(all[l - width]), b} : emu_pair{a, unsigned(all[l + width] >> 32)};
}
inline emu_pair __builtin_amdgcn_permlane32_swap(unsigned a, unsigned b, bool, bool) { return emu_swap(a, b, 32); }
inline emu_pair __builtin_amdgcn_permlane16_swap(unsigned a, unsigned b, bool, bool) { return emu_swap(a, b, 16); }

// the DPP controls the kernels use: quad_perm, row_half_mirror, row_mirror (every source lane
// valid, so `old` and the masks do not matter)
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int, int, bool) {
    (void)old;
    const int lane = int(threadIdx.x & 63u);
    int src;
    if (ctrl < 0x100)
        src = (lane & ~3) | ((ctrl >> (2 * (lane & 3))) & 3);
    else if (ctrl == 0x140)
        src = (lane & ~15) | (15 - (lane & 15));
    else if (ctrl == 0x141)
        src = (lane & ~7) | (7 - (lane & 7));
    else {
        std::fprintf(stderr, "emulated DPP control 0x%x not supported\n", ctrl);
        std::abort();
    }
    return emu_lane(v, src);
}
inline int __builtin_amdgcn_mov_dpp(int v, int ctrl, int a, int b, bool c) {
    return __builtin_amdgcn_update_dpp(0, v, ctrl, a, b, c);
}

// 16 x 16 x 4 FP64 product: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16], and holds rows 4 i + l / 16 of
// column l % 16 of the sum
template <class V>
V __builtin_amdgcn_mfma_f64_16x16x4f64(double a, double b, V c, int, int, int) {
    double A[64], B[64];
    uint64_t bits;
    std::memcpy(&bits, &a, 8);
    std::memcpy(A, emu::exchange_all(bits), sizeof(A));
    std::memcpy(&bits, &b, 8);
    std::memcpy(B, emu::exchange_all(bits), sizeof(B));
    const int n = int(threadIdx.x & 15u), g = int(threadIdx.x & 63u) / 16;
    for (int i = 0; i < 4; ++i)
        for (int k = 0; k < 4; ++k) c[i] = std::fma(A[16 * k + 4 * i + g], B[16 * k + n], c[i]);
    return c;
}

// lanes of the wave that have returned count as inactive
inline unsigned long long __ballot(int pred) {
    const int p = int(emu::S->f[emu::S->cur].count & 1);
    emu::S->buf[p][threadIdx.x] = pred ? 1u : 0u;
    emu::S->tag[p][threadIdx.x] = emu::S->f[emu::S->cur].count;
    emu::meet(emu::kBallot);
    unsigned long long m = 0;
    const unsigned w0 = threadIdx.x & ~63u;
    for (unsigned l = 0; l < 64 && w0 + l < blockDim.x; ++l)
        if (emu::attended(int(l)) && emu::S->buf[p][w0 + l]) m |= 1ull << l;
    return m;
}

inline unsigned long long __builtin_amdgcn_ballot_w64(bool pred) { return __ballot(pred); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline int __ffsll(long long x) { return __builtin_ffsll(x); }
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x; }
inline double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x); }
#define __constant__
#define __hip_atomic_load(p, order, scope) (*(p))
inline long long __double_as_longlong(double x) {
    long long r;
    std::memcpy(&r, &x, 8);
    return r;
}
inline double __longlong_as_double(long long x) {
    double r;
    std::memcpy(&r, &x, 8);
    return r;
}
inline unsigned long long atomicAdd(unsigned long long *p, unsigned long long v) {
    const unsigned long long o = *p;
    *p = o + v;
    return o;
}
inline int atomicAdd(int *p, int v) {
    const int o = *p;
    *p = o + v;
    return o;
}
