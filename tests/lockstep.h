// Runs one workgroup of device code on the CPU: every thread is a fiber that
// runs until it reaches an operation over its wavefront (ballot, shuffle, a
// wavefront barrier) or its workgroup (a barrier).  A wavefront's operation
// happens when all of its threads wait, over those that wait at it (the others
// wait at a workgroup barrier or have ended, as lanes masked off would).
#pragma once
#include <ucontext.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <vector>

namespace lockstep {

enum Op { kRun, kBallot, kShfl, kWave, kCount, kEnd };

struct Fiber {
    ucontext_t ctx;
    std::vector<char> stack;
    Op op = kRun;
    uint64_t value = 0, result = 0;
    int from = 0;
};

inline std::vector<Fiber> fibers;
inline ucontext_t back;
inline int self = 0, block = 0, grid = 1;
inline std::function<void()> body;

inline uint64_t wait(Op op, uint64_t value, int from = 0) {
    Fiber& f = fibers[self];
    f.op = op;
    f.value = value;
    f.from = from;
    swapcontext(&f.ctx, &back);
    return f.result;
}

inline void entry() {
    body();
    fibers[self].op = kEnd;
    swapcontext(&fibers[self].ctx, &back);
}

inline void run(int threads, const std::function<void()>& f) {
    body = f;
    fibers.resize(threads);
    for (Fiber& x : fibers) {
        x.stack.resize(1 << 18);
        getcontext(&x.ctx);
        x.ctx.uc_stack.ss_sp = x.stack.data();
        x.ctx.uc_stack.ss_size = x.stack.size();
        makecontext(&x.ctx, entry, 0);
        x.op = kRun;
    }
    for (;;) {
        for (self = 0; self < threads; ++self)
            if (fibers[self].op == kRun) swapcontext(&back, &fibers[self].ctx);
        bool moved = false;
        for (int w = 0; w < threads; w += 64) {
            Op op = kCount;
            for (int l = w; l < w + 64; ++l)
                if (fibers[l].op != kCount && fibers[l].op != kEnd) {
                    if (op != kCount && op != fibers[l].op) {
                        fprintf(stderr, "lanes of one wavefront at different operations\n");
                        abort();
                    }
                    op = fibers[l].op;
                }
            if (op == kCount) continue;
            uint64_t mask = 0;
            for (int l = 0; l < 64; ++l)
                if (fibers[w + l].op == op && fibers[w + l].value) mask |= 1ull << l;
            for (int l = 0; l < 64; ++l) {
                Fiber& x = fibers[w + l];
                if (x.op != op) continue;
                x.result = op == kBallot ? mask : op == kShfl ? fibers[w + (x.from & 63)].value : 0;
            }
            for (int l = 0; l < 64; ++l)
                if (fibers[w + l].op == op) fibers[w + l].op = kRun;
            moved = true;
        }
        if (moved) continue;
        uint64_t count = 0;
        bool any = false;
        for (Fiber& x : fibers)
            if (x.op == kCount) any = true, count += x.value != 0;
        if (!any) return;
        for (Fiber& x : fibers)
            if (x.op == kCount) x.result = count, x.op = kRun;
    }
}

struct ThreadIdx { struct { operator int() const { return self; } } x; };
struct BlockIdx { struct { operator int() const { return block; } } x; };
struct GridDim { struct { operator int() const { return grid; } } x; };

}  // namespace lockstep

#define __device__
#define __global__
#define __forceinline__ inline
#define __shared__
#define __launch_bounds__(...)
static const lockstep::ThreadIdx threadIdx;
static const lockstep::BlockIdx blockIdx;
static const lockstep::GridDim gridDim;
static inline uint64_t __ballot(bool p) { return lockstep::wait(lockstep::kBallot, p); }
template <class T>
static inline T __shfl(T v, int from, int = 64) {
    return (T)lockstep::wait(lockstep::kShfl, (uint64_t)v, from);
}
template <class T>
static inline T __shfl_up(T v, int d, int = 64) {
    const int l = lockstep::self & 63;
    return (T)lockstep::wait(lockstep::kShfl, (uint64_t)v, l >= d ? l - d : l);
}
static inline int __syncthreads_count(bool p) { return (int)lockstep::wait(lockstep::kCount, p); }
static inline void __syncthreads() { lockstep::wait(lockstep::kCount, 0); }
static inline int __popc(uint32_t x) { return __builtin_popcount(x); }
static inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
template <class T>
static inline T atomicOr(T* p, T v) {
    const T o = *p;
    *p |= v;
    return o;
}
template <class T>
static inline T atomicAdd(T* p, T v) {
    const T o = *p;
    *p += v;
    return o;
}
template <class T>
static inline T atomicMin(T* p, T v) {
    const T o = *p;
    if (v < o) *p = v;
    return o;
}
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (void)(*(p) = (v))
#define __builtin_amdgcn_wave_barrier() (void)lockstep::wait(lockstep::kWave, 0)
static inline uint32_t lockstep_alignbit(uint32_t hi, uint32_t lo, uint32_t s) {
    return (uint32_t)((((uint64_t)hi << 32) | lo) >> (s & 31));
}
#define __builtin_amdgcn_alignbit(hi, lo, s) lockstep_alignbit((hi), (lo), (s))
static inline uint32_t lockstep_perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint32_t r = 0;
    for (int i = 0; i < 4; ++i) r |= (uint32_t)((v >> (8 * ((sel >> (8 * i)) & 7))) & 0xff) << (8 * i);
    return r;
}
#define RX_PERM(hi, lo, sel) lockstep_perm((hi), (lo), (sel))
#define RX_SEL(a, b, m) ((((uint32_t)(a)) & (m)) | (((uint32_t)(b)) & ~(m)))
struct uint4 { uint32_t x, y, z, w; };
static inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
