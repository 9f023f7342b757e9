// Runs a kernel's workgroups on the CPU, one after the other, to check what a
// GPU run shows only by chance: that every thread of a workgroup meets the
// same barriers in whatever order its wavefronts run.  A thread is a
// coroutine that runs to its next barrier (or wavefront operation); of the
// wavefronts, `late` runs last after each barrier, when the others have
// already gone as far as the next.  A barrier that finds its threads at
// different places in the source ends the program with status 3.
//
// This is no model of memory or of partly active wavefronts: the wavefront
// operations want all 64 lanes.  Test code, compiled by g++ with the kernels'
// own source.
#pragma once

#include <limits.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <chrono>
#include <functional>
#include <new>
#include <random>
#include <string>
#include <vector>

namespace emu {

constexpr int kLanes = 64;
struct Dim {
    unsigned x = 0, y = 0, z = 0;
};
enum Wait { kReady, kWave, kBlock, kDone };
struct Thread {
    ucontext_t uc;
    std::vector<char> stack;
    Dim idx;
    Wait wait = kReady;
    int line = 0;   // of the barrier or the wavefront operation it waits at
};
inline std::vector<Thread> threads;
inline std::vector<uint64_t> lane_word;
inline Thread *self = nullptr;
inline ucontext_t home;
inline std::function<void()> body;
inline std::function<void(int)> after_wave;   // called when wavefront w has run as far as it can
inline Dim block, grid;
inline int late = 0, or_acc = 0, or_val = 0;

inline void yield(Wait w, int line) {
    self->wait = w;
    self->line = line;
    swapcontext(&self->uc, &home);
}
inline void entry() {
    body();
    self->wait = kDone;
    swapcontext(&self->uc, &home);
}
[[noreturn]] inline void diverged(const char *what, const Thread &a, const Thread &b) {
    printf("%s: thread %u waits at line %d, thread %u at line %d (state %d)\n", what, a.idx.x, a.line, b.idx.x, b.line,
           (int)b.wait);
    fflush(stdout);
    _Exit(3);
}
// Runs wavefront w until its lanes wait at a barrier of the workgroup or have ended.
inline void run_wave(int w) {
    Thread *t = &threads[(size_t)w * kLanes];
    while (true) {
        for (int l = 0; l < kLanes; l++)
            if (t[l].wait == kReady) {
                self = &t[l];
                swapcontext(&home, &t[l].uc);
            }
        int at_op = 0;
        for (int l = 0; l < kLanes; l++) at_op += t[l].wait == kWave;
        if (at_op == 0) return;
        for (int l = 0; l < kLanes; l++)
            if (t[l].wait != kWave || t[l].line != t[0].line) diverged("wavefront operation", t[0], t[l]);
        for (int l = 0; l < kLanes; l++) t[l].wait = kReady;
    }
}
inline void run_block() {
    const int waves = (int)threads.size() / kLanes;
    for (Thread &t : threads) {
        getcontext(&t.uc);
        t.stack.resize(1 << 16);
        t.uc.uc_stack.ss_sp = t.stack.data();
        t.uc.uc_stack.ss_size = t.stack.size();
        t.uc.uc_link = nullptr;
        makecontext(&t.uc, entry, 0);
        t.wait = kReady;
    }
    while (true) {
        for (int k = 0; k <= waves; k++) {   // the late wavefront last
            const int w = k < waves ? k : late;
            if (k < waves && w == late) continue;
            run_wave(w);
            if (after_wave) after_wave(w);
        }
        Thread *first = nullptr;
        for (Thread &t : threads) {
            if (t.wait == kDone) continue;
            if (!first) first = &t;
            if (t.line != first->line) diverged("barrier", *first, t);
        }
        if (!first) return;
        or_val = or_acc;
        or_acc = 0;
        for (Thread &t : threads)
            if (t.wait == kBlock) t.wait = kReady;
    }
}
// `blocks` workgroups of n threads each run f, wavefront `late_wave` always last.
inline void launch(unsigned blocks, unsigned n, int late_wave, std::function<void()> f) {
    threads = std::vector<Thread>(n);
    lane_word.assign(n, 0);
    for (unsigned k = 0; k < n; k++) threads[k].idx.x = k;
    late = late_wave;
    body = std::move(f);
    grid.x = blocks;
    for (block.x = 0; block.x < blocks; block.x++) run_block();
}
// Every lane's word to every lane of its wavefront.
template <class T, class F>
T exchange(T x, int line, F from) {
    static_assert(sizeof(T) <= 8, "a word");
    const unsigned me = self->idx.x, base = me / kLanes * kLanes;
    uint64_t u = 0;
    memcpy(&u, &x, sizeof(T));
    lane_word[me] = u;
    yield(kWave, line);
    const uint64_t r = lane_word[base + (unsigned)from((int)(me - base)) % kLanes];
    yield(kWave, line);   // nobody overwrites a word that is still to be read
    memcpy(&x, &r, sizeof(T));
    return x;
}
inline unsigned long long ballot(bool p, int line) {
    const unsigned me = self->idx.x, base = me / kLanes * kLanes;
    lane_word[me] = p;
    yield(kWave, line);
    unsigned long long m = 0;
    for (int l = 0; l < kLanes; l++) m |= (unsigned long long)(lane_word[base + l] & 1) << l;
    yield(kWave, line);
    return m;
}
inline int barrier_or(int x, int line) {
    or_acc |= x != 0;
    yield(kBlock, line);
    return or_val;
}
struct Pair {
    uint32_t v[2];
    uint32_t operator[](int k) const { return v[k]; }
};
template <class T>
T dpp(T x, int ctrl, int line) {
    return exchange(x, line, [=](int l) {
        return ctrl == 0xB1 ? l ^ 1 : ctrl == 0x4E ? l ^ 2 : ctrl == 0x141 ? l ^ 7 : l ^ 15;
    });
}
inline Pair swap(uint32_t x, int half, int line) {   // the lower rows' word, then the upper rows'
    return Pair{{exchange(x, line, [=](int l) { return l & ~half; }), exchange(x, line, [=](int l) { return l | half; })}};
}

}  // namespace emu

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __noinline__
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define threadIdx (emu::self->idx)
#define blockIdx (emu::block)
#define gridDim (emu::grid)
#define __syncthreads() emu::yield(emu::kBlock, __LINE__)
#define __syncthreads_or(x) emu::barrier_or((x) ? 1 : 0, __LINE__)
#define __ballot(p) emu::ballot((p), __LINE__)
#define __any(p) (emu::ballot((p), __LINE__) != 0)
#define __shfl(x, from, ...) emu::exchange((x), __LINE__, [=](int) { return (int)(from); })
#define __shfl_xor(x, o, ...) emu::exchange((x), __LINE__, [=](int l) { return l ^ (int)(o); })
#define __shfl_up(x, o, ...) emu::exchange((x), __LINE__, [=](int l) { return l < (int)(o) ? l : l - (int)(o); })
#define __builtin_amdgcn_update_dpp(old, x, ctrl, rows, banks, bound) emu::dpp((x), (ctrl), __LINE__)
#define __builtin_amdgcn_permlane16_swap(x, y, fi, bc) emu::swap((x), 16, __LINE__)
#define __builtin_amdgcn_permlane32_swap(x, y, fi, bc) emu::swap((x), 32, __LINE__)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() emu::yield(emu::kWave, __LINE__)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
#define __popc(x) __builtin_popcount(x)
#define __popcll(x) __builtin_popcountll(x)
#define __ffsll(x) __builtin_ffsll(x)
#define __threadfence() ((void)0)
#define __threadfence_system() ((void)0)

using hipStream_t = void *;
enum hipError_t { hipSuccess = 0 };
struct int4 {
    int x, y, z, w;
};
struct alignas(16) float4 {
    float x, y, z, w;
};
using std::max;
using std::min;
template <class T, class U>
T atomicAdd(T *p, U x) {
    const T old = *p;
    *p = old + (T)x;
    return old;
}
template <class T, class U>
T atomicSub(T *p, U x) {
    const T old = *p;
    *p = old - (T)x;
    return old;
}
template <class T, class U>
T unsafeAtomicAdd(T *p, U x) { return atomicAdd(p, x); }
template <class T>
T atomicCAS(T *p, T want, T to) {
    const T old = *p;
    if (old == want) *p = to;
    return old;
}
