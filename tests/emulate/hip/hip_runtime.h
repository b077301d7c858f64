// One workgroup of a kernel on the CPU: the kernel headers compiled as host C++.
//
// Every work-item is a fiber that runs until it reaches a barrier or a lane
// exchange, in an order that the test chooses, so a result that hangs on the order
// of the work-items between two barriers shows.  (On the device the order is the
// hardware's and the compiler's choice.)  An ended work-item no longer counts at a
// barrier, as on gfx950.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <type_traits>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define hipLaunchKernelGGL(...) ((void)0)
typedef void* hipStream_t;

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

template <typename T>
T min(T a, T b) { return a < b ? a : b; }
template <typename T>
T max(T a, T b) { return a > b ? a : b; }

namespace emu {
enum State { READY, AT_WORKGROUP, AT_WAVE, AT_EXCHANGE, ENDED };
struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    State st = READY;
    unsigned sent = 0;   // values put into box
    int box[2];
};
inline std::vector<Lane> lanes;
inline ucontext_t home;
inline unsigned cur;
inline const std::function<void()>* body;

inline void yield(State s) {
    lanes[cur].st = s;
    swapcontext(&lanes[cur].ctx, &home);
}
inline void entry() {
    (*body)();
    lanes[cur].st = ENDED;
    swapcontext(&lanes[cur].ctx, &home);
}
// x of the other lane of a pair (both of them take part).
template <int CTRL>
int exchange(int x) {
    static_assert(CTRL == 0xB1, "only the swap of lane pairs");
    Lane &me = lanes[cur], &other = lanes[cur ^ 1];
    const unsigned k = me.sent++;
    me.box[k & 1] = x;
    while (other.sent <= k) yield(AT_EXCHANGE);
    return other.box[k & 1];
}
// `fn` on every work-item of workgroup `blk`, each turn in the order `order`;
// `after(k)` once k work-items have had their first turn.
inline void run(unsigned nt, dim3 blk, dim3 grid, const std::vector<unsigned>& order,
                const std::function<void()>& fn, const std::function<void(unsigned)>& after) {
    lanes.clear();
    lanes.resize(nt);
    body = &fn;
    blockIdx = blk;
    gridDim = grid;
    blockDim = dim3(nt);
    for (Lane& l : lanes) {
        l.stack.resize(1 << 17);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = &home;
        makecontext(&l.ctx, entry, 0);
    }
    auto wave_is = [&](unsigned w, State s) {
        for (unsigned k = 64 * w; k < 64 * w + 64 && k < nt; ++k)
            if (lanes[k].st != ENDED && lanes[k].st != s) return false;
        return true;
    };
    for (bool first = true;; first = false) {
        bool ran = false;
        unsigned k = 0;
        for (unsigned l : order) {
            if (lanes[l].st == READY || lanes[l].st == AT_EXCHANGE) {
                const unsigned sent = lanes[l].sent;
                const State before = lanes[l].st;
                cur = l;
                threadIdx = dim3(l, 0, 0);
                swapcontext(&home, &lanes[l].ctx);
                ran = ran || lanes[l].sent != sent || lanes[l].st != before;
            }
            if (first) after(++k);
        }
        for (unsigned w = 0; 64 * w < nt; ++w)
            if (wave_is(w, AT_WAVE))
                for (unsigned j = 64 * w; j < 64 * w + 64 && j < nt; ++j)
                    if (lanes[j].st == AT_WAVE) { lanes[j].st = READY; ran = true; }
        bool all = true, ended = true;
        for (unsigned w = 0; 64 * w < nt; ++w) all = all && wave_is(w, AT_WORKGROUP);
        for (Lane& l : lanes) ended = ended && l.st == ENDED;
        if (ended) return;
        if (all) {
            for (Lane& l : lanes)
                if (l.st == AT_WORKGROUP) l.st = READY;
        } else if (!ran) {
            fprintf(stderr, "the workgroup hangs\n");
            exit(2);
        }
    }
}
}  // namespace emu

inline void __syncthreads() { emu::yield(emu::AT_WORKGROUP); }
#define __builtin_amdgcn_wave_barrier() emu::yield(emu::AT_WAVE)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_mov_dpp(x, ctrl, rows, banks, bound) \
    emu::exchange<ctrl>(x)
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_readfirstlane(x) (x)  // used on uniform values
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) ((void)(*(p) = (v)))
#define __HIP_MEMORY_SCOPE_AGENT 4

template <typename A, typename B>
A bits(B b) {
    static_assert(sizeof(A) == sizeof(B), "");
    A a;
    memcpy(&a, &b, sizeof a);
    return a;
}
inline int __double2hiint(double x) { return (int)(bits<uint64_t>(x) >> 32); }
inline int __double2loint(double x) { return (int)bits<uint64_t>(x); }
inline double __hiloint2double(int hi, int lo) {
    return bits<double>(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
}
inline int __float_as_int(float x) { return bits<int>(x); }
inline float __int_as_float(int x) { return bits<float>(x); }
inline double __shfl_down(double, int, int) {  // wave sums: not on the paths run here
    fprintf(stderr, "no cross-lane sums here\n");
    exit(2);
}
