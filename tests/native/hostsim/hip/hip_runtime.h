// The kernels' own headers and launchers compiled as plain C++: a workgroup's
// threads are fibers on one host thread, run from barrier to barrier in an
// order that the check chooses.  LDS starts filled with a chosen value, so a
// slot that is read before it is written, and an access that another wave's
// access of the same barrier interval conflicts with, change the result from
// one order or fill to the next.
//
// Lanes of a wave are not in lockstep here: a wave's lanes meet at
// __builtin_amdgcn_wave_barrier and in lane exchanges only.  skip_lane leaves
// out lanes whose work other lanes of the wave repeat in lockstep.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <random>
#include <string>
#include <type_traits>
#include <unordered_map>
#include <utility>
#include <vector>

#include "hip_runtime_api.h"

using std::fma;

struct dim3 {
    unsigned x, y, z;
    explicit dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace hostsim {

constexpr int kLds = 20480; // doubles: one compute unit's 160 KB
enum State { READY, AT_WAVE, AT_BLOCK, DONE };

struct Fiber {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    State state;
};
inline ucontext_t sched;
inline std::vector<Fiber> fibers;
inline int current;
inline const std::function<void()> *body;
inline double exchange[1024];

// what a check sets before a launch
inline int order = 0;                                    // 0 ascending, 1 descending, 2 random
inline double fill = 0.0;                                // value of unwritten LDS
inline bool (*skip_lane)(int lane) = nullptr;            // lanes left out
inline std::vector<double *> lds_arrays;                 // the kernels' LDS arrays
inline int errors = 0;

inline void yield(State s)
{
    Fiber &f = fibers[current];
    f.state = s;
    swapcontext(&f.ctx, &sched);
}
inline void entry()
{
    (*body)();
    fibers[current].state = DONE;
    swapcontext(&fibers[current].ctx, &sched);
}

inline void workgroup(int n)
{
    constexpr size_t kStack = 1 << 18;
    if (int(fibers.size()) < n) fibers.resize(n);
    std::vector<std::vector<int>> waves((n + 63) / 64);
    for (int t = 0; t < n; ++t) {
        Fiber &f = fibers[t];
        f.state = DONE;
        if (skip_lane && skip_lane(t & 63)) continue;
        if (!f.stack) f.stack.reset(new char[kStack]);
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = f.stack.get();
        f.ctx.uc_stack.ss_size = kStack;
        f.ctx.uc_link = nullptr;
        makecontext(&f.ctx, entry, 0);
        f.state = READY;
        waves[t / 64].push_back(t);
    }
    if (order == 1) {
        std::reverse(waves.begin(), waves.end());
        for (auto &w : waves) std::reverse(w.begin(), w.end());
    }
    std::mt19937 rng(7);
    for (;;) {
        if (order == 2) {
            std::shuffle(waves.begin(), waves.end(), rng);
            for (auto &w : waves) std::shuffle(w.begin(), w.end(), rng);
        }
        int blocked = 0, done = 0;
        for (const auto &w : waves) { // each wave as far as it gets
            for (int at_wave = 1; at_wave > 0;) {
                at_wave = 0;
                int left = 0;
                for (int t : w) {
                    if (fibers[t].state == READY) {
                        current = t;
                        threadIdx.x = unsigned(t);
                        swapcontext(&sched, &fibers[t].ctx);
                    }
                    (fibers[t].state == AT_WAVE ? at_wave : left) += 1;
                }
                if (at_wave > 0 && left > 0) {
                    std::fprintf(stderr, "lanes of one wave at different barriers\n");
                    std::exit(2);
                }
                if (at_wave > 0)
                    for (int t : w) fibers[t].state = READY;
            }
            for (int t : w) (fibers[t].state == AT_BLOCK ? blocked : done) += 1;
        }
        if (blocked == 0) return;
        if (done != 0) {
            std::fprintf(stderr, "%d threads at a barrier that %d have left\n", blocked, done);
            std::exit(2);
        }
        for (const auto &w : waves)
            for (int t : w) fibers[t].state = READY;
    }
}

inline void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()> &kernel)
{
    if (lds > sizeof(double) * kLds || block.x == 0 || block.x > 1024 || grid.x == 0) {
        std::fprintf(stderr, "launch of %u threads with %zu bytes of LDS\n", block.x, lds);
        std::exit(2);
    }
    body = &kernel;
    gridDim = grid;
    blockDim = block;
    const double mark = -fill - 1.0;
    for (unsigned b = 0; b < grid.x; ++b) {
        blockIdx.x = b;
        for (double *a : lds_arrays)
            for (int i = 0; i < kLds + 64; ++i) a[i] = size_t(i) < lds / sizeof(double) ? fill : mark;
        workgroup(int(block.x));
        for (double *a : lds_arrays)
            for (int i = int(lds / sizeof(double)); i < kLds + 64; ++i)
                if (std::memcmp(a + i, &mark, sizeof(mark)) != 0) ++errors;
    }
}

inline double shfl_xor(double x, int off)
{
    const int t = current, o = t ^ off;
    exchange[t] = x;
    yield(AT_WAVE);
    const double r = o < int(blockDim.x) && fibers[o].state != DONE ? exchange[o] : x;
    yield(AT_WAVE);
    return r;
}

} // namespace hostsim

#define __device__
#define __host__
#define __global__
#define __shared__
#define __constant__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define asm
#define volatile(...)
#define __syncthreads() hostsim::yield(hostsim::AT_BLOCK)
#define __shfl_xor(x, off) hostsim::shfl_xor(x, off)
#define __builtin_amdgcn_wave_barrier() hostsim::yield(hostsim::AT_WAVE)
#define __builtin_amdgcn_fence(...)
#define __builtin_amdgcn_sched_barrier(...)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / std::sqrt(x))
#define __builtin_amdgcn_sqrtf(x) std::sqrt(x)
#define __builtin_amdgcn_mov_dpp(x, ...) (x)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, ...) (c)
#define __hip_atomic_load(p, ...) (*(p))
#define __HIP_MEMORY_SCOPE_AGENT 0
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    hostsim::launch(grid, block, lds, [&] { (kernel)(__VA_ARGS__); })
inline hipError_t hipGetLastError() { return hipSuccess; }
inline void atomicMax(unsigned long long *p, unsigned long long v) { *p = std::max(*p, v); }
inline double __longlong_as_double(long long x) { double d; std::memcpy(&d, &x, 8); return d; }
inline long long __double_as_longlong(double x) { long long d; std::memcpy(&d, &x, 8); return d; }
inline int __double2loint(double x) { return int(__double_as_longlong(x)); }
inline int __double2hiint(double x) { return int(__double_as_longlong(x) >> 32); }
inline double __hiloint2double(int hi, int lo) { return __longlong_as_double((long long)(hi) << 32 | unsigned(lo)); }
