// Runs the kernels' own source on the CPU, one block per OS thread: every GPU
// thread is a fiber, barriers and cross-lane moves wait for the lanes that are
// still running, and LDS arrays belong to the OS thread (so they keep what the
// last block there left in them, as LDS does).  The order in which wavefronts
// reach a barrier is the caller's: run_block calls `between` after each
// wavefront has gone as far as it can for the first time, and anything may
// happen to global memory there, other blocks included.
//
// Include before the kernel source; compile as plain C++ with clang.
#pragma once

#define __HIP_PLATFORM_AMD__
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <vector>

namespace emu {

struct Idx {
    unsigned x = 0, y = 0, z = 0;
};
inline thread_local Idx tid, bid, bdim, gdim;

enum State { READY, BARRIER, XLANE, DONE };
struct Fiber {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    State state = READY;
};
struct Block {
    std::vector<Fiber> f;
    std::vector<int> post, seen;  // cross-lane operands: being posted, and of the last move
    ucontext_t main;
    std::function<void()> body;
    int cur = 0;
};
inline thread_local Block *blk = nullptr;

[[noreturn]] inline void fail(const char *what) {
    std::printf("emulation: %s\n", what);
    std::exit(1);
}

inline void yield(State s) {
    Block *b = blk;
    Fiber &f = b->f[b->cur];
    f.state = s;
    swapcontext(&f.ctx, &b->main);
}

inline void entry() {
    blk->body();
    blk->f[blk->cur].state = DONE;
    swapcontext(&blk->f[blk->cur].ctx, &blk->main);
}

// one block of `threads` threads, index `bx` of `nblocks`
inline void run_block(int bx, int nblocks, int threads, std::function<void()> body,
                      std::function<void(int)> between = nullptr) {
    Block b;
    b.f.resize(threads);
    b.post.resize(threads);
    b.seen.resize(threads);
    b.body = std::move(body);
    constexpr size_t kStack = 256 << 10;
    for (auto &f : b.f) {
        f.stack.reset(new char[kStack]);
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = f.stack.get();
        f.ctx.uc_stack.ss_size = kStack;
        f.ctx.uc_link = nullptr;
        makecontext(&f.ctx, entry, 0);
    }
    Block *outer = blk;
    const Idx t0 = tid, b0 = bid, d0 = bdim, g0 = gdim;
    bid.x = bx;
    bdim = Idx{(unsigned)threads, 1, 1};
    gdim = Idx{(unsigned)nblocks, 1, 1};
    blk = &b;
    const int waves = (threads + 63) / 64;
    // run one wavefront until each of its lanes waits at a barrier or has left
    auto advance = [&](int w) {
        const int lo = 64 * w, hi = std::min(threads, lo + 64);
        for (;;) {
            for (int l = lo; l < hi; l++)
                if (b.f[l].state == READY) {
                    b.cur = l;
                    tid.x = l;
                    swapcontext(&b.main, &b.f[l].ctx);
                }
            int x = 0, bar = 0;
            for (int l = lo; l < hi; l++) {
                x += b.f[l].state == XLANE;
                bar += b.f[l].state == BARRIER;
            }
            if (!x) return;
            if (bar) fail("a cross-lane move and a barrier in one wavefront");
            for (int l = lo; l < hi; l++) {
                b.seen[l] = b.post[l];
                if (b.f[l].state == XLANE) b.f[l].state = READY;
            }
        }
    };
    bool first = true;
    for (;;) {
        for (int w = 0; w < waves; w++) {
            advance(w);
            if (first && between) between(w);
        }
        first = false;
        bool left = false;
        for (auto &f : b.f)
            if (f.state == BARRIER) {
                f.state = READY;
                left = true;
            }
        if (!left) break;
    }
    blk = outer;
    tid = t0;
    bid = b0;
    bdim = d0;
    gdim = g0;
}

// a cross-lane move: this lane's operand goes out, all lanes' come back
inline const int *exchange(int v) {
    Block *b = blk;
    b->post[b->cur] = v;
    yield(XLANE);
    return b->seen.data() + (b->cur & ~63);
}
inline int readlane(int v, int lane) { return exchange(v)[lane]; }
inline int readfirstlane(int v) {
    const int *all = exchange(v);
    const int base = blk->cur & ~63;
    for (int l = 0; l < 64; l++)
        if (blk->f[base + l].state != DONE) return all[l];
    return v;
}
inline int update_dpp(int old, int src, int ctrl, int rows, int banks, bool bound) {
    const int *all = exchange(src);
    const int l = blk->cur & 63, row = l >> 4;
    if (!(rows >> row & 1) || !(banks >> (l >> 2 & 3) & 1)) return old;
    int from = -1;
    if (ctrl >= 0x111 && ctrl <= 0x11f) from = (l & 15) >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    else if (ctrl == 0x142) from = row ? 16 * row - 1 : -1;
    else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
    else fail("unknown dpp control");
    return from >= 0 ? all[from] : bound ? 0 : old;
}

struct Half2 {
    _Float16 x, y;
};
inline Half2 floats2half2(float a, float b) { return Half2{(_Float16)a, (_Float16)b}; }
inline float2 half22float2(Half2 h) { return make_float2((float)h.x, (float)h.y); }

}  // namespace emu

using std::isfinite;
using std::max;
using std::min;
using std::signbit;
inline void sincospif(float x, float *s, float *c) {
    *s = (float)std::sin(M_PI * (double)x);
    *c = (float)std::cos(M_PI * (double)x);
}

#define threadIdx emu::tid
#define blockIdx emu::bid
#define blockDim emu::bdim
#define gridDim emu::gdim
#undef __shared__
#define __shared__ static thread_local
#undef __launch_bounds__
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(...)
#define __syncthreads() emu::yield(emu::BARRIER)
#define __builtin_amdgcn_readlane emu::readlane
#define __builtin_amdgcn_readfirstlane emu::readfirstlane
#define __builtin_amdgcn_update_dpp emu::update_dpp
#define __half2 emu::Half2
#define __half22float2 emu::half22float2
#define __floats2half2_rn emu::floats2half2
inline long long emu_d2l(double v) {
    long long r;
    std::memcpy(&r, &v, 8);
    return r;
}
inline double emu_l2d(long long v) {
    double r;
    std::memcpy(&r, &v, 8);
    return r;
}
#define __double_as_longlong emu_d2l
#define __longlong_as_double emu_l2d
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) ((void)0)

// the one-launch loop's grid barrier is not emulated; these only let it compile
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, o, s) __atomic_load_n(p, o)
#define __hip_atomic_store(p, v, o, s) __atomic_store_n(p, v, o)
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
inline void __threadfence() {}
inline long long wall_clock64() { return 0; }
inline int __all(int) { emu::fail("__all"); }
namespace cooperative_groups {
struct Grid {
    void sync() { emu::fail("a grid barrier"); }
};
inline Grid this_grid() { return Grid(); }
}  // namespace cooperative_groups
