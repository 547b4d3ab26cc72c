// The device language as a workgroup of lanes on the CPU, for headers of
// kernels that use one workgroup.  Every lane is a fiber.  The lanes of a
// wavefront meet at each cross-lane operation, the wavefronts of the workgroup
// at each barrier, and nothing else orders one wavefront against another: the
// caller names the order in which the wavefronts are let run, and each runs as
// far as it can before the next.  So a use of shared memory that lacks a
// barrier gives different results under some orders.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <ucontext.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <vector>

#define __device__
#define __global__ static
#define __shared__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

namespace lanes {

struct Dim {
    unsigned x, y = 1, z = 1;
};

struct Lane {
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    unsigned id = 0;
    uint32_t value = 0;     // operand of the cross-lane operation it waits in
    enum { READY, CROSS, BARRIER, DONE } state = READY;
};

inline ucontext_t scheduler;
inline std::vector<Lane> all;
inline Lane *cur = nullptr;
inline Dim block{64}, grid{1}, at{0};
inline void (*entry)() = nullptr;

inline void wait_in(int state)
{
    cur->state = static_cast<decltype(cur->state)>(state);
    swapcontext(&cur->ctx, &scheduler);
}

inline void start()
{
    entry();
    cur->state = Lane::DONE;
    swapcontext(&cur->ctx, &scheduler);
}

// Run `kernel` (which calls the kernel with its arguments) as one workgroup of
// `waves` wavefronts; order: the wavefronts, first choice first.
inline void run(void (*kernel)(), int waves, const std::vector<int> &order)
{
    constexpr size_t kStack = 64 << 10;
    entry = kernel;
    block.x = 64u * (unsigned)waves;
    all.clear();
    all.resize(block.x);
    for (unsigned i = 0; i < block.x; ++i) {
        Lane &l = all[i];
        l.id = i;
        l.stack.reset(new char[kStack]);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.get();
        l.ctx.uc_stack.ss_size = kStack;
        l.ctx.uc_link = nullptr;
        makecontext(&l.ctx, start, 0);
    }
    auto state = [&](int w) { return all[64 * w].state; };
    // up to the wavefront's next meeting point
    auto advance = [&](int w) {
        for (int i = 64 * w; i < 64 * w + 64; ++i) {
            cur = &all[i];
            swapcontext(&scheduler, &cur->ctx);
        }
        for (int i = 64 * w; i < 64 * w + 64; ++i)
            if (all[i].state != state(w)) {
                std::fprintf(stderr, "lanes of a wavefront part\n");
                std::exit(2);
            }
    };
    for (;;) {
        bool ran = false, live = false;
        for (int w : order) {
            while (state(w) == Lane::READY || state(w) == Lane::CROSS) {
                advance(w);
                ran = true;
            }
            live |= state(w) != Lane::DONE;
        }
        if (!live) return;
        if (ran) continue;
        for (Lane &l : all)
            if (l.state == Lane::BARRIER) l.state = Lane::READY;
    }
}

// DPP move: lane i of the wavefront gets the source lane's value, or `old`
// (bound: 0) where there is none; `old` in rows of 16 that the mask leaves out.
inline int dpp(int old, int value, int ctrl, int rows, int, bool bound)
{
    Lane *const me = cur;
    me->value = (uint32_t)value;
    wait_in(Lane::CROSS);
    const int i = (int)(me->id & 63), base = (int)(me->id & ~63u), row = i & ~15, in = i & 15;
    int src = -1;
    if (ctrl <= 0xff) src = (i & ~3) + (ctrl >> 2 * (i & 3) & 3);         // quad_perm
    else if (ctrl > 0x100 && ctrl < 0x110) src = in + (ctrl & 15) < 16 ? i + (ctrl & 15) : -1;  // row_shl
    else if (ctrl > 0x110 && ctrl < 0x120) src = in - (ctrl & 15) >= 0 ? i - (ctrl & 15) : -1;  // row_shr
    else if (ctrl == 0x130) src = i < 63 ? i + 1 : -1;                    // wave_shl:1
    else if (ctrl == 0x138) src = i - 1;                                  // wave_shr:1
    else if (ctrl == 0x140) src = row + 15 - in;                          // row_mirror
    else if (ctrl == 0x141) src = row + (in < 8 ? 7 - in : 23 - in);      // row_half_mirror
    else if (ctrl == 0x142) src = row - 1;                                // row_bcast:15
    else if (ctrl == 0x143) src = i >= 32 ? 31 : -1;                      // row_bcast:31
    else std::exit(3);
    const uint32_t got = src >= 0 ? all[base + src].value : 0;
    wait_in(Lane::CROSS);  // every lane has read before any offers its next value
    if (!(rows >> (i >> 4) & 1)) return old;
    if (src < 0) return bound ? 0 : old;
    return (int)got;
}

inline void barrier() { wait_in(Lane::BARRIER); }

}  // namespace lanes

#define threadIdx (lanes::Dim{lanes::cur->id})
#define blockDim (lanes::block)
#define gridDim (lanes::grid)
#define blockIdx (lanes::at)
#define __syncthreads() lanes::barrier()
#define __builtin_amdgcn_update_dpp(o, v, c, r, b, z) lanes::dpp(o, v, c, r, b, z)
#define __builtin_amdgcn_mov_dpp(v, c, r, b, z) lanes::dpp(0, v, c, r, b, z)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_s_setprio(p) ((void)0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)

inline unsigned __umulhi(unsigned a, unsigned b) { return (unsigned)((uint64_t)a * b >> 32); }

template <typename T>
inline T min(T a, T b)
{
    return b < a ? b : a;
}

using std::isfinite;
using std::sqrt;
