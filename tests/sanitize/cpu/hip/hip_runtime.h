// A stand-in for the HIP runtime header that runs a kernel on the CPU, one
// block after another: every thread of the block is a fiber that runs until a
// barrier or a cross-lane operation, which wait for the threads of the block or
// of the wave that still run. `emu::last_wave_first` picks the order in which
// the waves go on behind a barrier, so that a result that depends on it shows.
// Kernels built with it see every index checked by the sanitizers of the host
// compiler (shared arrays are static arrays of their declared size). Only what
// the sources tested here use is defined. A wave's lanes are not in lockstep
// between two cross-lane operations.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <cmath>
#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __noinline__
#define __shared__ static
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct uint4 {
    uint32_t x, y, z, w;
} __attribute__((aligned(16)));
struct dim3 {
    uint32_t x, y, z;
    dim3(uint32_t a = 1, uint32_t b = 1, uint32_t c = 1) : x(a), y(b), z(c) {}
};
typedef int hipError_t;
typedef void *hipStream_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1;
inline hipError_t hipGetLastError() { return hipSuccess; }

using std::isfinite;
using std::isnan;

namespace emu {

inline dim3 thread_idx, block_idx, block_dim, grid_dim;
inline bool last_wave_first = false;

struct Fiber {
    ucontext_t ctx;
    std::vector<char> stack;
    bool done = false, blocked = false;
};
struct Group {   // the threads of a block, or of a wave
    uint32_t live = 0, here = 0;
    std::vector<uint32_t> waiting;
};
inline std::vector<Fiber> fibers;
inline std::vector<Group> waves;
inline Group block;
inline ucontext_t scheduler;
inline uint32_t running;
inline const std::function<void()> *body;
inline uint64_t slot[1024][2];   // the lanes' operands, by the parity of the operation
inline uint32_t parity[1024];

inline void release(Group &g)
{
    if (g.here < g.live) return;
    for (uint32_t t : g.waiting) fibers[t].blocked = false;
    g.waiting.clear();
    g.here = 0;
}

inline void wait(Group &g)
{
    const uint32_t t = running;
    g.here++;
    g.waiting.push_back(t);
    fibers[t].blocked = true;
    release(g);
    swapcontext(&fibers[t].ctx, &scheduler);
}

inline void thread_main()
{
    (*body)();
    const uint32_t t = running;
    fibers[t].done = true;
    block.live--;
    waves[t / 64].live--;
    release(block);
    release(waves[t / 64]);
    swapcontext(&fibers[t].ctx, &scheduler);
}

inline void run_block(uint32_t threads)
{
    fibers.resize(threads);
    waves.assign((threads + 63) / 64, Group());
    block = Group();
    for (uint32_t t = 0; t < threads; t++) {
        Fiber &f = fibers[t];
        f.done = f.blocked = false;
        f.stack.resize(256 << 10);
        getcontext(&f.ctx);
        f.ctx.uc_stack.ss_sp = f.stack.data();
        f.ctx.uc_stack.ss_size = f.stack.size();
        f.ctx.uc_link = nullptr;
        makecontext(&f.ctx, thread_main, 0);
        block.live++;
        waves[t / 64].live++;
    }
    // a wave goes on as long as one of its lanes can
    const uint32_t nw = (uint32_t)waves.size();
    for (bool any = true; any;) {
        any = false;
        for (uint32_t i = 0; i < nw; i++) {
            const uint32_t w = last_wave_first ? nw - 1 - i : i;
            for (bool more = true; more;) {
                more = false;
                for (uint32_t t = w * 64; t < w * 64 + 64 && t < threads; t++) {
                    if (fibers[t].done || fibers[t].blocked) continue;
                    running = t;
                    thread_idx = dim3(t);
                    swapcontext(&scheduler, &fibers[t].ctx);
                    more = any = true;
                }
            }
        }
    }
    if (block.live) {
        fprintf(stderr, "threads wait for each other\n");
        abort();
    }
}

inline void launch(const std::function<void()> &f, dim3 grid, dim3 threads)
{
    body = &f;
    grid_dim = grid;
    block_dim = threads;
    for (uint32_t b = 0; b < grid.x; b++) {
        block_idx = dim3(b);
        run_block(threads.x);
    }
}

// Every lane's operand, then the operation's result from all of the wave's.
inline const uint64_t (*exchange(uint64_t x, uint32_t &p))[2]
{
    const uint32_t t = running;
    p = parity[t] ^= 1u;
    slot[t][p] = x;
    wait(waves[t / 64]);
    return &slot[t & ~63u];
}
template <typename T> uint64_t bits(T v)
{
    uint64_t x = 0;
    memcpy(&x, &v, sizeof v);
    return x;
}
template <typename T> T from(uint64_t x)
{
    T v;
    memcpy(&v, &x, sizeof v);
    return v;
}
template <typename T> T lane_value(T v, uint32_t lane)
{
    uint32_t p;
    const uint64_t(*s)[2] = exchange(bits(v), p);
    return from<T>(s[lane & 63u][p]);
}
inline uint64_t ballot(bool b)
{
    uint32_t p;
    const uint64_t(*s)[2] = exchange(b, p);
    uint64_t m = 0;
    for (uint32_t l = 0; l < 64; l++) m |= s[l][p] << l;
    return m;
}
inline int dpp(int edge, int x, int ctrl, int row_mask, int, bool zero)
{
    uint32_t p;
    const int l = (int)(running & 63u);
    const uint64_t(*s)[2] = exchange(bits(x), p);
    int src = -1;
    if (ctrl > 0x110 && ctrl < 0x120) src = (l & 15) >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    else if (ctrl == 0x130) src = l < 63 ? l + 1 : -1;
    else if (ctrl == 0x138) src = l - 1;
    else if (ctrl == 0x142) src = l >= 16 ? (l & ~15) - 1 : -1;
    else if (ctrl == 0x143) src = l >= 32 ? 31 : -1;
    else abort();
    if (!((row_mask >> (l >> 4)) & 1)) return edge;
    return src < 0 ? (zero ? 0 : edge) : from<int>(s[src][p]);
}
inline uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c, uint32_t table)
{
    uint32_t r = 0;
    for (int i = 0; i < 8; i++)
        if ((table >> i) & 1u) r |= (i & 4 ? a : ~a) & (i & 2 ? b : ~b) & (i & 1 ? c : ~c);
    return r;
}
inline uint32_t sad_u8(uint32_t a, uint32_t b, uint32_t acc)
{
    for (int i = 0; i < 32; i += 8) acc += (uint32_t)abs((int)((a >> i) & 255u) - (int)((b >> i) & 255u));
    return acc;
}
template <typename T, typename U> T fetch_add(T *p, U v)
{
    const T old = *p;
    *p = (T)(old + v);
    return old;
}

}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define blockDim emu::block_dim
#define gridDim emu::grid_dim
#define hipLaunchKernelGGL(kernel, grid, threads, shared, stream, ...) \
    emu::launch([&] { (kernel)(__VA_ARGS__); }, grid, threads)

inline void __syncthreads() { emu::wait(emu::block); }
#define __builtin_amdgcn_s_barrier() emu::wait(emu::block)
#define __builtin_amdgcn_wave_barrier() ((void)emu::ballot(true))
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#define __builtin_amdgcn_readlane(v, l) emu::lane_value<int>(v, (uint32_t)(l))
#define __builtin_amdgcn_readfirstlane(v) emu::lane_value<int>(v, 0u)
#define __builtin_amdgcn_update_dpp(e, x, c, r, b, z) emu::dpp(e, x, c, r, b, z)
#define __builtin_amdgcn_sbfe(x, o, w) ((int)((uint32_t)(x) << (32 - (o) - (w))) >> (32 - (w)))
#define __builtin_amdgcn_bitop3_b32(a, b, c, t) emu::bitop3(a, b, c, t)
#define __builtin_amdgcn_sad_u8(a, b, c) emu::sad_u8(a, b, c)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) ((void)(*(p) = (v)))

inline uint64_t __ballot(bool b) { return emu::ballot(b); }
template <typename T> T __shfl(T v, int l, int) { return emu::lane_value(v, (uint32_t)l); }
template <typename T> T __shfl_xor(T v, int m, int) { return emu::lane_value(v, (emu::running ^ (uint32_t)m) & 63u); }
template <typename T> T __shfl_up(T v, int d, int)
{
    const int l = (int)(emu::running & 63u);
    return emu::lane_value(v, (uint32_t)(l >= d ? l - d : l));
}
template <typename T> T __shfl_down(T v, int d, int)
{
    const int l = (int)(emu::running & 63u);
    return emu::lane_value(v, (uint32_t)(l + d < 64 ? l + d : l));
}
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __clzll(long long x) { return x ? __builtin_clzll((unsigned long long)x) : 64; }
inline long long __double_as_longlong(double x) { return (long long)emu::bits(x); }
inline double __longlong_as_double(long long x) { return emu::from<double>((uint64_t)x); }
inline uint32_t atomicOr(uint32_t *p, uint32_t v)
{
    const uint32_t old = *p;
    *p |= v;
    return old;
}
inline uint32_t atomicAdd(uint32_t *p, uint32_t v) { return emu::fetch_add(p, v); }
