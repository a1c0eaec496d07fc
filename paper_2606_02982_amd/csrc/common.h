// Device helpers shared by the DriftSched kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ds {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

__device__ __forceinline__ uint32_t readlane32(uint32_t v, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int lane)
{
    uint32_t lo = readlane32((uint32_t)v, lane);
    uint32_t hi = readlane32((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t lanemask_lt()
{
    int l = lane_id();
    return l ? (~0ull >> (64 - l)) : 0ull;
}

// The lanes of `among` whose bits [kFrom, kFrom + kBits) of x equal this
// lane's. Per bit: the bit spread over a word, the ballot of it, and one
// three-input operation per half that collects the lanes that differ (four
// instructions; written with selects it compiled to nine).
template <int kBits, int kFrom = 0>
__device__ __forceinline__ uint64_t match_bits(uint32_t x, uint64_t among)
{
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int b = kFrom; b < kFrom + kBits; b++) {
        const uint32_t own = (uint32_t)__builtin_amdgcn_sbfe((int)x, b, 1);   // 0 or ~0
        const uint64_t m = __ballot(own != 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, own, 0xF6);          // lo | (m ^ own)
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), own, 0xF6);
    }
    return among & ~(((uint64_t)hi << 32) | lo);
}

// match_bits<kBits>, and in `mine` the number of lanes of `among` whose low
// bits of x equal the lane's index (lanes below 2^kBits).
template <int kBits>
__device__ __forceinline__ uint64_t match_count(uint32_t x, uint64_t among, uint32_t &mine)
{
    uint32_t lo = 0, hi = 0, clo = 0, chi = 0;
#pragma unroll
    for (int b = 0; b < kBits; b++) {
        const uint32_t own = (uint32_t)__builtin_amdgcn_sbfe((int)x, b, 1);
        const uint32_t ind = (uint32_t)__builtin_amdgcn_sbfe(lane_id(), b, 1);
        const uint64_t m = __ballot(own != 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, own, 0xF6);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), own, 0xF6);
        clo = __builtin_amdgcn_bitop3_b32(clo, (uint32_t)m, ind, 0xF6);
        chi = __builtin_amdgcn_bitop3_b32(chi, (uint32_t)(m >> 32), ind, 0xF6);
    }
    mine = (uint32_t)__popcll(among & ~(((uint64_t)chi << 32) | clo));
    return among & ~(((uint64_t)hi << 32) | lo);
}

// DPP lane moves (gfx9 wave shifts): lane i receives lane i-1 (shr) or
// lane i+1 (shl) of x; the lane without a source receives `edge`.
__device__ __forceinline__ uint32_t wave_shr1(uint32_t x, uint32_t edge)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)x, 0x138, 0xF, 0xF, false);
}

__device__ __forceinline__ uint32_t wave_shl1(uint32_t x, uint32_t edge)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)x, 0x130, 0xF, 0xF, false);
}

// Inclusive prefix sum over the wave with DPP row shifts and row broadcasts.
__device__ __forceinline__ uint32_t wave_incl_scan_dpp(uint32_t x)
{
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);   // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);   // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);   // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast:15
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return x;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Total order on doubles as unsigned integers: a < b  <=>  bits(a) < bits(b),
// with -0.0 and +0.0 mapped to the same key. NaN is outside the contract.
__device__ __forceinline__ uint64_t ordered_bits(double x)
{
    if (x == 0.0) x = 0.0;
    uint64_t u = (uint64_t)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Device-scope relaxed atomics on 32-bit words (used for decoupled
// look-back flags, whose payload is the word itself).
__device__ __forceinline__ uint32_t ld_relaxed(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_relaxed(uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Block barrier for LDS traffic alone (s_waitcnt lgkmcnt(0); s_barrier):
// global loads and stores may stay in flight across it, so it orders no
// global memory between waves.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__host__ __device__ constexpr uint64_t cdiv(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
__host__ __device__ constexpr uint64_t align_up(uint64_t a, uint64_t b) { return cdiv(a, b) * b; }

}  // namespace ds
