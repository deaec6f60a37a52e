// Accesses at a wave-uniform base plus a 32-bit lane offset in bytes, an addressing mode of the global memory instructions.
//
// The base is pinned to scalar registers: otherwise the compiler folds the lane offset into one loop-invariant 64-bit vector
// address per access, and dozens of such register pairs crowd out the accumulators (or push them out to scratch memory).  The pin goes
// through an integer, so the pointer has to be made one to global memory again: a generic one makes flat instructions, which may be
// LDS accesses for all that the hardware knows, so that every wait for an LDS read also waits for all of them, in whatever order
// they return.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace global_access {

typedef __attribute__((address_space(1))) char *bytes;

__device__ __forceinline__ uint64_t pinned(const void *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    uint64_t v = ((uint64_t)hi << 32) | lo;
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ bytes uniform_base(const void *p) { return (bytes)pinned(p); }
// A generic pointer, for kernels that were slower with global accesses or have not been tried with them.
__device__ __forceinline__ const char *uniform_flat(const void *p) { return (const char *)pinned(p); }

// V: float or a vector type
template <class V>
__device__ __forceinline__ void store(void *base, uint32_t lane_off, V v)
{
    *(__attribute__((address_space(1))) V *)(uniform_base(base) + lane_off) = v;
}
template <class V>
__device__ __forceinline__ void store_stream(void *base, uint32_t lane_off, V v)
{
    __builtin_nontemporal_store(v, (__attribute__((address_space(1))) V *)(uniform_base(base) + lane_off));
}

}  // namespace global_access
