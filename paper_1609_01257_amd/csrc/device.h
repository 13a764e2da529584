// Device functions that the generation and the batch kernels share.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rngx {

// Wait (bounded) until the device's constant-rate clock reaches `due`: at
// most about 2^16 polls of about 100 ns, so a wait ends whatever the clock
// does. Uniform across the wavefront: the clock is read by a scalar
// instruction.
__device__ __forceinline__ void wait_until(uint64_t due)
{
    uint32_t polls = 0;
#pragma nounroll
    while (__builtin_amdgcn_s_memrealtime() < due && ++polls < (1u << 16))
        __builtin_amdgcn_s_sleep(2);
}

// y = M x for a lane's own x, M given as 16 tables of 16 entries (entry v of
// table q is M (v << 4q)) held in LDS: the XOR of one lookup per nibble of x.
// Each table spans 128 bytes, so the lanes' lookups never share a bank.
__device__ __forceinline__ uint64_t nibble_product(const uint64_t *__restrict__ tab, uint64_t x)
{
    uint64_t y = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q)
        y ^= tab[16 * q + (uint32_t)((x >> (4 * q)) & 15u)];
    return y;
}

// Orders a wavefront's own LDS writes before its reads (and the reverse).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

} // namespace rngx
