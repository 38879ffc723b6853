// sse_guard.h -- values by the upper half of their absolute binary64 form, as the guard of
// the spectral form (SpecGuard) compares them.
#pragma once

#include <hip/hip_runtime.h>

#include "sse_internal.h"

namespace sse {

__device__ __forceinline__ uint32_t magnitude(double x) { return (uint32_t)__double2hiint(x) & 0x7fffffffu; }
__device__ __forceinline__ uint32_t magnitude(double2 v)
{
    const uint32_t x = magnitude(v.x), y = magnitude(v.y);
    return x > y ? x : y;
}
__device__ __forceinline__ uint32_t magnitude(float2 v) { return magnitude(make_double2(v.x, v.y)); }
// The least value that does not lie below the guard of a peak.
__device__ __forceinline__ uint32_t guard_floor(uint32_t peak, int bits)
{
    const uint32_t b = (uint32_t)bits << 20;
    return peak > b ? peak - b : 0u;
}
__device__ __forceinline__ uint32_t scaled(uint32_t peak, double scale)
{
    return magnitude(__hiloint2double((int)peak, 0) * scale);
}

// The word at the start of a spectral instance's workspace: a value was not finite, the direct
// kernel computes all; some outputs are marked as suspect.
constexpr uint32_t kFlagAll = 1u, kFlagSuspect = 2u;

// Momentum k's bit in an energy's suspect word; more momenta than bits share them all.
__device__ __forceinline__ uint32_t suspect_bit(int k, int Nkz) { return Nkz > 32 ? ~0u : 1u << (Nkz - 1 - k); }

}  // namespace sse
