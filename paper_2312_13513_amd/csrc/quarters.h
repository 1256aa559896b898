// A wave as four quarters of 16 lanes: exchanges and sums of doubles between
// the quarters, on the lane swaps of the target (no LDS).
#pragma once

#include <hip/hip_runtime.h>

namespace chem {

typedef unsigned ux2 __attribute__((ext_vector_type(2)));

struct DPair {
    double a, b;
};

// Halves: {a's lanes 0-31, b's lanes 0-31} and {a's 32-63, b's 32-63}.
__device__ __forceinline__ DPair swap_halves(double a, double b)
{
    const ux2 ua = __builtin_bit_cast(ux2, a), ub = __builtin_bit_cast(ux2, b);
    const auto lo = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
    return {__builtin_bit_cast(double, ux2{lo[0], hi[0]}), __builtin_bit_cast(double, ux2{lo[1], hi[1]})};
}

// Quarters: {a0, b0, a2, b2} and {a1, b1, a3, b3}.
__device__ __forceinline__ DPair swap_quarters(double a, double b)
{
    const ux2 ua = __builtin_bit_cast(ux2, a), ub = __builtin_bit_cast(ux2, b);
    const auto lo = __builtin_amdgcn_permlane16_swap(ua.x, ub.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(ua.y, ub.y, false, false);
    return {__builtin_bit_cast(double, ux2{lo[0], hi[0]}), __builtin_bit_cast(double, ux2{lo[1], hi[1]})};
}

// Sum over the four quarters, the same bits in each.
__device__ __forceinline__ double sum_quarters(double x)
{
    const DPair h = swap_halves(x, x);
    const double s = h.a + h.b;
    const DPair g = swap_quarters(s, s);
    return g.a + g.b;
}

__device__ __forceinline__ double min_quarters(double x)
{
    const DPair h = swap_halves(x, x);
    const double s = fmin(h.a, h.b);
    const DPair g = swap_quarters(s, s);
    return fmin(g.a, g.b);
}

}  // namespace chem
