// Sum over the lanes of a wavefront without the LDS unit.
#pragma once
#include <hip/hip_runtime.h>

namespace ivftq {

// The sum of a value over a wavefront, in every lane: lanes 32 apart first, then 16, 8, ... 1, as a butterfly of exchanges
// adds them (an addition does not depend on the order of its two sides), without a trip through the LDS unit: once the
// values repeat every 2 s lanes, turning a row of sixteen by s is the exchange over a distance of s.
template <int S>
__device__ __forceinline__ float add_turned(float v) {
    const int i = __builtin_bit_cast(int, v);
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, i, 0x120 + S, 0xf, 0xf, false));   // row_ror:S
}
__device__ __forceinline__ float wave_sum(float v) {
    unsigned a = __builtin_bit_cast(unsigned, v);
    const auto h = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const unsigned h0 = h[0], h1 = h[1];         // (a bit cast of an element of a vector casts the first one, whichever is named)
    v = __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1);
    a = __builtin_bit_cast(unsigned, v);
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    v = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
    return add_turned<1>(add_turned<2>(add_turned<4>(add_turned<8>(v))));
}

}  // namespace ivftq
