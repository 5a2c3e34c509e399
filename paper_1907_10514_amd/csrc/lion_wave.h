// Sums over a wavefront with lane exchanges that stay in the vector registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lion {

// v plus the value of the lane that the DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over the 8 lanes of an octet, in every lane: xor 1, xor 2, then the mirrored
// halves (every lane of a quad already holds the same sum).
__device__ __forceinline__ double row8_sum(double v) {
    v = dpp_add<0xB1>(v);      // quad_perm(1, 0, 3, 2)
    v = dpp_add<0x4E>(v);      // quad_perm(2, 3, 0, 1)
    return dpp_add<0x141>(v);  // row_half_mirror
}

// Sum over the 16 lanes of a row.
__device__ __forceinline__ double row16_sum(double v) {
    return dpp_add<0x140>(row8_sum(v));  // row_mirror
}

// Sum over the 64 lanes, in every lane: the rows, then rows 0 + 1 and 2 + 3 and the
// two halves by the row swaps (each leaves one operand in the first result and the
// other in the second).
__device__ __forceinline__ double wave_sum(double v) {
    v = row16_sum(v);
    auto swap_add = [](double x, auto swap) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const auto lo = swap((uint32_t)b), hi = swap((uint32_t)(b >> 32));
        return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
               __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
    };
    v = swap_add(v, [](uint32_t u) { return __builtin_amdgcn_permlane16_swap(u, u, false, false); });
    return swap_add(v, [](uint32_t u) { return __builtin_amdgcn_permlane32_swap(u, u, false, false); });
}

}  // namespace lion
