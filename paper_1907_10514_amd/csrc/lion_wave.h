// Sums over a wavefront with lane exchanges that stay in the vector registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lion {

// The value of the lane that the DPP control CTRL names.
template <int CTRL>
__device__ __forceinline__ double dpp_get(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    return v + dpp_get<CTRL>(v);
}

// v plus the value of lane ^ D, D = 1, 2 or 4 (4: from the lane four up in the lower
// quad of an octet, four down in the upper).
template <int D>
__device__ __forceinline__ double xor_add(double v) {
    if constexpr (D == 1) {
        return dpp_add<0xB1>(v);
    } else if constexpr (D == 2) {
        return dpp_add<0x4E>(v);
    } else {
        static_assert(D == 4, "within an octet");
        auto get = [](uint32_t u) {
            const int up = __builtin_amdgcn_update_dpp(0, (int)u, 0x104, 0xf, 0x5, false);
            return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)u, 0x114, 0xf, 0xa, false);
        };
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        return v + __builtin_bit_cast(double, ((uint64_t)get((uint32_t)(b >> 32)) << 32) | get((uint32_t)b));
    }
}

// The value of the lane above, lane 0's in lane 63.
__device__ __forceinline__ double lane_above(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, 0x134, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b >> 32), 0x134, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
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

// a and b with halves (swap_rows: rows 0 and 1, 2 and 3) exchanged and added: one half
// (the even rows) of the result holds a's sum over the pair, the other b's.
template <bool HALVES>
__device__ __forceinline__ double swap_add(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    auto swap = [](uint32_t u, uint32_t w) {
        if constexpr (HALVES)
            return __builtin_amdgcn_permlane32_swap(u, w, false, false);
        else
            return __builtin_amdgcn_permlane16_swap(u, w, false, false);
    };
    const auto lo = swap((uint32_t)x, (uint32_t)y);
    const auto hi = swap((uint32_t)(x >> 32), (uint32_t)(y >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi[0] << 32) | lo[0]) +
           __builtin_bit_cast(double, ((uint64_t)hi[1] << 32) | lo[1]);
}

// Sum over the 64 lanes, in every lane.
__device__ __forceinline__ double wave_sum(double v) {
    v = row16_sum(v);
    v = swap_add<false>(v, v);
    return swap_add<true>(v, v);
}

// The sums of N values over the 64 lanes into out[0 .. N): four at a time share the
// lanes (21 instructions for four values, 72 for four single sums).
template <int N>
__device__ __forceinline__ void wave_sums(const double (&v)[N], double* out) {
    const int lane = threadIdx.x & 63, row = lane >> 4;
#pragma unroll
    for (int g = 0; g < N; g += 4) {
        auto at = [&](int k) { return g + k < N ? v[g + k] : 0.0; };
        const double h0 = swap_add<true>(at(0), at(1)), h1 = swap_add<true>(at(2), at(3));
        const double s = row16_sum(swap_add<false>(h0, h1));  // rows: values 0, 2, 1, 3
        const int k = g + (row == 1 ? 2 : (row == 2 ? 1 : row));
        if ((lane & 15) == 0 && k < N) out[k] = s;
    }
}

}  // namespace lion
