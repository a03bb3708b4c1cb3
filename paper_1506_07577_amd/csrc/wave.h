// wave.h -- sums over the lanes of a wavefront (or of aligned groups of 2, 4, 8 or 16 lanes) with
// register lane exchanges.  An xor butterfly through __shfl_xor costs two LDS-crossbar round trips
// per FP64 step; here lane i meets lane i ^ M by v_permlane32_swap / v_permlane16_swap (M = 32, 16)
// or by DPP within a row of 16 lanes, all VALU.  The partners and so the sums are those of the
// butterfly, bit for bit.  Every lane of the group must be active.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ebbx {

template <int CTRL> __device__ __forceinline__ double dpp_mov(double x) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// x of this lane plus x of lane ^ M
template <int M> __device__ __forceinline__ double xor_add(double x) {
    if constexpr (M == 32 || M == 16) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
        // of two copies, the first ends with the lower partner's value in both lanes, the second
        // with the upper one's
        auto swap = [](uint32_t v) {
            if constexpr (M == 32) return __builtin_amdgcn_permlane32_swap(v, v, false, false);
            else return __builtin_amdgcn_permlane16_swap(v, v, false, false);
        };
        const auto l = swap(lo), h = swap(hi);
        return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
               __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
    } else if constexpr (M == 8) {
        return x + dpp_mov<0x128>(x);                  // row_ror:8
    } else if constexpr (M == 4) {
        return x + dpp_mov<0x1b>(dpp_mov<0x141>(x));   // row_half_mirror, then quad_perm [3,2,1,0]
    } else if constexpr (M == 2) {
        return x + dpp_mov<0x4e>(x);                   // quad_perm [2,3,0,1]
    } else {
        static_assert(M == 1, "a power of two below 64");
        return x + dpp_mov<0xb1>(x);                   // quad_perm [1,0,3,2]
    }
}

// Sum over aligned groups of L lanes, in every lane: partners L/2 apart first, then L/4, ...
template <int L> __device__ __forceinline__ double lanes_sum(double x) {
    if constexpr (L > 1) return lanes_sum<L / 2>(xor_add<L / 2>(x));
    return x;
}

}  // namespace ebbx
