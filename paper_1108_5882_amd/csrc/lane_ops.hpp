// Values of other lanes without LDS: lane ^ M of the 64-lane wave.
#pragma once

#include <hip/hip_runtime.h>

namespace pwa {

template <int M>
__device__ __forceinline__ unsigned lane_xor(unsigned x) {
    static_assert(M == 1 || M == 2 || M == 4 || M == 8 || M == 16 || M == 32, "one lane bit");
    if constexpr (M == 1) return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);     // quad_perm [1,0,3,2]
    if constexpr (M == 2) return __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);     // quad_perm [2,3,0,1]
    if constexpr (M == 4)                                                                     // lane ^ 3, then ^ 7
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, x, 0x1B, 0xF, 0xF, true), 0x141, 0xF, 0xF,
                                           true);
    if constexpr (M == 8) return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xF, 0xF, true);    // row_ror 8
    if constexpr (M == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    }
    if constexpr (M == 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    }
}

template <int M>
__device__ __forceinline__ unsigned long long lane_xor(unsigned long long x) {
    return ((unsigned long long)lane_xor<M>((unsigned)(x >> 32)) << 32) | lane_xor<M>((unsigned)x);
}

template <int M>
__device__ __forceinline__ double lane_xor(double x) {
    return __longlong_as_double((long long)lane_xor<M>((unsigned long long)__double_as_longlong(x)));
}

// Sum over groups of W consecutive lanes, bits of the lane number from the lowest
// up; every lane of a group ends with the same bits.
template <int W>
__device__ __forceinline__ double lane_sum(double x) {
    if constexpr (W >= 2) x += lane_xor<1>(x);
    if constexpr (W >= 4) x += lane_xor<2>(x);
    if constexpr (W >= 8) x += lane_xor<4>(x);
    if constexpr (W >= 16) x += lane_xor<8>(x);
    if constexpr (W >= 32) x += lane_xor<16>(x);
    if constexpr (W >= 64) x += lane_xor<32>(x);
    return x;
}

}  // namespace pwa
