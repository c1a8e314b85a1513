// sem_wave.h -- sums across the lanes of a wave, for the device sources.
#pragma once

#include <hip/hip_runtime.h>

namespace sem {

// Sum over the wave, to every lane, all 64 active: the tree of a butterfly over lane distances
// 32, 16, 8, 4, 2, 1, bit for bit.  Cross-lane moves of the vector unit (half-wave and row
// swaps, then shifts within a row, whose lane 0 ends with the sum) take a few cycles a step
// where shuffles through LDS take over a hundred: a step of the coarse solve in one workgroup
// 3.4 -> 3.1 us at 1331 vertices and 1.24 -> 0.95 us at 343, with the single-reduction form.
template <int ROWS>
__device__ __forceinline__ double swap_plus(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    if constexpr (ROWS == 2) {  // lane distance 32
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    } else {  // 16
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    }
}
template <int N>
__device__ __forceinline__ double shl_plus(double v)  // lane i of a row adds lane i + N
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x100 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x100 + N, 0xf, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = swap_plus<2>(v);
    v = swap_plus<1>(v);
    v = shl_plus<8>(v);
    v = shl_plus<4>(v);
    v = shl_plus<2>(v);
    v = shl_plus<1>(v);
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

}  // namespace sem
