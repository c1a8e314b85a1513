// sem_wave.h -- sums across the lanes of a wave, for the device sources.
#pragma once

#include <hip/hip_runtime.h>

namespace sem {

// Sum over the wave, to every lane, all 64 active.  Cross-lane moves of the vector unit take a
// few cycles a step where shuffles through LDS take over a hundred: a step of the coarse solve
// in one workgroup 3.4 -> 3.1 us at 1331 vertices and 1.24 -> 0.95 us at 343, with the
// single-reduction form.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_plus(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
    return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum(double v)
{
    v = dpp_plus<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 has its sum
    v = dpp_plus<0x112, 0xf>(v);
    v = dpp_plus<0x114, 0xf>(v);
    v = dpp_plus<0x118, 0xf>(v);
    v = dpp_plus<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
    v = dpp_plus<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

}  // namespace sem
