// Sum over a wave of 64 lanes by DPP row shifts and row broadcasts (an
// exchange through LDS costs a few hundred cycles more).
#pragma once

#include <hip/hip_runtime.h>

namespace ctqw {

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_part(double v) {
    return __builtin_amdgcn_update_dpp(0.0, v, CTRL, ROWS, 0xF, true);
}

// Sum over the wave, valid in lane 63.
__device__ __forceinline__ double wave_sum_last(double v) {
    v += dpp_part<0x111, 0xF>(v);   // row_shr:1
    v += dpp_part<0x112, 0xF>(v);   // row_shr:2
    v += dpp_part<0x114, 0xF>(v);   // row_shr:4
    v += dpp_part<0x118, 0xF>(v);   // row_shr:8
    v += dpp_part<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v += dpp_part<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

}  // namespace ctqw
