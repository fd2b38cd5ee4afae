// Wave-level helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace moe {

// Inclusive prefix sum over a wave with DPP row shifts (each 16-lane row), then the
// row totals read from lanes 15, 31, 47 and 63.  Returns the wave total.
__device__ inline int wave_inclusive_scan(int &v, int lane)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    const int t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31),
              t2 = __builtin_amdgcn_readlane(v, 47), t3 = __builtin_amdgcn_readlane(v, 63);
    const int row = lane >> 4;
    v += (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
    return t0 + t1 + t2 + t3;
}

// A chunk record, the same for every lane, in scalar registers.
__device__ inline int4 chunk_record(const int4 *recs, int i)
{
    const int4 r = recs[i];
    return make_int4(__builtin_amdgcn_readfirstlane(r.x), __builtin_amdgcn_readfirstlane(r.y),
                     __builtin_amdgcn_readfirstlane(r.z), 0);
}

}  // namespace moe
