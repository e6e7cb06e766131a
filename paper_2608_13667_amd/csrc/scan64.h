// A wave's scan.
#pragma once

#include <hip/hip_runtime.h>

namespace fka {

// Inclusive sum over the lanes up to this one, in vector-ALU steps (DPP: row_shr, then the sums of the rows
// below by row_bcast 15 and 31); a scan of six shuffles is as many LDS round trips.
__device__ inline int scan64(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

}  // namespace fka
