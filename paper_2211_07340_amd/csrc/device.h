// Device code shared by the library's kernels.
#pragma once
#include "common.h"

namespace sdtw {

// For kernels that are over in tens or hundreds of microseconds, at their start:
// their waves issue before those of long launches on other HIP streams.  A SIMD
// issues from its oldest wave first, so waves that join three of an alignment that
// takes it whole get a thirtieth of their speed (16 reads' normalisation: 0.04 ms
// alone, 1.1 ms beside chunks on 10 M columns, 0.06 so).
__device__ __forceinline__ void issue_first() { __builtin_amdgcn_s_setprio(3); }

}  // namespace sdtw
