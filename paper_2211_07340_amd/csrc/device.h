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
// The same for a wave of a row-lane launch on a segment of so many columns, if it
// is short.  (In one piece: with a branch of its own at the top of those kernels the
// compiler arranges the sweeps' registers otherwise, and one read of 1,827 rows x
// 158,130 columns takes 725 us instead of 689.)
__device__ __forceinline__ void issue_first_if_short(int32_t segcols) {
  asm volatile(
      "s_cmp_gt_i32 %0, %1\n\t"
      "s_cbranch_scc1 .Llong%=\n\t"
      "s_setprio 3\n"
      ".Llong%=:" ::"s"(segcols),
      "i"(kShortSegment)
      : "scc");
}

}  // namespace sdtw
