// Which variant of a kernel a call runs: rules on sizes alone, plain C++ that the
// device code, the host code and a CPU build share.
#pragma once

#ifdef __HIP__
#include <hip/hip_runtime.h>
#define FD_RULE __host__ __device__ __forceinline__
#else
#define FD_RULE inline
#endif

namespace fd {

// The score in one pass, a workgroup per region that writes the region's score itself, or
// regions cut into chunks whose sums a second launch adds up.  `values` = the largest
// region's tokens x channels.  One pass saves the second launch, but reads a region from
// one CU, so a few large regions leave the GPU idle.  Measured, us, cut / one pass: 64
// regions of 8192 values 5.0 / 4.5, of 16384 5.8 / 6.5, of 65536 10.8 / 18.0; 16 of 65536
// 7.8 / 16.1; 140 of 14976 7.1 / 6.6, of 24576 7.8 / 9.3; 256 of 65536 26.1 / 22.9.
FD_RULE bool score_one_pass(int regions, long long values, int cus) {
  if (regions >= 2 * cus || values <= 8192) return true;
  if (values <= 16384) return 2 * regions >= cus;
  return values <= 65536 && 4 * regions >= 3 * cus;
}

}  // namespace fd
