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

// What a cut costs, in tile-steps (1.3 us at head dim 64, 1.8 at 128): the extra pieces'
// queries, first tiles and stores, and the merge.  Measured, us per attention, whole / cut:
// head dim 128, 60 items of 64 key tiles 108 / 65, 24 of 16 36 / 31, 192 of 16 47 / 61, 144
// of 2 15 / 31; head dim 64, 12 of 16 26 / 20, 16 of 8 19 / 18, 16 of 4 15 / 17.
constexpr int kCutCost = 7;
constexpr int kMinShareSteps = 4;   // 2, 3, 4 and 6 measured: 24 / 24 / 21 / 26 us for 48 items of 16

// Shares cut items when the longest share gets shorter by more than the pieces' fixed cost;
// otherwise every share is a run of whole items: one of the longest at most while there are items
// for every workgroup no more than once, else up to one more than its part.
FD_RULE bool attn_cuts(int items, long long part, int nkv_max, int G) {
  const long long whole = items <= G ? nkv_max : part + nkv_max;
  return (part > kMinShareSteps ? part : kMinShareSteps) + kCutCost < whole;
}

}  // namespace fd
