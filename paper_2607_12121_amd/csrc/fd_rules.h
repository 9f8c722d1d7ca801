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

// Whether the attention's shares cut (head, query tile) items into pieces that a second pass
// merges.  `tiles` query tiles of every head, `items` of all, `work_head` tile-steps of one head (a
// tile-step: one query tile against 64 keys), `nkv_max` key tiles of the longest request, G workgroups.
//
// A cut costs the pieces' traffic, their extra first tiles and the merge; it gives what the
// longest share gets shorter by.  With at most one item per workgroup that is an item less a
// workgroup's equal part; with more, the last round's excess, less what the power limit takes
// back: a GPU whose idle CUs start working lowers its clock (head dim 128, which draws most:
// 468 items of 512 tile-steps 1697 us whole, 1725 cut, although the longest share is 1024
// against 936; 480 of 128 451 / 470; 384 of 128 414 / 370).  Measured, us, whole / cut with the
// merge (MI355X, 256 CUs; the merge's launch, which an uncut pass pays where it may cut, 3):
//   head dim 128: 12 items of 16 34 / 28, 96 of 16 32 / 41, 192 of 16 41 / 59, 96 of 24 47 / 51,
//     96 of 32 57 / 55, 144 of 32 58 / 67, 96 of 48 77 / 65, 192 of 64 109 / 120, 60 of 64 97 / 64,
//     84 of 512 668 / 336, 228 of 256 426 / 442, 384 of 24 105 / 108, 288 of 48 171 / 140
//   head dim 64: 16 items of 16 23 / 19, 128 of 16 26 / 26, 256 of 16 29 / 33, 96 of 24 33 / 30,
//     192 of 32 42 / 47, 160 of 64 70 / 65, 448 of 16 43 / 49, 384 of 32 77 / 72, 320 of 64 143 / 110
constexpr int kMinShareSteps = 4;   // tile-steps of a share when the work is little: 2, 3, 4, 6 measured 24 / 24 / 21 / 26 us
// `part` = tile-steps per share when cut, rounded up; `margin` tile-steps the gain must exceed that by.
FD_RULE bool attn_cuts(int dh, int items, int heads, long long work_head, int tiles, long long part, int nkv_max, int G,
                       int margin) {
  if (items <= G) {
    // the longest item: every query tile has a tile-step, so one has no more than the rest leaves
    const long long longest = nkv_max < work_head - tiles + 1 ? nkv_max : work_head - tiles + 1;
    const long long gain = longest - (part > kMinShareSteps ? part : kMinShareSteps) - margin;
    // items that are two shares each have no piece beyond those: 128 of 24 50 / 50 us, of 32 63 / 58
    return dh >= 128 ? 8 * gain > (2 * items == G ? 112 : 40 + items) : 40 * gain > 160 + items;
  }
  // Items of one length run in whole rounds; of a mixed batch the longest share is somewhere
  // between its part and one longest item more.
  const long long gain = (work_head == static_cast<long long>(tiles) * nkv_max ? (items + G - 1) / G * nkv_max - part
                                                                               : nkv_max / 3) - margin;
  return dh >= 128 ? 32 * gain > 352 + 3 * part : gain > 6;
}

// Whether a launch may cut: the merge's launch costs an uncut pass 3 to 4 us (head dim 128, 8
// requests of 1024 tokens: 34 us, 38 with it), so it is left out, with the code of the pieces, where
// no number of active rows that a step has in earnest (at least one of every request) leads to a
// cut worth three tile-steps more than that, and up to 12 key tiles (24 items 26.6 us whole, 27.3
// cut at head dim 128; 32 items 19.4 / 18.5, 128 items 19.9 / 22.2 at head dim 64).  The active
// rows are only known on the device.
FD_RULE bool attn_may_cut(int dh, int heads, int requests, long long tokens, int max_request_tokens, int query_tile, int G) {
  const int nkv_max = (max_request_tokens + 63) / 64;
  if (nkv_max <= 12) return false;
  const long long nkv = (tokens + 64LL * requests - 1) / (64LL * requests);   // of a mean request
  const int most = (max_request_tokens + query_tile - 1) / query_tile;
  for (int k = 1; k <= most; ++k) {
    const int tiles = requests * k;
    const long long work_head = tiles * nkv;
    if (attn_cuts(dh, tiles * heads, heads, work_head, tiles, (work_head * heads + G - 1) / G, nkv_max, G, 3)) return true;
  }
  return false;
}

}  // namespace fd
