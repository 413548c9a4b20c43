// What the tile kernel's persistent workgroups and its copies into LDS run through, apart from the kernel so that the host
// can check it without a GPU: the order of the work items, the copies' cursor, and how many workgroups a launch may have.
#pragma once
#include <hip/hip_runtime.h>

namespace dllm {

// The work items are dealt in contiguous runs to the 8 XCDs (workgroups go round-robin to XCDs), inside an XCD round-robin
// to its workgroups.  The it-th item of workgroup `wg`, or -1.
__host__ __device__ __forceinline__ int gt_item(int wg, int n_wg, int it, int n_items) {
  const int per_xcd = (n_items + 7) / 8, iw = (wg >> 3) + it * (n_wg >> 3);
  const int item = (wg & 7) * per_xcd + iw;
  return iw < per_xcd && item < n_items ? item : -1;
}

// The copies' cursor, one per operand, one stage on: k is the 64-deep stage that the next copies fetch, from `first` to the
// end of the item's range [begin, end), then from its beginning up to `first`, then (`take` is run) the stages of nxt, the
// item behind the one that is multiplied.  Past the last item it is the last stage again, fetched and never used.
// (A macro: as an inline function over the same variables it left the 256 x 256 rotary tile 68 bytes of scratch per lane
// instead of 28, and a refresh of 1184 tokens 0.5 % slower.)
#define GT_ADVANCE(k, first, begin, end, nxt, take)                               \
  do {                                                                            \
    k = k + 64 < end ? k + 64 : begin;                                            \
    if (k == first) {                                                             \
      if (nxt.ok) { take; k = first = nxt.k_first; begin = nxt.k_begin; end = nxt.k_end; } \
      else k = (k > begin ? k : end) - 64;                                        \
    }                                                                             \
  } while (0)

// Workgroups of a launch over n_items items, `slots` of which the chip holds at a time.  Copies run up to nsw - 1 stages
// ahead and a workgroup knows one item ahead.  Items of fewer than nsw stages would need more: the cursor would come to
// the next item's end while the one in front of it is still being multiplied, and fetch that item a second time in place
// of the one behind it.  Such launches have a workgroup per item, so that no copies run on into a next one.  (Weights of two stages
// together: nsw is one more than the ring.)
__host__ __device__ inline int gt_workgroups(int n_items, int slots, int stages, int nsw) {
  return n_items < slots || stages < nsw ? (n_items + 7) / 8 * 8 : slots;
}

}  // namespace dllm
