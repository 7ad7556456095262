// Data structures shared by the segmented-sort kernels and their host callers.
#pragma once

#include <stdint.h>

namespace aps {

constexpr int kSegBuckets = 32;  // work-list classes: ceil(log2(length))
constexpr int kSegGroups = 6;    // length groups, each sorted by its own kernel configuration

// Control block of the segmented sort (device memory, zero at first).  What k_seg_classify adds up
// (count, done, bad) and what the groups count (head, done2) is zero again when its kernel ends; the rest
// is set by k_seg_classify's last workgroup, so no kernel at the end of a call has to clear it.
struct SegCtl {
  uint32_t count[kSegBuckets];   // segments per length class, while they are counted
  uint32_t start[kSegBuckets];   // first slot of each class in the work order (longest first); class c ends
                                 // where class c - 1 starts (class 0 is empty)
  uint32_t cursor[kSegBuckets];  // fill cursors
  uint32_t done;                 // completion counter of k_seg_classify's last-workgroup pattern
  uint32_t bad;                  // some offsets were invalid, while they are checked
  uint32_t invalid;              // some offsets were invalid: nothing is sorted
  uint32_t pad0;
  uint32_t head[kSegGroups];     // next work item of each length group's kernel
  uint32_t done2[kSegGroups];    // exit counters of each group's kernel
  // long segments (sorted by device-wide passes over one flat tile space)
  unsigned long long long_cursor;  // (long segments << 32) | flat tiles, advanced by k_seg_tiles
  uint32_t long_ctr[4];            // tile claim counters of the four digit passes
};

// A long segment: keys[0..n) sorted in place by device-wide digit passes, through tmp[0..n); its
// tiles are flat tiles [first_tile, first_tile + ntiles) of the batch.  The plan is written by
// k_seg_long_hist from the segment's bucket counts.
enum LongRun : uint32_t { LONG_SKIP = 0, LONG_SORT = 1, LONG_COPY = 2 };
struct LongSeg {
  uint32_t* keys;
  uint32_t* tmp;
  uint32_t n;
  uint32_t first_tile;
  uint32_t ntiles;
  uint32_t counted;     // tiles whose keys are in the bucket counts
  uint32_t run[4];      // LongRun of pass d
  uint32_t rd_tmp[4];   // pass d reads tmp and writes keys (else reads keys, writes tmp)
  uint32_t pad[4];
};

// One unit of work of the persistent sort: sort src[0..n) into dst[0..n) (src == dst allowed),
// using tmp[0..n) as scratch when more than one tile is needed; when spl is not NULL also write
// the P-1 splitters of the n sorted keys spread over P cells.
struct SegDesc {
  const uint32_t* src;
  uint32_t* dst;
  uint32_t* tmp;
  uint32_t* spl;
  uint32_t n;
  uint32_t P;
  uint32_t pad[2];
};

}  // namespace aps
