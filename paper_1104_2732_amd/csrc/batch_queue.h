// Work order and descriptor checks of the batched selections.  Scalar code shared by the
// batched kernels and the host replays of their queues (tests/cpp), so both take the same
// decisions on the same descriptors.
#pragma once

#include <stdint.h>

#include "cp_state.h"

namespace cps {

constexpr int kBatchSortMax = 4096;  // arrays sorted largest-first in LDS up to this count

// Sort key of array j: its size (clamped to [0, 2^50]) above the complement of its index, so
// that a descending sort puts larger arrays first and, among equal sizes, lower indices first.
// Keys of the padding slots of the sort (j >= count) are 0, below every array's key.
CPS_HD inline uint64_t lpt_key(int64_t size, int64_t j) {
  int64_t sz = size < 0 ? 0 : size;
  if (sz > ((int64_t)1 << 50)) sz = (int64_t)1 << 50;
  return ((uint64_t)sz << 12) | (uint64_t)(kBatchSortMax - 1 - j);
}

CPS_HD inline int64_t lpt_index(uint64_t key) {
  return (int64_t)(kBatchSortMax - 1 - (key & (uint64_t)(kBatchSortMax - 1)));
}

// One compare-exchange of the descending bitonic network over order[0..m) (m a power of two),
// at stage (kk, jj), for element i: a no-op unless i is the lower index of its pair.
CPS_HD inline void bitonic_exchange(uint64_t *order, int64_t i, int64_t jj, int64_t kk) {
  const int64_t p = i ^ jj;
  if (p <= i) return;
  const uint64_t x0 = order[i], x1 = order[p];
  const bool desc = (i & kk) == 0;
  if (desc ? (x0 < x1) : (x0 > x1)) {
    order[i] = x1;
    order[p] = x0;
  }
}

// Workgroups of one array: arrays of more than `chunk` elements are split into contiguous
// parts of about `chunk` elements, one workgroup each, at most `tmax` of them (1 when teams
// are off: tmax <= 1 or chunk <= 0).  Non-increasing in the size, so in the largest-first
// order the arrays with more than one workgroup come first.
CPS_HD inline int32_t team_blocks(int64_t size, int64_t chunk, int32_t tmax) {
  if (tmax <= 1 || chunk <= 0 || size <= chunk) return 1;
  const int64_t b = (size + chunk - 1) / chunk;
  return b > tmax ? tmax : (int32_t)b;
}

// After the largest-first sort, slot j of the order holds (first work item of the array in
// slot j) << 32 | (its index): the work items are the arrays' workgroup parts in that order,
// the B parts of one array consecutive.  Work item q belongs to the last slot whose first item
// is <= q (a binary search over the slots), as part q - first.
CPS_HD inline uint64_t item_entry(int64_t first_item, int64_t index) {
  return ((uint64_t)first_item << 32) | (uint64_t)index;
}
CPS_HD inline int64_t item_first(uint64_t e) { return (int64_t)(e >> 32); }
CPS_HD inline int64_t item_index(uint64_t e) { return (int64_t)(e & 0xffffffffull); }

// The slot of work item q among slots [0, count) (entries from item_entry, first items
// non-decreasing, slot 0's first item 0).
CPS_HD inline int64_t item_slot(const uint64_t *order, int64_t count, int64_t q) {
  int64_t lo = 0, hi = count - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) / 2;
    if (item_first(order[mid]) <= q) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// An array descriptor the kernel can run: a non-null pointer aligned to the element size,
// at least one element and a rank in [1, n].  Anything else gets status BADARG and is never
// read.
CPS_HD inline bool batch_array_valid(uint64_t addr, int64_t n, int64_t k, uint32_t esize) {
  return addr != 0 && n >= 1 && k >= 1 && k <= n && (addr % esize) == 0;
}

// ------------------------------------------------------------------ the default selection
// (batchq.hip).  esize: 4 or 8, the element's bytes.

constexpr int64_t kBqMaxN = (int64_t)1 << 31;  // larger arrays go to the general kernel
constexpr int kBqBins = 2048;                  // key bins of one part of a shared array

// Up to here one workgroup's registers hold an array.
CPS_HD inline constexpr int64_t bq_small_max(uint32_t esize) { return esize == 4 ? 16384 : 8192; }
// Arrays from this many elements on are shared by workgroups: smaller ones keep their inside
// elements in LDS.  The interval holds 3.6 % of the elements at most with float32's large sample
// (4.1 % with float64's), 7.1 % with the small one: 9300 of 12288 places (2700 of 6144).
CPS_HD inline constexpr int64_t bq_share(uint32_t esize) { return (int64_t)1 << (esize == 4 ? 18 : 16); }
CPS_HD inline bool bq_shared(int64_t n, uint32_t esize) { return n >= bq_share(esize) && n <= kBqMaxN; }
// A shared array's region of the pool: room for a sixteenth of its elements (the interval holds
// 3.6 % of them, of float64 4.1 %, give or take 5 % of that), whose last places take each part's sum
// of the elements below the interval (two doubles), then the key bins of each part.  (A batch of
// 2^30 elements in parts of 2^20 fills the default pool to the last place.)  Arrays that find no region are left to the general kernel unread.
CPS_HD inline int64_t bq_room(int64_t n) { return (n / 16 + 63) / 64 * 64; }
CPS_HD inline int64_t bq_copy_room(int64_t n, uint32_t parts, uint32_t esize) {
  return bq_room(n) - (int64_t)parts * (int64_t)(2 * sizeof(double) / esize);
}
CPS_HD inline int64_t bq_region(int64_t n, uint32_t parts, uint32_t esize) {
  return bq_room(n) + (int64_t)parts * (int64_t)(kBqBins * sizeof(uint32_t) / esize);
}

// Eight size classes per power of two; the limit of sharing is a class limit, so the shared
// arrays come before all others (what is left to the general kernel comes last).
CPS_HD inline int bq_class(int64_t n) {
  if (n < 8 || n > kBqMaxN) return n < 0 || n > kBqMaxN ? 0 : (int)n;
  const int e = 63 - __builtin_clzll((unsigned long long)n);
  return (e - 2) * 8 + (int)((n >> (e - 3)) & 7);  // (at most 239)
}

// A shared array is cut into parts of half a workgroup's share of all elements (at least the limit
// of sharing), so that the chip has two items per workgroup or more of its largest arrays.
CPS_HD inline double bq_weight(int64_t n) { return n > 0 && n <= kBqMaxN ? (double)n : 0.0; }
CPS_HD inline int64_t bq_part(double all, int grid, uint32_t esize) {
  const int64_t half = (int64_t)(all / (2.0 * grid));
  return half > bq_share(esize) ? half : bq_share(esize);
}
CPS_HD inline uint32_t bq_parts(int64_t n, int64_t part) { return (uint32_t)((n + part - 1) / part); }

// Regions in units of 64 elements, at most `most` (which no region gets): 4096 slots of at most 2^20
// - 1 units stay below 2^32.
CPS_HD inline uint32_t bq_most_units(int64_t pool_elems) {
  const uint64_t u = (uint64_t)pool_elems / 64;
  return (uint32_t)(u < (1u << 20) - 2 ? u : (1u << 20) - 2) + 1;
}
CPS_HD inline uint32_t bq_units(int64_t n, uint32_t parts, uint32_t most, uint32_t esize) {
  const int64_t u = bq_region(n, parts, esize) / 64;
  return u < (int64_t)most ? (uint32_t)u : most;
}
CPS_HD inline bool bq_fits(uint32_t at, uint32_t units, uint32_t most, int64_t pool_elems) {
  return ((int64_t)at + units) * 64 <= pool_elems && units < most;
}

// The slot of work item q: the shared arrays' items come first, and the slot is the last shared one
// whose first item is not after q; every later item is the next slot's only one.  `count(s, w)`:
// how many of the 64 slots s, s + w, s + 2 w, ... are shared with a first item not after q (a
// wavefront's ballot).
template <typename Count>
CPS_HD inline uint32_t bq_slot(uint32_t q, uint32_t teams, uint32_t team_items, Count &&count) {
  uint32_t slot = q - team_items + teams;
  if (q < team_items) {
    slot = (count(0u, 64u) - 1) * 64;
    slot += count(slot, 1u) - 1;
  }
  return slot;
}

}  // namespace cps
