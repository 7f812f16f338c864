// Stand-alone replay of the default batched selection's order, parts, regions, slot search and
// routes (csrc/batch_queue.h, the kernels' own code), built with the address and
// undefined-behaviour sanitizers by the tests.
//   input: one line "esize grid pool_elems count", then count lines "addr size k".
//   output: "shared T items_of_shared F items N", a line "slot i index first parts region" per slot
//   (region -1: none), and a line "item q slot part route" per work item.
#include <algorithm>
#include <cstdio>
#include <numeric>
#include <vector>

#include "../../paper_1104_2732_amd/csrc/batch_queue.h"

using namespace cps;

int main(int argc, char **argv) {
  if (argc != 2) return 2;
  FILE *f = std::fopen(argv[1], "r");
  if (!f) return 3;
  unsigned esize;
  int grid, count;
  long long pool;
  if (std::fscanf(f, "%u %d %lld %d", &esize, &grid, &pool, &count) != 4) return 4;
  if ((esize != 4 && esize != 8) || grid < 1 || pool < 0 || count < 1 || count > kBatchSortMax) return 5;
  std::vector<uint64_t> addr((size_t)count);
  std::vector<int64_t> size((size_t)count), k((size_t)count);
  for (size_t i = 0; i < (size_t)count; ++i) {
    unsigned long long a;
    long long n, r;
    if (std::fscanf(f, "%llu %lld %lld", &a, &n, &r) != 3) return 6;
    addr[i] = a;
    size[i] = n;
    k[i] = r;
  }
  std::fclose(f);
  // ---- the order: larger size classes first (any order inside a class)
  double all = 0.0;
  for (int64_t n : size) {
    if (bq_class(n) < 0 || bq_class(n) > 255) return 7;
    all += bq_weight(n);
  }
  std::vector<uint32_t> order((size_t)count);
  std::iota(order.begin(), order.end(), 0u);
  std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
    return bq_class(size[x]) > bq_class(size[y]);
  });
  const int64_t part = bq_part(all, grid, esize);
  const uint32_t most = bq_most_units(pool);
  std::vector<uint32_t> first((size_t)count), parts((size_t)count);
  uint32_t at = 0, unit = 0, teams = 0, team_items = 0;
  std::vector<long long> region((size_t)count, -1);
  for (size_t i = 0; i < (size_t)count; ++i) {
    const int64_t n = size[order[i]];
    parts[i] = 1;
    uint32_t units = 0;
    if (bq_shared(n, esize)) {
      parts[i] = bq_parts(n, part);
      units = bq_units(n, parts[i], most, esize);
      teams += 1;
      team_items += parts[i];
      if (bq_fits(unit, units, most, pool)) region[i] = (long long)unit * 64;
    }
    first[i] = at;
    at += parts[i];
    unit += units;
  }
  std::printf("shared %u items_of_shared %u items %u\n", teams, team_items, at);
  for (size_t i = 0; i < (size_t)count; ++i)
    std::printf("slot %zu %u %u %u %lld\n", i, order[i], first[i], parts[i], region[i]);
  // ---- the items
  for (uint32_t q = 0; q < at; ++q) {
    const uint32_t s = bq_slot(q, teams, team_items, [&](uint32_t s0, uint32_t w) {
      uint32_t c = 0;
      for (uint32_t lane = 0; lane < 64; ++lane) {
        const uint32_t t = s0 + lane * w;
        c += t < teams && first[t < teams ? t : 0] <= q ? 1u : 0u;
      }
      return c;
    });
    if (s >= (uint32_t)count) return 8;
    const size_t j = order[s];
    // the kernel's chain: a bad descriptor, too large, in registers, one workgroup's, shared
    const int route = !batch_array_valid(addr[j], size[j], k[j], esize) ? 0
                      : size[j] > kBqMaxN                                ? 1
                      : size[j] <= bq_small_max(esize)                   ? 2
                      : !bq_shared(size[j], esize)                       ? 3
                                                                         : 4;
    std::printf("item %u %u %u %d\n", q, s, q - first[s], route);
  }
  return 0;
}
