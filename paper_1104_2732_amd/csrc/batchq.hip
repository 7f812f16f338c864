// The default batched selection: every array is read once.
//
// The general batched kernel (batched_kernel.h) gives an array to one workgroup, whose chain of sample,
// pass 0, histogram passes, gather and radix select costs ~40 us however small the array is, and
// whose LDS leaves one workgroup per CU, so nothing hides it.  Here:
//
// * an array of up to 16384 float32 (8192 float64) elements is held in one workgroup's registers and
//   selected there;
// * a larger one is read once against a likely interval of its rank (sample quantiles, as the
//   single-array filter, quick.hip): elements below are counted, those inside (8 % at most) kept
//   in LDS, and when the counts prove the interval the select runs among them;
// * an array of 2^18 float32 (2^16 float64) elements or more is cut into parts of at least that
//   many (half a workgroup's share of the batch where that is more), taken by any workgroups.  All
//   parts take the same sample and so the same interval; each adds its counts to the array's
//   record and its inside elements to the array's region of a pool, and the last to arrive
//   selects among them.  Few large arrays then fill the chip like many small ones.
//
// An array whose counts do not prove the interval, or whose inside elements found no room (or whose
// region found none in the pool), goes on a list that the general kernel works through afterwards,
// so no result depends on a sample.
//
// Two workgroups of 512 threads per CU: one's latencies (sample 9 us, ends 4, select 6 to 12, next
// item 3) hide behind the other's streaming.  Calls: 4096 float32 arrays of 10^3 to 10^6 elements
// (2.37 GB) 597 us, the general kernel 1156; 64 arrays of 2^22 elements 333 us, the general kernel
// 1592; of these the order kernel is 22 and 6, the general kernel's empty launch 4.  The
// comparisons that follow are of the selection's kernel alone, 576 and 314 us when they were made.
// Three smaller workgroups (half the tile, spills): 690 us for the 4096 arrays.  Of the 576, a
// workgroup spends 416 streaming, at the rate that reads mixed with the shared arrays' copies
// reach (60 us of it is the copies), 70 on samples and their ends, 42 on selects, 19 between
// items.  Comparing and appending element by element instead of by vectors (RowFilter): 690 us.
// With the key bins counted by a walk over the kept elements instead of on the way: 580 and 355
// us (the last array's select alone 100 us).  Many large float64 arrays gain least, as their
// copies are the widest writes: calls of 512 arrays of 2^20 elements 952 us (general 958; with a
// sample of 8192 for 12288, 970).
#include "batch_queue.h"
#include "cps_quick.h"

namespace cps {

constexpr int kBqBlock = 512;
constexpr int kBqWaves = kBqBlock / kWave;
template <typename T> constexpr int kBqPer = sizeof(T) == 4 ? 32 : 16;  // keys per lane, small arrays
template <typename T> constexpr int kBqSmall = kBqBlock * kBqPer<T>;
static_assert(kBqSmall<float> == bq_small_max(4) && kBqSmall<double> == bq_small_max(8), "the route's line");
constexpr int kBqSmpA = 8;                       // samples per lane: 4096 in all, or
template <typename T> constexpr int kBqSmpB = sizeof(T) == 4 ? 32 : 24;  // 16384 (12288)
constexpr int kBqU = 4;                          // vectors per lane and tile
constexpr size_t kBqListBytes = 49152;           // LDS for the inside elements
constexpr double kBqDev = 4.5;  // deviations of the interval's ends: a miss in 10^5 arrays
template <typename T> CPS_HD inline bool bq_big_sample(int64_t n) { return n >= bq_share(sizeof(T)) / 2; }
constexpr int kBqBinsLog2 = quick_bins_log2(kBqBlock);
static_assert(kBqBins == 4 * kBqBlock, "four bins per thread");

// ------------------------------------------------------------------ the order of the arrays

// One workgroup: the arrays by size class, larger first, with their work items.  A shared array is
// cut into parts of half a workgroup's share of all elements (at least kBqShare), so that the
// chip has two items per workgroup or more of its largest arrays.
template <typename T>
__global__ __launch_bounds__(1024) void batchq_order_kernel(BatchqArgs<T> a, int grid) {
  constexpr int BLOCK = 1024, PER = kBatchSortMax / BLOCK;
  __shared__ uint32_t cls[256];
  __shared__ uint32_t wsum[BLOCK / kWave];
  __shared__ uint32_t order[kBatchSortMax], first[kBatchSortMax], unit[kBatchSortMax], npart[kBatchSortMax];
  __shared__ int64_t size[kBatchSortMax];
  __shared__ uint32_t total[3];  // items, shared arrays, their items
  __shared__ double wtot[BLOCK / kWave];
  const int tid = threadIdx.x;
  const int count = (int)a.count;
  if (tid < 256) cls[tid] = 0u;
  if (tid < 3) total[tid] = 0u;
  __syncthreads();
  int64_t n[PER];
  double all = 0.0;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int j = tid + p * BLOCK;
    n[p] = a.sizes[j < count ? j : 0];
  }
#pragma unroll
  for (int p = 0; p < PER; ++p)
    if (tid + p * BLOCK < count) {
      size[tid + p * BLOCK] = n[p];
      atomicAdd(&cls[255 - bq_class(n[p])], 1u);
      all += bq_weight(n[p]);
    }
  all = wave_sum(all);
  if (tid % kWave == 0) wtot[tid / kWave] = all;
  __syncthreads();
  all = 0.0;
  for (int w = 0; w < BLOCK / kWave; ++w) all += wtot[w];
  const int64_t part = bq_part(all, grid, sizeof(T));
  const uint32_t c = tid < 256 ? cls[tid] : 0u;
  const uint32_t at = block_scan_u32<BLOCK>(c, wsum);
  if (tid < 256) cls[tid] = at;
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int j = tid + p * BLOCK;
    if (j < count) order[atomicAdd(&cls[255 - bq_class(n[p])], 1u)] = (uint32_t)j;
  }
  __syncthreads();
  // slots tid * PER ..: first items and regions (in units of 64 elements; what passes the pool's
  // end gets none; 4096 slots of at most 2^20 - 1 units stay below 2^32)
  uint32_t parts[PER], units[PER], sp = 0, su = 0, st = 0, sti = 0;
  const uint32_t most = bq_most_units(a.pool_elems);
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const int i = tid * PER + p;
    const int64_t m = i < count ? size[order[i]] : 0;
    parts[p] = i < count ? 1u : 0u;
    units[p] = 0;
    if (i < count && bq_shared(m, sizeof(T))) {
      parts[p] = bq_parts(m, part);
      units[p] = bq_units(m, parts[p], most, sizeof(T));
      st += 1;
      sti += parts[p];
    }
    sp += parts[p];
    su += units[p];
  }
  uint32_t f = block_scan_u32<BLOCK>(sp, wsum);
  uint32_t u = block_scan_u32<BLOCK>(su, wsum);
  if (st) {
    atomicAdd(&total[1], st);
    atomicAdd(&total[2], sti);
  }
  if (tid == BLOCK - 1) total[0] = f + sp;
#pragma unroll
  for (int p = 0; p < PER; ++p) {
    const bool fits = bq_fits(u, units[p], most, a.pool_elems);
    first[tid * PER + p] = f;
    unit[tid * PER + p] = fits ? u : ~0u;
    npart[tid * PER + p] = parts[p];
    f += parts[p];
    u += units[p];
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PER; ++p) {  // (neighbouring slots by neighbouring lanes)
    const int i = tid + p * BLOCK;
    if (i < count) {
      const uint32_t j = order[i];
      BatchqSlot s;
      s.x = (uint64_t)(uintptr_t)a.ptrs[j];
      s.n = size[j];
      s.k = a.ks[j];
      s.index = j;
      s.first = first[i];
      s.parts = npart[i];
      s.pad = 0u;
      a.slot[i] = s;
      if (bq_shared(s.n, sizeof(T))) {
        BatchqRec r = {};
        r.region = unit[i] != ~0u ? (int64_t)unit[i] * 64 : -1;
        a.rec[i] = r;
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    a.ctl->items = total[0];
    a.ctl->teams = total[1];
    a.ctl->team_items = total[2];
    a.ctl->queue = 0u;
    a.ctl->redo = 0u;
  }
}

// ------------------------------------------------------------------ the selection

template <typename T> struct BqShared {
  RegSelShared<kBqBlock> rs;
  T list[kBqWaves][kBqListBytes / sizeof(T) / kBqWaves];
  typename Traits<T>::Vec rows[kBqWaves][RowFilter<T>::kRows];
  uint32_t hist[kBqBins];
  typename Traits<T>::Key fin[kWalkFinal];
  uint64_t count[3];  // below, the ends' repeated values
  Sum2 sums[kBqWaves];
  uint32_t held[kBqWaves], over, item, last;
  BatchqSlot slot;
};

__device__ inline int64_t uniform_i64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <typename T>
__device__ inline void bq_redo(const BatchqArgs<T> &a, uint32_t j) {
  const uint32_t at = __hip_atomic_fetch_add(&a.ctl->redo, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  a.redo[at] = j;
}

template <typename T, bool SUM>
__device__ inline void bq_write(const BatchqArgs<T> &a, uint32_t j, typename Traits<T>::Key key,
                                int64_t less, int64_t equal, Sum2 below, int64_t n, int64_t k,
                                int32_t status) {
  write_key<T>(a.out + j, key, less, equal, n, 1, status);
  if (SUM)
    a.ksum[j] = status != ST_OK
                    ? __builtin_nan("")
                    : value(sum2(below, product2((double)(k - less), (double)(Traits<T>::unkey(key) + T(0)))));
}

// An array of at most 512 PER elements.
template <typename T, int PER, bool SUM>
__device__ inline void bq_small(const BatchqArgs<T> &a, uint32_t jj, const T *x, int n, int64_t k,
                                BqShared<T> &sh) {
  using Key = typename Traits<T>::Key;
  const int tid = threadIdx.x;
  const CPS_GLOBAL T *xg = (const CPS_GLOBAL T *)x;
  T v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = tid + j * kBqBlock;
    v[j] = xg[i < n ? i : 0];  // (past the end: the first element again)
  }
  bool nan = false;
  Key mn = (Key)~(Key)0, mx = 0, key[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    nan = nan || !(v[j] == v[j]);
    key[j] = Traits<T>::key(v[j]);
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
    if (tid + j * kBqBlock >= n) key[j] = (Key)~(Key)0;
  }
  nan = block_key_range<kBqBlock>(mn, mx, nan, sh.rs);
  if (nan) {  // (uniform)
    if (tid == 0) bq_write<T, SUM>(a, jj, 0, 0, 0, Sum2{}, n, k, ST_NAN);
    return;
  }
  const RegSel<Key> r =
      regs_select<T, kBqBlock, PER>(key, (uint32_t)k, (uint32_t)n, mn, mx, sh.hist, sh.rs);
  Sum2 below = {0.0, 0.0};
  if (SUM) {
#pragma unroll
    for (int j = 0; j < PER; ++j) below.hi += key[j] < r.key ? (double)Traits<T>::unkey(key[j]) : 0.0;
    below = block_sum2<kBqBlock>(below, sh.sums);
  }
  if (tid == 0) bq_write<T, SUM>(a, jj, r.key, r.less, r.equal, below, n, k, ST_OK);
}

// The likely interval from 512 PER samples (runs of kPropRun neighbours at even distances, as
// 16-byte vectors); false: they hold NaN.
template <typename T, int PER>
__device__ inline bool bq_ends(const Span<T> &sp, int64_t n, int64_t k, BqShared<T> &sh,
                               SampleEnds<typename Traits<T>::Key> &e) {
  using Key = typename Traits<T>::Key;
  using Vec = typename Traits<T>::Vec;
  constexpr int V = Traits<T>::kVec, S = kBqBlock * PER, RV = kPropRun / V;
  const int tid = threadIdx.x;
  const int64_t stride = sp.nvec / (S / kPropRun);
  Vec v[PER / V];
#pragma unroll
  for (int j = 0; j < PER / V; ++j) {
    const int i = tid + j * kBqBlock;
    v[j] = sp.V[(int64_t)(i / RV) * stride + i % RV];
  }
  bool nan = false;
  Key mn = (Key)~(Key)0, mx = 0, key[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const T w = v[j / V][j % V];
    nan = nan || !(w == w);
    key[j] = Traits<T>::key(w);
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
  }
  if (block_key_range<kBqBlock>(mn, mx, nan, sh.rs)) return false;
  e = sample_ends<T, kBqBlock, PER>(key, mn, mx, n, k, kBqDev, sh.hist, sh.rs);
  return true;
}

// One part (of `parts`) of an array that does not fit the registers; rec: a shared array's record.
template <typename T, bool SUM>
__device__ inline void bq_large(const BatchqArgs<T> &a, uint32_t jj, const T *x, int64_t n, int64_t k,
                                uint32_t part, uint32_t parts, BatchqRec *rec, BqShared<T> &sh) {
  using Key = typename Traits<T>::Key;
  using Vec = typename Traits<T>::Vec;
  constexpr int V = Traits<T>::kVec, U = kBqU, BLOCK = kBqBlock;
  constexpr uint32_t kSeg = (uint32_t)(kBqListBytes / sizeof(T) / kBqWaves);  // places per wavefront
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (rec && rec->region < 0) {  // (uniform)
    if (tid == 0 && part == 0) bq_redo<T>(a, jj);
    return;
  }
  SampleEnds<Key> e;
  const Span<T> sp = make_span(x, n);
  const bool num = bq_big_sample<T>(n) ? bq_ends<T, kBqSmpB<T>>(sp, n, k, sh, e)
                                       : bq_ends<T, kBqSmpA>(sp, n, k, sh, e);
  if (!num) {  // (uniform, and the same in every part)
    if (tid == 0 && part == 0) bq_write<T, SUM>(a, jj, 0, 0, 0, Sum2{}, n, k, ST_NAN);
    return;
  }
  RowFilter<T> f(e, sh.rows[wv]);
  const int64_t region = rec ? rec->region : 0, room = bq_copy_room(n, parts, sizeof(T));
  CPS_GLOBAL T *z = (CPS_GLOBAL T *)(a.pool + region);
  if (tid < 3) sh.count[tid] = 0ull;
  if (tid == 0) sh.over = 0u;  // (1: no room; 2: NaN)
  *reinterpret_cast<uint4 *>(&sh.hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
  const int shift = range_shift((uint64_t)(e.ib - e.ia), kBqBinsLog2);
  __syncthreads();
  uint32_t held = 0;  // in the wavefront's list
  double sum = 0.0;  // per lane: of the elements below the interval
  // the wavefront's elements to the array's region (a shared array only)
  auto flush = [&]() {
    unsigned long long at = 0;
    if (lane == 0)
      at = __hip_atomic_fetch_add(&rec->cursor, (uint64_t)held, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t off = (int64_t)__shfl(at, 0);
    __builtin_amdgcn_wave_barrier();
    if (off + held <= room) {
      for (uint32_t i = lane; i < held; i += kWave) z[off + i] = sh.list[wv][i];
    } else if (lane == 0) {
      atomicOr(&sh.over, 1u);
    }
    __builtin_amdgcn_wave_barrier();
    held = 0;
  };
  bool bad = false;
  auto put = [&](T v, uint64_t m) {
    if (__builtin_amdgcn_inverse_ballot_w64(m)) {
      const uint32_t at = held + lane_rank(m);  // (what finds no place overwrites the last)
      sh.list[wv][at < kSeg ? at : kSeg - 1] = v;
      const bool num = v == v;
      bad = bad | !num;
      if (num) atomicAdd(&sh.hist[(uint32_t)((Traits<T>::key(v) - e.ia) >> shift)], 1u);
    }
    held += popc(m);
  };
  auto add = [&](const Vec &v, bool ok) {
#pragma unroll
    for (int j = 0; j < V; ++j) sum += ok && v[j] < f.va ? (double)v[j] : 0.0;
  };
  // a tile's at most, with what the filter held and the edges
  constexpr uint32_t kTile = (uint32_t)(V * (U + 1) + 1) * kWave;
  static_assert(kTile < kSeg, "room for a tile after a flush");
  const int64_t v0 = sp.nvec * part / parts, v1 = sp.nvec * (part + 1) / parts;
  constexpr int64_t step = (int64_t)BLOCK * U;
  int64_t base = v0;
  Vec cur[U];
  auto load = [&](Vec(&w)[U], int64_t at) {  // (places past the end: the part's first again)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t vi = at + u * BLOCK + tid;
      w[u] = __builtin_nontemporal_load(&sp.V[vi < v1 ? vi : v0]);
    }
  };
  load(cur, base);
  // Every pass issues the next tile's loads: a conditional load would make the wait before the
  // current tile's use one for the next tile's first load as well.
  for (; base + 2 * step <= v1; base += step) {
    Vec nxt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) nxt[u] = __builtin_nontemporal_load(&sp.V[base + step + u * BLOCK + tid]);
    if (rec && held > kSeg - kTile) flush();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      f.row(cur[u], ~0ull, put);
      if (SUM) add(cur[u], true);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
  }
  for (; base < v1; base += step) {  // the last one or two tiles
    if (rec && held > kSeg - kTile) flush();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool valid = base + u * BLOCK + tid < v1;
      f.row(cur[u], ballot(valid), put);
      if (SUM) add(cur[u], valid);
    }
    load(cur, base + step);
  }
  if (f.held > 0) f.drain(f.held, put);
  if (sp.nedge > 0 && part == 0 && wv == 0) {  // the unaligned head and tail
    const uint64_t ok = (1ull << sp.nedge) - 1ull;
    const T v = sp.W[lane < sp.nedge ? edge_index(sp, lane) : 0];
    put(v, ok & ~f.outside(v, ok));
    if (SUM) sum += lane < sp.nedge && v < f.va ? (double)v : 0.0;
  }
  if (held > kSeg) {
    if (lane == 0) atomicOr(&sh.over, 1u);
    held = 0;
  }
  if (ballot(bad) != 0 && lane == 0) atomicOr(&sh.over, 2u);
  if (rec && held > 0) flush();
  Sum2 blw = {sum, 0.0};  // (per thread, summed over the workgroup at the end)
  if (lane == 0) {
    sh.held[wv] = held;
    atomicAdd((unsigned long long *)&sh.count[0], (unsigned long long)(f.below - f.ea));
    if (f.ea) atomicAdd((unsigned long long *)&sh.count[1], (unsigned long long)f.ea);
    if (f.eb) atomicAdd((unsigned long long *)&sh.count[2], (unsigned long long)f.eb);
  }
  __syncthreads();
  int64_t lt = (int64_t)sh.count[0], ca = (int64_t)sh.count[1], cb = (int64_t)sh.count[2], inner = 0;
  uint32_t over = sh.over;
  uint32_t h[4];
  {
    const uint4 q = *reinterpret_cast<const uint4 *>(&sh.hist[4 * tid]);
    h[0] = q.x;
    h[1] = q.y;
    h[2] = q.z;
    h[3] = q.w;
  }
  if (rec) {
    uint4 *bins = reinterpret_cast<uint4 *>(a.pool + region + bq_room(n));
    Sum2 *psum = reinterpret_cast<Sum2 *>(a.pool + region + room);
    if (parts > 1) {
      bins[(int64_t)part * kBqBlock + tid] = uint4{h[0], h[1], h[2], h[3]};
      if (SUM) blw = block_sum2<BLOCK>(blw, sh.sums);
      if (SUM && tid == 0) psum[part] = blw;
      __syncthreads();
    }
    if (tid == 0) {
      if (lt) __hip_atomic_fetch_add(&rec->lt, (uint64_t)lt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (ca) __hip_atomic_fetch_add(&rec->ea, (uint64_t)ca, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (cb) __hip_atomic_fetch_add(&rec->eb, (uint64_t)cb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (over) __hip_atomic_fetch_or(&rec->over, over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t p = atomic_add_release(&rec->arrived, 1u);
      sh.last = p == parts - 1 ? 1u : 0u;
      if (sh.last) fence_acquire();
    }
    __syncthreads();
    if (!sh.last) return;
    lt = (int64_t)load_relaxed(&rec->lt);
    ca = (int64_t)load_relaxed(&rec->ea);
    cb = (int64_t)load_relaxed(&rec->eb);
    inner = (int64_t)load_relaxed(&rec->cursor);
    over = load_relaxed(&rec->over);
    if (parts > 1) {
      h[0] = h[1] = h[2] = h[3] = 0u;
      for (uint32_t p = 0; p < parts; p += 8) {
        uint4 w[8];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
          w[i] = bins[(int64_t)(p + i < parts ? p + i : p) * kBqBlock + tid];
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i)
          if (p + i < parts) {
            h[0] += w[i].x;
            h[1] += w[i].y;
            h[2] += w[i].z;
            h[3] += w[i].w;
          }
      }
    }
    if (SUM && parts > 1) {
      blw = Sum2{0.0, 0.0};
      for (uint32_t p = tid; p < parts; p += BLOCK) blw = sum2(blw, psum[p]);
    }
  } else {
    for (int w = 0; w < kBqWaves; ++w) inner += sh.held[w];
  }
  const int64_t r = k - lt;
  const bool nan = (over & 2u) != 0;
  if (!nan && (over || r < 1 || r > ca + inner + cb)) {  // (uniform)
    if (tid == 0) bq_redo<T>(a, jj);
    return;
  }
  // the inside elements: the rank's if it is there
  const int64_t ri = r - ca;
  const int64_t rank = ri < 1 ? 1 : (ri > inner ? inner : ri);
  Key key = e.ka;
  int64_t less = 0, equal = 0;
  if (inner > 0 && !nan) {
    auto seg_walk = [&](auto &&one) {
      for (uint32_t i = lane; i < (held + kWave - 1) / kWave * kWave; i += kWave)
        one(sh.list[wv][i], i < held);
    };
    const CPS_GLOBAL Vec *zv = (const CPS_GLOBAL Vec *)z;  // (regions begin at multiples of 64)
    const int64_t nv = (inner + V - 1) / V;
    auto region_walk = [&](auto &&one) {
      constexpr int RU = 8;
      for (int64_t b = 0; b < nv; b += (int64_t)RU * BLOCK) {
        Vec w[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const int64_t i = b + u * BLOCK + tid;
          w[u] = zv[i < nv ? i : 0];
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          const int64_t i = (b + u * BLOCK + tid) * V;
#pragma unroll
          for (int j = 0; j < V; ++j) one(w[u][j], i + j < inner);
        }
      }
    };
    // (SUM: the inside elements below the key, all of them when the rank is above, none when below)
    double lsum = 0.0;
    auto add_inside = [&](T v, bool ok) {
      lsum += ok && (ri > inner || Traits<T>::key(v) < key) ? (double)v : 0.0;
    };
    if (rec) {
      walk_select<T, BLOCK>(region_walk, h, rank, e.ia, e.ib, sh.hist, sh.fin, sh.rs, key, less, equal);
      if (SUM) region_walk(add_inside);
    } else {
      walk_select<T, BLOCK>(seg_walk, h, rank, e.ia, e.ib, sh.hist, sh.fin, sh.rs, key, less, equal);
      if (SUM) seg_walk(add_inside);
    }
    if (SUM) blw = sum2(blw, Sum2{lsum, 0.0});
  }
  if (SUM) blw = block_sum2<BLOCK>(blw, sh.sums);
  if (tid == 0) {
    // at the lower end, inside or at the upper end
    if (SUM && ri >= 1 && ca) blw = sum2(blw, product2((double)ca, (double)f.va));
    if (ri < 1) {
      key = e.ka;
      less = lt;
      equal = ca;
    } else {
      less = lt + ca + (ri <= inner ? less : inner);
      key = ri <= inner ? key : e.kb;
      equal = ri <= inner ? equal : cb;
    }
    bq_write<T, SUM>(a, jj, key, less, equal, blw, n, k, nan ? ST_NAN : (equal ? ST_OK : ST_INTERNAL));
  }
}

template <typename T, bool SUM>
__global__ __launch_bounds__(kBqBlock, 4) void batchq_kernel(BatchqArgs<T> a) {
  __shared__ BqShared<T> sh;
  const int tid = threadIdx.x, lane = tid % kWave;
  const uint32_t items = a.ctl->items, teams = a.ctl->teams, team_items = a.ctl->team_items;
  auto take = [&]() -> uint32_t {
    return __hip_atomic_fetch_add(&a.ctl->queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  uint32_t next = 0;  // (thread 0: the next item, taken while this one runs)
  if (tid == 0) next = take();
  for (;;) {
    if (tid < kWave) {
      const uint32_t q = (uint32_t)__builtin_amdgcn_readfirstlane((int)next);
      const uint32_t slot = bq_slot(q, teams, team_items, [&](uint32_t s, uint32_t w) {
        const uint32_t t = s + lane * w;
        return popc(ballot(t < teams && a.slot[t < teams ? t : 0].first <= q));
      });
      if (lane == 0) {
        sh.item = q;
        if (q < items) {
          sh.slot = a.slot[slot];
          sh.slot.pad = slot;
        }
      }
    }
    __syncthreads();
    if (sh.item >= items) break;
    if (tid == 0) next = take();
    const uint32_t j = sh.slot.index, part = sh.item - sh.slot.first, parts = sh.slot.parts;
    const T *x = (const T *)uniform_ptr((const T *)(uintptr_t)sh.slot.x);
    const int64_t n = uniform_i64(sh.slot.n), k = uniform_i64(sh.slot.k);
    if (!batch_array_valid((uint64_t)(uintptr_t)x, n, k, (uint32_t)sizeof(T))) {
      if (tid == 0 && part == 0) {
        cps_result r = {};
        r.status = ST_BADARG;
        a.out[j] = r;
        if (SUM) a.ksum[j] = __builtin_nan("");
      }
    } else if (n > kBqMaxN) {
      if (tid == 0) bq_redo<T>(a, j);
    } else if (n <= kBqSmall<T> / 4) {
      bq_small<T, kBqPer<T> / 4, SUM>(a, j, x, (int)n, k, sh);
    } else if (n <= kBqSmall<T>) {
      bq_small<T, kBqPer<T>, SUM>(a, j, x, (int)n, k, sh);
    } else {
      bq_large<T, SUM>(a, j, x, n, k, part, parts, bq_shared(n, sizeof(T)) ? a.rec + sh.slot.pad : nullptr, sh);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ launchers

size_t batchq_bytes() {
  return sizeof(BatchqCtl) +
         kBatchSortMax * (sizeof(BatchqSlot) + sizeof(BatchqRec) + sizeof(uint32_t));
}

template <typename T>
hipError_t launch_batchq(const BatchqArgs<T> &a, int grid, hipStream_t stream) {
  batchq_order_kernel<T><<<1, 1024, 0, stream>>>(a, grid);
  if (a.ksum) batchq_kernel<T, true><<<grid, kBqBlock, 0, stream>>>(a);
  else batchq_kernel<T, false><<<grid, kBqBlock, 0, stream>>>(a);
  return hipGetLastError();
}

template <typename T> int batchq_max_blocks_per_cu() {
  int n0 = 0, n1 = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n0, batchq_kernel<T, false>, kBqBlock, 0) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n1, batchq_kernel<T, true>, kBqBlock, 0) != hipSuccess)
    return 0;
  return n0 < n1 ? n0 : n1;
}

template hipError_t launch_batchq<float>(const BatchqArgs<float> &, int, hipStream_t);
template hipError_t launch_batchq<double>(const BatchqArgs<double> &, int, hipStream_t);
template int batchq_max_blocks_per_cu<float>();
template int batchq_max_blocks_per_cu<double>();

}  // namespace cps
