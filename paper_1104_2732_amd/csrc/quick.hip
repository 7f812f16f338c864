// The default selection's own kernels: arrays that one workgroup holds in registers, and the
// filter that reads a larger array once.
//
// Larger arrays.  The general kernel (select_kernel.h) reads x two or three times and its small
// passes cost 10-15 us each, most of it waiting for the grid.  Here one kernel reads x once
// against a likely interval of the k-th smallest (sample quantiles, so the paper's
// count-and-compact needs no iterations first): it counts the elements below the interval,
// counts those inside in key bins, and copies them (inputs the caches do not hold) or leaves
// them to be read again (inputs they do).  The kernel after it (the first part of the general
// kernel, quick_enter) adds the workgroups' counts, proves the interval by them, narrows to
// the bin of the rank, gathers that bin's elements and selects among them.  Where the counts
// do not prove the interval the general kernel runs as before, so the result never depends on
// the sample.  The two kernels meet at a launch boundary (2.7 us) instead of a wait of the
// whole grid.
#include "cps_quick.h"

namespace cps {

// ------------------------------------------------------------------ one workgroup

// n <= BLOCK PER elements, all in registers: the key range, then histograms of the keys until
// the rank's bin holds at most 64 (regs_select).  One launch and no other workgroup to wait
// for: latency-bound (1000 float32 elements 6.6 us, the general kernel 21;
// 32768 elements 9.5 us in float32 and 17 in float64, the general kernel 68 and 97).  The
// largest float32 instance (64 keys per lane) spills a few registers and takes 22 us for 65536
// elements, still less than the filter and its second kernel (25 us from there on); in float64 the
// filter (26 us) takes over where the registers end.
template <typename T, int BLOCK, int PER>
__global__ __launch_bounds__(BLOCK) void quick_small_kernel(const T *__restrict__ x, int64_t n,
                                                            int64_t k, cps_result *out) {
  using Key = typename Traits<T>::Key;
  __shared__ uint32_t hist[4 * BLOCK];
  __shared__ RegSelShared<BLOCK> sh;
  const int tid = threadIdx.x;
  const CPS_GLOBAL T *xg = (const CPS_GLOBAL T *)x;
  T v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = tid + j * BLOCK;
    v[j] = xg[i < (int)n ? i : 0];  // (past the end: the first element again)
  }
  bool nan = false;
  Key mn = (Key)~(Key)0, mx = 0;
  Key key[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    nan = nan || !(v[j] == v[j]);
    key[j] = Traits<T>::key(v[j]);
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
    if (tid + j * BLOCK >= (int)n) key[j] = (Key)~(Key)0;
  }
  nan = block_key_range<BLOCK>(mn, mx, nan, sh);
  if (nan) {  // (uniform)
    if (tid == 0) write_key<T>(out, 0, 0, 0, n, 1, ST_NAN);
    return;
  }
  const RegSel<Key> r =
      regs_select<T, BLOCK, PER>(key, (uint32_t)k, (uint32_t)n, mn, mx, hist, sh);
  if (tid == 0) write_key<T>(out, r.key, r.less, r.equal, n, 1, ST_OK);
}

// ------------------------------------------------------------------ the filter

// Pass 0 of the one-read selection over x (n elements, at least the sample's 1024 SPER): every
// workgroup takes the sample and its ends by itself (the same everywhere, so nothing waits),
// then its tiles of x as the general kernel deals them (RowFilter).  An inside element that is NaN
// is counted, any other's key bin is, and with COPY all go to the wavefront's region of the split
// buffer (which holds the wavefront's whole share, so the copy always fits).  An end that is one
// repeated value is counted apart, by comparisons, and neither binned nor copied.
//
// Bound: HBM.  2^28 float32 197 us, float64 391 us; without the copy's stores 172 and 332, which is
// the sample (9 us) and the read (158 us per GiB): the ~3 % of the elements that are inside (4
// deviations of a 16384 sample either way) are cheap to find, but writing them between reads
// costs five times their share of the traffic.
constexpr int kQuickBlock = kSelectBlock;
constexpr int kQuickU = kSelectUnroll;

template <typename T, int SPER, bool COPY>
__global__ __launch_bounds__(kQuickBlock) __attribute__((amdgpu_num_vgpr(128)))
void quick_filter_kernel(QuickArgs<T> a) {
  using Key = typename Traits<T>::Key;
  using Vec = typename Traits<T>::Vec;
  constexpr int U = kQuickU, BLOCK = kQuickBlock, NW = BLOCK / kWave;
  __shared__ uint32_t hist[kHistMaxBins];
  __shared__ RegSelShared<BLOCK> sh;
  __shared__ Vec buf[NW][RowFilter<T>::kRows];
  __shared__ unsigned long long scount[4];  // below, the ends' repeated values, NaN
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int bid = blockIdx.x, G = gridDim.x;
  // the sample: runs of kPropRun neighbours at even distances
  constexpr int S = BLOCK * SPER;
  const int64_t stride = a.n / (S / kPropRun);
  const CPS_GLOBAL T *xg = (const CPS_GLOBAL T *)a.x;
  Key sk[SPER];
  Key mn = (Key)~(Key)0, mx = 0;
  bool nan = false;
  {
    T v[SPER];
#pragma unroll
    for (int j = 0; j < SPER; ++j) {
      const int i = tid + j * BLOCK;
      v[j] = xg[(int64_t)(i / kPropRun) * stride + i % kPropRun];
    }
#pragma unroll
    for (int j = 0; j < SPER; ++j) {
      nan = nan || !(v[j] == v[j]);
      sk[j] = Traits<T>::key(v[j]);
      mn = sk[j] < mn ? sk[j] : mn;
      mx = sk[j] > mx ? sk[j] : mx;
    }
  }
  nan = block_key_range<BLOCK>(mn, mx, nan, sh);
  if (nan) {  // (uniform, and the same in every workgroup)
    if (bid == 0 && tid == 0) a.rec->nan = 1;
    return;
  }
  const SampleEnds<Key> e = sample_ends<T, BLOCK, SPER>(sk, mn, mx, a.n, a.k, 4.0, hist, sh);
  if (bid == 0 && tid == 0) {
    QuickRec r;
    r.ka = (uint64_t)e.ka;
    r.kb = (uint64_t)e.kb;
    r.ia = (uint64_t)e.ia;
    r.ib = (uint64_t)e.ib;
    r.nan = 0;
    r.copied = COPY ? 1 : 0;
    *a.rec = r;
  }
  const int shift = range_shift((uint64_t)(e.ib - e.ia), 12);
  *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
  if (tid < 4) scount[tid] = 0ull;
  __syncthreads();
  RowFilter<T> f(e, buf[wv]);
  uint32_t nn = 0;   // per lane: NaN
  uint32_t out = 0;  // per wavefront: in the region
  CPS_GLOBAL T *region = nullptr;
  if (COPY) region = (CPS_GLOBAL T *)uniform_ptr(a.z0 + ((int64_t)bid * NW + wv) * a.seg_R);
  auto put = [&](T v, uint64_t m) {
    const bool num = v == v;
    if (__builtin_amdgcn_inverse_ballot_w64(m)) {
      nn += num ? 0u : 1u;
      if (num) atomicAdd(&hist[(uint32_t)((Traits<T>::key(v) - e.ia) >> shift)], 1u);
      if (COPY) region[out + lane_rank(m)] = v;
    }
    if (COPY) out += popc(m);
  };
  const Span<T> sp = make_span(a.x, a.n);
  const int64_t step = (int64_t)BLOCK * U, hop = (int64_t)G * step;
  int64_t base = (int64_t)bid * step;
  Vec cur[U];
  auto load = [&](int64_t at) {  // (places past the end: the first vector)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t vi = at + u * BLOCK + tid;
      cur[u] = __builtin_nontemporal_load(&sp.V[vi < sp.nvec ? vi : 0]);
    }
  };
  load(base);
  // Every pass issues the next tile's loads: a conditional load would make the wait before the
  // current tile's use one for the next tile's first load as well.
  for (; base + hop + step <= sp.nvec; base += hop) {
    Vec nxt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) nxt[u] = __builtin_nontemporal_load(&sp.V[base + hop + u * BLOCK + tid]);
#pragma unroll
    for (int u = 0; u < U; ++u) f.row(cur[u], ~0ull, put);
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = nxt[u];
  }
  for (; base < sp.nvec; base += hop) {  // the last one or two tiles
#pragma unroll
    for (int u = 0; u < U; ++u) f.row(cur[u], ballot(base + u * BLOCK + tid < sp.nvec), put);
    load(base + hop);
  }
  if (sp.nedge > 0 && bid == 0 && wv == 0) {  // the unaligned head and tail
    const uint64_t ok = (1ull << sp.nedge) - 1ull;
    const T v = sp.W[lane < sp.nedge ? edge_index(sp, lane) : 0];
    put(v, ok & ~f.outside(v, ok));
  }
  if (f.held > 0) f.drain(f.held, put);
  if (COPY && lane == 0) a.kept[(int64_t)bid * NW + wv] = out;
  const double fnn = wave_sum((double)nn);
  if (lane == 0) {
    atomicAdd(&scount[0], (unsigned long long)(f.below - f.ea));
    if (f.ea) atomicAdd(&scount[1], (unsigned long long)f.ea);
    if (f.eb) atomicAdd(&scount[2], (unsigned long long)f.eb);
    if (fnn > 0.0) atomicAdd(&scount[3], (unsigned long long)fnn);
  }
  __syncthreads();
  if (tid < 4) a.slot[(int64_t)tid * a.slot_stride + bid] = (int64_t)scount[tid];
  // (workgroups that end together would wait for each other at every line of one set of bins)
  uint32_t *gh = a.hist + (int64_t)(bid % kQuickCopies) * kHistMaxBins;
#pragma unroll
  for (int j = 0; j < kHistMaxBins / BLOCK; ++j) {
    const uint32_t c = hist[tid + j * BLOCK];
    if (c) __hip_atomic_fetch_add(&gh[tid + j * BLOCK], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ------------------------------------------------------------------ launchers

template <typename T> int64_t quick_small_max() { return sizeof(T) == 4 ? 65536 : 32768; }

template <typename T>
hipError_t launch_quick_small(const T *x, int64_t n, int64_t k, cps_result *out, hipStream_t stream) {
  if (n <= 1024) quick_small_kernel<T, 256, 4><<<1, 256, 0, stream>>>(x, n, k, out);
  else if (n <= 4096) quick_small_kernel<T, 1024, 4><<<1, 1024, 0, stream>>>(x, n, k, out);
  else if (n <= 16384) quick_small_kernel<T, 1024, 16><<<1, 1024, 0, stream>>>(x, n, k, out);
  else if (sizeof(T) == 8 || n <= 32768) quick_small_kernel<T, 1024, 32><<<1, 1024, 0, stream>>>(x, n, k, out);
  else quick_small_kernel<T, 1024, sizeof(T) == 4 ? 64 : 32><<<1, 1024, 0, stream>>>(x, n, k, out);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_quick_filter(const QuickArgs<T> &a, bool copy, int grid, hipStream_t stream) {
  const dim3 g(grid), b(kQuickBlock);
  if (a.n < kPropBigN) {
    if (copy) quick_filter_kernel<T, 4, true><<<g, b, 0, stream>>>(a);
    else quick_filter_kernel<T, 4, false><<<g, b, 0, stream>>>(a);
  } else {
    if (copy) quick_filter_kernel<T, 16, true><<<g, b, 0, stream>>>(a);
    else quick_filter_kernel<T, 16, false><<<g, b, 0, stream>>>(a);
  }
  return hipGetLastError();
}

template int64_t quick_small_max<float>();
template int64_t quick_small_max<double>();
template hipError_t launch_quick_small<float>(const float *, int64_t, int64_t, cps_result *, hipStream_t);
template hipError_t launch_quick_small<double>(const double *, int64_t, int64_t, cps_result *, hipStream_t);
template hipError_t launch_quick_filter<float>(const QuickArgs<float> &, bool, int, hipStream_t);
template hipError_t launch_quick_filter<double>(const QuickArgs<double> &, bool, int, hipStream_t);

}  // namespace cps
