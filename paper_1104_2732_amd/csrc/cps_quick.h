// Building blocks of the one-read selection (quick.hip and the first part of the general
// kernel): what the filter leaves for the kernel after it, and exact selects and sample
// quantiles over keys that one workgroup holds in registers.
#pragma once

#include "cps_device.h"
#include "cps_kernels.h"
#include "cps_passes.h"
#include "cps_sample.h"

namespace cps {

// ------------------------------------------------------------------ scans and folds

// Inclusive prefix sum over the wavefront: four row shifts, then two row broadcasts.
template <int CTRL, int ROWS> __device__ inline uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ inline uint32_t wave_scan_u32(uint32_t v) {
  v += dpp_or_zero<0x111, 0xF>(v);
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);
  v += dpp_or_zero<0x143, 0xC>(v);
  return v;
}

// Exclusive prefix sum over the workgroup in thread order (wsum: a word per wavefront).
template <int BLOCK> __device__ inline uint32_t block_scan_u32(uint32_t v, uint32_t *wsum) {
  const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  const uint32_t x = wave_scan_u32(v);
  if (lane == kWave - 1) wsum[wv] = x;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < BLOCK / kWave; ++w) off += w < wv ? wsum[w] : 0u;
  __syncthreads();
  return off + x - v;
}

// A sum in two parts: hi, and in lo what its additions rounded off (two-sum, Knuth, The Art of
// Computer Programming vol. 2, 4.2.2).  The sums of the k smallest are folded this way from the lanes
// on, and rounded once at the end: the lanes' own sums are short and their errors average out, but
// some fifteen further additions of the whole size left the result 0.8 to 1.9 units of 2^-53 off
// (rms, float64 arrays), the general kernel's fewer ones 0.4 to 1.2, this way 0 to 0.4.
struct Sum2 {
  double hi, lo;
};
__device__ inline Sum2 sum2(double a, double b) {
  const double s = a + b, c = s - a, e = (a - (s - c)) + (b - c);
  return {s, e - e == 0.0 ? e : 0.0};  // (an infinite sum has no error)
}
__device__ inline Sum2 sum2(Sum2 a, Sum2 b) {
  Sum2 t = sum2(a.hi, b.hi);
  t.lo += a.lo + b.lo;
  return t;
}
__device__ inline Sum2 product2(double a, double b) {
  const double p = a * b, e = __builtin_fma(a, b, -p);
  return {p, e - e == 0.0 ? e : 0.0};
}
__device__ inline double value(Sum2 s) { return s.hi + s.lo; }

template <int CTRL, int ROWS> __device__ inline Sum2 sum2_move(Sum2 v) {
  return sum2(v, Sum2{dpp_move<CTRL, ROWS>(v.hi, 0.0), dpp_move<CTRL, ROWS>(v.lo, 0.0)});
}
template <int LANE> __device__ inline double lane_value(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, LANE);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), LANE);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Over the workgroup, in every thread, in a fixed order (`red`: one per wavefront).
template <int BLOCK> __device__ inline Sum2 block_sum2(Sum2 v, Sum2 *red) {
  v = sum2_move<0x111, 0xF>(v);
  v = sum2_move<0x112, 0xF>(v);
  v = sum2_move<0x114, 0xF>(v);
  v = sum2_move<0x118, 0xF>(v);
  v = sum2_move<0x142, 0xA>(v);
  v = sum2_move<0x143, 0xC>(v);
  __syncthreads();
  if (threadIdx.x % kWave == kWave - 1) red[threadIdx.x / kWave] = v;
  __syncthreads();
  constexpr int NW = BLOCK / kWave;  // (one row of lanes holds them)
  static_assert(NW <= 16 && (NW & (NW - 1)) == 0, "a power of two of wavefronts");
  const int lane = threadIdx.x % kWave;
  v = red[lane % NW];
  if (NW > 1) v = sum2_move<0x111, 0xF>(v);
  if (NW > 2) v = sum2_move<0x112, 0xF>(v);
  if (NW > 4) v = sum2_move<0x114, 0xF>(v);
  if (NW > 8) v = sum2_move<0x118, 0xF>(v);
  return {lane_value<NW - 1>(v.hi), lane_value<NW - 1>(v.lo)};
}

__device__ inline uint32_t shfl_xor_key(uint32_t v, int o) { return (uint32_t)__shfl_xor((int)v, o); }
__device__ inline uint64_t shfl_xor_key(uint64_t v, int o) {
  return (uint64_t)__shfl_xor((unsigned long long)v, o);
}

template <int BLOCK> struct RegSelShared {
  uint32_t wsum[BLOCK / kWave];
  uint64_t kmin[BLOCK / kWave], kmax[BLOCK / kWave];
  uint32_t flag[BLOCK / kWave];
  uint32_t bin[2], below[2], inb[2];  // a pick's bin, the count below it and its own
  uint32_t cursor, less, equal;
  uint64_t key, list[kWave];
};

// Minimum and maximum of the workgroup's keys (a thread without one: mn = ~0, mx = 0), and
// whether any thread's flag is set.
template <int BLOCK, typename Key>
__device__ inline bool block_key_range(Key &mn, Key &mx, bool flag, RegSelShared<BLOCK> &sh) {
  const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const Key a = shfl_xor_key(mn, o), b = shfl_xor_key(mx, o);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  const bool any = ballot(flag) != 0;
  if (lane == 0) {
    sh.kmin[wv] = (uint64_t)mn;
    sh.kmax[wv] = (uint64_t)mx;
    sh.flag[wv] = any ? 1u : 0u;
  }
  __syncthreads();
  uint32_t f = 0;
#pragma unroll
  for (int w = 0; w < BLOCK / kWave; ++w) {
    const Key a = (Key)sh.kmin[w], b = (Key)sh.kmax[w];
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
    f |= sh.flag[w];
  }
  return f != 0;
}

// The smallest shift that brings a key range into `bins` bins.
__device__ inline int range_shift(uint64_t span, int bins_log2) {
  const int bits = span == 0 ? 0 : 64 - __builtin_clzll(span);
  return bits > bins_log2 ? bits - bins_log2 : 0;
}

// The bin that holds rank r (1-based) of `hist` (4 bins per thread, in thread order), left in
// slot `s` of the shared picks.  Callers pass the scan of their four bins.
template <int BLOCK>
__device__ inline void pick4(const uint32_t (&h)[4], uint32_t cum, uint32_t r, int s,
                             RegSelShared<BLOCK> &sh) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (cum < r && r <= cum + h[j]) {
      sh.bin[s] = threadIdx.x * 4 + j;
      sh.below[s] = cum;
      sh.inb[s] = h[j];
    }
    cum += h[j];
  }
}

template <typename Key> struct RegSel {
  Key key;
  uint32_t less, equal;
};

// The r-th smallest (1-based) of the workgroup's keys (cnt of them in [klo, khi], r <= cnt; an
// empty place holds ~0, which no number has), with its counts: histograms of 4 BLOCK bins narrow
// the key range to the bin of the rank until the range is one key or holds at most 64 keys,
// which one wavefront ranks by comparing each with all.  `hist` is 4 BLOCK words of LDS.
template <typename T, int BLOCK, int PER>
__device__ inline RegSel<typename Traits<T>::Key> regs_select(
    const typename Traits<T>::Key (&k)[PER], uint32_t r, uint32_t cnt,
    typename Traits<T>::Key klo, typename Traits<T>::Key khi, uint32_t *hist,
    RegSelShared<BLOCK> &sh) {
  using Key = typename Traits<T>::Key;
  constexpr int kBinsLog2 = BLOCK == 1024 ? 12 : (BLOCK == 512 ? 11 : 10);
  static_assert((4 * BLOCK) == (1 << kBinsLog2), "four bins per thread");
  const int tid = threadIdx.x, lane = tid % kWave;
  uint32_t base = 0;
  while (klo != khi && cnt > (uint32_t)kWave) {
    const int shift = range_shift((uint64_t)(khi - klo), kBinsLog2);
    *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const Key d = k[j] - klo;
      if (d <= khi - klo) atomicAdd(&hist[(uint32_t)(d >> shift)], 1u);
    }
    __syncthreads();
    const uint4 q = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    const uint32_t h[4] = {q.x, q.y, q.z, q.w};
    const uint32_t cum = block_scan_u32<BLOCK>(h[0] + h[1] + h[2] + h[3], sh.wsum);
    pick4<BLOCK>(h, cum, r, 0, sh);
    __syncthreads();
    base += sh.below[0];
    r -= sh.below[0];
    cnt = sh.inb[0];
    const Key lo = klo + ((Key)sh.bin[0] << shift);
    const Key hi = lo + (((Key)1 << shift) - 1);
    khi = hi < khi && hi >= lo ? hi : khi;
    klo = lo;
  }
  if (klo == khi) return {klo, base, cnt};
  // at most 64 keys in [klo, khi]
  __syncthreads();
  if (tid == 0) sh.cursor = 0u;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if (k[j] - klo <= khi - klo) {
      const uint32_t at = atomicAdd(&sh.cursor, 1u);
      if (at < (uint32_t)kWave) sh.list[at] = (uint64_t)k[j];
    }
  }
  __syncthreads();
  if (tid < kWave) {
    const Key mine = lane < (int)cnt ? (Key)sh.list[lane] : (Key)~(Key)0;
    uint32_t less = 0, eq = 0;
    for (uint32_t i = 0; i < cnt; ++i) {
      const Key o = (Key)sh.list[i];
      less += o < mine ? 1u : 0u;
      eq += o == mine ? 1u : 0u;
    }
    if (lane < (int)cnt && less < r && r <= less + eq) {
      sh.key = (uint64_t)mine;
      sh.less = less;
      sh.equal = eq;
    }
  }
  __syncthreads();
  return {(Key)sh.key, base + sh.less, sh.equal};
}

__device__ inline void write_selection(cps_result *out, uint64_t bits, double value, int64_t less,
                                       int64_t equal, int64_t n, int32_t passes, int32_t status) {
  cps_result r;
  r.value_bits = bits;
  r.value = value;
  r.less = less;
  r.equal = equal;
  r.greater = status == ST_OK ? n - less - equal : 0;
  r.passes = passes;
  r.status = status;
  *out = r;
}
// ... of the element with this key, or (a status other than ok) of none: NaN.
template <typename T>
__device__ inline void write_key(cps_result *out, typename Traits<T>::Key key, int64_t less,
                                 int64_t equal, int64_t n, int32_t passes, int32_t status) {
  const bool none = status != ST_OK;
  const T v = none ? (T)__builtin_nan("") : Traits<T>::unkey(key) + T(0);
  uint64_t bits;
  if (sizeof(T) == 4) bits = (uint64_t)__builtin_bit_cast(uint32_t, (float)v);
  else bits = __builtin_bit_cast(uint64_t, (double)v);
  write_selection(out, bits, (double)v, none ? 0 : less, none ? 0 : equal, n, passes, status);
}

// The element of rank r (1-based) among the elements that `walk` visits, all with keys in [klo,
// khi], from their counts in this thread's four key bins (range_shift of the range): the rank's
// bin, split again while it holds many elements, then ranked by comparing each with all.
// `hist` is 4 BLOCK words of LDS, `fin` kWalkFinal keys.  `equal` is 0 where the counts and the
// elements disagree, as when the input changes during the call (no bin holds the rank, or not as
// many elements as its bin counted).
constexpr uint32_t kWalkFinal = 256;
CPS_HD constexpr int quick_bins_log2(int block) { return block == 1024 ? 12 : (block == 512 ? 11 : 10); }
template <typename T, int BLOCK, typename Walk>
__device__ inline void walk_select(Walk &&walk, uint32_t (&h)[4], int64_t r,
                                   typename Traits<T>::Key klo, typename Traits<T>::Key khi,
                                   uint32_t *hist, typename Traits<T>::Key *fin,
                                   RegSelShared<BLOCK> &sh, typename Traits<T>::Key &key,
                                   int64_t &less, int64_t &equal) {
  using Key = typename Traits<T>::Key;
  const int tid = threadIdx.x;
  less = 0;
  int64_t cnt = 0;
  // (each round narrows the range by the bins' bits: seven at most)
  for (int round = 0; round < 8; ++round) {
    const int shift = range_shift((uint64_t)(khi - klo), quick_bins_log2(BLOCK));
    if (tid == 0) sh.inb[0] = 0u;
    const uint32_t cum = block_scan_u32<BLOCK>(h[0] + h[1] + h[2] + h[3], sh.wsum);
    pick4<BLOCK>(h, cum, (uint32_t)r, 0, sh);
    __syncthreads();
    less += sh.below[0];
    r -= sh.below[0];
    cnt = sh.inb[0];
    const Key lo = klo + ((Key)sh.bin[0] << shift);
    const Key hi = lo + (((Key)1 << shift) - 1);
    khi = hi < khi && hi >= lo ? hi : khi;
    klo = lo;
    if (klo == khi) {
      key = klo;
      equal = cnt;
      return;
    }
    if (cnt <= (int64_t)kWalkFinal) break;
    const int next = range_shift((uint64_t)(khi - klo), quick_bins_log2(BLOCK));
    __syncthreads();
    *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    walk([&](T v, bool ok) {
      const Key d = Traits<T>::key(v) - klo;
      if (ok & (d <= khi - klo)) atomicAdd(&hist[(uint32_t)(d >> next)], 1u);
    });
    __syncthreads();
    const uint4 q = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    h[0] = q.x;
    h[1] = q.y;
    h[2] = q.z;
    h[3] = q.w;
  }
  if (cnt > (int64_t)kWalkFinal) cnt = kWalkFinal;
  if (tid == 0) sh.cursor = sh.equal = 0u;
  __syncthreads();
  walk([&](T v, bool ok) {
    const Key q = Traits<T>::key(v), d = q - klo;
    if (ok & (d <= khi - klo)) {
      const uint32_t at = atomicAdd(&sh.cursor, 1u);
      if (at < kWalkFinal) fin[at] = q;
    }
  });
  __syncthreads();
  if (tid < (int)cnt) {
    const Key mine = fin[tid];
    uint32_t lo = 0, eq = 0;
    for (int i = 0; i < (int)cnt; ++i) {
      const Key o = fin[i];
      lo += o < mine ? 1u : 0u;
      eq += o == mine ? 1u : 0u;
    }
    if ((int64_t)lo < r && r <= (int64_t)(lo + eq)) {  // (one key: all its threads write the same)
      sh.key = (uint64_t)mine;
      sh.less = lo;
      sh.equal = eq;
    }
  }
  __syncthreads();
  key = (Key)sh.key;
  less += sh.less;
  equal = sh.cursor == (uint32_t)cnt ? sh.equal : 0u;
}

// A value every lane of the wavefront holds, moved to scalar registers.
__device__ inline float uniform_value(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ inline double uniform_value(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <typename Key> struct SampleEnds {
  Key ka, kb;  // the likely interval, as closed keys
  Key ia, ib;  // ... without an end that is one repeated value (its elements are counted apart)
};

// ------------------------------------------------------------------ the filter's inner loop

// One wavefront's elements against a likely interval, a vector per lane at a time.  Per vector
// only comparisons, scalar counts and one LDS write of the vectors that hold an inside element
// (a tenth to a fifth of them); 64 of these at a time are taken apart element by element, by full
// lanes.  Masks are combined as scalars: per-lane booleans cost two vector instructions each time
// they become a mask.  (Element by element, each with its own branch: 2^24 float32 45 us a call,
// this way 43; the default batch of 4096 arrays 690 us, this way 620.)
template <typename T> struct RowFilter {
  using Vec = typename Traits<T>::Vec;
  static constexpr int V = Traits<T>::kVec;
  static constexpr uint32_t kRows = 2 * kWave;  // LDS vectors per wavefront
  T va, vb, wa, wb;      // the interval's ends, and without repeated ends (uniform)
  bool ties;             // they differ (uniform)
  uint64_t below, ea, eb;  // per wavefront: below wa, of these equal to va, above wb equal to vb
  uint32_t held;
  CPS_LDS Vec *buf;

  __device__ inline RowFilter(const SampleEnds<typename Traits<T>::Key> &e, Vec *lds) {
    va = uniform_value(Traits<T>::unkey(e.ka));
    vb = uniform_value(Traits<T>::unkey(e.kb));
    wa = uniform_value(Traits<T>::unkey(e.ia));
    wb = uniform_value(Traits<T>::unkey(e.ib));
    ties = __builtin_amdgcn_readfirstlane(e.ia != e.ka || e.ib != e.kb) != 0;
    below = ea = eb = 0;
    held = 0;
    buf = (CPS_LDS Vec *)lds;
  }
  __device__ inline uint64_t outside(T v, uint64_t ok) {
    const uint64_t lo = ballot(v < wa), hi = ballot(v > wb);
    below += popc(lo & ok);
    if (ties) {
      ea += popc(lo & ~ballot(v < va) & ok);
      eb += popc(hi & ~ballot(v > vb) & ok);
    }
    return lo | hi;
  }
  // A vector per lane (those of the mask): put(v, mask) gets inside elements when 64 are held.
  template <typename Put> __device__ inline void row(Vec v, uint64_t ok, Put &&put) {
    uint64_t out = ~0ull;
#pragma unroll
    for (int j = 0; j < V; ++j) out &= outside(v[j], ok);
    const uint64_t m = ok & ~out;
    if (__builtin_amdgcn_inverse_ballot_w64(m)) buf[held + lane_rank(m)] = v;
    held += popc(m);
    if (held >= (uint32_t)kWave) drain(kWave, put);
  }
  // The last m (<= 64) vectors held.
  template <typename Put> __device__ inline void drain(uint32_t m, Put &&put) {
    __builtin_amdgcn_wave_barrier();
    held -= m;
    const int lane = threadIdx.x % kWave;
    const Vec v = buf[held + lane];
    const uint64_t ok = m >= (uint32_t)kWave ? ~0ull : (1ull << m) - 1ull;
#pragma unroll
    for (int j = 0; j < V; ++j) put(v[j], ok & ~(ballot(v[j] < wa) | ballot(v[j] > wb)));
    __builtin_amdgcn_wave_barrier();
  }
};

// ------------------------------------------------------------------ the sample's ends


// The likely interval of rank k of n values from S of their keys, PER per thread in registers
// (S = BLOCK PER; no NaN): the bins of sample ranks floor(q - d) and ceil(q + d), q = S p, p = (k -
// 1/2) / n, d = dev sqrt(S p (1 - p)) + 2 (dev binomial standard deviations), each end's bin
// split again (2 BLOCK sub-bins) until it holds at most a sixteenth of the samples between the
// ranks or is one key (a value that repeats).  An end whose rank falls outside the sample is
// open: the key of -inf or +inf.  Every workgroup that calls it on the same sample gets the
// same interval.
template <typename T, int BLOCK, int PER>
__device__ inline SampleEnds<typename Traits<T>::Key> sample_ends(
    const typename Traits<T>::Key (&v)[PER], typename Traits<T>::Key klo,
    typename Traits<T>::Key khi, int64_t n, int64_t k, double dev, uint32_t *hist,
    RegSelShared<BLOCK> &sh) {
  using Key = typename Traits<T>::Key;
  constexpr int kBinsLog2 = BLOCK == 1024 ? 12 : (BLOCK == 512 ? 11 : 10);
  constexpr uint32_t S = BLOCK * PER;
  const int tid = threadIdx.x;
  const double Sd = (double)S, p = ((double)k - 0.5) / (double)n;
  const double q = Sd * p, d = dev * __builtin_sqrt(Sd * p * (1.0 - p)) + 2.0;
  const double r0 = __builtin_floor(q - d), r1 = __builtin_ceil(q + d);
  const bool open0 = r0 < 1.0, open1 = r1 > Sd;
  const uint32_t rank0 = open0 ? 1u : (uint32_t)r0, rank1 = open1 ? S : (uint32_t)r1;
  const uint32_t most = (rank1 - rank0 + 1) / 16 + 4;
  int sh0 = range_shift((uint64_t)(khi - klo), kBinsLog2), sh1 = sh0;
  *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) atomicAdd(&hist[(uint32_t)((v[j] - klo) >> sh0)], 1u);
  __syncthreads();
  {
    const uint4 w = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    const uint32_t h[4] = {w.x, w.y, w.z, w.w};
    const uint32_t cum = block_scan_u32<BLOCK>(h[0] + h[1] + h[2] + h[3], sh.wsum);
    pick4<BLOCK>(h, cum, rank0, 0, sh);
    pick4<BLOCK>(h, cum, rank1, 1, sh);
  }
  __syncthreads();
  Key f0 = klo + ((Key)sh.bin[0] << sh0), f1 = klo + ((Key)sh.bin[1] << sh1);  // first keys
  uint32_t t0 = rank0 - sh.below[0], t1 = rank1 - sh.below[1];  // ranks inside the bins
  uint32_t in0 = sh.inb[0], in1 = sh.inb[1];
  for (;;) {
    const bool s0 = !open0 && sh0 > 0 && in0 > most, s1 = !open1 && sh1 > 0 && in1 > most;
    if (!s0 && !s1) break;  // (uniform)
    constexpr int kHalf = 2 * BLOCK;  // sub-bins per end, the upper end's after the lower's
    const int n0 = sh0 > kBinsLog2 - 1 ? sh0 - (kBinsLog2 - 1) : 0;
    const int n1 = sh1 > kBinsLog2 - 1 ? sh1 - (kBinsLog2 - 1) : 0;
    __syncthreads();
    *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
    __syncthreads();
    const Key m0 = ((Key)1 << sh0) - 1, m1 = ((Key)1 << sh1) - 1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const Key d0 = v[j] - f0, d1 = v[j] - f1;
      if (s0 && d0 <= m0) atomicAdd(&hist[(uint32_t)(d0 >> n0)], 1u);
      if (s1 && d1 <= m1) atomicAdd(&hist[kHalf + (uint32_t)(d1 >> n1)], 1u);
    }
    __syncthreads();
    const uint4 w = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    const uint32_t h[4] = {w.x, w.y, w.z, w.w};
    const uint32_t cum = block_scan_u32<BLOCK>(h[0] + h[1] + h[2] + h[3], sh.wsum);
    // (the upper half follows the lower bin's samples in the scan, where they were counted)
    if (s0 && tid < BLOCK / 2) pick4<BLOCK>(h, cum, t0, 0, sh);
    if (s1 && tid >= BLOCK / 2) pick4<BLOCK>(h, cum, t1 + (s0 ? in0 : 0u), 1, sh);
    __syncthreads();
    if (s0) {
      f0 += (Key)sh.bin[0] << n0;
      t0 -= sh.below[0];
      sh0 = n0;
    }
    if (s1) {
      f1 += (Key)(sh.bin[1] - kHalf) << n1;
      t1 -= sh.below[1] - (s0 ? in0 : 0u);
      sh1 = n1;
    }
    if (s0) in0 = sh.inb[0];
    if (s1) in1 = sh.inb[1];
  }
  const Key kneg = Traits<T>::key(-t_inf<T>()), kpos = Traits<T>::key(t_inf<T>());
  SampleEnds<Key> e;
  // (-0's own key is no element's: +0 compares equal to it and has the next key)
  const Key hole = Traits<T>::key(T(0)) - 1;
  e.ka = open0 ? kneg : f0;
  if (e.ka == hole) ++e.ka;
  const Key l1 = f1 + (((Key)1 << sh1) - 1);
  e.kb = open1 || l1 > kpos || l1 < f1 ? kpos : l1;
  if (e.kb == hole) --e.kb;
  e.ia = e.ka;
  e.ib = e.kb;
  if (e.ka == kpos) {
    --e.ib;  // (nothing lies above +inf: repeated, it is the upper end)
  } else {
    if (!open0 && sh0 == 0) {
      ++e.ia;
      if (e.ia == hole) ++e.ia;
    }
    if (!open1 && sh1 == 0 && e.kb != e.ka) {
      --e.ib;
      if (e.ib == hole) --e.ib;
    }
  }
  __syncthreads();
  return e;
}

}  // namespace cps
