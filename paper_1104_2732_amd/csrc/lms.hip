// Least median of squares (Section 6): the lower median of the squared residuals of many
// candidate parameter vectors, via the batched selection.
//
// The residual kernels form r_i = (y_i - sum_j X_ij b_j)^2 for a group of candidates per
// thread row: each X row and y_i are read once per group, the sum runs left to right in
// j with every product and sum rounded on its own (the library is built without fused
// multiply-add).
//
// Two forms.  The materialised form writes every square candidate-major in the workspace,
// one array of n per candidate, and the batched kernel selects rank floor((n+1)/2) of every
// array.  The filtered form never writes the whole arrays: a first kernel takes each
// candidate's sampled bracket (a, b) from the squares of a fixed sample of rows, the filter
// kernel forms every square once and keeps only those in (a, b), with #(r <= a), and a select
// kernel reads the kept squares of each candidate.  Where #(r <= a) < k <= #(r <= a) +
// #(a < r < b) the k-th smallest of all n squares is the (k - #(r <= a))-th smallest of the
// kept ones; a candidate whose bracket misses gets its full array written and selected as in
// the materialised form.  Both give the same value and counts.
#include "cps_device.h"
#include "cps_kernels.h"
#include "cps_quick.h"
#include "cps_sample.h"
#include "cps_wgsel.h"

namespace cps {

#ifndef CPS_LMS_GROUP
#define CPS_LMS_GROUP 64
#endif
constexpr int kLmsGroup = CPS_LMS_GROUP;  // candidates per thread row (X read once per group)
constexpr int kLmsBlock = 256;
#ifndef CPS_LMS_ROWS
#define CPS_LMS_ROWS 2
#endif
constexpr int kLmsRows = CPS_LMS_ROWS;  // rows per thread of the 16-byte residual kernel

// ONLY: write only the candidates whose flag in `only` is set (the filtered form's
// fallback); a workgroup whose candidates have none returns at once.
template <int P, bool ONLY>
__global__ __launch_bounds__(kLmsBlock) void lms_residual_kernel(
    const double *__restrict__ X, const double *__restrict__ y, const double *__restrict__ betas,
    int64_t n, int32_t p, int64_t m, double *__restrict__ R, const int32_t *__restrict__ only) {
  __shared__ double sb[kLmsGroup * 16];
  __shared__ int32_t sf[kLmsGroup];
  const int64_t c0 = (int64_t)blockIdx.y * kLmsGroup;
  const int nc = (int)((m - c0) < kLmsGroup ? (m - c0) : kLmsGroup);
  for (int q = threadIdx.x; q < nc * p; q += kLmsBlock) sb[q] = betas[c0 * p + q];
  if (ONLY && threadIdx.x < nc) sf[threadIdx.x] = only[c0 + threadIdx.x];
  if (ONLY) {
    if (!__syncthreads_or(threadIdx.x < nc && only[c0 + threadIdx.x] != 0)) return;
  } else {
    __syncthreads();
  }
  const CPS_GLOBAL double *Xg = (const CPS_GLOBAL double *)X;
  const CPS_GLOBAL double *yg = (const CPS_GLOBAL double *)y;
  CPS_GLOBAL double *Rg = (CPS_GLOBAL double *)R;
  for (int64_t i = (int64_t)blockIdx.x * kLmsBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kLmsBlock) {
    double row[P > 0 ? P : 16];
    const int pp = P > 0 ? P : p;
#pragma unroll
    for (int j = 0; j < (P > 0 ? P : 16); ++j)
      if (j < pp) row[j] = Xg[i * pp + j];
    const double yi = yg[i];
    for (int c = 0; c < nc; ++c) {
      if (ONLY && sf[c] == 0) continue;
      const double *b = sb + c * pp;
      double s = row[0] * b[0];
#pragma unroll
      for (int j = 1; j < (P > 0 ? P : 16); ++j) {
        if (j < pp) {
          const double prod = row[j] * b[j];
          s = s + prod;
        }
      }
      const double d = yi - s;
      __builtin_nontemporal_store(d * d, &Rg[(c0 + c) * n + i]);  // written once, read later
    }
  }
}

// The same residuals for p = P columns, R consecutive rows per thread: each thread's X rows
// are R*P contiguous doubles (16-byte loads) and each candidate's R residuals one or two
// 16-byte stores, so a wavefront writes R*512 contiguous bytes per candidate.  Needs n to be a
// multiple of R (every candidate's array then starts 16-byte aligned).
template <int P, int R, bool ONLY>
__global__ __launch_bounds__(kLmsBlock) void lms_residual_rows_kernel(
    const double *__restrict__ X, const double *__restrict__ y, const double *__restrict__ betas,
    int64_t n, int64_t m, double *__restrict__ R_out, const int32_t *__restrict__ only) {
  static_assert(R % 2 == 0 && (P * R) % 2 == 0, "16-byte groups");
  __shared__ double sb[kLmsGroup * P];
  __shared__ int32_t sf[kLmsGroup];
  const int64_t c0 = (int64_t)blockIdx.y * kLmsGroup;
  const int nc = (int)((m - c0) < kLmsGroup ? (m - c0) : kLmsGroup);
  for (int q = threadIdx.x; q < nc * P; q += kLmsBlock) sb[q] = betas[c0 * P + q];
  if (ONLY && threadIdx.x < nc) sf[threadIdx.x] = only[c0 + threadIdx.x];
  if (ONLY) {
    if (!__syncthreads_or(threadIdx.x < nc && only[c0 + threadIdx.x] != 0)) return;
  } else {
    __syncthreads();
  }
  using D2 = double __attribute__((ext_vector_type(2)));
  const CPS_GLOBAL D2 *Xg = (const CPS_GLOBAL D2 *)X;
  const CPS_GLOBAL D2 *yg = (const CPS_GLOBAL D2 *)y;
  CPS_GLOBAL double *Rg = (CPS_GLOBAL double *)R_out;
  const int64_t groups = n / R;
  for (int64_t g = (int64_t)blockIdx.x * kLmsBlock + threadIdx.x; g < groups;
       g += (int64_t)gridDim.x * kLmsBlock) {
    const int64_t i0 = g * R;
    double row[R][P];
#pragma unroll
    for (int v = 0; v < R * P / 2; ++v) {
      const D2 w = Xg[i0 * P / 2 + v];
      row[(2 * v) / P][(2 * v) % P] = w.x;
      row[(2 * v + 1) / P][(2 * v + 1) % P] = w.y;
    }
    double yi[R];
#pragma unroll
    for (int v = 0; v < R / 2; ++v) {
      const D2 w = yg[i0 / 2 + v];
      yi[2 * v] = w.x;
      yi[2 * v + 1] = w.y;
    }
    for (int c = 0; c < nc; ++c) {
      if (ONLY && sf[c] == 0) continue;
      const double *b = sb + c * P;
      double r[R];
#pragma unroll
      for (int q = 0; q < R; ++q) {
        double s = row[q][0] * b[0];
#pragma unroll
        for (int j = 1; j < P; ++j) {
          const double prod = row[q][j] * b[j];
          s = s + prod;
        }
        const double d = yi[q] - s;
        r[q] = d * d;
      }
      CPS_GLOBAL D2 *dst = (CPS_GLOBAL D2 *)(Rg + (c0 + c) * n + i0);
#pragma unroll
      for (int v = 0; v < R / 2; ++v) {
        D2 w;
        w.x = r[2 * v];
        w.y = r[2 * v + 1];
        __builtin_nontemporal_store(w, dst + v);  // written once, read later
      }
    }
  }
}

// ------------------------------------------------------------------ the filtered form

// One squared residual, in the order of the materialised kernels (bit-identical to them).
template <int P>
__device__ __forceinline__ double sq_residual(const double *row, double yi, const double *b, int p) {
  const int pp = P > 0 ? P : p;
  double s = row[0] * b[0];
#pragma unroll
  for (int j = 1; j < (P > 0 ? P : 16); ++j) {
    if (j < pp) {
      const double prod = row[j] * b[j];
      s = s + prod;
    }
  }
  const double d = yi - s;
  return d * d;
}

// The three kernels below give a lane a row (T rows: 64 neighbours per T) and loop over the
// candidates, whose coefficients are scalar loads.  A candidate per lane instead (rows by scalar
// loads) left most lanes idle with few candidates, and every lane appended to its own candidate's
// array: a branch for each square, and 8-byte stores into 64 arrays at a time.
template <int P> constexpr int kLmsTiles = P <= 10 ? 4 : 2;
constexpr int64_t lms_seg(int p) { return kWave * (p <= 10 ? 4 : 2); }

// The squares of the sampled rows (runs of kPropRun neighbours at sample_stride apart), to
// Rs[c * S + i].
template <int P>
__global__ __launch_bounds__(kLmsBlock, 4) void lms_sample_kernel(
    const double *__restrict__ X, const double *__restrict__ y, const double *__restrict__ betas,
    int64_t n, int64_t m, int64_t chunk, double *__restrict__ Rs) {
  constexpr int T = kLmsTiles<P>;
  const int lane = threadIdx.x % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int S = sample_size(n);
  const int64_t stride = sample_stride(n, S);
  const int i0 = ((int)blockIdx.x * (kLmsBlock / kWave) + wv) * T * kWave;  // (S is a multiple)
  if (i0 >= S) return;
  double x[T][P], yv[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int i = i0 + t * kWave + lane;
    const int64_t row = (int64_t)(i / kPropRun) * stride + i % kPropRun;
#pragma unroll
    for (int j = 0; j < P; ++j) x[t][j] = X[row * P + j];
    yv[t] = y[row];
  }
  const int64_t c0 = (int64_t)blockIdx.y * chunk, c1 = c0 + chunk < m ? c0 + chunk : m;
  CPS_GLOBAL double *dst = (CPS_GLOBAL double *)Rs + c0 * S + i0 + lane;
  for (int64_t c = c0; c < c1; ++c) {
    double b[P];
#pragma unroll
    for (int j = 0; j < P; ++j) b[j] = betas[c * P + j];
#pragma unroll
    for (int t = 0; t < T; ++t) dst[t * kWave] = sq_residual<P>(x[t], yv[t], b, P);
    dst += S;
  }
}

// One workgroup per candidate: the likely interval [ka, kb] of its squares' rank from the sampled
// squares, in registers (sample_ends, 4.5 deviations: a miss in 10^5, and each costs a select
// over n), as the open interval (a, b) to ab[2c], ab[2c+1].  A candidate whose sample holds NaN gets
// (+inf, -inf): the filter then keeps nothing of it but NaN, and it goes down the materialised
// path.  1024 candidates: 76 us with the samples read again for every histogram, 51 us
// this way.
template <int PER>
__global__ __launch_bounds__(1024) void lms_bracket_kernel(const double *__restrict__ Rs, int64_t n,
                                                           int64_t k, double *__restrict__ ab) {
  constexpr int BLOCK = 1024;
  __shared__ uint32_t hist[4 * BLOCK];
  __shared__ RegSelShared<BLOCK> sh;
  const int64_t c = blockIdx.x;
  const CPS_GLOBAL double *src = (const CPS_GLOBAL double *)Rs + c * (BLOCK * PER) + threadIdx.x;
  double v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = src[j * BLOCK];
  uint64_t mn = ~0ull, mx = 0ull, key[PER];
  bool nan = false;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    nan = nan || !(v[j] == v[j]);
    key[j] = Traits<double>::key(v[j]);
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
  }
  nan = block_key_range<BLOCK>(mn, mx, nan, sh);
  double a = __builtin_inf(), b = -__builtin_inf();
  if (!nan) {  // (uniform)
    const SampleEnds<uint64_t> e = sample_ends<double, BLOCK, PER>(key, mn, mx, n, k, 4.5, hist, sh);
    // (squares are not negative: -1 lies below an open lower end, and below 0)
    const uint64_t kpos = Traits<double>::key(__builtin_inf());
    a = e.ka <= Traits<double>::key(0.0) ? -1.0 : Traits<double>::unkey(e.ka - 1);
    b = e.kb == kpos ? __builtin_inf() : Traits<double>::unkey(e.kb + 1);
  }
  if (threadIdx.x == 0) {
    ab[2 * c] = a;
    ab[2 * c + 1] = b;
  }
}

// The filter: every square r of the wavefront's rows (a segment of 64 T) and of `chunk`
// candidates.  Per candidate #(r <= a) is counted in scalar registers (SUM: their sum as well),
// and the r in (a, b), or NaN, are appended to the wavefront's region of R, one candidate's after
// another's, so that all stores are contiguous; the candidate's first place there, the number
// kept and the count below go to info[segment * m + candidate], 64 candidates at a time.
// A region holds all squares of the wavefront's rows and candidates: segment sg's and the
// candidates' from c0 on begin at (sg m + c0) rows per segment.  The kept squares pass through a
// wavefront's LDS list and are stored 64 at a time.
//
// Bound: double-precision arithmetic (2 p + 1 operations per square, each rounded as in the
// materialised form) and what keeping costs.  2^20 rows, p = 8, 1024 candidates: 0.54 ms of
// arithmetic at the rate measured (33.5 T/s), 640 us with its loads, 740 with the two
// comparisons, 975 with the keeping (1080 with a candidate per lane).  200003 rows, p = 5, 300
// candidates, with sums: 124 us a candidate per lane, 74 this way.
template <int P, bool SUM>
__global__ __launch_bounds__(kLmsBlock, 4) void lms_filter_kernel(
    const double *__restrict__ X, const double *__restrict__ y, const double *__restrict__ betas,
    const double *__restrict__ ab, int64_t n, int64_t m, int64_t chunk, double *__restrict__ R,
    uint2 *__restrict__ info, double *__restrict__ psum) {
  constexpr int T = kLmsTiles<P>;
  const int lane = threadIdx.x % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int64_t sg = (int64_t)blockIdx.x * (kLmsBlock / kWave) + wv, r0 = sg * (T * kWave);
  if (r0 >= n) return;
  const int64_t rows = n - r0 < T * kWave ? n - r0 : T * kWave;
  constexpr uint32_t kList = (T + 1) * kWave;
  __shared__ double lists[kLmsBlock / kWave][kList];
  CPS_LDS double *list = (CPS_LDS double *)lists[wv];
  double x[T][P], yv[T];
  uint64_t ok[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const bool valid = t * kWave + lane < rows;
    ok[t] = ballot(valid);
    const int64_t row = r0 + (valid ? t * kWave + lane : 0);
#pragma unroll
    for (int j = 0; j < P; ++j) x[t][j] = X[row * P + j];
    yv[t] = y[row];
  }
  const int64_t c0 = (int64_t)blockIdx.y * chunk, c1 = c0 + chunk < m ? c0 + chunk : m;
  CPS_GLOBAL double *region = (CPS_GLOBAL double *)uniform_ptr(R + (sg * m + c0) * (T * kWave));
  uint32_t out = 0, held = 0;  // stored, and in the list (below 64 before a candidate)
  // all whole wavefronts of the list, from its front; the rest moves there
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
    uint32_t at = 0;
    for (; held - at >= (uint32_t)kWave; at += kWave) region[out + at + lane] = list[at + lane];
    const double rest = list[at + lane < kList ? at + lane : 0];
    out += at;
    held -= at;
    __builtin_amdgcn_wave_barrier();
    if ((uint32_t)lane < held) list[lane] = rest;
    __builtin_amdgcn_wave_barrier();
  };
  for (int64_t cg = c0; cg < c1; cg += kWave) {
    const int lim = (int)(c1 - cg < kWave ? c1 - cg : kWave);
    uint32_t first = 0, num = 0;  // lane k: candidate cg + k's
    double sums = 0.0;
    for (int k = 0; k < lim; ++k) {
      const int64_t c = cg + k;
      double b[P];
#pragma unroll
      for (int j = 0; j < P; ++j) b[j] = betas[c * P + j];
      const double lo = ab[2 * c], hi = ab[2 * c + 1];
      double r[T], sum = 0.0;
#pragma unroll
      for (int t = 0; t < T; ++t) r[t] = x[t][0] * b[0];
#pragma unroll
      for (int j = 1; j < P; ++j) {  // (T independent sums advance together)
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const double q = x[t][j] * b[j];
          r[t] = r[t] + q;
        }
      }
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const double d = yv[t] - r[t];
        r[t] = d * d;
      }
      uint32_t below = 0;
      const uint32_t at = out + held;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint64_t le = ballot(r[t] <= lo) & ok[t];
        const uint64_t in = ok[t] & ~(le | ballot(r[t] >= hi));
        below += popc(le);
        if (SUM) sum += __builtin_amdgcn_inverse_ballot_w64(le) ? r[t] : 0.0;
        if (__builtin_amdgcn_inverse_ballot_w64(in))
          list[__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, held))] = r[t];
        held += popc(in);
      }
      const uint32_t num_kept = out + held - at;
      const bool mine = __builtin_amdgcn_inverse_ballot_w64(1ull << k);
      first = mine ? at : first;
      num = mine ? num_kept | (below << 16) : num;
      if (held >= (uint32_t)kWave) flush();
      if (SUM) {
        sum = wave_sum(sum);
        sums = mine ? sum : sums;
      }
    }
    if (lane < lim) {
      info[sg * m + cg + lane] = uint2{first, num};
      if (SUM) psum[sg * m + cg + lane] = sums;
    }
  }
  __builtin_amdgcn_wave_barrier();
  if ((uint32_t)lane < held) region[out + lane] = list[lane];
}

constexpr int kLmsGatherBlock = 256;

// ---- the filtered form's finish: one workgroup's exact select (cps_wgsel.h) over an array

// elements a narrowed key range may hold to finish in LDS (a candidate selected over all its n
// squares)
constexpr int kLmsSelCap = 992;
using WgSelLds = WgSelShared<kLmsGatherBlock>;

// The k-th smallest of W[0, len) (wg_select_pass over the array, eight loads per step).
template <int BLOCK>
__device__ __forceinline__ WgSelOut wg_select(const double *W, int64_t len, int64_t k, uint64_t klo,
                              uint64_t khi, int64_t below0, int64_t inrange0, uint32_t *hist,
                              double *buf, WgSelLds &sh) {
  const CPS_GLOBAL double *Wg = (const CPS_GLOBAL double *)W;
  auto pass = [&](auto f) { for_each8<BLOCK>(Wg, len, f); };
  return wg_select_pass<double, BLOCK>(pass, k, klo, khi, below0, inrange0, hist, buf,
                                       kLmsSelCap, sh);
}

// The record of a selection among all n squares.
__device__ inline void lms_write_result(cps_result *out, uint64_t key, int64_t less,
                                        int64_t equal, int64_t n, int32_t passes) {
  cps_result r;
  const double v = Traits<double>::unkey(key);
  r.value_bits = __builtin_bit_cast(uint64_t, v);
  r.value = v;
  r.less = less;
  r.equal = equal;
  r.greater = n - less - equal;
  r.passes = passes;
  r.status = CPS_STATUS_OK;
  *out = r;
}

__device__ inline void lms_write_nan(cps_result *out, int32_t passes) {
  cps_result r;
  r.value = __builtin_nan("");
  r.value_bits = __builtin_bit_cast(uint64_t, r.value);
  r.less = r.equal = r.greater = 0;
  r.passes = passes;
  r.status = CPS_STATUS_NAN;
  *out = r;
}

// The sum of the k smallest of a candidate's n squares: below (the squares under the
// selection's bracket, if any) plus those of W[0, len) below the selected value v, plus
// (k - #(r < v)) v (Section 6's trimmed sum with the multiplicity of v); one more pass over W.
template <int BLOCK>
__device__ inline double lms_ksum(const CPS_GLOBAL double *W, int64_t len, double v, int64_t k,
                                  int64_t less, double below, Sum2 *red) {
  double part = 0.0;
  for_each8<BLOCK>(W, len, [&](double r) {
    if (r < v) part += r;
  });
  const Sum2 s = block_sum2<BLOCK>(Sum2{part, 0.0}, red);
  return value(sum2(sum2(Sum2{below, 0.0}, s), product2((double)(k - less), v)));
}

// One workgroup per candidate: the segments' counts and the bracket's test; where it holds, the
// kept squares, read where the filter left them (eight lanes per segment, whose ~8 squares are
// contiguous; the next candidate's follow, so neighbouring candidates run on one XCD and share
// the lines), counted in 2^11 key bins over the bracket, and the rank's bin once more to rank
// its few squares.  Where it does not hold, full[c] = 1 and the candidate's whole array is formed and
// selected by the two kernels that follow.  passes: the filter and the two readings.
// (1024 candidates of 37 000 squares: 252 us; 300 of 14 000 with sums: 56, where packing
// the squares first and selecting among those took 86.)
constexpr int kLmsSelBlock = 512, kLmsSelSegs = 4096;
__global__ __launch_bounds__(kLmsSelBlock, 8) void lms_select_kernel(
    const double *__restrict__ R, const uint2 *__restrict__ info, const double *__restrict__ ab,
    int64_t n, int64_t m, int64_t nseg, int64_t seg, int64_t chunk, int64_t k,
    const double *__restrict__ psum, cps_result *__restrict__ out, double *__restrict__ ksum,
    int32_t *__restrict__ full) {
  constexpr int BLOCK = kLmsSelBlock, G = 8, NG = BLOCK / G, U = 4;
  __shared__ uint32_t first[kLmsSelSegs];
  __shared__ uint16_t kept[kLmsSelSegs];
  __shared__ uint32_t hist[4 * BLOCK];
  __shared__ uint64_t fin[kWalkFinal];
  __shared__ RegSelShared<BLOCK> sh;
  __shared__ double wred[BLOCK / kWave];
  __shared__ Sum2 sums[BLOCK / kWave];
  const int64_t per = (m + 7) / 8, c = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (c >= m) return;
  const int tid = threadIdx.x;
  const int64_t hop = seg * m;
  const CPS_GLOBAL double *Rc = (const CPS_GLOBAL double *)R + c / chunk * chunk * seg;
  auto load = [&](int64_t s0, uint64_t &in, uint64_t &bel) {
    const int cnt = (int)(nseg - s0 < kLmsSelSegs ? nseg - s0 : kLmsSelSegs);
    for (int i0 = tid; i0 < cnt; i0 += U * BLOCK) {
      uint2 w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * BLOCK;
        w[u] = info[(s0 + (i < cnt ? i : 0)) * m + c];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * BLOCK;
        if (i < cnt) {
          first[i] = w[u].x;
          kept[i] = (uint16_t)(w[u].y & 0xffffu);
          in += w[u].y & 0xffffu;
          bel += w[u].y >> 16;
        }
      }
    }
    return cnt;
  };
  const int grp = tid / G, l = tid % G;
  auto walk = [&](auto &&one) {
    for (int64_t s0 = 0; s0 < nseg; s0 += kLmsSelSegs) {
      int cnt = (int)nseg;
      if (nseg > kLmsSelSegs) {  // (not all in LDS: read again)
        uint64_t a = 0, b = 0;
        __syncthreads();
        cnt = load(s0, a, b);
        __syncthreads();
      }
      for (int i0 = grp; i0 < cnt; i0 += U * NG) {
        const CPS_GLOBAL double *p[U];
        int num[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int i = i0 + u * NG < cnt ? i0 + u * NG : i0;
          num[u] = i0 + u * NG < cnt ? (int)kept[i] : 0;
          p[u] = Rc + (s0 + i) * hop + first[i];
          v[u] = p[u][l < num[u] ? l : 0];  // (with none kept: a place inside the workspace)
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          one(v[u], l < num[u]);
          for (int e = l + G; e < num[u]; e += G) one(p[u][e], true);
        }
      }
    }
  };
  uint64_t in = 0, bel = 0;
  for (int64_t s0 = 0; s0 < nseg; s0 += kLmsSelSegs) load(s0, in, bel);
  const int64_t inside = (int64_t)block_sum_fixed<BLOCK>((double)in, wred);
  const int64_t below = (int64_t)block_sum_fixed<BLOCK>((double)bel, wred);
  const double lo = ab[2 * c], hi = ab[2 * c + 1];
  const bool holds = lo < hi && below < k && k <= below + inside;
  if (tid == 0) full[c] = holds ? 0 : 1;
  if (!holds) return;  // (uniform)
  // the keys of a < r < b
  const uint64_t ka = Traits<double>::key(lo) + 1, kb = Traits<double>::key(hi) - 1;
  const int shift = range_shift(kb - ka, quick_bins_log2(BLOCK));
  *reinterpret_cast<uint4 *>(&hist[4 * tid]) = uint4{0u, 0u, 0u, 0u};
  __syncthreads();
  bool nan = false;
  walk([&](double v, bool ok) {
    nan = nan | (ok & !(v == v));
    const uint64_t d = Traits<double>::key(v) - ka;
    if (ok & (d <= kb - ka)) atomicAdd(&hist[(uint32_t)(d >> shift)], 1u);
  });
  if (__syncthreads_or(nan)) {  // (uniform)
    if (tid == 0) {
      lms_write_nan(out + c, 2);
      if (ksum) ksum[c] = __builtin_nan("");
    }
    return;
  }
  const uint4 q = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
  uint32_t h[4] = {q.x, q.y, q.z, q.w};
  uint64_t key;
  int64_t less, equal;
  walk_select<double, BLOCK>(walk, h, k - below, ka, kb, hist, fin, sh, key, less, equal);
  if (equal == 0) {  // (uniform)
    if (tid == 0) {
      write_selection(out + c, 0, __builtin_nan(""), 0, 0, n, 3, CPS_STATUS_INTERNAL);
      if (ksum) ksum[c] = __builtin_nan("");
    }
    return;
  }
  if (tid == 0) lms_write_result(out + c, key, below + less, equal, n, 3);
  if (ksum) {  // (uniform)
    const double v = Traits<double>::unkey(key);
    double sb = 0.0, part = 0.0;
    for (int64_t s = tid; s < nseg; s += BLOCK) sb += psum[s * m + c];
    walk([&](double r, bool ok) { part += ok && r < v ? r : 0.0; });
    const Sum2 under = block_sum2<BLOCK>(Sum2{sb, 0.0}, sums);
    const Sum2 mid = block_sum2<BLOCK>(Sum2{part, 0.0}, sums);
    if (tid == 0) ksum[c] = value(sum2(sum2(under, mid), product2((double)(k - below - less), v)));
  }
}

// After the fallback residual kernel: the candidates whose bracket missed, over their whole
// arrays of n squares (a first pass for the key range and NaN, then wg_select); the others'
// workgroups return at once.
__global__ __launch_bounds__(kLmsGatherBlock) void lms_full_select_kernel(
    const double *__restrict__ R, int64_t n, int64_t k, const int32_t *__restrict__ full,
    cps_result *__restrict__ out, double *__restrict__ ksum) {
  __shared__ uint32_t hist[kHistMaxBins];
  __shared__ double buf[kLmsSelCap];
  __shared__ WgSelLds sh;
  __shared__ Sum2 sums[kLmsGatherBlock / kWave];
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  if (full[c] == 0) return;  // (uniform)
  if (tid == 0) {
    sh.kext[0] = ~0ull;
    sh.kext[1] = 0ull;
    sh.flag = 0u;
  }
  __syncthreads();
  const CPS_GLOBAL double *Rc = (const CPS_GLOBAL double *)(R + c * n);
  uint64_t kmn = ~0ull, kmx = 0ull;
  bool nan = false;
  for_each8<kLmsGatherBlock>(Rc, n, [&](double v) {
    const uint64_t kk = Traits<double>::key(v);
    nan = nan || !(v == v);
    kmn = kk < kmn ? kk : kmn;
    kmx = kk > kmx ? kk : kmx;
  });
  atomicMin(&sh.kext[0], (unsigned long long)kmn);
  atomicMax(&sh.kext[1], (unsigned long long)kmx);
  if (nan) atomicOr(&sh.flag, 1u);
  __syncthreads();
  if (sh.flag != 0u) {  // (uniform)
    if (tid == 0) {
      lms_write_nan(out + c, 3);
      if (ksum) ksum[c] = __builtin_nan("");
    }
    return;
  }
  const WgSelOut r = wg_select<kLmsGatherBlock>(R + c * n, n, k, sh.kext[0], sh.kext[1], 0, n,
                                                hist, buf, sh);
  if (tid == 0) lms_write_result(out + c, r.key, r.less, r.equal, n, 3 + r.passes);
  if (ksum) {  // (uniform)
    const double t = lms_ksum<kLmsGatherBlock>(Rc, n, Traits<double>::unkey(r.key), k, r.less,
                                               0.0, sums);
    if (tid == 0) ksum[c] = t;
  }
}

__global__ void lms_descriptor_kernel(const double *R, int64_t n, int64_t m, int64_t rank,
                                      const double **ptrs, int64_t *sizes, int64_t *ks) {
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < m;
       c += (int64_t)gridDim.x * blockDim.x) {
    ptrs[c] = R + c * n;
    sizes[c] = n;
    ks[c] = rank;
  }
}

// Least trimmed squares (Section 6): from the selection of rank h among a candidate's squared
// residuals (m = r_(h), #(r < m), #(r = m)) and the sum of its h smallest, the record with
// a = h - #(r < m), the weight of m in Section 6's rho.
__global__ void lts_finish_kernel(const cps_result *__restrict__ sel, const double *__restrict__ ksum,
                                  int64_t m, int64_t h, cps_trim *__restrict__ out) {
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < m;
       c += (int64_t)gridDim.x * blockDim.x) {
    const cps_result r = sel[c];
    cps_trim t;
    t.F = r.status == 0 ? ksum[c] : __builtin_nan("");
    t.m = r.value;
    t.below = r.less;
    t.a = r.status == 0 ? h - r.less : 0;
    t.b = r.equal;
    t.status = r.status;
    t.pad = 0;
    out[c] = t;
  }
}

hipError_t launch_lts_finish(const cps_result *sel, const double *ksum, int64_t m, int64_t h,
                             cps_trim *out, hipStream_t stream) {
  lts_finish_kernel<<<dim3((unsigned)((m + 255) / 256)), dim3(256), 0, stream>>>(sel, ksum, m, h, out);
  return hipGetLastError();
}

hipError_t launch_lms_residuals(const double *X, const double *y, const double *betas, int64_t n,
                                int32_t p, int64_t m, int64_t rank, double *R, const double **ptrs,
                                int64_t *sizes, int64_t *ks, int cu_count, hipStream_t stream) {
  const int64_t groups = (m + kLmsGroup - 1) / kLmsGroup;
  int64_t bx = (n + kLmsBlock - 1) / kLmsBlock;
  const int64_t want = (int64_t)cu_count * 8 / (groups < 1 ? 1 : groups) + 1;
  if (bx > want) bx = want;
  if (bx < 1) bx = 1;
  const dim3 grid((unsigned)bx, (unsigned)groups);
  const bool aligned = ((uintptr_t)X % 16 == 0) && ((uintptr_t)y % 16 == 0) && ((uintptr_t)R % 16 == 0);
  if (p == 8 && aligned && n % kLmsRows == 0) {
    const int64_t rb = (n / kLmsRows + kLmsBlock - 1) / kLmsBlock;
    const dim3 g2((unsigned)(bx < rb ? bx : rb), (unsigned)groups);
    lms_residual_rows_kernel<8, kLmsRows, false>
        <<<g2, dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, m, R, nullptr);
  } else if (p == 8) {
    lms_residual_kernel<8, false><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, p, m, R, nullptr);
  } else {
    lms_residual_kernel<0, false><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, p, m, R, nullptr);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  lms_descriptor_kernel<<<dim3((unsigned)((m + 255) / 256)), dim3(256), 0, stream>>>(R, n, m, rank,
                                                                                    ptrs, sizes, ks);
  return hipGetLastError();
}

void lms_filter_shape(int64_t n, int64_t m, int32_t p, int cu_count, int64_t *bx, int64_t *nseg,
                      int64_t *seg, int64_t *chunk) {
  // the filter: a wavefront per segment and chunk of candidates (a multiple of 64), two rounds of
  // four wavefronts per SIMD or more where there are that many
  *seg = lms_seg(p);
  *nseg = (n + *seg - 1) / *seg;
  const int64_t want = (2 * 16 * (int64_t)cu_count + *nseg - 1) / *nseg;
  const int64_t most = (m + kWave - 1) / kWave;
  const int64_t chunks = want < 1 ? 1 : (want < most ? want : most);
  *chunk = ((m + chunks - 1) / chunks + kWave - 1) / kWave * kWave;
  // the fallback residual kernel's grid, as the materialised form's
  const int64_t groups = (m + kLmsGroup - 1) / kLmsGroup;
  int64_t b = (n + kLmsBlock - 1) / kLmsBlock;
  const int64_t fb = (int64_t)cu_count * 8 / groups + 1;
  if (b > fb) b = fb;
  *bx = b < 1 ? 1 : b;
}

// The sample's and the filter's kernels have an instance for every p: the columns' loops unroll.
template <int P>
static void launch_lms_sample(const double *X, const double *y, const double *betas, int64_t n,
                              int32_t p, int64_t m, double *Rs, hipStream_t stream) {
  if constexpr (P > 1)
    if (p < P) return launch_lms_sample<P - 1>(X, y, betas, n, p, m, Rs, stream);
  constexpr int64_t chunk = 32;
  const int per = kLmsBlock * kLmsTiles<P>;
  const dim3 grid((unsigned)((sample_runs(n) * kPropRun + per - 1) / per), (unsigned)((m + chunk - 1) / chunk));
  lms_sample_kernel<P><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, m, chunk, Rs);
}
template <int P>
static void launch_lms_filter(const double *X, const double *y, const double *betas, int64_t n,
                              int32_t p, int64_t m, const LmsFilterBufs &w, bool sum,
                              hipStream_t stream) {
  if constexpr (P > 1)
    if (p < P) return launch_lms_filter<P - 1>(X, y, betas, n, p, m, w, sum, stream);
  constexpr int W = kLmsBlock / kWave;
  const dim3 grid((unsigned)((w.nseg + W - 1) / W), (unsigned)((m + w.chunk - 1) / w.chunk));
  if (sum)
    lms_filter_kernel<P, true><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, w.ab, n, m, w.chunk,
                                                                      w.R, w.info, w.psum);
  else
    lms_filter_kernel<P, false><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, w.ab, n, m, w.chunk,
                                                                       w.R, w.info, nullptr);
}

hipError_t launch_lms_filtered(const double *X, const double *y, const double *betas, int64_t n,
                               int32_t p, int64_t m, int64_t rank, const LmsFilterBufs &w,
                               cps_result *out, double *ksum, hipStream_t stream) {
  const int64_t groups = (m + kLmsGroup - 1) / kLmsGroup;
  launch_lms_sample<16>(X, y, betas, n, p, m, w.Rs, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (sample_runs(n) * kPropRun == kPropSampleBig)
    lms_bracket_kernel<kPropSampleBig / 1024><<<dim3((unsigned)m), dim3(1024), 0, stream>>>(w.Rs, n, rank, w.ab);
  else
    lms_bracket_kernel<kPropSample / 1024><<<dim3((unsigned)m), dim3(1024), 0, stream>>>(w.Rs, n, rank, w.ab);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool aligned = ((uintptr_t)X % 16 == 0) && ((uintptr_t)y % 16 == 0);
  launch_lms_filter<16>(X, y, betas, n, p, m, w, ksum != nullptr, stream);
  const dim3 grid((unsigned)w.bx, (unsigned)groups);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  lms_select_kernel<<<dim3((unsigned)((m + 7) / 8 * 8)), dim3(kLmsSelBlock), 0, stream>>>(
      w.R, w.info, w.ab, n, m, w.nseg, w.seg, w.chunk, rank, w.psum, out, ksum, w.full);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the candidates whose bracket missed: their whole arrays (workgroups without one return)
  if (p == 8 && aligned && (uintptr_t)w.R % 16 == 0 && n % kLmsRows == 0) {
    int64_t rb = (n / kLmsRows + kLmsBlock - 1) / kLmsBlock;
    if (rb > w.bx) rb = w.bx;
    lms_residual_rows_kernel<8, kLmsRows, true>
        <<<dim3((unsigned)rb, (unsigned)groups), dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, m, w.R,
                                                                           w.full);
  } else {
    lms_residual_kernel<0, true><<<grid, dim3(kLmsBlock), 0, stream>>>(X, y, betas, n, p, m, w.R,
                                                                        w.full);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  lms_full_select_kernel<<<dim3((unsigned)m), dim3(kLmsGatherBlock), 0, stream>>>(w.R, n, rank,
                                                                                w.full, out, ksum);
  return hipGetLastError();
}

}  // namespace cps
