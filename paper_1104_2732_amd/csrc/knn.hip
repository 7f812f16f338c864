// k nearest neighbours (Section 6, last paragraph): for each query point, the squared
// Euclidean distances to every data point, their k-th smallest d_k by the batched selection,
// and the mean ordinate of the k nearest points, formed by a reduction with the weight of
// Section 6's rho adapted to an indicator: 1 below d_k, a/b at d_k (b points at d_k, a = k -
// #(d < d_k) of them count), 0 above.
//
// The distance kernel forms d_i = sum_j (P_ij - q_j)^2 for a group of queries per thread row
// (each data point read once per group), left to right in j with every difference, square
// and sum rounded on its own in float (the library is built without fused multiply-add), and
// writes them query-major, one array of n per query.  The reduction reads the distance
// arrays back (one read of 4 bytes per distance; recomputing them from the points instead
// reads the points once per query from the caches and measured 13 % slower in all) and sums
// the ordinates below and at d_k in double precision, per block in a fixed order, then per
// query in block order.
#include "cps_device.h"
#include "cps_kernels.h"
#include "cps_quick.h"
#include "cps_passes.h"
#include "cps_sample.h"
#include "cps_wgsel.h"

namespace cps {

#ifndef CPS_KNN_GROUP
#define CPS_KNN_GROUP 64
#endif
#ifndef CPS_KNN_READ
#define CPS_KNN_READ 1
#endif
constexpr int kKnnGroup = CPS_KNN_GROUP;  // queries per thread row of the distance kernel
// the reduction reads the distance arrays back (1) or recomputes the distances (0)
constexpr bool kKnnRead = CPS_KNN_READ != 0;
constexpr int kKnnBlock = 256;
constexpr int kKnnRedBlocks = 8;  // reduction blocks per query

template <int D>
__device__ inline float knn_dist(const float (&row)[D > 0 ? D : 16], const float *q, int dim) {
  const int dd = D > 0 ? D : dim;
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < (D > 0 ? D : 16); ++j) {
    if (j < dd) {
      const float e = row[j] - q[j];
      const float sq = e * e;
      s = j == 0 ? sq : s + sq;
    }
  }
  return s;
}

template <int D>
__global__ __launch_bounds__(kKnnBlock) void knn_distance_kernel(
    const float *__restrict__ P, const float *__restrict__ Q, int64_t n, int32_t dim, int64_t nq,
    float *__restrict__ Dst) {
  __shared__ float sq[kKnnGroup * 16];  // (up to 16 coordinates per query)
  const int64_t c0 = (int64_t)blockIdx.y * kKnnGroup;
  const int nc = (int)((nq - c0) < kKnnGroup ? (nq - c0) : kKnnGroup);
  for (int t = threadIdx.x; t < nc * dim; t += kKnnBlock) sq[t] = Q[c0 * dim + t];
  __syncthreads();
  const CPS_GLOBAL float *Pg = (const CPS_GLOBAL float *)P;
  CPS_GLOBAL float *Dg = (CPS_GLOBAL float *)Dst;
  for (int64_t i = (int64_t)blockIdx.x * kKnnBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kKnnBlock) {
    float row[D > 0 ? D : 16];
    const int dd = D > 0 ? D : dim;
#pragma unroll
    for (int j = 0; j < (D > 0 ? D : 16); ++j)
      if (j < dd) row[j] = Pg[i * dd + j];
    for (int c = 0; c < nc; ++c)
      __builtin_nontemporal_store(knn_dist<D>(row, sq + c * dd, dim), &Dg[(c0 + c) * n + i]);
  }
}

__global__ void knn_descriptor_kernel(const float *Dst, int64_t n, int64_t nq, int64_t k,
                                      const float **ptrs, int64_t *sizes, int64_t *ks) {
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nq;
       c += (int64_t)gridDim.x * blockDim.x) {
    ptrs[c] = Dst + c * n;
    sizes[c] = n;
    ks[c] = k;
  }
}

// Partial sums of the ordinates below and at d_k over this block's slice of the points.
template <int D>
__global__ __launch_bounds__(kKnnBlock) void knn_partial_kernel(
    const float *__restrict__ P, const float *__restrict__ f, const float *__restrict__ Q,
    int64_t n, int32_t dim, const cps_result *__restrict__ sel, double *__restrict__ pd,
    int64_t *__restrict__ pi) {
  __shared__ double sd[8][kKnnBlock / kWave];
  __shared__ int64_t si[8][kKnnBlock / kWave];
  __shared__ float sq[16];
  const int64_t c = blockIdx.y;
  if (threadIdx.x < dim) sq[threadIdx.x] = Q[c * dim + threadIdx.x];
  __syncthreads();
  const float dk = (float)sel[c].value;
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < n ? lo + per : n;
  double sb = 0.0, se = 0.0;
  int64_t nb = 0, ne = 0;
  const int dd = D > 0 ? D : dim;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kKnnBlock) {
    float row[D > 0 ? D : 16];
#pragma unroll
    for (int j = 0; j < (D > 0 ? D : 16); ++j)
      if (j < dd) row[j] = P[i * dd + j];
    const float d = knn_dist<D>(row, sq, dim);
    const double fi = (double)f[i];
    if (d < dk) {
      sb += fi;
      ++nb;
    } else if (d == dk) {
      se += fi;
      ++ne;
    }
  }
  double dv[8] = {sb, se, 0, 0, 0, 0, 0, 0};
  int dop[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int64_t iv[8] = {nb, ne, 0, 0, 0, 0, 0, 0};
  block_reduce<kKnnBlock, 2, 2>(dv, dop, iv, false, sd, si);
  if (threadIdx.x == 0) {
    const int64_t slot = c * gridDim.x + blockIdx.x;
    pd[2 * slot] = dv[0];
    pd[2 * slot + 1] = dv[1];
    pi[2 * slot] = iv[0];
    pi[2 * slot + 1] = iv[1];
  }
}

// The same partial sums from the distance arrays the distance kernel wrote (query c's at
// D + c n): 16-byte loads of distances and ordinates when n is a multiple of 4.
template <bool VEC>
__global__ __launch_bounds__(kKnnBlock) void knn_partial_read_kernel(
    const float *__restrict__ D, const float *__restrict__ f, int64_t n,
    const cps_result *__restrict__ sel, double *__restrict__ pd, int64_t *__restrict__ pi) {
  __shared__ double sd[8][kKnnBlock / kWave];
  __shared__ int64_t si[8][kKnnBlock / kWave];
  const int64_t c = blockIdx.y;
  const float dk = (float)sel[c].value;
  int64_t per = (n + gridDim.x - 1) / gridDim.x;
  per = (per + 3) / 4 * 4;
  const int64_t lo = (int64_t)blockIdx.x * per;
  const int64_t hi = lo + per < n ? lo + per : n;
  const float *Dr = D + c * n;
  double sb = 0.0, se = 0.0;
  int64_t nb = 0, ne = 0;
  auto one = [&](float d, float fi) {
    if (d < dk) {
      sb += (double)fi;
      ++nb;
    } else if (d == dk) {
      se += (double)fi;
      ++ne;
    }
  };
  if (VEC) {
    using F4 = float __attribute__((ext_vector_type(4)));
    for (int64_t i = lo + 4 * (int64_t)threadIdx.x; i < hi; i += 4 * (int64_t)kKnnBlock) {
      const F4 d = __builtin_nontemporal_load((const F4 *)(Dr + i));
      const F4 fv = *(const F4 *)(f + i);
      one(d.x, fv.x);
      one(d.y, fv.y);
      one(d.z, fv.z);
      one(d.w, fv.w);
    }
  } else {
    for (int64_t i = lo + threadIdx.x; i < hi; i += kKnnBlock) one(Dr[i], f[i]);
  }
  double dv[8] = {sb, se, 0, 0, 0, 0, 0, 0};
  int dop[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int64_t iv[8] = {nb, ne, 0, 0, 0, 0, 0, 0};
  block_reduce<kKnnBlock, 2, 2>(dv, dop, iv, false, sd, si);
  if (threadIdx.x == 0) {
    const int64_t slot = c * gridDim.x + blockIdx.x;
    pd[2 * slot] = dv[0];
    pd[2 * slot + 1] = dv[1];
    pi[2 * slot] = iv[0];
    pi[2 * slot + 1] = iv[1];
  }
}

__global__ void knn_final_kernel(int64_t nq, int64_t k, int nb, const cps_result *__restrict__ sel,
                                 const double *__restrict__ pd, const int64_t *__restrict__ pi,
                                 cps_knn *__restrict__ out) {
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nq;
       c += (int64_t)gridDim.x * blockDim.x) {
    double sb = 0.0, se = 0.0;
    int64_t below = 0, eq = 0;
    for (int b = 0; b < nb; ++b) {
      sb += pd[2 * (c * nb + b)];
      se += pd[2 * (c * nb + b) + 1];
      below += pi[2 * (c * nb + b)];
      eq += pi[2 * (c * nb + b) + 1];
    }
    const cps_result r = sel[c];
    cps_knn o;
    o.dk = (float)r.value;
    o.status = r.status;
    o.below = below;
    o.equal = eq;
    // the reduction's counts are the selection's (anything else: the data changed)
    if (r.status == 0 && (below != r.less || eq != r.equal)) o.status = CPS_STATUS_INTERNAL;
    const double a = (double)(k - below);
    o.mean = (o.status == 0 && eq > 0) ? (sb + a * se / (double)eq) / (double)k
                                       : __builtin_nan("");
    out[c] = o;
  }
}

// ------------------------------------------------------------------ the filtered form
//
// For small k the k nearest are a sliver of the n points: a sampled bracket (a, b) of each
// query's distances (the batched kernel's rule over the distances of the sampled points)
// keeps only the distances in (a, b), with their ordinates, and the selection and the
// reductions run over those.  #(d <= a) and the ordinates' sum there come from the same
// pass; a query whose bracket does not hold d_k (or keeps more than kKnnCap) is selected by
// its own workgroup over recomputed distances.  Results equal the materialised form's.

constexpr int kKnnCap = (int)kKnnKeptCap;  // (the select holds them in LDS)

// d = sum_j (P_ij - q_j)^2 for a row and a query both in registers, in the order knn_dist uses
template <int D>
__device__ __forceinline__ float knn_dist_reg(const float (&row)[D > 0 ? D : 16],
                                              const float (&qv)[D > 0 ? D : 16], int dim) {
  const int dd = D > 0 ? D : dim;
  float s = 0.0f;
#pragma unroll
  for (int j = 0; j < (D > 0 ? D : 16); ++j) {
    if (j < dd) {
      const float e = row[j] - qv[j];
      const float sq = e * e;
      s = j == 0 ? sq : s + sq;
    }
  }
  return s;
}

// ---- the screen's constants and operands (see knn_screen_kernel)

constexpr int kScrWaves = 4;
constexpr int kScrBlock = kScrWaves * kWave;
constexpr int kScrTile = 32;         // points and queries per tile
constexpr int kScrK = 16;            // terms per matrix instruction
constexpr int kScrList = 2 * kWave;  // pairs a wavefront's list holds
constexpr float kScrNormMax = 1e37f;
constexpr float kScrMargin = 0x1p-14f;
constexpr int kScrQt = 4;            // query tiles per wavefront (one where there are few queries)
constexpr int kScrPerCu = 4;         // workgroups per CU, all resident at once
constexpr double kScrPart = 1.0 / 24.0;  // see knn_use_screen

// The terms of the screen: slot s < 3 dim is coordinate s % dim of the products hi.hi (s / dim
// = 0), hi.lo (1) and lo.hi (2), points first; the next two are the point's norm in two parts
// times one; the slots up to a whole instruction are zero.
struct ScreenSlot {
  int j;
  bool product, lo_p, lo_q;
  int norm;  // 1, 2: the norm's parts
};
__host__ __device__ constexpr __forceinline__ int screen_steps(int dim) { return (3 * dim + 2 + kScrK - 1) / kScrK; }
__device__ __forceinline__ ScreenSlot screen_slot(int s, int dim) {
  const int g = s < dim ? 0 : (s < 2 * dim ? 1 : 2);
  const bool pr = s < 3 * dim;
  return {pr ? s - g * dim : 0, pr, g == 2, g == 1, !pr && s < 3 * dim + 2 ? s - 3 * dim + 1 : 0};
}
__device__ __forceinline__ __bf16 bf16_part(float v, bool lo) {
  const __bf16 hi = (__bf16)v;
  return lo ? (__bf16)(v - (float)hi) : hi;
}
using BF8 = __bf16 __attribute__((ext_vector_type(8)));

// The distances of the sampled points (runs of kPropRun at sample_stride apart) to
// Ds[query * S + i]: kSmpTiles points per lane, the queries of a chunk as scalar loads, so that a
// store is a whole line of one query's array (a query per lane, its run as 16-byte stores of one
// 64-byte line: 34 us for 1024 queries x 16384 samples, this 18).  The first workgroup
// also leaves the mean of 64 points spread over P in centre[0, dim) (a coordinate whose mean
// is not an ordinary number: 0), which the screen takes as its origin; any origin gives the
// same results.
constexpr int kSmpTiles = 4, kSmpChunk = 32;
template <int D>
__global__ __launch_bounds__(kKnnBlock) void knn_sample_kernel(
    const float *__restrict__ P, const float *__restrict__ Q, int64_t n, int32_t dim, int64_t nq,
    float *__restrict__ Ds, float *__restrict__ centre) {
  constexpr int DM = D > 0 ? D : 16;
  const int dd = D > 0 ? D : dim;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kWave) {
    const int64_t i = (int64_t)threadIdx.x * (n / kWave);
    for (int j = 0; j < dd; ++j) {
      const double s = wave_sum((double)P[i * dd + j]) / kWave;
      if (threadIdx.x == 0) centre[j] = fabs(s) < 1e18 ? (float)s : 0.0f;
    }
  }
  const int S = sample_size(n);
  const int64_t stride = sample_stride(n, S);
  const int i0 = (int)blockIdx.x * kKnnBlock * kSmpTiles + threadIdx.x;  // (S is a multiple)
  float row[kSmpTiles][DM];
#pragma unroll
  for (int t = 0; t < kSmpTiles; ++t) {
    const int i = i0 + t * kKnnBlock;
    const int64_t r = (int64_t)(i / kPropRun) * stride + i % kPropRun;
#pragma unroll
    for (int j = 0; j < DM; ++j) row[t][j] = j < dd ? P[r * dd + j] : 0.0f;
  }
  const int64_t q0 = (int64_t)blockIdx.y * kSmpChunk, q1 = q0 + kSmpChunk < nq ? q0 + kSmpChunk : nq;
  CPS_GLOBAL float *dst = (CPS_GLOBAL float *)Ds + q0 * S + i0;
  for (int64_t q = q0; q < q1; ++q) {
    float qv[DM];
#pragma unroll
    for (int j = 0; j < DM; ++j) qv[j] = j < dd ? Q[q * dd + j] : 0.0f;
#pragma unroll
    for (int t = 0; t < kSmpTiles; ++t) dst[t * kKnnBlock] = knn_dist_reg<D>(row[t], qv, dim);
    dst += S;
  }
}

// One workgroup per query: its sampled bracket to ab[2c], ab[2c+1] ((+inf, -inf) where there
// is none: the filter then keeps nothing but NaN and the select recomputes), and the filter's
// counters of c cleared.  The sample stays in registers (sample_ends); read again for every
// histogram by 256 threads, 1024 queries took 45 us, this way 21.
// With the screen (nm > 0), also the query's operands: -2 q' (exact scaling) in slot order and
// the threshold (a query that is not screened: zero terms, and everything passes).
template <int PER>
__global__ __launch_bounds__(1024) void knn_bracket_kernel(
    const float *__restrict__ Ds, const float *__restrict__ Q, const float *__restrict__ centre,
    int64_t n, int32_t dim, int64_t k, int64_t nq, int32_t nm, float *__restrict__ ab,
    uint32_t *__restrict__ cnt, double *__restrict__ fsum, __bf16 *__restrict__ B,
    float *__restrict__ T) {
  constexpr int BLOCK = 1024;
  __shared__ uint32_t hist[4 * BLOCK];
  __shared__ RegSelShared<BLOCK> sh;
  const int64_t c = blockIdx.x;
  if (threadIdx.x < 2) cnt[c * kKnnCntStride + threadIdx.x] = 0u;
  if (threadIdx.x == 2) fsum[c] = 0.0;
  using F4 = float __attribute__((ext_vector_type(4)));
  const CPS_GLOBAL F4 *src = (const CPS_GLOBAL F4 *)(Ds + c * (BLOCK * PER)) + threadIdx.x;
  F4 v[PER / 4];
#pragma unroll
  for (int j = 0; j < PER / 4; ++j) v[j] = src[j * BLOCK];
  uint32_t mn = ~0u, mx = 0u, key[PER];
  bool bad = false;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const float w = v[j / 4][j % 4];
    bad = bad || !(w < __builtin_inff());
    key[j] = Traits<float>::key(w);
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
  }
  bad = block_key_range<BLOCK>(mn, mx, bad, sh);
  float a = 0.0f, b = 0.0f;
  bool use = !bad && mn < mx;  // (uniform)
  if (use) {
    const SampleEnds<uint32_t> e = sample_ends<float, BLOCK, PER>(key, mn, mx, n, k, 4.0, hist, sh);
    // (distances are not negative: nothing lies below 0)
    const uint32_t kpos = Traits<float>::key(__builtin_inff());
    a = e.ka <= Traits<float>::key(0.0f) ? -__builtin_inff() : Traits<float>::unkey(e.ka - 1u);
    b = e.kb == kpos ? __builtin_inff() : Traits<float>::unkey(e.kb + 1u);
    use = a > -__builtin_inff() || b < __builtin_inff();
  }
  if (threadIdx.x == 0) {
    ab[2 * c] = use ? a : __builtin_inff();
    ab[2 * c + 1] = use ? b : -__builtin_inff();
  }
  if (nm > 0 && threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    const float *Qr = Q + c * dim;
    const float e = lane < dim ? Qr[lane < dim ? lane : 0] - centre[lane < dim ? lane : 0] : 0.0f;
    const double n2 = wave_sum((double)e * (double)e);
    const bool wild = !(n2 < (double)kScrNormMax);
    if (lane < nm * kScrK) {
      const ScreenSlot sl = screen_slot(lane, dim);
      const float v = -2.0f * (Qr[sl.j] - centre[sl.j]);
      B[c * nm * kScrK + lane] =
          sl.norm ? (__bf16)1.0f : (sl.product && !wild ? bf16_part(v, sl.lo_q) : (__bf16)0.0f);
    }
    if (lane == 0) {
      const double hi = use ? (double)b : -__builtin_inf();
      const double v = hi * (1.0 + (dim + 8) * 0x1p-24) - n2 * (1.0 - (double)kScrMargin) + 1e-36;
      T[c] = hi == -__builtin_inf() ? -__builtin_inff()
                                    : (wild ? __builtin_inff() : (float)(v + fabs(v) * 0x1p-23));
    }
  }
}

// The filter on the matrix cores, for queries whose k nearest are a small part of the points.
// Nearly every distance lies above b, and that can be seen without forming it: with a centre
// c near the data, p' = fl(p - c) and q' = fl(q - c),
//     d = |p'|^2 - 2 p'.q' + |q'|^2  up to the rounding of p', q' and of the sums,
// and |p'|^2 - 2 p'.q' with every value split in two bfloat16 parts (hi.hi + hi.lo + lo.hi per
// product and the norm's two, 3 dim + 2 terms added in float) is a matrix product.  A pair whose screen exceeds b - |q'|^2 by more than the margin below is above b for
// certain; every other pair's distance is formed in float in the fixed order (knn_dist) and
// tested as in knn_filter_kernel, so the kept distances and the counts are the same bits: the
// screen only decides which pairs need not be formed.  (The ordinates' sums add the same terms, in
// another order, in double; in either filter the order of the last additions is not fixed.)
//
// The margin, u = 2^-24, D = dim.  (1) An exact-order d below b has a true value below
// b (1 + (D + 4) u) (D + 2 roundings, each relative, as every term is positive).  (2) p' and q'
// are off by u |p'| and u |q'|, which moves the true distance by at most a factor 1 + u and
// 2.01 u (|p'|^2 + |q'|^2) more.  (3) hi is off by 2^-9 and hi + lo by 2^-18 of the value, so the
// terms left out of 2 p'.q' are below 3.1 * 2^-18 (|p'|^2 + |q'|^2).  (4) The at most 50 float
// additions, in whatever order and however the matrix instruction aligns its terms (2^-22 of
// the terms' sum each), are off by less than 2^-16 (2 |p'|^2 + |q'|^2), the norms by D u and
// their parts by 2^-18.  Together below 2^-14 (|p'|^2 + |q'|^2) with room to spare: the norm is
// lowered by 2^-14 of itself, so each point carries its own share, and the threshold is
// b (1 + (D + 8) u) - |q'|^2 (1 - 2^-14) + 1e-36, formed in double and rounded up.  A point or
// query whose norm is not below 1e37 (NaN, infinities) is not screened: all its distances are
// formed.
//
// Why this shape.  On gfx950 the vector instructions of a SIMD wait while its matrix pipe
// runs, so what counts is the sum of both.  A tile of 32 x 32 pairs takes 64 cycles of
// matrix instructions for dim 5 to 10 (the same product in float: 256, as many as 8 vector FMAs
// per pair), and its sixteen results per lane fold to their minimum and one compare;
// forming every distance takes 16 x 28 vector instructions.  The split operands of the points
// are laid out once per call (knn_split_kernel: one 16-byte load per lane and instruction),
// a wavefront keeps QT tiles of 32 queries, and the wavefronts of a workgroup take other
// queries of the same points, so that a point's line is read from the caches once.
// 1024 queries x 2^20 points in 8 dimensions, k = 64: the plain filter 745 us, the screen
// 106 us after the split's 20 us (the same screen with float matrix instructions and the
// norms as start values took 235 us); the whole call 849 -> 232 us.
// The points' operands: for every point the 16 nm terms in slot order (a lane of the screen
// loads eight at once), the norm as |p'|^2 (1 - 2^-14); the points past n - 1 of the last tile
// repeat it.  A workgroup takes kSplitRows points through LDS, so that both its loads and its
// stores are whole lines.  A point that is not screened gets zero terms and a norm of -inf:
// it passes for every query.
// (The dimension is a template argument: places in the tile divide by it, and with a runtime
// divisor the divisions took longer than the memory, 38 us against 20 us at 2^20 x 8.)
constexpr int kSplitRows = 128;
template <int dim>
__global__ __launch_bounds__(kKnnBlock) void knn_split_kernel(const float *__restrict__ P,
                                                              const float *__restrict__ centre,
                                                              int64_t n, __bf16 *__restrict__ A) {
  constexpr int nm = screen_steps(dim), ld = dim + 1;
  __shared__ float sp[kSplitRows * ld];  // rows of dim + 1 words: a row per lane hits all banks
  __shared__ float sn[kSplitRows];
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kSplitRows;
  const int64_t rows = (n + kScrTile - 1) / kScrTile * kScrTile;
  const int nr = (int)(rows - r0 < kSplitRows ? rows - r0 : kSplitRows);
  for (int t = tid; t < nr * dim; t += kKnnBlock) {
    const int r = t / dim, j = t - r * dim;
    const int64_t i = r0 + r < n ? r0 + r : n - 1;
    sp[r * ld + j] = P[i * dim + j] - centre[j];
  }
  __syncthreads();
  if (tid < nr) {
    float nx = 0.0f;
    for (int j = 0; j < dim; ++j) nx = nx + sp[tid * ld + j] * sp[tid * ld + j];
    sn[tid] = nx < kScrNormMax ? nx * (1.0f - kScrMargin) : -__builtin_inff();
  }
  __syncthreads();
  constexpr int groups = 2 * nm;
  for (int t = tid; t < nr * groups; t += kKnnBlock) {
    const int r = t / groups, g = t - r * groups;
    const float nr2 = sn[r];
    const bool wild = nr2 < 0.0f;
    BF8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const ScreenSlot sl = screen_slot(8 * g + e, dim);
      const float v = sl.norm ? nr2 : sp[r * ld + sl.j];
      const bool on = wild ? sl.norm == 1 : sl.norm || sl.product;
      out[e] = on ? bf16_part(v, sl.norm ? sl.norm == 2 : sl.lo_p) : (__bf16)0.0f;
    }
    *(BF8 *)(A + ((r0 + r) * groups + g) * 8) = out;
  }
}

// NM matrix instructions per tile (16 terms each), QT query tiles per wavefront.  wq wavefronts
// of the workgroup take other queries (wq QT 32 per workgroup), kScrWaves / wq other points.
template <int NM, int QT>
__global__ __launch_bounds__(kScrBlock, 4) void knn_screen_kernel(
    const float *__restrict__ P, const float *__restrict__ f, const float *__restrict__ Q,
    const float *__restrict__ ab, const __bf16 *__restrict__ Bq, const float *__restrict__ Tq,
    const __bf16 *__restrict__ A, int64_t n, int32_t dim, int64_t nq, int32_t wq, int64_t seg,
    float *__restrict__ K, uint32_t *__restrict__ cnt, double *__restrict__ fsum) {
  using F16 = float __attribute__((ext_vector_type(16)));
  constexpr int NQ = QT * kScrTile;      // queries per wavefront
  __shared__ uint32_t list[kScrWaves][kScrList];
  __shared__ float slo[kScrWaves][NQ], shi[kScrWaves][NQ];
  __shared__ double sfb[kScrWaves][NQ];  // the ordinates' sum over d <= a, and their count
  __shared__ uint32_t sbelow[kScrWaves][NQ];
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int col = lane % kScrTile, half = lane / kScrTile;
  const int64_t q0 = ((int64_t)blockIdx.y * wq + wv % wq) * NQ;
  for (int t = lane; t < NQ; t += kWave) {
    const bool live = q0 + t < nq;
    const int64_t q = live ? q0 + t : 0;
    slo[wv][t] = live ? ab[2 * q] : __builtin_inff();
    shi[wv][t] = live ? ab[2 * q + 1] : -__builtin_inff();
    sfb[wv][t] = 0.0;
    sbelow[wv][t] = 0u;
  }
  // the query operands and thresholds (a query past the last one: nothing passes)
  BF8 B[QT][NM];
  float T[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int64_t q = q0 + t * kScrTile + col;
    const int64_t qc = q < nq ? q : nq - 1;
#pragma unroll
    for (int m = 0; m < NM; ++m) B[t][m] = ((const BF8 *)Bq)[qc * (2 * NM) + 2 * m + half];
    const float v = Tq[qc];
    T[t] = q < nq ? v : -__builtin_inff();
  }
  const int64_t rb = (int64_t)blockIdx.x * seg;
  const int64_t re = rb + seg < n ? rb + seg : n;
  // the exact distance and tests of one pair per lane: point rb + r, query ql of the wavefront
  auto exact = [&](bool on, uint32_t r, int ql) {
    const int64_t i = rb + r, q = q0 + ql;
    if (!on || i >= re || q >= nq) return;
    const float fi = f[i];
    float d = 0.0f;  // (knn_dist's order)
    for (int j0 = 0; j0 < dim; j0 += 4) {
      float pv[4], qv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + e < dim ? j0 + e : j0;
        pv[e] = P[i * dim + j];
        qv[e] = Q[q * dim + j];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float dif = pv[e] - qv[e];
        const float sq = dif * dif;
        if (j0 + e < dim) d = j0 + e == 0 ? sq : d + sq;
      }
    }
    if (d <= slo[wv][ql]) {
      atomicAdd(&sbelow[wv][ql], 1u);
      atomicAdd(&sfb[wv][ql], (double)fi);
    } else if (!(d >= shi[wv][ql])) {
      const uint32_t at = atomicAdd(&cnt[q * kKnnCntStride], 1u);
      if (at < (uint32_t)kKnnCap) {
        K[2 * (q * kKnnCap + at)] = d;
        K[2 * (q * kKnnCap + at) + 1] = fi;
      }
    }
  };
  uint32_t held = 0;  // pairs in the list (uniform)
  auto drain = [&](uint32_t count) {  // the list's last `count` (<= 64) pairs
    __builtin_amdgcn_wave_barrier();
    const uint32_t e = lane < count ? list[wv][held - count + lane] : 0u;
    held -= count;
    exact(lane < count, e / NQ, (int)(e % NQ));
    __builtin_amdgcn_wave_barrier();
  };
  // this wavefront's tiles of the segment
  const uint32_t tiles = (uint32_t)((re - rb + kScrTile - 1) / kScrTile);
  const uint32_t step = kScrWaves / wq;
  const BF8 *Ab = (const BF8 *)A + (rb + col) * (2 * NM) + half;
  BF8 a[NM];
  auto load = [&](uint32_t tile, BF8 (&av)[NM]) {
#pragma unroll
    for (int m = 0; m < NM; ++m) av[m] = Ab[(int64_t)tile * (kScrTile * 2 * NM) + 2 * m];
  };
  uint32_t tile = wv / wq;
  if (tile < tiles) load(tile, a);
  for (; tile < tiles; tile += step) {
    BF8 an[NM];
    load(tile + step < tiles ? tile + step : tile, an);
    // (result i of a lane is point 8 (i / 4) + 4 half + i % 4 of the tile)
    // the pairs that pass: bit i of tile t's sixteen for result i
    uint32_t hit[(QT + 1) / 2] = {};
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      F16 R = {};
#pragma unroll
      for (int m = 0; m < NM; ++m)
        R = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m], B[t][m], R, 0, 0, 0);
      float mm = R[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mm = __builtin_fminf(mm, R[i]);
      if (ballot(mm <= T[t]) != 0) {  // (a tile in three has a pair that passes, mostly one)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float mg = __builtin_fminf(
              __builtin_fminf(__builtin_fminf(R[4 * g], R[4 * g + 1]), R[4 * g + 2]), R[4 * g + 3]);
          if (ballot(mg <= T[t]) == 0) continue;
          uint32_t w = 0;
#pragma unroll
          for (int j = 3; j >= 0; --j) w = 2 * w + (R[4 * g + j] <= T[t] ? 1u : 0u);
          hit[t / 2] |= w << (16 * (t % 2) + 4 * g);
        }
      }
    }
    for (int h = 0; h < (QT + 1) / 2; ++h) {
      uint32_t w = hit[h];
      for (;;) {  // each lane's next pair, until none has one
        const uint64_t mask = ballot(w != 0);
        if (mask == 0) break;
        if (w != 0) {
          const uint32_t b = (uint32_t)__builtin_ctz(w);
          const uint32_t i = b % 16, ql = (2 * h + b / 16) * kScrTile + col;
          list[wv][held + lane_rank(mask)] =
              (tile * kScrTile + 8 * (i / 4) + 4 * half + i % 4) * NQ + ql;
          w &= w - 1;
        }
        held += popc(mask);
        if (held >= (uint32_t)kWave) drain(kWave);
      }
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) a[m] = an[m];
  }
  if (held) drain(held);
  __builtin_amdgcn_wave_barrier();
  for (int t = lane; t < NQ; t += kWave)
    if (q0 + t < nq && sbelow[wv][t]) {
      atomicAdd(&cnt[(q0 + t) * kKnnCntStride + 1], sbelow[wv][t]);
      atomicAdd(&fsum[q0 + t], sfb[wv][t]);
    }
}

template <int D>
__global__ __launch_bounds__(kKnnBlock) void knn_filter_kernel(
    const float *__restrict__ P, const float *__restrict__ f, const float *__restrict__ Q,
    const float *__restrict__ ab, int64_t n, int32_t dim, int64_t nq, int64_t seg,
    float *__restrict__ K, uint32_t *__restrict__ cnt, double *__restrict__ fsum) {
  constexpr int DM = D > 0 ? D : 16;
  const int dd = D > 0 ? D : dim;
  const int64_t q = (int64_t)blockIdx.y * kKnnBlock + threadIdx.x;
  const bool live = q < nq;
  float qv[DM];
#pragma unroll
  for (int j = 0; j < DM; ++j) qv[j] = live && j < dd ? Q[q * dd + j] : 0.0f;
  const float lo = live ? ab[2 * q] : __builtin_inff();
  const float hi = live ? ab[2 * q + 1] : -__builtin_inff();
  const int64_t rb = (int64_t)blockIdx.x * seg;
  const int64_t re = rb + seg < n ? rb + seg : n;
  uint32_t below = 0;
  double fb = 0.0;
  for (int64_t i = rb; i < re; ++i) {
    float row[DM];
#pragma unroll
    for (int j = 0; j < DM; ++j) row[j] = j < dd ? P[i * dd + j] : 0.0f;
    const float fi = f[i];
    const float d = knn_dist_reg<D>(row, qv, dim);
    const bool le = d <= lo;
    if (live && !le && !(d >= hi)) {
      const uint32_t at = atomicAdd(&cnt[q * kKnnCntStride], 1u);
      if (at < (uint32_t)kKnnCap) {
        K[2 * (q * kKnnCap + at)] = d;
        K[2 * (q * kKnnCap + at) + 1] = fi;
      }
    }
    if (le) {
      ++below;
      fb += (double)fi;
    }
  }
  if (live && below) {
    atomicAdd(&cnt[q * kKnnCntStride + 1], below);
    atomicAdd(&fsum[q], fb);
  }
}

__device__ inline void knn_write(cps_knn *out, double mean, float dk, int32_t status,
                                 int64_t below, int64_t equal) {
  cps_knn o;
  o.mean = mean;
  o.dk = dk;
  o.status = status;
  o.below = below;
  o.equal = equal;
  *out = o;
}

// One workgroup per query: where the bracket holds d_k (#(d <= a) < k <= #(d <= a) + kept,
// kept <= kKnnCap), the kept distances and ordinates in LDS, d_k by a radix select of rank
// k - #(d <= a) among them, and the sums of the ordinates below and at d_k (fixed order);
// else the same over the query's n distances recomputed (key range, histogram narrowing,
// a last pass for the sums).  The mean as the materialised form's final kernel forms it.
template <int D>
__global__ __launch_bounds__(kKnnBlock) void knn_select_kernel(
    const float *__restrict__ K, const uint32_t *__restrict__ cnt,
    const double *__restrict__ fsum, const float *__restrict__ ab, const float *__restrict__ P,
    const float *__restrict__ f, const float *__restrict__ Q, int64_t n, int32_t dim, int64_t nq,
    int64_t k, cps_knn *__restrict__ out) {
  constexpr int DM = D > 0 ? D : 16;
  __shared__ float kd[kKnnCap];
  __shared__ float kf[kKnnCap];
  __shared__ uint32_t hist[kHistMaxBins];
  __shared__ WgSelShared<kKnnBlock> sh;
  __shared__ double wred[kKnnBlock / kWave];
  __shared__ float sq[16];
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  const int dd = D > 0 ? D : dim;
  const int64_t len = cnt[c * kKnnCntStride], below = cnt[c * kKnnCntStride + 1];
  const float lo = ab[2 * c], hi = ab[2 * c + 1];
  const bool holds = lo < hi && below < k && k <= below + len && len <= kKnnCap;
  if (tid < dd) sq[tid] = Q[c * dd + tid];
  if (tid == 0) {
    sh.flag = 0u;
    sh.kext[0] = ~0ull;
    sh.kext[1] = 0ull;
  }
  __syncthreads();
  if (holds) {  // (uniform)
    bool nan = false;
    for (int64_t i = tid; i < len; i += kKnnBlock) {
      const float d = K[2 * (c * kKnnCap + i)];
      kd[i] = d;
      kf[i] = K[2 * (c * kKnnCap + i) + 1];
      nan = nan || !(d == d);
    }
    if (nan) atomicOr(&sh.flag, 1u);
    __syncthreads();
    if (sh.flag != 0u) {
      if (tid == 0) knn_write(out + c, __builtin_nan(""), __builtin_nanf(""), CPS_STATUS_NAN, 0, 0);
      return;
    }
    uint32_t key;
    int64_t b_in, eq;
    block_radix_select<float, kKnnBlock>(kd, len, false, 0.0f, 0.0f, k - below, hist, sh.misc,
                                         key, b_in, eq);
    const float dk = Traits<float>::unkey(key);
    double slt = 0.0, seq = 0.0;
    for (int64_t i = tid; i < len; i += kKnnBlock) {
      if (kd[i] < dk) slt += (double)kf[i];
      else if (kd[i] == dk) seq += (double)kf[i];
    }
    slt = block_sum_fixed<kKnnBlock>(slt, wred);
    seq = block_sum_fixed<kKnnBlock>(seq, wred);
    const int64_t less = below + b_in;
    if (tid == 0) {
      const double a = (double)(k - less);
      const double mean = (fsum[c] + slt + a * seq / (double)eq) / (double)k;
      knn_write(out + c, mean, dk, CPS_STATUS_OK, less, eq);
    }
    return;
  }
  // the query's distances, recomputed in point order from its share
  float qv[DM];
#pragma unroll
  for (int j = 0; j < DM; ++j) qv[j] = j < dd ? sq[j] : 0.0f;
  auto pass = [&](auto fn) {
    for (int64_t i = tid; i < n; i += kKnnBlock) {
      float row[DM];
#pragma unroll
      for (int j = 0; j < DM; ++j) row[j] = j < dd ? P[i * dd + j] : 0.0f;
      fn(knn_dist_reg<D>(row, qv, dim));
    }
  };
  uint32_t kmn = ~0u, kmx = 0u;
  bool nan = false;
  pass([&](float d) {
    const uint32_t kk = Traits<float>::key(d);
    nan = nan || !(d == d);
    kmn = kk < kmn ? kk : kmn;
    kmx = kk > kmx ? kk : kmx;
  });
  atomicMin(&sh.kext[0], (unsigned long long)kmn);
  atomicMax(&sh.kext[1], (unsigned long long)kmx);
  if (nan) atomicOr(&sh.flag, 1u);
  __syncthreads();
  if (sh.flag != 0u) {  // (uniform)
    if (tid == 0) knn_write(out + c, __builtin_nan(""), __builtin_nanf(""), CPS_STATUS_NAN, 0, 0);
    return;
  }
  const WgSelOut r = wg_select_pass<float, kKnnBlock>(pass, k, sh.kext[0], sh.kext[1], 0, n, hist,
                                                      kd, kKnnCap, sh);
  const float dk = Traits<float>::unkey((uint32_t)r.key);
  double slt = 0.0, seq = 0.0;
  for (int64_t i = tid; i < n; i += kKnnBlock) {
    float row[DM];
#pragma unroll
    for (int j = 0; j < DM; ++j) row[j] = j < dd ? P[i * dd + j] : 0.0f;
    const float d = knn_dist_reg<D>(row, qv, dim);
    if (d < dk) slt += (double)f[i];
    else if (d == dk) seq += (double)f[i];
  }
  slt = block_sum_fixed<kKnnBlock>(slt, wred);
  seq = block_sum_fixed<kKnnBlock>(seq, wred);
  if (tid == 0) {
    const double a = (double)(k - r.less);
    knn_write(out + c, (slt + a * seq / (double)r.equal) / (double)k, dk, CPS_STATUS_OK, r.less,
              r.equal);
  }
}

// Whether the screen serves a call: by the part of the points expected below the bracket's
// upper end (rank k and four standard deviations of the sample, as sample_bracket_rule), since
// a pair that passes costs more than in the plain filter.  Whole calls, screen against plain
// filter: 1024 queries x 2^17 points x 8, 3.6 % of the points below the end 216 against 245 us,
// 4.3 % 271 against 274, 6.6 % 326 against 300; 1024 x 40000 x 5, 4.3 % 147 against 245, 14 %
// 224 against 268; the line is at the first one's crossing.
bool knn_use_screen(int64_t n, int64_t k) {
  const double S = (double)sample_runs(n) * kPropRun, p = ((double)k - 0.5) / (double)n;
  return p + 4.0 * sqrt(p * (1.0 - p) / S) + 2.0 / S <= kScrPart;
}

// The screen's shape: matrix instructions per tile, query tiles per wavefront, and wavefronts
// of a workgroup that take other queries (as many as the queries fill).
struct ScreenShape {
  int nm, qt, wq;
  int64_t groups;
};
static ScreenShape knn_screen_shape(int32_t dim, int64_t nq) {
  ScreenShape s;
  s.nm = screen_steps(dim);
  s.qt = nq > 2 * kScrTile ? kScrQt : 1;
  const int64_t waves = (nq + s.qt * kScrTile - 1) / (s.qt * kScrTile);
  s.wq = waves > 2 ? 4 : (waves > 1 ? 2 : 1);
  s.groups = (waves + s.wq - 1) / s.wq;
  return s;
}

int64_t knn_split_elems(int64_t n, int32_t dim) {
  const int64_t rows = (n + kScrTile - 1) / kScrTile * kScrTile;
  return rows * screen_steps(dim) * kScrK;
}

void knn_filter_shape(int64_t n, int32_t dim, int64_t nq, bool screen, int cu_count, int64_t *nseg,
                      int64_t *seg) {
  if (screen) {
    // kScrPerCu workgroups per CU over (segments x groups of queries);
    // segments of whole tiles, at most 2^24 points (a pair's place in its 32-bit list word)
    const ScreenShape s = knn_screen_shape(dim, nq);
    int64_t ns = (int64_t)cu_count * kScrPerCu / s.groups;
    if (ns < 1) ns = 1;
    const int64_t round = (int64_t)kScrTile * (kScrWaves / s.wq);
    int64_t sl = ((n + ns - 1) / ns + round - 1) / round * round;
    if (sl > ((int64_t)1 << 24)) sl = (int64_t)1 << 24;
    *nseg = (n + sl - 1) / sl;
    *seg = sl;
    return;
  }
  // about 4 x 8 workgroups per CU over (segments x groups of kKnnBlock queries), segments of
  // at least 256 points
  const int64_t groups = (nq + kKnnBlock - 1) / kKnnBlock;
  int64_t ns = (int64_t)cu_count * 32 / groups;
  const int64_t nmax = (n + 255) / 256;
  if (ns > nmax) ns = nmax;
  if (ns > 65535) ns = 65535;
  if (ns < 1) ns = 1;
  const int64_t sl = (n + ns - 1) / ns;
  *nseg = (n + sl - 1) / sl;
  *seg = sl;
}

template <int D>
static void launch_knn_split(const float *P, const float *centre, int64_t n, int32_t dim, __bf16 *A,
                             hipStream_t stream) {
  if constexpr (D > 1)
    if (dim < D) return launch_knn_split<D - 1>(P, centre, n, dim, A, stream);
  const int64_t rows = (n + kScrTile - 1) / kScrTile * kScrTile;
  knn_split_kernel<D><<<dim3((unsigned)((rows + kSplitRows - 1) / kSplitRows)), dim3(kKnnBlock), 0,
                        stream>>>(P, centre, n, A);
}

template <int NM>
static void launch_knn_screen_nm(const float *P, const float *f, const float *Q, int64_t n,
                                 int32_t dim, int64_t nq, const ScreenShape &s,
                                 const KnnFilterBufs &w, hipStream_t stream) {
  const dim3 grid((unsigned)w.nseg, (unsigned)s.groups);
  const __bf16 *A = (const __bf16 *)w.A;
  if (s.qt == kScrQt)
    knn_screen_kernel<NM, kScrQt><<<grid, dim3(kScrBlock), 0, stream>>>(
        P, f, Q, w.ab, (const __bf16 *)w.Bq, w.Tq, A, n, dim, nq, s.wq, w.seg, w.K, w.cnt, w.fsum);
  else
    knn_screen_kernel<NM, 1><<<grid, dim3(kScrBlock), 0, stream>>>(
        P, f, Q, w.ab, (const __bf16 *)w.Bq, w.Tq, A, n, dim, nq, s.wq, w.seg, w.K, w.cnt, w.fsum);
}

static hipError_t launch_knn_screen(const float *P, const float *f, const float *Q, int64_t n,
                                    int32_t dim, int64_t nq, const KnnFilterBufs &w,
                                    hipStream_t stream) {
  const ScreenShape s = knn_screen_shape(dim, nq);
  launch_knn_split<16>(P, w.centre, n, dim, (__bf16 *)w.A, stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (s.nm == 1) launch_knn_screen_nm<1>(P, f, Q, n, dim, nq, s, w, stream);
  else if (s.nm == 2) launch_knn_screen_nm<2>(P, f, Q, n, dim, nq, s, w, stream);
  else if (s.nm == 3) launch_knn_screen_nm<3>(P, f, Q, n, dim, nq, s, w, stream);
  else launch_knn_screen_nm<4>(P, f, Q, n, dim, nq, s, w, stream);
  return hipGetLastError();
}

// (8 dimensions have instances of the sample, filter and select kernels of their own: 1024 queries
// x 2^20 points 181 us a call, with the 16-wide guarded loops of the other dimensions 194.)
hipError_t launch_knn_filtered(const float *P, const float *f, const float *Q, int64_t n,
                               int32_t dim, int64_t nq, int64_t k, const KnnFilterBufs &w,
                               cps_knn *out, hipStream_t stream) {
  const int64_t groups = (nq + kKnnBlock - 1) / kKnnBlock;
  static_assert(kPropSample % (kKnnBlock * kSmpTiles) == 0, "whole workgroups of samples");
  const dim3 sg((unsigned)(sample_runs(n) * kPropRun / (kKnnBlock * kSmpTiles)),
                (unsigned)((nq + kSmpChunk - 1) / kSmpChunk));
  if (dim == 8)
    knn_sample_kernel<8><<<sg, dim3(kKnnBlock), 0, stream>>>(P, Q, n, dim, nq, w.Ds, w.centre);
  else
    knn_sample_kernel<0><<<sg, dim3(kKnnBlock), 0, stream>>>(P, Q, n, dim, nq, w.Ds, w.centre);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool big = sample_runs(n) * kPropRun == kPropSampleBig;
  (big ? knn_bracket_kernel<kPropSampleBig / 1024> : knn_bracket_kernel<kPropSample / 1024>)
      <<<dim3((unsigned)nq), dim3(1024), 0, stream>>>(
      w.Ds, Q, w.centre, n, dim, k, nq, w.A ? knn_screen_shape(dim, nq).nm : 0, w.ab, w.cnt, w.fsum,
      (__bf16 *)w.Bq, w.Tq);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 fg((unsigned)w.nseg, (unsigned)groups);
  if (w.A) {
    e = launch_knn_screen(P, f, Q, n, dim, nq, w, stream);
    if (e != hipSuccess) return e;
  } else if (dim == 8)
    knn_filter_kernel<8><<<fg, dim3(kKnnBlock), 0, stream>>>(P, f, Q, w.ab, n, dim, nq, w.seg, w.K,
                                                              w.cnt, w.fsum);
  else
    knn_filter_kernel<0><<<fg, dim3(kKnnBlock), 0, stream>>>(P, f, Q, w.ab, n, dim, nq, w.seg, w.K,
                                                              w.cnt, w.fsum);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dim == 8)
    knn_select_kernel<8><<<dim3((unsigned)nq), dim3(kKnnBlock), 0, stream>>>(
        w.K, w.cnt, w.fsum, w.ab, P, f, Q, n, dim, nq, k, out);
  else
    knn_select_kernel<0><<<dim3((unsigned)nq), dim3(kKnnBlock), 0, stream>>>(
        w.K, w.cnt, w.fsum, w.ab, P, f, Q, n, dim, nq, k, out);
  return hipGetLastError();
}

hipError_t launch_knn_distances(const float *P, const float *Q, int64_t n, int32_t dim, int64_t nq,
                                int64_t k, float *Dst, const float **ptrs, int64_t *sizes,
                                int64_t *ks, int cu_count, hipStream_t stream) {
  const int64_t groups = (nq + kKnnGroup - 1) / kKnnGroup;
  int64_t bx = (n + kKnnBlock - 1) / kKnnBlock;
  const int64_t want = (int64_t)cu_count * 8 / (groups < 1 ? 1 : groups) + 1;
  if (bx > want) bx = want;
  if (bx < 1) bx = 1;
  const dim3 grid((unsigned)bx, (unsigned)groups);
  if (dim == 8)
    knn_distance_kernel<8><<<grid, dim3(kKnnBlock), 0, stream>>>(P, Q, n, dim, nq, Dst);
  else
    knn_distance_kernel<0><<<grid, dim3(kKnnBlock), 0, stream>>>(P, Q, n, dim, nq, Dst);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  knn_descriptor_kernel<<<dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, stream>>>(
      Dst, n, nq, k, ptrs, sizes, ks);
  return hipGetLastError();
}

hipError_t launch_knn_reduce(const float *P, const float *f, const float *Q, const float *Dst,
                             int64_t n, int32_t dim, int64_t nq, int64_t k, const cps_result *sel,
                             double *pd, int64_t *pi, cps_knn *out, hipStream_t stream) {
  const dim3 grid((unsigned)kKnnRedBlocks, (unsigned)nq);
  const bool vec = n % 4 == 0 && (uintptr_t)f % 16 == 0 && (uintptr_t)Dst % 16 == 0;
  if (kKnnRead && vec)
    knn_partial_read_kernel<true><<<grid, dim3(kKnnBlock), 0, stream>>>(Dst, f, n, sel, pd, pi);
  else if (kKnnRead)
    knn_partial_read_kernel<false><<<grid, dim3(kKnnBlock), 0, stream>>>(Dst, f, n, sel, pd, pi);
  else if (dim == 8)
    knn_partial_kernel<8><<<grid, dim3(kKnnBlock), 0, stream>>>(P, f, Q, n, dim, sel, pd, pi);
  else
    knn_partial_kernel<0><<<grid, dim3(kKnnBlock), 0, stream>>>(P, f, Q, n, dim, sel, pd, pi);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  knn_final_kernel<<<dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, stream>>>(
      nq, k, kKnnRedBlocks, sel, pd, pi, out);
  return hipGetLastError();
}

}  // namespace cps
