// The selection kernel's general instance and its launch, and the objective at given points.
#include "select_kernel.h"

namespace cps {

// ------------------------------------------------------------------ objective at given y

// Partial sums of the objective pieces at ys[blockIdx.y] over this block's slice of x.
template <typename T, int BLOCK>
__global__ __launch_bounds__(BLOCK) void objective_partial_kernel(const T *__restrict__ x,
                                                                  int64_t n,
                                                                  const double *__restrict__ ys,
                                                                  double *__restrict__ pd,
                                                                  int64_t *__restrict__ pi) {
  __shared__ double sd[8][BLOCK / kWave];
  __shared__ int64_t si[8][BLOCK / kWave];
  const double y = ys[blockIdx.y];
  double A = 0, B = 0, pred = -__builtin_inf(), succ = __builtin_inf();
  int64_t L = 0, E = 0, Gc = 0;
  for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * BLOCK) {
    const double v = (double)x[i];
    const double d = v - y;
    if (v > y) { A += d; Gc++; succ = fmin(succ, v); }
    else if (v < y) { B -= d; L++; pred = fmax(pred, v); }
    else if (v == y) { E++; }
  }
  double dv[8] = {A, B, pred, succ, 0, 0, 0, 0};
  int dop[8] = {0, 0, 2, 1, 0, 0, 0, 0};
  int64_t iv[8] = {L, E, Gc, 0, 0, 0, 0, 0};
  block_reduce<BLOCK, 4, 3>(dv, dop, iv, false, sd, si);
  if (threadIdx.x == 0) {
    const int64_t slot = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    for (int f = 0; f < 4; ++f) pd[slot * 4 + f] = dv[f];
    for (int f = 0; f < 3; ++f) pi[slot * 3 + f] = iv[f];
  }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void objective_final_kernel(int64_t n, int64_t k, int nb,
                                                                const double *__restrict__ pd,
                                                                const int64_t *__restrict__ pi,
                                                                cps_eval *__restrict__ out) {
  __shared__ double sd[8][BLOCK / kWave];
  __shared__ int64_t si[8][BLOCK / kWave];
  const int64_t y = blockIdx.x;
  double dv[8] = {0, 0, -__builtin_inf(), __builtin_inf(), 0, 0, 0, 0};
  int dop[8] = {0, 0, 2, 1, 0, 0, 0, 0};
  int64_t iv[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < nb; b += BLOCK) {
    const int64_t slot = y * nb + b;
    dv[0] += pd[slot * 4 + 0];
    dv[1] += pd[slot * 4 + 1];
    dv[2] = fmax(dv[2], pd[slot * 4 + 2]);
    dv[3] = fmin(dv[3], pd[slot * 4 + 3]);
    iv[0] += pi[slot * 3 + 0];
    iv[1] += pi[slot * 3 + 1];
    iv[2] += pi[slot * 3 + 2];
  }
  block_reduce<BLOCK, 4, 3>(dv, dop, iv, false, sd, si);
  if (threadIdx.x == 0) {
    const double alpha = (double)k - 0.5, beta = (double)n - (double)k + 0.5;
    cps_eval e;
    e.A = dv[0];
    e.B = dv[1];
    e.f = alpha * dv[0] + beta * dv[1];
    e.L = iv[0];
    e.E = iv[1];
    e.G = iv[2];
    e.pred = dv[2];
    e.succ = dv[3];
    e.gminus = (double)n * ((double)iv[0] - (double)k + 0.5);
    e.gplus = (double)n * ((double)(iv[0] + iv[1]) - (double)k + 0.5);
    out[y] = e;
  }
}

// ------------------------------------------------------------------ launchers

template <typename T>
hipError_t launch_select(const SelectArgs<T> &a, int grid, bool cooperative, hipStream_t stream) {
  SelectParams<T, false> p;
  static_cast<SelectArgs<T> &>(p) = a;
  // The grid never exceeds the workgroups that fit at once (one per CU), so an ordinary launch
  // on a GPU not running another grid-synchronising kernel has them all resident; the
  // cooperative launch guarantees it in every case but costs ~17 us more per call (measured:
  // an empty kernel takes ~2.5 us per ordinary launch and ~20 us per cooperative one).
  if (!cooperative) {
    cp_select_kernel<T, kSelectBlock, kSelectUnroll, false><<<dim3(grid), dim3(kSelectBlock), 0, stream>>>(p);
    return hipGetLastError();
  }
  void *args[] = {&p};
  return hipLaunchCooperativeKernel((const void *)cp_select_kernel<T, kSelectBlock, kSelectUnroll, false>,
                                    dim3(grid), dim3(kSelectBlock), args, 0, stream);
}

template <typename T> int select_max_blocks_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &nb, cp_select_kernel<T, kSelectBlock, kSelectUnroll, false>, kSelectBlock, 0) != hipSuccess)
    return 0;
  const int quick = select_quick_max_blocks_per_cu<T>();
  return nb < quick ? nb : quick;
}

template <typename T>
hipError_t launch_objective(const T *x, int64_t n, int64_t k, const double *ys, int64_t ny,
                            cps_eval *out, double *pd, int64_t *pi, int nb, hipStream_t stream) {
  constexpr int BLOCK = 256;
  objective_partial_kernel<T, BLOCK><<<dim3(nb, (unsigned)ny), dim3(BLOCK), 0, stream>>>(x, n, ys, pd, pi);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  objective_final_kernel<BLOCK><<<dim3((unsigned)ny), dim3(BLOCK), 0, stream>>>(n, k, nb, pd, pi, out);
  return hipGetLastError();
}

template hipError_t launch_select<float>(const SelectArgs<float> &, int, bool, hipStream_t);
template hipError_t launch_select<double>(const SelectArgs<double> &, int, bool, hipStream_t);
template int select_max_blocks_per_cu<float>();
template int select_max_blocks_per_cu<double>();
template hipError_t launch_objective<float>(const float *, int64_t, int64_t, const double *,
                                            int64_t, cps_eval *, double *, int64_t *, int,
                                            hipStream_t);
template hipError_t launch_objective<double>(const double *, int64_t, int64_t, const double *,
                                             int64_t, cps_eval *, double *, int64_t *, int,
                                             hipStream_t);

}  // namespace cps
