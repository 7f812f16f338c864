// The general batched kernel's instance for the arrays that the default selection (batchq.hip) left.
#include "batched_kernel.h"

namespace cps {

template <typename T> hipError_t launch_batched_list(const BatchArgs<T> &a, int grid, hipStream_t stream) {
  batched_select_kernel<T, 1024, kSelectUnroll, true><<<dim3(grid), dim3(1024), 0, stream>>>(a);
  return hipGetLastError();
}

template hipError_t launch_batched_list<float>(const BatchArgs<float> &, int, hipStream_t);
template hipError_t launch_batched_list<double>(const BatchArgs<double> &, int, hipStream_t);

}  // namespace cps
