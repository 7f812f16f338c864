// The general batched kernel's instances and their launch.
#include "batched_kernel.h"

namespace cps {

template <typename T>
hipError_t launch_batched(const BatchArgs<T> &a, int grid, int block, hipStream_t stream) {
  if (block == 256)
    batched_select_kernel<T, 256, kSelectUnroll, false><<<dim3(grid), dim3(256), 0, stream>>>(a);
  else if (block == 512)
    batched_select_kernel<T, 512, kSelectUnroll, false><<<dim3(grid), dim3(512), 0, stream>>>(a);
  else
    batched_select_kernel<T, 1024, kSelectUnroll, false><<<dim3(grid), dim3(1024), 0, stream>>>(a);
  return hipGetLastError();
}

template <typename T> int batched_max_blocks_per_cu(int block) {
  int nb = 0;
  hipError_t e;
  if (block == 256)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batched_select_kernel<T, 256, kSelectUnroll, false>, 256, 0);
  else if (block == 512)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batched_select_kernel<T, 512, kSelectUnroll, false>, 512, 0);
  else
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batched_select_kernel<T, 1024, kSelectUnroll, false>, 1024, 0);
  return e == hipSuccess ? nb : 0;
}

template hipError_t launch_batched<float>(const BatchArgs<float> &, int, int, hipStream_t);
template hipError_t launch_batched<double>(const BatchArgs<double> &, int, int, hipStream_t);
template int batched_max_blocks_per_cu<float>(int);
template int batched_max_blocks_per_cu<double>(int);

}  // namespace cps
