// The selection kernel's instance that follows the one-read filter (quick.hip).
#include "select_kernel.h"

namespace cps {

template <typename T>
hipError_t launch_select_quick(const SelectArgs<T> &a, const QuickArgs<T> &quick, int grid,
                               hipStream_t stream) {
  SelectParams<T, true> p;
  static_cast<SelectArgs<T> &>(p) = a;
  p.quick = quick;
  cp_select_kernel<T, kSelectBlock, kSelectUnroll, true><<<dim3(grid), dim3(kSelectBlock), 0, stream>>>(p);
  return hipGetLastError();
}

template <typename T> int select_quick_max_blocks_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &nb, cp_select_kernel<T, kSelectBlock, kSelectUnroll, true>, kSelectBlock, 0) != hipSuccess)
    return 0;
  return nb;
}

template hipError_t launch_select_quick<float>(const SelectArgs<float> &, const QuickArgs<float> &, int,
                                               hipStream_t);
template hipError_t launch_select_quick<double>(const SelectArgs<double> &, const QuickArgs<double> &, int,
                                                hipStream_t);
template int select_quick_max_blocks_per_cu<float>();
template int select_quick_max_blocks_per_cu<double>();

}  // namespace cps
