// Steps of model 1 in FP64 on grids that take them two at a time; contraction as
// launch_paired_of asks.
#pragma clang fp contract(on)
#include "step_kernel.h"
#include "twostep_kernel.h"

namespace lbm {

template <>
hipError_t launch_paired<1, double>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return launch_paired_of<1, double>(h, src, dst, st);
}

}  // namespace lbm
