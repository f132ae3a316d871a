// Steps of model 2 in FP32 on grids that take them two at a time; contraction as
// launch_paired_of asks.
#pragma clang fp contract(on)
#include "step_kernel.h"
#include "twostep_kernel.h"

namespace lbm {

template <>
hipError_t launch_paired<2, float>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return launch_paired_of<2, float>(h, src, dst, st);
}

}  // namespace lbm
