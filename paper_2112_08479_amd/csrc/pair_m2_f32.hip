// Steps of model 2 in FP32 on grids that take them two at a time: pairs, and the
// single steps of an odd count. Multiply-adds are contracted within an
// expression only, not where the optimiser happens to see one, which differs
// between kernels: the two then round alike, and a run gives the same bits
// however it is split into calls.
#pragma clang fp contract(on)
#include "step_kernel.h"
#include "twostep_kernel.h"

namespace lbm {

template <>
hipError_t launch_paired<2, float>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return launch_paired_of<2, float>(h, src, dst, st);
}

}  // namespace lbm
