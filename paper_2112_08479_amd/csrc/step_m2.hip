// FP32 and FP64 step kernels of model 2. Multiply-adds are contracted within an
// expression only, not where the optimiser happens to see one: single steps and
// steps two at a time then round alike, and a run gives the same bits however
// its steps are grouped.
#pragma clang fp contract(on)
#include "step_kernel.h"
#include "twostep_kernel.h"

namespace lbm {

template <>
hipError_t launch_step_real<2>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return h->cfg.storage == LBM_F64 ? launch_step_of<2, double, double, double>(h, src, dst, nullptr, st)
                                   : launch_step_of<2, float, float, float>(h, src, dst, nullptr, st);
}

template <>
hipError_t launch_step2_real<2>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return launch_step2_of<2, float>(h, src, dst, st);
}

}  // namespace lbm
