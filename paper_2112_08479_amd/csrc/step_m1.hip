// FP32 and FP64 single steps of model 1
#include "step_kernel.h"

namespace lbm {

template <>
hipError_t launch_step_real<1>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  return h->cfg.storage == LBM_F64 ? launch_step_of<1, double, double, double>(h, src, dst, nullptr, st)
                                   : launch_step_of<1, float, float, float>(h, src, dst, nullptr, st);
}

}  // namespace lbm
