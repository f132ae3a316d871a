// The adjoint's forward steps (FP32, FP64): the single step that also writes the
// wall-layer sums of F_w.
#include "step_kernel.h"

namespace lbm {

template <int M>
static hipError_t fw_step(lbm_handle* h, const void* src, void* dst, double* fw, hipStream_t st) {
  return h->cfg.storage == LBM_F64 ? launch_step_of<M, double, double, double, true>(h, src, dst, fw, st)
                                   : launch_step_of<M, float, float, float, true>(h, src, dst, fw, st);
}

hipError_t launch_step_fw(lbm_handle* h, const void* src, void* dst, double* fw, hipStream_t st) {
  if (h->cfg.storage != LBM_F64 && h->cfg.storage != LBM_F32) return hipErrorInvalidValue;
  switch (h->cfg.model) {
    case LBM_CUMULANT27_Q7: return fw_step<0>(h, src, dst, fw, st);
    case LBM_BGK19_SMAG_Q6: return fw_step<1>(h, src, dst, fw, st);
    case LBM_CUMULANT27_FCM27: return fw_step<2>(h, src, dst, fw, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
