// Which step kernel a handle takes; the kernels are in step_m*.hip (FP32, FP64),
// step16_m*.hip (16-bit storage) and pair_m*.hip (grids that take steps two at a
// time), one translation unit per model, and stepfw.hip (the adjoint's forward
// steps).
#include "runtime.h"

namespace lbm {

hipError_t launch_step(lbm_handle* h, const void* src, void* dst, double* fw, hipStream_t st) {
  if (!st) st = h->stream;
  if (fw) return launch_step_fw(h, src, dst, fw, st);
  if (h->paired) {
    const bool f64 = h->cfg.storage == LBM_F64;
    switch (h->cfg.model) {
      case LBM_CUMULANT27_Q7:
        return f64 ? launch_paired<0, double>(h, src, dst, st) : launch_paired<0, float>(h, src, dst, st);
      case LBM_BGK19_SMAG_Q6: return launch_paired<1, double>(h, src, dst, st);
      case LBM_CUMULANT27_FCM27: return launch_paired<2, float>(h, src, dst, st);
    }
    return hipErrorInvalidValue;
  }
  const bool real = h->cfg.storage == LBM_F64 || h->cfg.storage == LBM_F32;
  switch (h->cfg.model) {
    case LBM_CUMULANT27_Q7:
      return real ? launch_step_real<0>(h, src, dst, st) : launch_step_16<0>(h, src, dst, st);
    case LBM_BGK19_SMAG_Q6:
      return real ? launch_step_real<1>(h, src, dst, st) : launch_step_16<1>(h, src, dst, st);
    case LBM_CUMULANT27_FCM27:
      return real ? launch_step_real<2>(h, src, dst, st) : launch_step_16<2>(h, src, dst, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
