// 16-bit storage step kernels of model 1
#include "step_kernel.h"

namespace lbm {

template <>
hipError_t launch_step_16<1>(lbm_handle* h, const void* src, void* dst, hipStream_t st) {
  switch (h->cfg.storage) {
    case LBM_F16: return launch_step_of<1, __half, __half, float>(h, src, dst, nullptr, st);
    case LBM_BF16: return launch_step_of<1, bf16_t, bf16_t, float>(h, src, dst, nullptr, st);
    case LBM_BF16_F16S: return launch_step_of<1, bf16_t, __half, float>(h, src, dst, nullptr, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace lbm
