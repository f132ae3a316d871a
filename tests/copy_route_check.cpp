// Host check of the state copy's route (csrc/copy.cpp) with the runtime's calls
// replaced: the copy kernel only where both sides are device memory of the
// handle's GPU, on 16 bytes, and hold the whole state; the runtime's copy, which
// checks its own ranges, everywhere else.
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "runtime.h"

static struct { hipMemoryType type; int device; uintptr_t base; size_t size; } mem[2];
static int side(const void* p) { return (uintptr_t)p >= mem[1].base ? 1 : 0; }
static int kernel_copies, runtime_copies;

extern "C" {
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const auto& m = mem[side(p)];
  if (!m.size) return hipErrorInvalidValue;
  memset(a, 0, sizeof(*a));
  a->type = m.type;
  a->device = m.device;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* b, size_t* n, hipDeviceptr_t p) {
  const auto& m = mem[side(p)];
  *b = (hipDeviceptr_t)m.base;
  *n = m.size;
  return m.size ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
  ++runtime_copies;
  return hipErrorInvalidValue;
}
}
namespace lbm {
hipError_t launch_stream_copy(void*, const void*, size_t, hipStream_t) {
  ++kernel_copies;
  return hipSuccess;
}
}  // namespace lbm

int main() {
  int fails = 0;
  const size_t state = 4096;
  const auto run = [&](bool kernel, size_t at_src, size_t at_dst, const char* what) {
    lbm_handle h{};
    h.state_bytes = state;
    h.device = 1;
    kernel_copies = runtime_copies = 0;
    const hipError_t e = lbm::launch_copy_state(&h, (void*)(mem[0].base + at_src), (void*)(mem[1].base + at_dst));
    const bool ok = kernel ? kernel_copies == 1 && !runtime_copies && e == hipSuccess
                           : !kernel_copies && runtime_copies == 1 && e == hipErrorInvalidValue;
    if (!ok) ++fails, printf("FAIL %s\n", what);
  };
  const auto reset = [&] {
    mem[0] = {hipMemoryTypeDevice, 1, 1 << 20, 3 * state};
    mem[1] = {hipMemoryTypeDevice, 1, 1 << 24, 256 + state};
  };
  reset();
  run(true, 256, 256, "both hold the state, to the last byte");
  run(true, 2 * state, 0, "the end of the source");
  run(false, 0, 272, "the slot's allocation ends 16 bytes too early");
  run(false, 2 * state + 16, 256, "the source ends too early");
  run(false, 0, 8, "not on 16 bytes");
  mem[1].size = state / 2;
  run(false, 0, 256, "half a slot");
  mem[1].size = 128;
  run(false, 0, 256, "a slot shorter than its header");
  for (int s = 0; s < 2; ++s) {
    reset();
    mem[s].type = hipMemoryTypeHost;
    run(false, 0, 256, "host memory");
    reset();
    mem[s].type = hipMemoryTypeManaged;
    run(false, 0, 256, "managed memory");
    reset();
    mem[s].device = 0;
    run(false, 0, 256, "another GPU");
    reset();
    mem[s].size = 0;
    run(false, 0, 0, "unknown to the runtime");
  }
  printf("fails %d\n", fails);
  return fails != 0;
}
