// Handle and launcher interface shared by the C ABI (abi.cpp) and the kernel
// translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "../../include/lbm.h"

struct lbm_handle {
  lbm_config cfg;
  lbm_params prm;
  int qf, qs, qt;     // flow, scalar, total populations
  int64_t n;          // nodes
  size_t esize;       // bytes per stored population value
  size_t state_bytes; // bytes of one population buffer (x-blocked, padded rows)
  int device;
  int cu_count;       // compute units of the device
  hipStream_t stream;
  char* ws;
  size_t ws_bytes;
  void* buf[2];       // population buffers (post-collision values, pull layout)
  int cur;            // index of the buffer holding the current state
  double* chibar;     // nx * nz span sums of chi (diagnostics)
  double* partials;   // diagnostic partial sums (diag_partials doubles)
  double* dres;       // 8 doubles: current diagnostics
  double* d0;         // 8 doubles: diagnostics at initialisation
  double* scratch;    // n doubles (get/set hooks, wall shear)
  int64_t step;
  bool paired;        // the grid takes steps two at a time
  int per_launch;     // steps that the next launch makes where it is: 1 or 2
  bool pinned;        // a captured graph names the population buffers
  bool initialised;
  int x0;             // gate index
  // the adjoint run's second stream (default priority) and its events, made
  // on first use for a grid whose recomputation overlaps the reverse sweep
  hipStream_t side;
  hipEvent_t ev_fork, ev_rec[2], ev_rev[2];
};

namespace lbm {

constexpr int kBlock = 256;  // threads per block along x (multiple of 64)
constexpr int kNodesPerThread = 2;  // step kernel: nodes per thread along x (FP32, FP64)
// The cumulant + D3Q27-scalar model holds 54 populations per node: one node
// per thread keeps its register count (and so its occupancy) near the others'.
// With 16-bit storage one node per thread also measured faster (FP16 +5 %,
// BF16 +13 % at 2048 x 128 x 256); FP32 is faster at two.
template <int MODEL, typename ST>
constexpr int nodes_per_thread() {
  return MODEL == 2 ? 1 : (sizeof(ST) == 2 ? 1 : kNodesPerThread);
}

// step.cpp
// one step src -> dst; fw (the adjoint's forward pass, FP32 / FP64 storage):
// also the wall-layer sums of F_w of the gathered state into
// fw[2 fw_blocks], as launch_fw_layers writes them. st: the stream to launch
// on (null: the handle's). With h->paired and no fw the launch makes
// h->per_launch steps; pairs and single steps of such a handle round alike.
hipError_t launch_step(lbm_handle* h, const void* src, void* dst, double* fw = nullptr,
                       hipStream_t st = nullptr);
hipError_t launch_step_fw(lbm_handle* h, const void* src, void* dst, double* fw, hipStream_t st);
// by model: step_m*.hip, step16_m*.hip, pair_m*.hip (models and types that take pairs)
template <int MODEL>
hipError_t launch_step_real(lbm_handle* h, const void* src, void* dst, hipStream_t st);
// h->per_launch steps of a handle with h->paired
template <int MODEL, typename T>
hipError_t launch_paired(lbm_handle* h, const void* src, void* dst, hipStream_t st);
template <int MODEL>
hipError_t launch_step_16(lbm_handle* h, const void* src, void* dst, hipStream_t st);
template <>
hipError_t launch_step_real<0>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_step_real<1>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_step_real<2>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_paired<0, float>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_paired<0, double>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_paired<1, double>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_paired<2, float>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_step_16<0>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_step_16<1>(lbm_handle*, const void*, void*, hipStream_t);
template <>
hipError_t launch_step_16<2>(lbm_handle*, const void*, void*, hipStream_t);

// init.hip; both also take the initial diagnostics into h->d0
hipError_t launch_init_lock(lbm_handle* h, double lock_fraction, double amp, uint64_t seed);
hipError_t launch_init_field(lbm_handle* h, const double* chi0);
// observe.hip
hipError_t launch_moments(lbm_handle* h, int dtype, void* rho, void* ux, void* uy, void* uz,
                          void* chi);
hipError_t launch_wall_shear(lbm_handle* h, int dtype, void* tau, void* tau_bar);
hipError_t launch_diag(lbm_handle* h, double* out);
// the second half of launch_diag: the column pass's partial sums and span means
// (h->partials, h->chibar) into out
hipError_t launch_diag_reduce(lbm_handle* h, double* out);
// One block reads small concentration fields for their depth maxima faster than
// a second launch takes (128 x 16: about 6 us either way); of large ones it
// makes a serial chain (1024 x 128: 21 us, 2048 x 256: 87 us), so those are
// reduced by x-block first. Shallow grids have no chain to cut.
inline bool diag_depth_first(int nx, int nz) { return nz >= 16 && (int64_t)nx * nz >= 16384; }
// doubles of h->partials: one slot per x-block and z, then, for the depth pass,
// one per x-block and the columns' maxima
constexpr int kDiagSlots = 8;
inline size_t diag_partials(int nx, int nxb, int nz) {
  return (size_t)nxb * nz * kDiagSlots + (diag_depth_first(nx, nz) ? (size_t)nxb * kDiagSlots + nx : 0);
}
// kernels.hip
hipError_t launch_get_pop(lbm_handle* h, int q, double* dst);
hipError_t launch_set_pop(lbm_handle* h, int q, const double* src);
// device address, on the current device, of the static scratch array of the
// allocation-free diagnostics (kStaticScratchDoubles doubles: the grids that
// the entry point takes, whose span means and 8 doubles per 256 columns fit
// 2^22, need up to 1.17 of that with the 8 doubles per 64 columns and the
// columns' maxima that the kernels keep)
constexpr size_t kStaticScratchDoubles = ((size_t)1 << 22) + ((size_t)1 << 20);
hipError_t static_scratch(double** ptr);
// copy.cpp
hipError_t launch_copy_state(lbm_handle* h, const void* src, void* dst);
// util.hip
hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t stream);

// adjoint.hip
int adjoint_blocks(const lbm_handle* h);
int fw_blocks(const lbm_handle* h);
hipError_t launch_adjoint_step(lbm_handle* h, const void* state, const void* lam_next,
                               void* lam_out, double a0, double a1, double* gpart, double* dchi0);
hipError_t launch_adjoint_seed(lbm_handle* h, const void* state, void* lam, double a0, double a1,
                               const double* fs);
hipError_t launch_front_seed(lbm_handle* h, double w_front, double* out);
// wall-layer sums of F_w of the current state into part[2 fw_blocks]
hipError_t launch_fw_layers(lbm_handle* h, const void* state, double* part);
// out[0] += nu0 (9 S0 - S1) / 3 over nparts partial pairs (fixed order)
hipError_t launch_fw_reduce(lbm_handle* h, const double* part, int64_t nparts, double* out);
hipError_t launch_sum_pairs(lbm_handle* h, const double* part, int nparts, double* out);
hipError_t launch_zero(lbm_handle* h, double* p, int64_t n);

}  // namespace lbm
