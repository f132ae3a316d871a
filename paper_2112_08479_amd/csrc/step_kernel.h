// The single step: fused gather + collide + store. Included by one translation
// unit per model and storage width, which instantiates the launchers.
#pragma once

#include "dispatch.h"

namespace lbm {

// ------------------------------------------------------------------- step
// one tile: NPT * blockDim.x consecutive nodes of one row; KIND: kCumFast
// (omega3..omega6 = 1), kCumGeneral (given rates), kCumParam (parametrised).
// FW (the adjoint's forward pass): the tiles of the wall layers z = 0, 1 also
// write the x-velocity sums of their x-blocks that F_w (Eq. 62, 64) needs for
// the state they gather, as the separate wall-layer kernel does: per x-block
// the wave sum of u_x = j_x / rho (FP64, populations in order) into
// fwp[2 b + z], with b = xb + nxb (y + ny z), and 0 into the other slot.
// PAIRED: the collision of the paired steps. NT: the stores pass the caches.
template <int MODEL, typename ST, typename SS, typename CT, bool LES, int KIND, int NPT, bool FW,
          bool PAIRED, bool NT>
__device__ __forceinline__ void step_tile(const ST* __restrict__ src, ST* __restrict__ dst,
                                          const Grid& g, const Phys<CT>& p, int nbx, int b,
                                          double* __restrict__ fwp) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  const int row = b / nbx;
  const int x0 = (b - row * nbx) * (int)blockDim.x * NPT;
  // lanes with no node at all; the wave sums of FW need every lane of a wave
  if (!FW && x0 + (int)threadIdx.x >= g.nx) return;
  const int y = row % g.ny, z = row / g.ny;
  constexpr int QT = LF::Q + LS::Q;
  const TileLanes<QT, NPT> t = tile_lanes<QT, NPT>(g, x0, (int)threadIdx.x, (int)blockDim.x);
  CT fg[NPT][LF::Q], ph[NPT][LS::Q];
  gather_rows<LF, LS, NPT, ST, CT, SS>(src, g, t, y, z, fg, ph);
  if constexpr (FW) {
    if (z < 2) {  // uniform per block
      const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
#pragma unroll
      for (int k = 0; k < NPT; ++k) {
        double v = 0.0;
        if (t.x[k] < g.nx) {
          double drho = 0.0, jx = 0.0;
          static_for<0, LF::Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            drho += (double)fg[k][q];
            if (LF::cx[q]) jx += LF::cx[q] * (double)fg[k][q];
          });
          v = jx / (1.0 + drho);
        }
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        const int xb = ((x0 + k * (int)blockDim.x) >> kXBShift) + wave;
        if (lane == 0 && xb < g.nxb) {
          const int64_t fb = xb + (int64_t)g.nxb * (y + (int64_t)g.ny * z);
          fwp[2 * fb] = z == 0 ? v : 0.0;
          fwp[2 * fb + 1] = z == 0 ? 0.0 : v;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NPT; ++k) collide_node<MODEL, LES, KIND, PAIRED>(fg[k], ph[k], p);
  // block-uniform segment pointers + the lane's own offset, as for the loads
  ST* drow = dst + (int64_t)row * g.nxb * (QT * kXB);
  static_for<0, QT>([&](auto qc) {
    constexpr int a = decltype(qc)::value;
    ST* pa = drow + a * kXB;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      if ((k == 0 && !FW) || t.x[k] < g.nx) {
        if constexpr (a < LF::Q)
          store_val<NT>(&pa[t.own[k]], Conv<ST, CT>::store(fg[k][a]));
        else
          store_val<NT>(&reinterpret_cast<SS*>(pa)[t.own[k]], Conv<SS, CT>::store(ph[k][a - LF::Q]));
      }
    }
  });
}

// PAIRED: the instance of the translation units of paired steps, which contract
// multiply-adds in their own way and must not be merged with the others'.
template <int MODEL, typename ST, typename SS, typename CT, bool LES, int KIND, int NPT,
          bool FW, bool PAIRED, bool NT>
__global__ __launch_bounds__(kBlock) void k_step(const ST* __restrict__ src, ST* __restrict__ dst,
                                                 Grid g, Phys<CT> p, int nbx,
                                                 double* __restrict__ fwp) {
  step_tile<MODEL, ST, SS, CT, LES, KIND, NPT, FW, PAIRED, NT>(src, dst, g, p, nbx,
                                                   xcd_row_order(blockIdx.x, gridDim.x, nbx), fwp);
}

template <int M, typename ST, typename SS, typename CT, int NPT, bool FW, bool PAIRED = false>
static hipError_t launch_step_npt(lbm_handle* h, const Grid& g, const void* src, void* dst,
                                  double* fw, hipStream_t st) {
  // The two nodes of a thread are compiled with their own contractions, so the
  // block size, which pairs the nodes, moves FP32's last bits; the span velocity
  // of BGK shows these at the 1e-5 level. Threads of two nodes that stand alone
  // take full blocks whatever the row leaves idle.
  const int lanes = (g.nx + NPT - 1) / NPT;
  const int bx = NPT > 1 && !PAIRED ? std::min(kBlock, (lanes + 63) / 64 * 64)
                                    : tile_threads(g.nx, (int64_t)g.ny * g.nz, NPT, h->cu_count);
  const int nbx = (g.nx + bx * NPT - 1) / (bx * NPT);
  const unsigned blocks = (unsigned)((int64_t)nbx * g.ny * g.nz);
  const Phys<CT> p = phys_of<CT>(h);
  const ST* s = static_cast<const ST*>(src);
  ST* d = static_cast<ST*>(dst);
  return with_collision<M>(h, [&](auto les, auto kind) {
    constexpr bool LES = decltype(les)::value;
    constexpr int KIND = decltype(kind)::value;
    if constexpr (FW && KIND == kCumGeneral) {  // not differentiated
      return hipErrorInvalidValue;
    } else {
      if (stores_past_caches(h->state_bytes))
        hipLaunchKernelGGL((k_step<M, ST, SS, CT, LES, KIND, NPT, FW, PAIRED, true>), dim3(blocks), dim3(bx), 0, st, s, d, g, p, nbx, fw);
      else
        hipLaunchKernelGGL((k_step<M, ST, SS, CT, LES, KIND, NPT, FW, PAIRED, false>), dim3(blocks), dim3(bx), 0, st, s, d, g, p, nbx, fw);
      return hipGetLastError();
    }
  });
}

// Grids too small to give every SIMD four waves at the preferred nodes per
// thread (cache-resident, latency-bound runs such as a 256 x 16 x 32
// adjoint) take one node per thread: twice the waves.
static bool few_waves(const lbm_handle* h, int npt) {
  const int64_t waves = (h->n + (int64_t)64 * npt - 1) / ((int64_t)64 * npt);
  return waves < (int64_t)16 * h->cu_count;
}

template <int M, typename ST, typename SS, typename CT, bool FW = false, bool PAIRED = false>
static hipError_t launch_step_of(lbm_handle* h, const void* src, void* dst, double* fw,
                                 hipStream_t stream) {
  const Grid g = grid_of(h);
  constexpr int NPT = nodes_per_thread<M, ST>();
  if constexpr (NPT > 1) {
    if (few_waves(h, NPT)) return launch_step_npt<M, ST, SS, CT, 1, FW, PAIRED>(h, g, src, dst, fw, stream);
  }
  return launch_step_npt<M, ST, SS, CT, NPT, FW, PAIRED>(h, g, src, dst, fw, stream);
}

}  // namespace lbm
