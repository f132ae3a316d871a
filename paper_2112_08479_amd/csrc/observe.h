// The diagnostics' column pass, shared by the state's and the initial state's
// kernels.
#pragma once

#include "dispatch.h"

namespace lbm {

// at most 8 waves per x-block and z, which share its span rows: enough loads in
// flight on small grids, and a grid of any span keeps them busy. A launch holds
// fewer than 2^32 threads.
constexpr int kDiagThreads = 512;
static inline int diag_threads(const Grid& g) {
  const int64_t threads = (int64_t)g.nxb * g.nz * 64;
  int w = 1;
  while (w < 8 && w < g.ny && threads * (2 * w) < ((int64_t)1 << 32)) w *= 2;
  return 64 * w;
}

// moments of a node before the collision, FP64
struct NodeSums {
  double drho = 0, jx = 0, jy = 0, jz = 0, c = 0;
};

// whether population q is the first of its (c_y, c_z), or of c_x != 0
template <class L>
constexpr bool first_of_yz(int q) {
  for (int p = 0; p < q; ++p)
    if (L::cy[p] == L::cy[q] && L::cz[p] == L::cz[q]) return false;
  return true;
}

// Sums of the flow deviations: over x first, so that the nine (c_y, c_z) sums
// serve the density and two momenta (about 50 additions against 80).
template <class LF, typename CT>
__device__ __forceinline__ void flow_sums(const CT* fg, NodeSums& s) {
  double S[3][3];
  s.jx = 0;
  static_for<0, LF::Q>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    const double v = to_d(fg[q]);
    double& t = S[LF::cy[q] + 1][LF::cz[q] + 1];
    t = first_of_yz<LF>(q) ? v : t + v;
    if (LF::cx[q]) s.jx += LF::cx[q] * v;
  });
  const double m = S[0][0] + S[0][1] + S[0][2], p = S[2][0] + S[2][1] + S[2][2];
  s.drho = m + p + (S[1][0] + S[1][1] + S[1][2]);
  s.jy = p - m;
  s.jz = (S[0][2] - S[0][0]) + (S[1][2] - S[1][0]) + (S[2][2] - S[2][0]);
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// block-wide reduction of NV values (sum, except index imax: max); result in
// thread 0. Fixed order, so the result is reproducible.
template <int NV>
__device__ void block_reduce(double (&v)[NV], int imax) {
  __shared__ double red[kDiagThreads / 64 * NV];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = (k == imax) ? wave_max(v[k]) : wave_sum(v[k]);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wid * NV + k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w)
#pragma unroll
      for (int k = 0; k < NV; ++k)
        v[k] = (k == imax) ? fmax(v[k], red[w * NV + k]) : v[k] + red[w * NV + k];
  }
  __syncthreads();
}

// Bound by reading the state: 1024 x 64 x 128 FP32 233 -> 185 us (6.2 TB/s), bf16
// 185 -> 130 (4.4), 128 x 8 x 16 FP64 16 -> 9, against one thread per column with
// 64-bit addresses per population and a square root per node.
// One block per x-block and z; its waves take the span rows in turn. node(x, y,
// z, sums) gives a node's moments; it is called by every lane of a wave, with x
// held inside the grid. Writes the span mean of chi, and the block's partial
// sums {drho, chi, u_x(z=0), u_x(z=1), max |u|^2, nonfinite} in slot z nxb + xb.
template <class Node>
__device__ __forceinline__ void column_sums(const Grid& g, double gp, double* __restrict__ chibar,
                                            double* __restrict__ partials, Node&& node) {
  __shared__ double cols[kDiagThreads];
  const int lane = (int)threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
  // a z row's x-blocks on one XCD: their pulls share lines at the seams
  const int b = xcd_row_order(blockIdx.x, gridDim.x, g.nxb);
  const int z = b / g.nxb, xb = b - z * g.nxb;
  const int x = xb * kXB + lane;
  double v[6] = {0, 0, 0, 0, 0, 0};
  double col = 0;
  for (int y = w; y < g.ny; y += nw) {
    NodeSums s;
    node(x < g.nx ? x : g.nx - 1, y, z, s);
    if (x < g.nx) {
      const double r = 1.0 + s.drho;
      const double ux = s.jx / r, uy = s.jy / r, uz = (s.jz - 0.5 * gp * s.c) / r;
      const bool fin = isfinite(r) && isfinite(s.c) && isfinite(ux) && isfinite(uy) && isfinite(uz);
      v[0] += s.drho;
      col += s.c;
      if (z == 0) v[2] += ux;
      if (z == 1) v[3] += ux;
      if (fin)
        v[4] = fmax(v[4], ux * ux + uy * uy + uz * uz);
      else
        v[5] += 1.0;
    }
  }
  v[1] = col;
  cols[threadIdx.x] = col;
  __syncthreads();
  if (w == 0 && x < g.nx) {
    for (int i = 1; i < nw; ++i) col += cols[i * 64 + lane];
    chibar[(int64_t)z * g.nx + x] = col / g.ny;
  }
  block_reduce<6>(v, 4);
  if (threadIdx.x == 0) {
    double* o = partials + (int64_t)b * kDiagSlots;
    for (int k = 0; k < 6; ++k) o[k] = v[k];
  }
}

}  // namespace lbm
