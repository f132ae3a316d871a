// What a run reports: moments, the bottom-wall shear stress and the FP64
// diagnostics.
#include "observe.h"

namespace lbm {

// ----------------------------------------------------------------- moments
// outputs are not read again soon: past the caches
template <typename OT>
__device__ __forceinline__ void put_out(void* p, int64_t i, double v) {
  if (p) __builtin_nontemporal_store((OT)v, &static_cast<OT*>(p)[i]);
}

// the step kernel's tiles and pulls, one node per thread: 2048 x 128 x 256 FP16
// 1198 -> 1020 us (5.8 TB/s with its FP32 outputs)
template <int MODEL, typename ST, typename SS, typename CT, typename OT>
__global__ __launch_bounds__(kBlock) void k_moments(const ST* __restrict__ src, Grid g, double gp,
                                                    int nbx, void* rho, void* ux, void* uy,
                                                    void* uz, void* chi) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  constexpr int QT = LF::Q + LS::Q;
  const int b = xcd_row_order(blockIdx.x, gridDim.x, nbx);
  const int row = b / nbx;
  const int x0 = (b - row * nbx) * (int)blockDim.x;
  if (x0 + (int)threadIdx.x >= g.nx) return;
  const int y = row % g.ny, z = row / g.ny;
  const int xb0 = x0 >> kXBShift;
  const TileLanes<QT, 1> t = tile_lanes<QT, 1>(g, x0, (int)threadIdx.x, (int)blockDim.x, xb0);
  src += (int64_t)xb0 * (QT * kXB);
  CT fg[1][LF::Q], ph[1][LS::Q];
  gather_rows<LF, LS, 1, ST, CT, SS>(src, g, t, y, z, fg, ph);
  NodeSums s;
  flow_sums<LF>(fg[0], s);
  static_for<0, LS::Q>([&](auto qc) { s.c += to_d(ph[0][decltype(qc)::value]); });
  const int64_t node = (int64_t)row * g.nx + t.x[0];
  const double r = 1.0 + s.drho;
  put_out<OT>(rho, node, r);
  put_out<OT>(ux, node, s.jx / r);
  put_out<OT>(uy, node, s.jy / r);
  put_out<OT>(uz, node, (s.jz - 0.5 * gp * s.c) / r);
  put_out<OT>(chi, node, s.c);
}

// -------------------------------------------------------------- wall shear
// Bottom-wall shear stress (Eq. 62, lattice units, rho_bar = 1): the slope at
// the half-way wall of the quadratic through u = 0 at the wall and the nodes at
// distances 1/2 and 3/2, tau_w = nu0 (9 u_x(z=0) - u_x(z=1)) / 3, from the
// pre-collision u_x = j_x / rho of the two nodes. One wavefront per x-block and
// span row, so that the whole wall is in flight at once.
template <int MODEL, typename ST, typename CT>
__device__ __forceinline__ double wall_value(const ST* __restrict__ src, const Grid& g, int xb, int y,
                                             double nu0, int& x) {
  using LF = typename ModelT<MODEL>::LF;
  constexpr int QT = LF::Q + ModelT<MODEL>::LS::Q;
  const int lane = (int)threadIdx.x & 63;
  const TileLanes<QT, 1> t = tile_lanes<QT, 1>(g, xb * kXB, lane, 64, xb);
  src += (int64_t)xb * (QT * kXB);
  x = t.x[0];
  const bool wall = __builtin_amdgcn_ballot_w64(x == 0 || x == g.nx - 1) != 0;
  double u[2];
#pragma unroll
  for (int z = 0; z < 2; ++z) {
    CT fg[1][LF::Q];
    pull_lattice<LF, 0, QT, 1, ST, CT>(src, g, y, z, t, wall, fg);
    NodeSums s;
    flow_sums<LF>(fg[0], s);
    u[z] = s.jx / (1.0 + s.drho);
  }
  return nu0 * (9.0 * u[0] - u[1]) / 3.0;
}

// Any wall; tw (ny x nx, FP64) keeps the values for the mean, which a second
// launch takes (1024 x 64, 16-bit: 188 -> 10 us for both).
template <int MODEL, typename ST, typename CT, typename OT>
__global__ __launch_bounds__(kBlock) void k_wall_shear(const ST* __restrict__ src, Grid g, double nu0,
                                                       double* __restrict__ tw, void* tau) {
  const int b = (int)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (b >= g.nxb * g.ny) return;
  const int y = b / g.nxb;
  int x;
  const double v = wall_value<MODEL, ST, CT>(src, g, b - y * g.nxb, y, nu0, x);
  if (x >= g.nx) return;
  tw[(int64_t)y * g.nx + x] = v;
  put_out<OT>(tau, (int64_t)y * g.nx + x, v);
}

// A wall of few span rows in one launch: a block holds an x-block's rows, one
// wave each, and its first wave takes the mean of the values in LDS.
constexpr int kWallRows = 8;
template <int MODEL, typename ST, typename CT, typename OT>
__global__ __launch_bounds__(kWallRows * 64) void k_wall_shear_rows(const ST* __restrict__ src, Grid g,
                                                                    double nu0, void* tau, void* tau_bar) {
  __shared__ double tw[kWallRows * kXB];
  const int y = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  int x;
  const double v = wall_value<MODEL, ST, CT>(src, g, (int)blockIdx.x, y, nu0, x);
  tw[threadIdx.x] = v;
  if (x < g.nx) put_out<OT>(tau, (int64_t)y * g.nx + x, v);
  __syncthreads();
  if (y != 0 || x >= g.nx) return;
  double s = 0;
  for (int r = 0; r < g.ny; ++r) s += tw[r * kXB + lane];
  put_out<OT>(tau_bar, x, s / g.ny);
}

// span mean (the integrand of Eq. 66), rows in order
template <typename OT>
__global__ __launch_bounds__(64) void k_span_mean(const double* __restrict__ tw, Grid g, void* tau_bar) {
  const int x = (int)blockIdx.x * 64 + (int)threadIdx.x;
  if (x >= g.nx) return;
  double s = 0;
#pragma unroll 8
  for (int y = 0; y < g.ny; ++y) s += tw[(int64_t)y * g.nx + x];
  put_out<OT>(tau_bar, x, s / g.ny);
}

// ------------------------------------------------------------- diagnostics
template <int MODEL, typename ST, typename SS, typename CT>
__global__ __launch_bounds__(kDiagThreads) void k_diag_columns(const ST* __restrict__ src, Grid g,
                                                               double gp, double* __restrict__ chibar,
                                                               double* __restrict__ partials) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  constexpr int QT = LF::Q + LS::Q;
  const int b = xcd_row_order(blockIdx.x, gridDim.x, g.nxb);
  const int xb = b % g.nxb;
  const TileLanes<QT, 1> t = tile_lanes<QT, 1>(g, xb * kXB, (int)threadIdx.x & 63, 64, xb);
  src += (int64_t)xb * (QT * kXB);
  column_sums(g, gp, chibar, partials, [&](int, int y, int z, NodeSums& s) {
    CT fg[1][LF::Q], ph[1][LS::Q];
    gather_rows<LF, LS, 1, ST, CT, SS>(src, g, t, y, z, fg, ph);
    flow_sums<LF>(fg[0], s);
    static_for<0, LS::Q>([&](auto qc) { s.c += to_d(ph[0][decltype(qc)::value]); });
  });
}

// One block per x-block: the partial sums and the depth maxima of its columns.
__global__ __launch_bounds__(kDiagThreads) void k_diag_depth(const double* __restrict__ partials,
                                                             const double* __restrict__ chibar, Grid g,
                                                             double* __restrict__ part2,
                                                             double* __restrict__ colmax) {
  __shared__ double m[kDiagThreads];
  const int t = (int)threadIdx.x, lane = t & 63, w = t >> 6, nw = (int)blockDim.x >> 6;
  const int xb = (int)blockIdx.x, x = xb * kXB + lane;
  double v[6] = {0, 0, 0, 0, 0, 0};
  for (int z = t; z < g.nz; z += (int)blockDim.x) {
    const double* p = partials + ((int64_t)z * g.nxb + xb) * kDiagSlots;
    for (int k = 0; k < 6; ++k) v[k] = (k == 4) ? fmax(v[k], p[k]) : v[k] + p[k];
  }
  double c = -INFINITY;
  if (x < g.nx) {
#pragma unroll 4
    for (int z = w; z < g.nz; z += nw) c = fmax(c, chibar[(int64_t)z * g.nx + x]);
  }
  m[t] = c;
  block_reduce<6>(v, 4);
  if (w == 0 && x < g.nx) {
    for (int i = 1; i < nw; ++i) c = fmax(c, m[i * 64 + lane]);
    colmax[x] = c;
  }
  if (t == 0)
    for (int k = 0; k < 6; ++k) part2[(int64_t)xb * kDiagSlots + k] = v[k];
}

// single block: reduce the partials, locate the front, write out[8] =
// {mass, chi_mass, fw, x_front, umax, nonfinite, i_star, 0}. colmax: the depth
// maxima if k_diag_depth made them, else NULL.
__global__ __launch_bounds__(1024) void k_diag_final(const double* __restrict__ partials, int nparts,
                                                     const double* __restrict__ chibar,
                                                     const double* __restrict__ colmax, Grid g,
                                                     double nu0, double* __restrict__ out) {
  __shared__ double red[16 * 6];
  __shared__ int ired[16];
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  double v[6] = {0, 0, 0, 0, 0, 0};
  for (int b = t; b < nparts; b += blockDim.x) {
    const double* p = partials + (int64_t)b * kDiagSlots;
    for (int k = 0; k < 6; ++k) v[k] = (k == 4) ? fmax(v[k], p[k]) : v[k] + p[k];
  }
  const double theta = 0.02;
  int best = -1;
  for (int i = t; i < g.nx; i += blockDim.x) {
    double top;
    if (colmax) {
      top = colmax[i];
    } else {
      // the depth maximum of column i, in four independent chains so that
      // the loads overlap (max is exact: the order does not matter)
      double m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      int k = 0;
      for (; k + 3 < g.nz; k += 4)
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = fmax(m[j], chibar[(int64_t)(k + j) * g.nx + i]);
      for (; k < g.nz; ++k) m[0] = fmax(m[0], chibar[(int64_t)k * g.nx + i]);
      top = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
    }
    if (top >= theta) best = i;
  }
  for (int k = 0; k < 6; ++k) v[k] = (k == 4) ? wave_max(v[k]) : wave_sum(v[k]);
  for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
  if (lane == 0) {
    for (int k = 0; k < 6; ++k) red[wid * 6 + k] = v[k];
    ired[wid] = best;
  }
  __syncthreads();
  if (wid != 0) return;
  // wave 0: the sums in fixed order (lane 0), then the depth maxima of the
  // front column and its neighbour across the wave
  const int nw = blockDim.x >> 6;
  for (int w = 1; w < nw; ++w) {
    for (int k = 0; k < 6; ++k) v[k] = (k == 4) ? fmax(v[k], red[w * 6 + k]) : v[k] + red[w * 6 + k];
    best = max(best, ired[w]);
  }
  double m0 = -INFINITY, m1 = -INFINITY;
  if (best >= 0 && best < g.nx - 1) {
    if (colmax) {
      m0 = colmax[best];
      m1 = colmax[best + 1];
    } else {
      for (int k = lane; k < g.nz; k += 64) {
        m0 = fmax(m0, chibar[(int64_t)k * g.nx + best]);
        m1 = fmax(m1, chibar[(int64_t)k * g.nx + best + 1]);
      }
    }
  }
  m0 = wave_max(m0);
  m1 = wave_max(m1);
  if (lane == 0) {
    double xf;
    if (best < 0) {
      xf = 0.0;
    } else if (best == g.nx - 1) {
      xf = (double)g.nx;
    } else {
      xf = best + 0.5 + (m0 - theta) / (m0 - m1);
    }
    out[0] = (double)g.n + v[0];
    out[1] = v[1];
    out[2] = g.nz >= 2 ? nu0 * (9.0 * v[2] - v[3]) / 3.0 : 0.0;
    out[3] = xf;
    out[4] = sqrt(v[4]);  // the root of the largest square is the largest root
    out[5] = v[5];
    out[6] = (double)best;
    out[7] = 0.0;
  }
}

// --------------------------------------------------------------- launchers
hipError_t launch_moments(lbm_handle* h, int dtype, void* rho, void* ux, void* uy, void* uz,
                          void* chi) {
  const Grid g = grid_of(h);
  const int bx = tile_threads(g.nx, (int64_t)g.ny * g.nz, 1, h->cu_count);
  const int nbx = (g.nx + bx - 1) / bx;
  const unsigned blocks = (unsigned)((int64_t)nbx * g.ny * g.nz);
  const double gp = h->prm.g_prime;
  return with_model(h, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    return with_storage(h, [&](auto st, auto ss, auto ct) {
      using ST = decltype(st);
      using SS = decltype(ss);
      using CT = decltype(ct);
      const ST* s = static_cast<const ST*>(h->buf[h->cur]);
      if (dtype == LBM_OUT_F64)
        hipLaunchKernelGGL((k_moments<M, ST, SS, CT, double>), dim3(blocks), dim3(bx), 0, h->stream, s, g, gp, nbx, rho, ux, uy, uz, chi);
      else
        hipLaunchKernelGGL((k_moments<M, ST, SS, CT, float>), dim3(blocks), dim3(bx), 0, h->stream, s, g, gp, nbx, rho, ux, uy, uz, chi);
      return hipGetLastError();
    });
  });
}

// The mean in the same launch where a block holds the whole span: a second launch
// costs 2 us (64 x 4 BGK FP32: 6.3 us with the mean, 8.5 in two launches).
hipError_t launch_wall_shear(lbm_handle* h, int dtype, void* tau, void* tau_bar) {
  const Grid g = grid_of(h);
  const int64_t waves = (int64_t)g.nxb * g.ny;
  const unsigned blocks = (unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64));
  const double nu0 = h->prm.nu0;
  const bool rows = tau_bar && g.ny <= kWallRows;
  auto launch = [&](auto out) {
    using OT = decltype(out);
    const hipError_t e = with_model(h, [&](auto mc) {
      constexpr int M = decltype(mc)::value;
      return with_storage(h, [&](auto st, auto, auto ct) {
        using ST = decltype(st);
        using CT = decltype(ct);
        const ST* s = static_cast<const ST*>(h->buf[h->cur]);
        if (rows)
          hipLaunchKernelGGL((k_wall_shear_rows<M, ST, CT, OT>), dim3(g.nxb), dim3(64 * g.ny), 0, h->stream, s, g, nu0, tau, tau_bar);
        else
          hipLaunchKernelGGL((k_wall_shear<M, ST, CT, OT>), dim3(blocks), dim3(kBlock), 0, h->stream, s, g, nu0, h->scratch, tau);
        return hipGetLastError();
      });
    });
    if (e != hipSuccess || !tau_bar || rows) return e;
    hipLaunchKernelGGL((k_span_mean<OT>), dim3(g.nxb), dim3(64), 0, h->stream, h->scratch, g, tau_bar);
    return hipGetLastError();
  };
  return dtype == LBM_OUT_F64 ? launch(double{}) : launch(float{});
}

hipError_t launch_diag_reduce(lbm_handle* h, double* out) {
  const Grid g = grid_of(h);
  const int nparts = g.nxb * g.nz;
  double* part2 = h->partials + (int64_t)nparts * kDiagSlots;
  double* colmax = part2 + (int64_t)g.nxb * kDiagSlots;
  const bool depth = diag_depth_first(g.nx, g.nz);
  if (depth)
    hipLaunchKernelGGL(k_diag_depth, dim3(g.nxb), dim3(kDiagThreads), 0, h->stream, h->partials, h->chibar, g, part2, colmax);
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(1024), 0, h->stream, depth ? part2 : h->partials,
                     depth ? g.nxb : nparts, h->chibar, depth ? colmax : nullptr, g, h->prm.nu0, out);
  return hipGetLastError();
}

hipError_t launch_diag(lbm_handle* h, double* out) {
  const Grid g = grid_of(h);
  const double gp = h->prm.g_prime;
  const hipError_t e = with_model(h, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    return with_storage(h, [&](auto st, auto ss, auto ct) {
      using ST = decltype(st);
      using SS = decltype(ss);
      using CT = decltype(ct);
      hipLaunchKernelGGL((k_diag_columns<M, ST, SS, CT>), dim3(g.nxb * g.nz), dim3(diag_threads(g)), 0,
                         h->stream, static_cast<const ST*>(h->buf[h->cur]), g, gp, h->chibar, h->partials);
      return hipGetLastError();
    });
  });
  if (e != hipSuccess) return e;
  return launch_diag_reduce(h, out);
}

}  // namespace lbm
