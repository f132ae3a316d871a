// Test hooks (populations in and out) and the static scratch.
//
// State convention. A population buffer holds post-collision values at the
// node where they were produced. One step pulls them (the gather with
// half-way bounce-back and periodic span, i.e. streaming of Eq. 17), collides
// at the node and writes the result to the other buffer. The pre-collision
// populations at step n are therefore gather(buffer). The gather is a
// permutation of the (population, node) slots, so every state has exactly one
// buffer representation; the init kernels and the set hook write the inverse
// permutation.
#include <math.h>

#include <mutex>

#include "dispatch.h"

namespace lbm {

// -------------------------------------------------------------- test hooks
template <class L>
__device__ __forceinline__ void vel(int q, int& cx, int& cy, int& cz) {
  cx = L::cx[q];
  cy = L::cy[q];
  cz = L::cz[q];
}

// pre-collision population a (0..qt-1) at every node, full value, float64
template <int MODEL, typename ST, typename SS>
__global__ __launch_bounds__(kBlock) void k_get_pop(const ST* __restrict__ src, Grid g, int a,
                                                    int nbx, double* __restrict__ out) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  using CT = typename std::conditional<std::is_same<ST, double>::value, double, float>::type;
  const int b = blockIdx.x;
  const int row = b / nbx;
  const int x = (b - row * nbx) * blockDim.x + threadIdx.x;
  if (x >= g.nx) return;
  const int y = row % g.ny, z = row / g.ny;
  const int64_t node = (int64_t)row * g.nx + x;
  const bool flow = a < LF::Q;
  const int q = flow ? a : a - LF::Q;
  int cx, cy, cz, o;
  double w;
  if (flow) {
    vel<LF>(q, cx, cy, cz);
    o = opp<LF>(q);
    w = weight<LF>(q);
  } else {
    vel<LS>(q, cx, cy, cz);
    o = opp<LS>(q);
    w = 0.0;
  }
  const int base = flow ? 0 : LF::Q;
  const int xs = x - cx, zs = z - cz;
  int ys = y - cy;
  ys = ys < 0 ? g.ny - 1 : (ys >= g.ny ? 0 : ys);
  const bool wall = (unsigned)xs >= (unsigned)g.nx || (unsigned)zs >= (unsigned)g.nz;
  constexpr int QT = LF::Q + LS::Q;
  const int64_t off = wall ? elem_index<QT>(g, base + o, row, x)
                           : elem_index<QT>(g, base + q, (int64_t)zs * g.ny + ys, xs);
  out[node] = (flow ? to_d(Conv<ST, CT>::load(src[off]))
                    : to_d(Conv<SS, CT>::load(reinterpret_cast<const SS*>(src)[off]))) + w;
}

// inverse of the gather for population a given its pre-collision values v
// (full values, float64): slot (a, y) <- v(y + c_a) when that node is fluid;
// slot (opp a, y) <- v(y) when y - c_a is outside.
template <int MODEL, typename ST, typename SS>
__global__ __launch_bounds__(kBlock) void k_set_pop(ST* __restrict__ dst, Grid g, int a, int nbx,
                                                    const double* __restrict__ v) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  using CT = typename std::conditional<std::is_same<ST, double>::value, double, float>::type;
  const int b = blockIdx.x;
  const int row = b / nbx;
  const int x = (b - row * nbx) * blockDim.x + threadIdx.x;
  if (x >= g.nx) return;
  const int y = row % g.ny, z = row / g.ny;
  const int64_t node = (int64_t)row * g.nx + x;
  const bool flow = a < LF::Q;
  const int q = flow ? a : a - LF::Q;
  int cx, cy, cz, o;
  double w;
  if (flow) {
    vel<LF>(q, cx, cy, cz);
    o = opp<LF>(q);
    w = weight<LF>(q);
  } else {
    vel<LS>(q, cx, cy, cz);
    o = opp<LS>(q);
    w = 0.0;
  }
  const int base = flow ? 0 : LF::Q;
  auto put = [&](int64_t i, double val) {
    if (flow)
      dst[i] = Conv<ST, CT>::store(CT(val));
    else
      reinterpret_cast<SS*>(dst)[i] = Conv<SS, CT>::store(CT(val));
  };
  {
    const int xn = x + cx, zn = z + cz;
    int yn = y + cy;
    yn = yn < 0 ? g.ny - 1 : (yn >= g.ny ? 0 : yn);
    if ((unsigned)xn < (unsigned)g.nx && (unsigned)zn < (unsigned)g.nz)
      put(elem_index<LF::Q + LS::Q>(g, base + q, row, x), v[((int64_t)zn * g.ny + yn) * g.nx + xn] - w);
  }
  {
    const int xs = x - cx, zs = z - cz;
    if ((unsigned)xs >= (unsigned)g.nx || (unsigned)zs >= (unsigned)g.nz)
      put(elem_index<LF::Q + LS::Q>(g, base + o, row, x), v[node] - w);
  }
}

// ------------------------------------------- allocation-free diagnostics
// Scratch of lbm_checkpoint_diagnostics: the span-averaged concentration, the
// per-block partial sums and the result slot of the diagnostics kernels,
// which a handle keeps in its workspace. A file-scope device array, so that
// the entry point allocates nothing; every GPU the library runs on holds its
// own copy until the process ends. In host code its name is only a stand-in
// for the symbol: its device address comes from hipGetSymbolAddress, taken
// once per device with that device current, and only that address is used.
static __device__ __align__(256) double scratch[kStaticScratchDoubles];

hipError_t static_scratch(double** ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = static_cast<double*>(p);
  }
  *ptr = addr[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------- dispatch

hipError_t launch_get_pop(lbm_handle* h, int a, double* dst) {
  const Grid g = grid_of(h);
  const int bx = block_x(h);
  const int nbx = (g.nx + bx - 1) / bx;
  const unsigned blocks = (unsigned)((int64_t)nbx * g.ny * g.nz);
  return with_model(h, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    return with_storage(h, [&](auto st, auto ss, auto) {
      using ST = decltype(st);
      using SS = decltype(ss);
      hipLaunchKernelGGL((k_get_pop<M, ST, SS>), dim3(blocks), dim3(bx), 0, h->stream,
                         static_cast<const ST*>(h->buf[h->cur]), g, a, nbx, dst);
      return hipGetLastError();
    });
  });
}

hipError_t launch_set_pop(lbm_handle* h, int a, const double* src) {
  const Grid g = grid_of(h);
  const int bx = block_x(h);
  const int nbx = (g.nx + bx - 1) / bx;
  const unsigned blocks = (unsigned)((int64_t)nbx * g.ny * g.nz);
  return with_model(h, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    return with_storage(h, [&](auto st, auto ss, auto) {
      using ST = decltype(st);
      using SS = decltype(ss);
      hipLaunchKernelGGL((k_set_pop<M, ST, SS>), dim3(blocks), dim3(bx), 0, h->stream,
                         static_cast<ST*>(h->buf[h->cur]), g, a, nbx, src);
      return hipGetLastError();
    });
  });
}

}  // namespace lbm
