// Initial states and their diagnostics.
#include "dispatch.h"
#include "observe.h"

namespace lbm {

__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

struct LockInit {
  int gate;
  double amp;
  uint64_t seed;
  __device__ double chi0(const Grid& g, int i, int j, int k) const {
    double c = (i < gate) ? 1.0 : 0.0;
    if (amp != 0.0 && (i == gate - 1 || i == gate)) {
      const uint64_t lin = (uint64_t)i + (uint64_t)g.nx * ((uint64_t)j + (uint64_t)g.ny * (uint64_t)k);
      const uint64_t r = splitmix64(seed ^ (lin * 0x9E3779B97F4A7C15ull));
      const double U = (double)(r >> 11) * 0x1.0p-53;
      c += amp * (2.0 * U - 1.0);
    }
    return c;
  }
};
struct FieldInit {
  const double* chi;
  __device__ double chi0(const Grid& g, int i, int j, int k) const {
    return chi[((int64_t)k * g.ny + j) * g.nx + i];
  }
};

// Buffer slot (q, node) is read by node + c_q when that node is fluid, else by
// the node itself for population opp(q) (bounce-back). Initial populations:
// flow f = w (stored deviation 0), scalar phi_p = w_p chi0.
//
// One wavefront per x-block. Mostly writes: the flow part of an x-block is QF 64
// zeros in one span and goes out as 16-byte vectors past the caches (the padding
// of a ragged last block too, which nothing reads). 1024 x 64 x 128: FP32 245 ->
// 201 us (5.7 TB/s), 16-bit 160 -> 106. Beyond the last-level cache the up to
// nine reads of each concentration row show: FP16 2048 x 128 x 256 1439 -> 1375.
template <int MODEL, typename ST, typename SS, class Init>
__global__ __launch_bounds__(kBlock) void k_init(ST* __restrict__ dst, Grid g, Init init, int64_t nblk) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  using CT = typename std::conditional<std::is_same<ST, double>::value, double, float>::type;
  constexpr int QT = LF::Q + LS::Q;
  const int lane = (int)threadIdx.x & 63;
  const int64_t b = (int64_t)blockIdx.x * (kBlock / 64) + ((int)threadIdx.x >> 6);
  if (b >= nblk) return;
  const int64_t row = b / g.nxb;
  const int x = (int)(b - row * g.nxb) * kXB + lane;
  ST* blk = dst + b * (QT * kXB);
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kVec = LF::Q * kXB * (int)sizeof(ST) / 16;
  static_assert(LF::Q * kXB * sizeof(ST) % 16 == 0 && QT * kXB * sizeof(ST) % 16 == 0, "16-byte spans");
  u32x4* v = reinterpret_cast<u32x4*>(blk);
#pragma unroll
  for (int i = 0; i < kVec; i += 64)
    if (i + lane < kVec) __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, &v[i + lane]);
  if (x >= g.nx) return;
  const int y = (int)(row % g.ny), z = (int)(row / g.ny);
  static_for<0, LS::Q>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    const int xn = x + LS::cx[q], zn = z + LS::cz[q];
    int yn = y + LS::cy[q];
    yn = yn < 0 ? g.ny - 1 : (yn >= g.ny ? 0 : yn);
    const bool fluid = (unsigned)xn < (unsigned)g.nx && (unsigned)zn < (unsigned)g.nz;
    const double c = fluid ? init.chi0(g, xn, yn, zn) : init.chi0(g, x, y, z);
    store_val(&reinterpret_cast<SS*>(blk)[(LF::Q + q) * kXB + lane],
              Conv<SS, CT>::store(CT(weight<LS>(q) * c)));
  });
}

// Diagnostics of the initial state without reading it: every node's scalar
// populations are the stored w_p chi0 of the node itself, the flow is at rest.
// The sums are those that the state's column pass would make.
template <int MODEL, typename ST, typename SS, class Init>
__global__ __launch_bounds__(kDiagThreads) void k_diag_init(Grid g, Init init, double gp,
                                                            double* __restrict__ chibar,
                                                            double* __restrict__ partials) {
  using LS = typename ModelT<MODEL>::LS;
  using CT = typename std::conditional<std::is_same<ST, double>::value, double, float>::type;
  column_sums(g, gp, chibar, partials, [&](int x, int y, int z, NodeSums& s) {
    const double c0 = init.chi0(g, x, y, z);
    s = NodeSums{};
    static_for<0, LS::Q>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      s.c += to_d(Conv<SS, CT>::load(Conv<SS, CT>::store(CT(weight<LS>(q) * c0))));
    });
  });
}

template <class Init>
static hipError_t launch_init_any(lbm_handle* h, Init init) {
  const Grid g = grid_of(h);
  const int64_t nblk = (int64_t)g.nxb * g.ny * g.nz;
  const unsigned blocks = (unsigned)((nblk + kBlock / 64 - 1) / (kBlock / 64));
  const double gp = h->prm.g_prime;
  const hipError_t e = with_model(h, [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    return with_storage(h, [&](auto st, auto ss, auto) {
      using ST = decltype(st);
      using SS = decltype(ss);
      hipLaunchKernelGGL((k_init<M, ST, SS, Init>), dim3(blocks), dim3(kBlock), 0, h->stream,
                         static_cast<ST*>(h->buf[h->cur]), g, init, nblk);
      hipLaunchKernelGGL((k_diag_init<M, ST, SS, Init>), dim3(g.nxb * g.nz), dim3(diag_threads(g)), 0,
                         h->stream, g, init, gp, h->chibar, h->partials);
      return hipGetLastError();
    });
  });
  if (e != hipSuccess) return e;
  return launch_diag_reduce(h, h->d0);
}

hipError_t launch_init_lock(lbm_handle* h, double lock_fraction, double amp, uint64_t seed) {
  LockInit init{(int)floor(lock_fraction * h->cfg.nx), amp, seed};
  return launch_init_any(h, init);
}

hipError_t launch_init_field(lbm_handle* h, const double* chi0) {
  return launch_init_any(h, FieldInit{chi0});
}

}  // namespace lbm
