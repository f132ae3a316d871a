// Two time steps in one launch: half the memory traffic of two single steps.
//
// A single step is bound by its nine-row pull (about 5.8 of the copy's 6.3 TB/s,
// the vector units 41 % busy in FP32), so what is left to gain is traffic. The
// tile of 64 x TY nodes marching in z computes 19 waves of collisions for 16
// (TY = 8: ten rows and the ring's columns, then eight rows) and reads 1.17
// times the state (1.23 with the D3Q27 scalar). Measured at 1024 x 64 x 128 with
// LES, us per step, single -> paired: cumulant + D3Q7 FP32 394 -> 255, given rates
// 393 -> 322, parametrised 394 -> 275, FP64 820 -> 560, 885 -> 652 and 845 -> 594;
// cumulant + D3Q27 FP32 656 -> 401, 649 -> 488 and 657 -> 433; BGK FP64 599 -> 443.
// The vector units are 52 % busy (46 % with the D3Q27 scalar, 49 % parametrised);
// the rest of the time goes to the phases between the barriers, in which every
// wave moves data (the lean collisions of collide.h took 283 to 255). Measured and
// not taken: TY = 5 or 3 with two blocks per CU (670 and 890 us per pair against
// 558), pulling before the first step's collision (579 against 560), half the
// waves with their two steps in the other order (the registers spill: 612), four
// or eight chunks in z for two (598 and 630).
#pragma once

#include "dispatch.h"
#include "twostep.h"

namespace lbm {

// waves per SIMD that the block's registers must allow
template <typename T>
constexpr int tile_waves() {
  return sizeof(T) == 8 ? 2 : 3;
}
// Populations of the next plane that are pulled before the second step is
// computed: all, and already before the barriers, where the registers hold
// them; the D3Q27 scalar's 27 after it in the model with 54.
template <int MODEL>
constexpr int pulled_ahead() {
  return MODEL == 2 ? 27 : ModelT<MODEL>::LF::Q + ModelT<MODEL>::LS::Q;
}

// A z plane of populations as a buffer resource: loads and stores take a
// scalar offset (the population) and a 32-bit lane offset, so that no 64-bit
// lane addresses are kept or computed. Accesses beyond `bytes` are dropped by
// the hardware.
using Rsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Rsrc plane_rsrc(const void* p, uint32_t bytes) {
  // uniform values: said so outright, they stay in scalar registers
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(lo | (hi << 32)), 0,
                                           __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}
template <typename T>
__device__ __forceinline__ T load_at(Rsrc r, uint32_t lane, int scalar) {
  if constexpr (sizeof(T) == 8) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(T, (u32x2)__builtin_amdgcn_raw_buffer_load_b64(r, lane, scalar, 0));
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, lane, scalar, 0));
  }
}
// a lane offset beyond every plane (three planes are below 2 GiB)
constexpr uint32_t kDropped = 0x80000000u;
template <bool NT, typename T>
__device__ __forceinline__ void store_at(Rsrc r, uint32_t lane, int scalar, T v) {
  constexpr int kNt = NT ? 2 : 0;
  if constexpr (sizeof(T) == 8) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, lane, scalar, kNt);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, lane, scalar, kNt);
  }
}

template <typename CT, int N>
__device__ __forceinline__ void keep(CT (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm("" : "+v"(v[i]));
}

// LDS contents before the barrier are seen after it; global loads and stores
// stay in flight across it
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The z planes a pull reads: m, 0, p (z - 1, z, z + 1; z itself beyond a wall)
// for a node with no wall beside it, and all three from one resource for the
// others, where `lo` is the first of them.
struct Planes {
  Rsrc m, z, p, all;
  uint32_t to_m, to_z, to_p;  // bytes from `all` to each plane
};
template <typename ST>
__device__ __forceinline__ Planes planes_at(const ST* src, const Grid& g, int64_t plane,
                                            uint32_t bytes, int z) {
  const int zm = z == 0 ? z : z - 1, zp = z == g.nz - 1 ? z : z + 1;
  Planes s;
  s.m = plane_rsrc(src + zm * plane, bytes);
  s.z = plane_rsrc(src + z * plane, bytes);
  s.p = plane_rsrc(src + zp * plane, bytes);
  s.all = plane_rsrc(src + zm * plane, bytes * (uint32_t)(zp - zm + 1));
  s.to_m = 0;
  s.to_z = bytes * (uint32_t)(z - zm);
  s.to_p = bytes * (uint32_t)(zp - zm);
  return s;
}

// pull of the populations A .. B - 1 of a node of plane z. At a wall the
// lane's address itself turns to the node's own opposite population, so that
// these loads fly as freely as the others.
template <class P, int A, int B, typename T, int QF, int QS>
__device__ __forceinline__ void pull_plane(const Planes& s, const Grid& g, int z, int x, bool wall,
                                           const uint32_t (&off)[3][3], T (&f)[QF], T (&ph)[QS]) {
  constexpr int kSeg = kXB * (int)sizeof(T);
  auto load = [&](auto ac, Rsrc r, uint32_t lane, int scalar) __attribute__((always_inline)) {
    constexpr int a = decltype(ac)::value;
    if constexpr (P::flow(a))
      f[a] = load_at<T>(r, lane, scalar);
    else
      ph[a - QF] = load_at<T>(r, lane, scalar);
  };
  if (!wall) {
    static_for<A, B>([&](auto ac) {
      constexpr int a = decltype(ac)::value;
      load(ac, P::cz(a) > 0 ? s.m : (P::cz(a) < 0 ? s.p : s.z), off[P::cy(a) + 1][P::cx(a) + 1], a * kSeg);
    });
  } else {
    // hidden, so that no sums are kept over the planes for this rare path
    uint32_t o[3][3];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      o[i / 3][i % 3] = off[i / 3][i % 3];
      asm volatile("" : "+v"(o[i / 3][i % 3]));
    }
    static_for<A, B>([&](auto ac) {
      constexpr int a = decltype(ac)::value;
      constexpr int cx = P::cx(a), cz = P::cz(a);
      bool back = false;
      if constexpr (cz != 0) back = z == (cz > 0 ? 0 : g.nz - 1);
      if constexpr (cx != 0) back = back || x == (cx > 0 ? 0 : g.nx - 1);
      const uint32_t there = o[P::cy(a) + 1][cx + 1] + (cz > 0 ? s.to_m : (cz < 0 ? s.to_p : s.to_z)) +
                             (uint32_t)(a * kSeg);
      const uint32_t here = o[1][1] + s.to_z + (uint32_t)(P::opposite(a) * kSeg);
      load(ac, s.all, back ? here : there, 0);
    });
  }
}

template <int MODEL, typename T, bool LES, int KIND, int TY, bool NT>
__global__ __launch_bounds__(64 * (TY + 3), tile_waves<T>()) void k_step2(const T* __restrict__ src,
                                                                          T* __restrict__ dst, Grid g,
                                                                          Phys<T> p, TwoStep ts) {
  using LF = typename ModelT<MODEL>::LF;
  using LS = typename ModelT<MODEL>::LS;
  using P = Pops<LF, LS>;
  constexpr int QT = P::Q;
  static_assert(2 * (TY + 2) <= 64, "the ring's columns share one wave");
  __shared__ T lds[P::kSlots * TY * kPitch];
  const int lane = (int)threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const Tile tile = tile_of(g, ts, TY, (int)blockIdx.x);
  const Lane l = lane_of(g, tile, TY, w, lane);
  const bool wave_at_wall =
      __builtin_amdgcn_ballot_w64(l.active && (l.x == 0 || l.x == g.nx - 1)) != 0;
  const bool row = w < TY + 2, own = (unsigned)(w - 1) < (unsigned)tile.rows;
  const bool second = w < tile.rows;
  const int x2 = tile.xb * kXB + lane;  // the second step's node, row w of the tile
  const int64_t plane = (int64_t)g.ny * g.nxb * (QT * kXB);
  const uint32_t bytes = (uint32_t)(plane * (int64_t)sizeof(T));
  uint32_t off[3][3];
  plane_offsets<QT, T>(g, l.x, l.y, off);
  const uint32_t out = (uint32_t)(((int64_t)(tile.y0 + w) * g.nxb + tile.xb) * (QT * kXB) + lane) *
                       (uint32_t)sizeof(T);
  // LDS places of the lane for the first step's pushes and the second step's
  // reads; the resting class's as well, which lies beyond the reach of an
  // instruction's constant offset (hidden so that no sums are kept instead)
  int at = lds_lane(l, lane), at2 = w * kPitch + 1 + lane;
  int rest = at + class_base<P, TY>(0, 0), rest2 = at2 + class_base<P, TY>(0, 0);
  asm("" : "+v"(at), "+v"(at2), "+v"(rest), "+v"(rest2));
  T fin[LF::Q], pin[LS::Q];  // pulled populations of the next plane
  T fg[LF::Q], ph[LS::Q];    // the first step's results
  // populations from .. to - 1 of plane k + 1 (the last plane again past the end)
  auto pull = [&](int k, auto from, auto to) __attribute__((always_inline)) {
    const int z = k + 1 < g.nz ? k + 1 : g.nz - 1;
    const Planes s = planes_at(src, g, plane, bytes, z);
    pull_plane<P, decltype(from)::value, decltype(to)::value, T>(
        s, g, z, l.x, wave_at_wall || z == 0 || z == g.nz - 1, off, fin, pin);
  };
  using I0 = std::integral_constant<int, 0>;
  using IQ = std::integral_constant<int, QT>;
  constexpr int kAhead = pulled_ahead<MODEL>();
  using IE = std::integral_constant<int, kAhead>;
  auto put = [&](auto ac, int i) __attribute__((always_inline)) {
    constexpr int a = decltype(ac)::value;
    if constexpr (P::flow(a))
      lds[i] = fg[a];
    else
      lds[i] = ph[a - LF::Q];
  };
  // First step of plane k, up to its downward pushes, and then the pulls of the
  // plane after it, which fly over the barriers and the second step. Every wave
  // makes it, also where its values are not wanted (rows past a ragged tile,
  // the plane past the last): a branch here would make the pulled values'
  // arrival uncertain to the compiler, which then waits for the stores behind
  // them too.
  bool push;
  auto first_step = [&](int k) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LF::Q; ++q) fg[q] = fin[q];
#pragma unroll
    for (int q = 0; q < LS::Q; ++q) ph[q] = pin[q];
    collide_node<MODEL, LES, KIND, true>(fg, ph, p);
    // all of it before the barriers: none is left over for after them
    keep(fg);
    keep(ph);
    if (kAhead == QT) pull(k, I0{}, IQ{});
    push = l.active && k < g.nz;
    if (push) push_class<P, TY, -1>(l, row, w - 1, tile.rows, at, at, put);
  };
  const int ks = tile.z0 > 0 ? tile.z0 - 1 : 0;
  pull(ks - 1, I0{}, IQ{});
  first_step(ks);
  for (int k = ks;; ++k) {
    const bool two = second && k > tile.z0;  // second step of plane k - 1
    lds_barrier();
    T f2[LF::Q], p2[LS::Q];
    if (two) {
      int up2 = at2 + class_base<P, TY>(1, k - 1);
      asm("" : "+v"(up2));
      static_for<0, QT>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        const int i = (P::cz(a) < 0 ? at2 : (P::cz(a) > 0 ? up2 : rest2)) + class_offset<P, TY>(a, 0, 0);
        if constexpr (P::flow(a))
          f2[a] = lds[i];
        else
          p2[a - LF::Q] = lds[i];
      });
    }
    lds_barrier();
    if (push) {
      int up = at + class_base<P, TY>(1, k + 1);
      asm("" : "+v"(up));
      push_class<P, TY, 0>(l, row, w - 1, tile.rows, rest, at, put);
      push_class<P, TY, 1>(l, row, w - 1, tile.rows, up, at, put);
      if ((wave_at_wall || k == 0 || k == g.nz - 1) && row && own)
        push_bounce<P, TY>(g, l, {at, rest, at + class_base<P, TY>(1, k)}, k, put);
    }
    if (kAhead < QT) pull(k, I0{}, IE{});
    const Rsrc rd = plane_rsrc(dst + (two ? k - 1 : tile.z0) * plane, bytes);
    auto store = [&](uint32_t to) __attribute__((always_inline)) {
      static_for<0, QT>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        constexpr int seg = a * kXB * (int)sizeof(T);
        if constexpr (P::flow(a))
          store_at<NT>(rd, to, seg, f2[a]);
        else
          store_at<NT>(rd, to, seg, p2[a - LF::Q]);
      });
    };
    // Stores by every wave, those of lanes without a second-step node out of
    // bounds and so dropped: the loads in flight are then followed by a known
    // number of stores, and waiting for the loads need not wait for these.
    if (two) {
      collide_node<MODEL, LES, KIND, true>(f2, p2, p);
      store(x2 < g.nx ? out : kDropped);
    } else {
      store(kDropped);
    }
    if (k == tile.z1) break;
    if (kAhead < QT) pull(k, IE{}, IQ{});
    first_step(k + 1);
  }
}

// Steps of a grid that takes them two at a time: pairs, and the single steps of
// an odd count. Included by translation units of their own with `#pragma clang fp
// contract(on)` before the includes: multiply-adds are contracted within an
// expression only, not where the optimiser happens to see one, which differs
// between kernels. The two then round alike, and a run gives the same bits
// however it is split into calls.
template <int M, typename T>
static hipError_t launch_paired_of(lbm_handle* h, const void* src, void* dst, hipStream_t stream) {
  const Grid g = grid_of(h);
  if (h->per_launch == 1) return launch_step_of<M, T, T, T, false, true>(h, src, dst, nullptr, stream);
  return with_collision<M>(h, [&](auto les, auto kind) {
    constexpr int TY = two_step_rows(sizeof(T));
    TwoStep ts;
    two_step_plan(g, TY, h->cu_count, ts);
    auto launch = [&](auto nt) {
      hipLaunchKernelGGL((k_step2<M, T, decltype(les)::value, decltype(kind)::value, TY, decltype(nt)::value>),
                         dim3(ts.nblocks), dim3(64 * (TY + 3)), 0, stream, static_cast<const T*>(src),
                         static_cast<T*>(dst), g, phys_of<T>(h), ts);
    };
    if (stores_past_caches(h->state_bytes))
      launch(std::true_type{});
    else
      launch(std::false_type{});
    return hipGetLastError();
  });
}

}  // namespace lbm
