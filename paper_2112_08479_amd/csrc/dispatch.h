// What the forward kernels' translation units share: the models' lattices, the
// local collision by model and kind, kernel parameters from a handle and the
// dispatch over storage modes and models.
#pragma once

#include <math.h>

#include <type_traits>

#include "collide.h"
#include "lattice.h"
#include "runtime.h"

namespace lbm {

template <int MODEL>
struct ModelT;
template <>
struct ModelT<0> {
  using LF = Q27;
  using LS = Q7;
};
template <>
struct ModelT<1> {
  using LF = Q19;
  using LS = Q6;
};
template <>
struct ModelT<2> {
  using LF = Q27;
  using LS = Q27;
};

// collision kinds of the cumulant models: omega3..omega6 = 1, given rates,
// parametrised
enum { kCumFast = 0, kCumGeneral = 1, kCumParam = 2 };

// LEAN: the lean forms (cumulant models)
template <int MODEL, bool LES, int KIND, bool LEAN, typename CT>
LBM_HD void collide_node(CT* fg, CT* ph, const Phys<CT>& p) {
  using LS = typename ModelT<MODEL>::LS;
  if constexpr (MODEL == 1)
    collide_bgk_q19_q6<LES, CT>(fg, ph, p);
  else if constexpr (KIND == kCumParam)
    collide_cumulant27_param<LS, LEAN>(fg, ph, p);
  else if constexpr (KIND == kCumGeneral)
    collide_cumulant27_general<LS, LES, LEAN>(fg, ph, p);
  else
    collide_cumulant27<LS, LES, LEAN>(fg, ph, p);
}

template <typename T>
LBM_HD double to_d(T v);
template <>
LBM_HD double to_d<double>(double v) { return v; }
template <>
LBM_HD double to_d<float>(float v) { return (double)v; }

// Post-collision values are not read again before the next launch, so they
// may bypass the caches on the way to HBM (NT; see stores_past_caches).
template <bool NT = true, typename ST>
__device__ __forceinline__ void store_val(ST* p, ST v) {
  if constexpr (!NT) {
    *p = v;
  } else if constexpr (std::is_same<ST, double>::value || std::is_same<ST, float>::value) {
    __builtin_nontemporal_store(v, p);
  } else {
    uint16_t bits;
    __builtin_memcpy(&bits, &v, 2);
    __builtin_nontemporal_store(bits, reinterpret_cast<uint16_t*>(p));
  }
}

static inline Grid grid_of(const lbm_handle* h) {
  return Grid{h->cfg.nx, h->cfg.ny, h->cfg.nz, h->n, xblocks(h->cfg.nx)};
}

static inline int block_x(const lbm_handle* h) {
  const int nx = h->cfg.nx;
  return nx >= kBlock ? kBlock : ((nx + 63) / 64) * 64;
}

template <typename CT>
static inline Phys<CT> phys_of(const lbm_handle* h) {
  const lbm_params& p = h->prm;
  const lbm_config& c = h->cfg;
  Phys<CT> r;
  r.g = (CT)p.g_prime;
  r.tau0 = (CT)p.tau0;
  r.tau_phi0 = (CT)p.tau_phi0;
  // 18 sqrt(2) C_s^2 (standard closure) or 18 sqrt(2) C_s (as printed in Eq. 32)
  r.c_les = (CT)(18.0 * sqrt(2.0) * (c.smag_paper_form ? c.cs_smag : c.cs_smag * c.cs_smag));
  r.d0 = (CT)p.d0;
  r.inv_sct = (CT)(1.0 / c.sc_t);
  r.inv_cs2phi = (CT)(1.0 / p.cs2_phi);
  r.omega2 = (CT)c.omega_bulk;
  r.omega3 = (CT)c.omega3;
  r.omega4 = (CT)c.omega4;
  r.omega5 = (CT)c.omega5;
  r.omega6 = (CT)c.omega6;
  const double h4 = p.tau0 - 0.5;  // 1/omega1 - 1/2
  r.w_plus = (CT)p.w_plus;
  r.w_minus = (CT)p.w_minus;
  r.w_111 = (CT)p.w_111;
  r.a4 = (CT)(-2.0 / 3.0 * h4 * p.coef_a);
  r.b4 = (CT)(-1.0 / 3.0 * h4 * p.coef_b);
  r.lam = c.limiter > 0.0 ? (CT)c.limiter : (CT)INFINITY;
  return r;
}

// calls f(ST{}, SS{}, CT{}) for the handle's storage mode: flow element
// type, scalar element type, arithmetic type
template <class F>
static hipError_t with_storage(const lbm_handle* h, F&& f) {
  switch (h->cfg.storage) {
    case LBM_F64: return f(double{}, double{}, double{});
    case LBM_F32: return f(float{}, float{}, float{});
    case LBM_F16: return f(__half{}, __half{}, float{});
    case LBM_BF16: return f(bf16_t{}, bf16_t{}, float{});
    case LBM_BF16_F16S: return f(bf16_t{}, __half{}, float{});
  }
  return hipErrorInvalidValue;
}
template <class F>
static hipError_t with_model(const lbm_handle* h, F&& f) {
  switch (h->cfg.model) {
    case LBM_CUMULANT27_Q7: return f(std::integral_constant<int, 0>{});
    case LBM_BGK19_SMAG_Q6: return f(std::integral_constant<int, 1>{});
    case LBM_CUMULANT27_FCM27: return f(std::integral_constant<int, 2>{});
  }
  return hipErrorInvalidValue;
}

static inline int cumulant_kind(const lbm_handle* h) {
  const lbm_config& c = h->cfg;
  if (c.parametrized) return kCumParam;
  return (c.omega3 != 1.0 || c.omega4 != 1.0 || c.omega5 != 1.0 || c.omega6 != 1.0) ? kCumGeneral
                                                                                   : kCumFast;
}

// calls f(LES, KIND) with integral constants for the handle's collision: one
// kind for the BGK model; the parametrised kind never has the LES (rejected
// when the handle is made)
template <int MODEL, class F>
static hipError_t with_collision(const lbm_handle* h, F&& f) {
  const bool les = h->cfg.cs_smag > 0.0;
  using T = std::true_type;
  using N = std::false_type;
  using Fast = std::integral_constant<int, kCumFast>;
  if constexpr (MODEL == 1) {
    return les ? f(T{}, Fast{}) : f(N{}, Fast{});
  } else {
    using General = std::integral_constant<int, kCumGeneral>;
    const int kind = cumulant_kind(h);
    if (kind == kCumParam) return f(N{}, std::integral_constant<int, kCumParam>{});
    if (kind == kCumGeneral) return les ? f(T{}, General{}) : f(N{}, General{});
    return les ? f(T{}, Fast{}) : f(N{}, Fast{});
  }
}

}  // namespace lbm
