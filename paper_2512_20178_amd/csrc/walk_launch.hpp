// Choice of a walk instance from a launch's arguments (one source file per
// pair of element types instantiates it).
#pragma once

#include "walk.hpp"

namespace shiro {

template <typename TIN, typename TOUT, int VEC, bool DOT, int SCAT, bool EDGE>
int walk_go(const SpmmArgs& a, dim3 grid, hipStream_t s) {
  if constexpr (VEC * (int)sizeof(TIN) >= 4) {
    if (walk_narrow(a, sizeof(TIN), VEC)) {
      if constexpr (EDGE && SCAT >= 0 && std::is_same<TIN, TOUT>::value) {
        if (a.vperm) {
          k_walk<TIN, TOUT, VEC, DOT, SCAT, EDGE, false, true><<<grid, kBlock, 0, s>>>(SHIRO_SPMM_ARGS(TIN, TOUT, a));
          SHIRO_LAUNCH_CHECK();
          return SHIRO_OK;
        }
      }
      k_walk<TIN, TOUT, VEC, DOT, SCAT, EDGE, false, false><<<grid, kBlock, 0, s>>>(SHIRO_SPMM_ARGS(TIN, TOUT, a));
      SHIRO_LAUNCH_CHECK();
      return SHIRO_OK;
    }
  }
  k_walk<TIN, TOUT, VEC, DOT, SCAT, EDGE, true, false><<<grid, kBlock, 0, s>>>(SHIRO_SPMM_ARGS(TIN, TOUT, a));
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

// The dots sum over lanes, so whole tiles are worth an instance of their own;
// without dots idle lanes cost one exec mask per stored row.
template <typename TIN, typename TOUT, int VEC, int SCAT>
int walk_dot(const SpmmArgs& a, dim3 grid, hipStream_t s) {
  if (a.N % (kWave * VEC) == 0 && !a.vperm) return walk_go<TIN, TOUT, VEC, true, SCAT, false>(a, grid, s);
  return walk_go<TIN, TOUT, VEC, true, SCAT, true>(a, grid, s);
}

// The transposed product (dots, overwritten scatter rows) has one type for
// all its dense operands; only the sums into other rows' types mix them.
// Dots without carry slots: the sampled product.
template <typename TIN, typename TOUT, int VEC>
int walk_form(const SpmmArgs& a, dim3 grid, hipStream_t s) {
  if (a.vperm && !walk_narrow(a, sizeof(TIN), VEC))
    return set_error(SHIRO_ERR_UNSUPPORTED, "walk: values through a permutation need 32-bit row offsets");
  if (a.N < VEC) return set_error(SHIRO_ERR_UNSUPPORTED, "walk: more columns per lane than the matrix has");
  const int scat = a.scat ? a.scat_mode : 0;
  if constexpr (std::is_same<TIN, TOUT>::value) {
    if (a.dot_out) {
      if (!a.carry) return walk_dot<TIN, TOUT, VEC, -1>(a, grid, s);
      if (scat == 2) return walk_dot<TIN, TOUT, VEC, 2>(a, grid, s);
      if (scat == 1) return walk_dot<TIN, TOUT, VEC, 1>(a, grid, s);
      return walk_dot<TIN, TOUT, VEC, 0>(a, grid, s);
    }
    if (scat == 2) return walk_go<TIN, TOUT, VEC, false, 2, true>(a, grid, s);
  } else if (a.dot_out || scat == 2) {
    return set_error(SHIRO_ERR_UNSUPPORTED, "walk: one dtype for all operands of the transposed product");
  }
  if (scat == 1) return walk_go<TIN, TOUT, VEC, false, 1, true>(a, grid, s);
  return walk_go<TIN, TOUT, VEC, false, 0, true>(a, grid, s);
}

}  // namespace shiro
