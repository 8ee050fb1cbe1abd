// The nonzero walk over bfloat16 rows.
#include "walk_launch.hpp"

namespace shiro {

int launch_walk_bf16(const SpmmArgs& a, int vec, dim3 grid, hipStream_t s) {
  if (vec == 1) return walk_form<bf16_t, bf16_t, 1>(a, grid, s);
  if (vec == 2) return walk_form<bf16_t, bf16_t, 2>(a, grid, s);
  if (vec == 4) return walk_form<bf16_t, bf16_t, 4>(a, grid, s);
  return set_error(SHIRO_ERR_UNSUPPORTED, "walk: no kernel for this tile width");
}

}  // namespace shiro
