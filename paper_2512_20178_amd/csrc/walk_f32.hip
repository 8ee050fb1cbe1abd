// The nonzero walk over float32 rows.
#include "walk_launch.hpp"

namespace shiro {

int launch_walk_f32(const SpmmArgs& a, int vec, dim3 grid, hipStream_t s) {
  if (vec == 1) return walk_form<float, float, 1>(a, grid, s);
  if (vec == 2) return walk_form<float, float, 2>(a, grid, s);
  return set_error(SHIRO_ERR_UNSUPPORTED, "walk: no kernel for this tile width");
}

}  // namespace shiro
