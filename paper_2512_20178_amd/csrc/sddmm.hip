// The row kernel of the sampled product: a wavefront per row, its lane groups
// on the row's nonzeros, UNROLL deep, LANES lanes of 16 bytes on each gathered
// row; the first column tile of the dY row stays in registers.  What bounds it
// are the gathers.  It takes every width and stride and needs no buffer; where
// it is the default and where the nonzero walk is: default_tuning.
#include "spmm_args.hpp"

namespace shiro {

namespace {

template <typename TIN, int LANES, int VEC, int UNROLL>
__global__ __launch_bounds__(kBlock) void k_sddmm(
    const int64_t* __restrict__ ptr, const int32_t* __restrict__ idx, const TIN* __restrict__ dY,
    int64_t lddy, const TIN* __restrict__ Bp, int64_t ldp, float* __restrict__ dvals,
    const int32_t* __restrict__ out_map, const int32_t* __restrict__ chunk_row,
    const int32_t* __restrict__ chunk_nz, int32_t W, int32_t R, int32_t N, int32_t cpw, int32_t xcd_remap) {
  constexpr int G = kWave / LANES;
  constexpr int TW = LANES * VEC;
  constexpr int STEP = G * UNROLL;
  const int lane = lane_id();
  const int g = lane / LANES;
  const int li = lane % LANES;
  const int ntiles = (N + TW - 1) / TW;
  const int64_t c0 = (int64_t)li * VEC;

  const int32_t gw = uniform(logical_block(xcd_remap) * kWavesPerBlock + wave_id());
  const int32_t w_begin = gw * cpw;
  const int32_t w_end = min(w_begin + cpw, W);

  for (int32_t w = w_begin; w < w_end; ++w) {
    const int32_t i0 = chunk_row[w], i1 = chunk_row[w + 1];
    const int64_t j0 = chunk_nz[w], j1 = chunk_nz[w + 1];
    int64_t rs = i0 < R ? ptr[i0] : 0;
    for (int32_t r = i0; r <= i1 && r < R; ++r) {
      const int64_t re = ptr[r + 1];
      const int64_t kb = rs > j0 ? rs : j0;
      const int64_t ke = re < j1 ? re : j1;
      rs = re;
      if (kb >= ke) continue;
      // first column tile of dY row r stays in registers for the whole row
      float y0[VEC];
      Elem<TIN>::template load<VEC>(dY + (int64_t)r * lddy + (c0 < N ? c0 : 0), y0);
      if (c0 >= N) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) y0[e] = 0.f;
      }
      for (int64_t k = kb; k < ke; k += STEP) {
        int32_t xi[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
          const int64_t kk = k + u * G + g;
          xi[u] = idx[kk < ke ? kk : ke - 1];
        }
        float part[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
          float b[VEC];
          Elem<TIN>::template load<VEC>(Bp + (int64_t)xi[u] * ldp + (c0 < N ? c0 : 0), b);
          part[u] = 0.f;
#pragma unroll
          for (int e = 0; e < VEC; ++e) part[u] = fmaf(y0[e], b[e], part[u]);
        }
        for (int t = 1; t < ntiles; ++t) {
          const int64_t ct = (int64_t)t * TW + c0;
          const bool cv = ct < N;
          float y[VEC];
          Elem<TIN>::template load<VEC>(dY + (int64_t)r * lddy + (cv ? ct : 0), y);
#pragma unroll
          for (int u = 0; u < UNROLL; ++u) {
            float b[VEC];
            Elem<TIN>::template load<VEC>(Bp + (int64_t)xi[u] * ldp + (cv ? ct : 0), b);
            float q = 0.f;
#pragma unroll
            for (int e = 0; e < VEC; ++e) q = fmaf(y[e], b[e], q);
            part[u] += cv ? q : 0.f;
          }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
          part[u] = group_sum<LANES>(part[u]);
          const int64_t kk = k + u * G + g;
          if (li == LANES - 1 && kk < ke) dvals[out_map ? (int64_t)out_map[kk] : kk] = part[u];
        }
      }
    }
  }
}

template <typename TIN, int VEC>
int go(const SddmmArgs& a, int lanes, int unroll, dim3 grid, hipStream_t s) {
#define SHIRO_SDDMM_CASE(L, U)                                                                                   \
  if (lanes == L && unroll == U) {                                                                               \
    k_sddmm<TIN, L, VEC, U><<<grid, kBlock, 0, s>>>(                                                             \
        a.ptr, a.idx, reinterpret_cast<const TIN*>(a.dY), a.lddy, reinterpret_cast<const TIN*>(a.Bp), a.ldp,     \
        a.dvals, a.out_map, a.chunk_row, a.chunk_nz, a.W, a.R, a.N, a.chunks_per_wave, a.xcd_remap);             \
    SHIRO_LAUNCH_CHECK();                                                                                        \
    return SHIRO_OK;                                                                                             \
  }
  SHIRO_SDDMM_CASE(8, 1) SHIRO_SDDMM_CASE(8, 2) SHIRO_SDDMM_CASE(8, 4)
  SHIRO_SDDMM_CASE(16, 1) SHIRO_SDDMM_CASE(16, 2) SHIRO_SDDMM_CASE(16, 4)
  SHIRO_SDDMM_CASE(32, 1) SHIRO_SDDMM_CASE(32, 2) SHIRO_SDDMM_CASE(32, 4)
  SHIRO_SDDMM_CASE(64, 1) SHIRO_SDDMM_CASE(64, 2) SHIRO_SDDMM_CASE(64, 4)
#undef SHIRO_SDDMM_CASE
  return set_error(SHIRO_ERR_UNSUPPORTED, "sddmm: no kernel for lanes/unroll");
}

}  // namespace

int launch_sddmm_rows(const SddmmArgs& a, shiro_dtype dt, int vec, int lanes, int unroll, dim3 grid, hipStream_t s) {
  if (dt == SHIRO_F32) return vec == 4 ? go<float, 4>(a, lanes, unroll, grid, s) : go<float, 1>(a, lanes, unroll, grid, s);
  return vec == 8 ? go<bf16_t, 8>(a, lanes, unroll, grid, s) : go<bf16_t, 1>(a, lanes, unroll, grid, s);
}

}  // namespace shiro
