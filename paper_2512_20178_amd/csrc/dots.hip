// Value gradients alone over narrow rows: dvals[k] = dY[row(k), :] . Bp[idx[k], :].
//
// The walk gives a gathered row a whole wavefront, which leaves most lanes idle
// at 64 columns and fewer. Without sums the nonzeros are independent, so here
// L lanes (8 up to 32 columns, 16 up to 64) take one nonzero each step: a
// wavefront takes a window of 64 consecutive nonzeros (one coalesced load of
// their indices and row ids), 64 / L at a time, both dense rows gathered, and
// stores the window's dots together.  No work list: 256 nonzeros a wavefront.
// Four columns a lane, one below 4 columns (a row is then shorter than a lane).
// Bound by its gathers' L2 requests. dvals alone, us, wavefront-per-row kernel /
// walk / this: 2^18 R-MAT (4.9M nonzeros) at N = 32 183 / 109 / 49, at N = 1
// 140 / 84 / 27; 2^18 ER (3.1M) at N = 3 in bfloat16 65 / 96 / 24; ER panel
// (4.2M) at N = 16 in bfloat16 95 / 113 / 89; 2^19 R-MAT (15.5M) at N = 64
// 710 / 342 / 334; from 65 columns on the walk's gathers are full wavefronts.
#include "plan.hpp"
#include "walk.hpp"

namespace shiro {

namespace {

constexpr int kDotWindows = 4;  // windows per wavefront

// VEC columns per lane; the last active lane of a row whose width is no
// multiple of VEC starts at N - VEC and leaves out the columns it shares.
template <typename TIN, int L, int VEC>
__global__ __launch_bounds__(kBlock) void k_dots(const int32_t* __restrict__ idx, const int32_t* __restrict__ rid,
                                                 const TIN* __restrict__ D, int64_t ldd, const TIN* __restrict__ X,
                                                 int64_t ldx, const int32_t* __restrict__ out_map,
                                                 float* __restrict__ out, int64_t nnz, int32_t N) {
  typedef RowVec<TIN, VEC> RI;
  typedef typename RI::V VI;
  constexpr int G = kWave / L;  // nonzeros per step
  const int lane = lane_id();
  const int g = lane / L, li = lane % L;
  const int32_t c0 = li * VEC;
  const bool active = c0 < N;
  const int32_t c = c0 + VEC <= N ? c0 : N - VEC;
  const int32_t dup = c0 - c;
  // the lane whose group sum belongs to this lane's nonzero of a step
  const int from = (lane % G) * L + L - 1;
  const int my_step = lane / G;
  const int64_t w0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave_id()) * kDotWindows;
  for (int64_t w = w0; w < w0 + kDotWindows && w * kWave < nnz; ++w) {
    const int64_t kw = w * kWave;
    const int64_t kk = kw + lane < nnz ? kw + lane : nnz - 1;
    const int32_t wi = idx[kk], wr = rid[kk];
    float mine = 0.f;
#pragma unroll 4
    for (int s = 0; s < kWave / G; ++s) {
      const int src = s * G + g;
      const int32_t xi = __builtin_amdgcn_ds_bpermute(src << 2, wi);
      const int32_t ri = __builtin_amdgcn_ds_bpermute(src << 2, wr);
      const VI xv = *reinterpret_cast<const VI*>(X + (int64_t)xi * ldx + c);
      const VI dv = *reinterpret_cast<const VI*>(D + (int64_t)ri * ldd + c);
      float x[VEC], d[VEC];
      RI::unpack(xv, x);
      RI::unpack(dv, d);
      float q = 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float t = fmaf(d[e], x[e], q);
        q = e >= dup ? t : q;
      }
      q = group_sum<L>(active ? q : 0.f);
      const float t = __int_as_float(__builtin_amdgcn_ds_bpermute(from << 2, __float_as_int(q)));
      mine = s == my_step ? t : mine;
    }
    if (kw + lane < nnz) out[out_map ? (int64_t)out_map[kk] : kk] = mine;
  }
}

template <typename TIN>
int go(const int32_t* idx, const int32_t* rid, const void* D, int64_t ldd, const void* X, int64_t ldx,
       const int32_t* map, float* out, int64_t nnz, int32_t N, hipStream_t s) {
  const int64_t blocks = ceil_div(nnz, (int64_t)kWave * kDotWindows * kWavesPerBlock);
  const TIN *d = reinterpret_cast<const TIN*>(D), *x = reinterpret_cast<const TIN*>(X);
  if (N < 4) k_dots<TIN, 8, 1><<<dim3((unsigned)blocks), kBlock, 0, s>>>(idx, rid, d, ldd, x, ldx, map, out, nnz, N);
  else if (N <= 32) k_dots<TIN, 8, 4><<<dim3((unsigned)blocks), kBlock, 0, s>>>(idx, rid, d, ldd, x, ldx, map, out, nnz, N);
  else k_dots<TIN, 16, 4><<<dim3((unsigned)blocks), kBlock, 0, s>>>(idx, rid, d, ldd, x, ldx, map, out, nnz, N);
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

}  // namespace

bool dots_narrow(int32_t N) { return N >= 1 && N <= 64; }

int launch_dots(const int32_t* idx, const int32_t* rid, const void* D, int64_t ldd, const void* X, int64_t ldx,
                const int32_t* map, float* out, int64_t nnz, int32_t N, shiro_dtype dt, hipStream_t s) {
  if (nnz <= 0) return SHIRO_OK;
  if (!dots_narrow(N)) return set_error(SHIRO_ERR_UNSUPPORTED, "dots: 1 to 64 columns");
  if (dt == SHIRO_F32) return go<float>(idx, rid, D, ldd, X, ldx, map, out, nnz, N, s);
  return go<bf16_t>(idx, rid, D, ldd, X, ldx, map, out, nnz, N, s);
}

}  // namespace shiro
