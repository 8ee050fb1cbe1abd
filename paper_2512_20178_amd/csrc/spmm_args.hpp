// Arguments shared by the product kernels, and the fixed parts of their launch.
#pragma once

#include "plan.hpp"

namespace shiro {

// Host-side bundle of the kernel arguments.  The kernels take them as
// separate __restrict__ parameters: that tells the compiler the pattern
// arrays are never written, so wave-uniform reads of them (row pointers,
// chunk bounds) become scalar loads.
struct SpmmArgs {
  const int64_t* ptr;       // R + 1
  const int32_t* idx;       // nnz: row of X to gather
  const float* vals;        // values in pattern order, or (the walk) through vperm
  const int32_t* vperm;     // optional (the walk): where vals and dot_out hold nonzero k
  const void* D;            // optional: dense row per pattern row, dotted with each gathered row
  int64_t ldd;
  float* dot_out;           // nnz: the dots, in pattern order (when D is set)
  int64_t dot_ld;           // between the dots of one column tile and the next (the walk)
  const void* X;            // gathered dense rows
  int64_t x_rows;           // rows of X
  int64_t ldx;
  void* out;                // R x N, may be null (transposed: dBpacked optional)
  int64_t ldo;
  void* scat;               // transposed only: dB, rows scat_idx[r] (see scat_mode)
  int64_t lds;
  int32_t scat_mode;        // 1: add the row into dB, 2: overwrite the dB row
  const int32_t* scat_idx;  // R
  const int32_t* chunk_row;  // W + 1
  const int32_t* chunk_nz;   // W + 1
  const int32_t* rid;       // nnz: row of each nonzero (both walks; without it the row kernel)
  const int32_t* hot_src;   // windowed walk: rows of X kept in LDS (idx = -(slot + 1) reads slot)
  int32_t n_hot;
  float* carry;             // [W][2][N]
  int32_t W, R, N;
  int32_t chunks_per_wave;
  int32_t xcd_remap;
};

#define SHIRO_SPMM_PARAMS(TIN, TOUT)                                                          \
  const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,                           \
      const float *__restrict__ vals, const int32_t *__restrict__ vperm,                      \
      const TIN *__restrict__ D, int64_t ldd,                                                 \
      float *__restrict__ dot_out, int64_t dot_ld,                                            \
      const TIN *__restrict__ X, int64_t ldx, TOUT *__restrict__ out, int64_t ldo,           \
      TOUT *__restrict__ scat, int64_t lds, const int32_t *__restrict__ scat_idx,             \
      const int32_t *__restrict__ chunk_row, const int32_t *__restrict__ chunk_nz,            \
      const int32_t *__restrict__ rid, float *__restrict__ carry, int32_t W, int32_t R,         \
      int32_t N, int32_t cpw, int32_t xcd_remap, int32_t scat_mode,                             \
      const int32_t *__restrict__ hot_src, int32_t n_hot

#define SHIRO_SPMM_ARGS(TIN, TOUT, a)                                                          \
  (a).ptr, (a).idx, (a).vals, (a).vperm, reinterpret_cast<const TIN*>((a).D), (a).ldd, (a).dot_out, (a).dot_ld, \
      reinterpret_cast<const TIN*>((a).X), (a).ldx,                                            \
      reinterpret_cast<TOUT*>((a).out), (a).ldo, reinterpret_cast<TOUT*>((a).scat), (a).lds,   \
      (a).scat_idx, (a).chunk_row, (a).chunk_nz, (a).rid, (a).carry, (a).W, (a).R, (a).N,     \
      (a).chunks_per_wave, (a).xcd_remap, (a).scat_mode, (a).hot_src, (a).n_hot

#define SHIRO_SPMM_NAMES                                                                       \
  ptr, idx, vals, vperm, D, ldd, dot_out, dot_ld, X, ldx, out, ldo, scat, lds, scat_idx, chunk_row, chunk_nz, rid, \
      carry, W, R, N, cpw, xcd_remap, scat_mode, hot_src, n_hot

// Logical workgroup index: with xcd_remap, workgroups that the dispatcher
// places on the same XCD (round robin over 8) get a contiguous index range,
// so each XCD's L2 serves a contiguous range of rows.
__device__ __forceinline__ int32_t logical_block(int32_t remap) {
  const int32_t b = blockIdx.x, g = gridDim.x;
  if (!remap || (g & 7)) return b;
  return (b & 7) * (g >> 3) + (b >> 3);
}

// The walk gathers by 32-bit row offsets of whole dwords: elements of `size`
// bytes, vec of them per lane.
inline bool walk_narrow(const SpmmArgs& a, int64_t size, int vec) {
  const int64_t xb = a.ldx * size;
  return a.x_rows * xb < ((int64_t)1 << 32) && (uintptr_t)a.X % 4 == 0 && xb % 4 == 0 && a.N * size % 4 == 0 &&
         vec * size >= 4;
}

// The row kernel of the sampled product (sddmm.hip): dvals[k] = dY[row(k), :] . Bp[idx[k], :].
struct SddmmArgs {
  const int64_t* ptr;
  const int32_t* idx;
  const void* dY;
  int64_t lddy;
  const void* Bp;
  int64_t ldp;
  float* dvals;
  const int32_t* out_map;  // optional: dvals index of each pattern nonzero (subset plans)
  const int32_t* chunk_row;
  const int32_t* chunk_nz;
  int32_t W, R, N;
  int32_t chunks_per_wave;
  int32_t xcd_remap;
};
int launch_sddmm_rows(const SddmmArgs& a, shiro_dtype dt, int vec, int lanes, int unroll, dim3 grid, hipStream_t s);

// The nonzero walk (walk_*.hip).  The grid covers a.W chunks, a.chunks_per_wave
// consecutive ones per wavefront, and `tiles` column tiles of 64 * vec columns.
int launch_walk_f32(const SpmmArgs& a, int vec, dim3 grid, hipStream_t s);
int launch_walk_bf16(const SpmmArgs& a, int vec, dim3 grid, hipStream_t s);
int launch_walk_bf16_f32(const SpmmArgs& a, int vec, dim3 grid, hipStream_t s);

}  // namespace shiro
