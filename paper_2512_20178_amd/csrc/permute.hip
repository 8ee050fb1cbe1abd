// Values between the CSR's order and the transposed pattern's.
//
// perm[j] is the CSR position of transposed entry j.  Through perm every value
// is one 4-byte access at random: 1.63 ms in and 2.15 ms out for the 97.6M
// nonzeros of the 2^21 GCN matrix, because each moves a whole line across the
// fabric.  Large patterns go through a staged order instead: the transposed
// entries are cut into windows of 2^18 (1 MB of values), and the staged order
// is window by window, CSR order inside a window.  Between CSR and staged
// order a workgroup's run of consecutive CSR positions touches one short run
// per window; between staged and transposed order everything happens inside
// one window, which the workgroups of one XCD handle together, so its lines
// are in that XCD's L2 from the first touch to the last.  Measured (2^21 GCN
// matrix): in 1.63 -> 0.67 + 0.63 ms, out 2.15 -> 0.69 + 0.54 ms; 31M nonzeros
// (2^20 R-MAT) 0.40 -> 0.36 and 0.58 -> 0.35 ms.  Each pass moves 12 bytes per
// value and is bound by the L2's rate of 4-byte requests (155 G/s), no longer
// by the fabric.
#include <algorithm>

#include "plan.hpp"

namespace shiro {

namespace {

constexpr int kWinShift = 18;            // entries per window: 2^18
constexpr int kPart = 4096;              // entries per workgroup inside a window
constexpr int kParts = (1 << kWinShift) / kPart;
constexpr int kRun = 16384;              // CSR positions per workgroup
constexpr int kFlight = 8;               // values in flight per thread

// Patterns from here on use the staged order.  Below about 4M nonzeros the value
// array and perm are mostly in the MALL and one pass is faster; from 8M on two
// are, and the order costs its set-up once.  Direct / staged, backward with value
// gradients at N = 128 in us, and what the set-up adds to prepare in ms:
//    3.9M (2^18 R-MAT)   330 / 351,      0.2
//    8.4M (2^19 ER)     1053 / 951,      0.4   paid back after 5 backwards
//   10.2M (2^20 R-MAT)  1111 / 1056,     0.4                   8
//   12.6M (2^19 ER)     1523 / 1389,     0.6                   5
//   16.8M (2^20 ER)     2108 / 1915,     0.8                   5
//   20.0M (2^20 R-MAT)  1962 / 1917,     0.8                  19
//   31.4M (2^20 R-MAT)  3221 / 2903,     1.4                   5
//   97.6M (2^21 GCN)   11804 / 10577,    6.0                   5
// The line lies above the crossing, so that patterns of a few million nonzeros,
// which a program may make often (a rank's panel), do not pay the set-up.
constexpr int64_t kStagedMin = (int64_t)12 << 20;

__global__ __launch_bounds__(kBlock) void k_gather_vals(const int32_t* __restrict__ perm,
                                                        const float* __restrict__ vals, int64_t n,
                                                        float* __restrict__ out) {
  for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock)
    out[j] = vals[perm[j]];
}

// One value per thread: with four per thread (16-byte index loads) the
// scattered stores ran slower on the MI355X (55 against 44 us for 4.2M
// values), as did a gather through the inverse permutation.
__global__ __launch_bounds__(kBlock) void k_scatter_vals(const int32_t* __restrict__ perm,
                                                         const float* __restrict__ in, int sets, int64_t n,
                                                         float* __restrict__ out) {
  for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock) {
    float s = in[j];
    for (int t = 1; t < sets; ++t) s += in[j + t * n];
    out[perm ? (int64_t)perm[j] : j] = s;
  }
}

// [begin, end) of this workgroup inside the windows: workgroups that the
// dispatcher places on one XCD (round robin over 8) share a window.
__device__ __forceinline__ void window_part(int64_t n, int64_t* begin, int64_t* end) {
  const int64_t b = blockIdx.x, r = b >> 3;
  const int64_t win = (r / kParts) * 8 + (b & 7);
  *begin = (win << kWinShift) + (r % kParts) * kPart;
  *end = *begin + kPart < n ? *begin + kPart : n;
}

// Staged -> transposed, or (GATHER) transposed -> staged with the sets summed.
template <bool GATHER>
__global__ __launch_bounds__(kBlock) void k_stage_window(const int32_t* __restrict__ entry,
                                                         const float* __restrict__ in, int sets, int64_t n,
                                                         float* __restrict__ out) {
  int64_t b, e;
  window_part(n, &b, &e);
  for (int64_t q0 = b + threadIdx.x; q0 < e; q0 += kBlock * kFlight) {
    int32_t j[kFlight];
    float v[kFlight];
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t q = q0 + u * kBlock;
      j[u] = __builtin_nontemporal_load(entry + (q < e ? q : e - 1));
    }
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t q = q0 + u * kBlock;
      v[u] = GATHER ? in[j[u]] : __builtin_nontemporal_load(in + (q < e ? q : e - 1));
    }
    for (int t = 1; GATHER && t < sets; ++t)
#pragma unroll
      for (int u = 0; u < kFlight; ++u) v[u] += in[j[u] + t * n];
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t q = q0 + u * kBlock;
      if (q < e) out[GATHER ? q : (int64_t)j[u]] = v[u];
    }
  }
}

// CSR -> staged, or (GATHER) staged -> CSR.
template <bool GATHER>
__global__ __launch_bounds__(kBlock) void k_stage_runs(const int32_t* __restrict__ place,
                                                       const float* __restrict__ in, int64_t n,
                                                       float* __restrict__ out) {
  const int64_t b = (int64_t)blockIdx.x * kRun;
  const int64_t e = b + kRun < n ? b + kRun : n;
  for (int64_t k0 = b + threadIdx.x; k0 < e; k0 += kBlock * kFlight) {
    int32_t q[kFlight];
    float v[kFlight];
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t k = k0 + u * kBlock;
      q[u] = __builtin_nontemporal_load(place + (k < e ? k : e - 1));
    }
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t k = k0 + u * kBlock;
      v[u] = GATHER ? in[q[u]] : __builtin_nontemporal_load(in + (k < e ? k : e - 1));
    }
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      const int64_t k = k0 + u * kBlock;
      if (k < e) out[GATHER ? k : (int64_t)q[u]] = v[u];
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_invert(const int32_t* __restrict__ perm, int64_t n,
                                                   uint32_t* __restrict__ inv) {
  for (int64_t j = blockIdx.x * (int64_t)kBlock + threadIdx.x; j < n; j += (int64_t)gridDim.x * kBlock)
    inv[perm[j]] = (uint32_t)j;
}

__global__ __launch_bounds__(kBlock) void k_places(const int32_t* __restrict__ entry, const int32_t* __restrict__ perm,
                                                   int64_t n, int32_t* __restrict__ place) {
  for (int64_t q = blockIdx.x * (int64_t)kBlock + threadIdx.x; q < n; q += (int64_t)gridDim.x * kBlock)
    place[perm[entry[q]]] = (int32_t)q;
}

unsigned grid_for(int64_t n, int64_t cap = 65536) { return (unsigned)std::min<int64_t>(ceil_div(std::max<int64_t>(n, 1), kBlock), cap); }
unsigned window_blocks(int64_t n) {
  const int64_t wins = ceil_div(n, (int64_t)1 << kWinShift);
  return (unsigned)(ceil_div(wins, 8) * 8 * kParts);
}

}  // namespace

bool staged_values(shiro_plan plan) { return plan->nnz >= kStagedMin && !plan->vmap; }

// After plan->tr.perm: the staged order of large whole-panel patterns (subset
// plans read the caller's array through a map that skips positions).  One
// array more than the direct permutation needs: the inverse permutation and,
// after the sort, the places live in the scratch that the transposed pattern's
// own sort has just used, and the places end in perm's memory.
int build_value_permutation(shiro_plan plan, hipStream_t s) {
  Transposed& tr = plan->tr;
  const int64_t n = plan->nnz;
  if (!staged_values(plan)) return SHIRO_OK;
  SHIRO_TRY(ensure_scratch(plan, sort_scratch_bytes(n)));
  // without memory for it the direct permutation stays
  const int rc = dev_alloc_n(&tr.entry_of_stage, n);
  if (rc == SHIRO_ERR_OOM) return SHIRO_OK;
  SHIRO_TRY(rc);
  uint32_t* inv = reinterpret_cast<uint32_t*>(plan->scratch);  // the sort's first n words, which it only reads
  k_invert<<<grid_for(n), kBlock, 0, s>>>(tr.perm, n, inv);
  SHIRO_LAUNCH_CHECK();
  int bits = 0;
  while (((int64_t)1 << bits) < ceil_div(n, (int64_t)1 << kWinShift)) ++bits;
  SHIRO_TRY(radix_sort_keys(inv, reinterpret_cast<uint32_t*>(tr.entry_of_stage), n, kWinShift, bits, plan->scratch, s));
  int32_t* place = reinterpret_cast<int32_t*>(inv);
  k_places<<<grid_for(n), kBlock, 0, s>>>(tr.entry_of_stage, tr.perm, n, place);
  SHIRO_LAUNCH_CHECK();
  SHIRO_HIP(hipMemcpyAsync(tr.perm, place, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
  SHIRO_HIP(hipStreamSynchronize(s));
  tr.stage_of_csr = tr.perm;
  tr.perm = nullptr;
  return SHIRO_OK;
}

int gather_values(const int32_t* map, const float* vals, int64_t n, float* out, hipStream_t s) {
  if (n <= 0) return SHIRO_OK;
  k_gather_vals<<<grid_for(n), kBlock, 0, s>>>(map, vals, n, out);
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

int scatter_values(const int32_t* map, const float* in, int sets, int64_t n, float* out, hipStream_t s) {
  if (n <= 0) return SHIRO_OK;
  k_scatter_vals<<<grid_for(n), kBlock, 0, s>>>(map, in, sets, n, out);
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

int values_to_transposed(shiro_plan plan, const float* vals, float* tvals, float* stage, hipStream_t s) {
  const Transposed& tr = plan->tr;
  const int64_t n = plan->nnz;
  if (!tr.stage_of_csr) return gather_values(tr.perm, vals, n, tvals, s);
  k_stage_runs<false><<<(unsigned)ceil_div(n, kRun), kBlock, 0, s>>>(tr.stage_of_csr, vals, n, stage);
  SHIRO_LAUNCH_CHECK();
  k_stage_window<false><<<window_blocks(n), kBlock, 0, s>>>(tr.entry_of_stage, stage, 1, n, tvals);
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

int values_from_transposed(shiro_plan plan, const float* tvals, int sets, float* vals, float* stage, hipStream_t s) {
  const Transposed& tr = plan->tr;
  const int64_t n = plan->nnz;
  if (!tr.stage_of_csr) return scatter_values(tr.perm, tvals, sets, n, vals, s);
  k_stage_window<true><<<window_blocks(n), kBlock, 0, s>>>(tr.entry_of_stage, tvals, sets, n, stage);
  SHIRO_LAUNCH_CHECK();
  k_stage_runs<true><<<(unsigned)ceil_div(n, kRun), kBlock, 0, s>>>(tr.stage_of_csr, stage, n, vals);
  SHIRO_LAUNCH_CHECK();
  return SHIRO_OK;
}

}  // namespace shiro
