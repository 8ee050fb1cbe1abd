// The nonzero walk of the product kernels (forward, transposed, row-based):
// one wavefront per chunk, one nonzero per gather, all bookkeeping scalar.
//
// A wavefront walks the nonzeros of its merge-path chunk in pattern order.
// Their indices, values and row ids come in as windows of 64 (one coalesced
// load per stream, a window ahead, lane l holding nonzero l) and go to scalar
// registers one by one with readlane; every gathered row is one load
// instruction of the whole wavefront (lane l holds columns [l VEC, l VEC +
// VEC)), whose address is a scalar row base plus a lane offset that never
// changes.  Where rows end is one bit mask per window (a row id compared with
// its neighbour lane's).
//
// What bounds it: on matrices larger than the caches the rows that miss L2.
// Counted (fetched and written bytes over the kernel's time): forwards 7.0 TB/s
// on the 2^24 R-MAT panel, 6.8 in bfloat16, 7.2 on the 2^21 GCN matrix, which is
// the rate of random rows across the fabric; backwards with dots 5.8 and 5.3
// (they also wait for the rows they dot with), 7.0 on the ER panel at N = 128.  On L2-resident rows (8192 of them, 512 uses
// each) the L2 itself at N >= 128 (16 TB/s of rows) and latency below (11 cycles
// a nonzero and CU from 16 to 64 columns).  Why this split: the walk it
// replaced gave every lane group a chunk of its own, with three vector loads
// of indices per gather, divergent row ends, 118 registers, and one column
// per lane at widths that are no multiple of 16 bytes.  Scalar loads of the
// three streams instead of the windows were tried first: the scalar cache
// fills one 64-byte line in about 36 cycles, 14 to 17 cycles per nonzero and
// CU on L2-resident rows against 11.
//   before -> after, us (MI355X, each call repeated alone; backwards with both
//   value permutations)
//   2^24 R-MAT panel, N = 128  f32 forward 323 -> 306, backward 646 -> 467
//                              bf16 forward 208 -> 172, backward 453 -> 298
//   ER panel, N = 64           f32 forward 281 -> 238, backward 614 -> 557 (the
//                              forward 276 when the pack has just run)
//   2^18 R-MAT, N = 47         f32 forward 331 -> 97, backward 418 -> 208
//   2^21 GCN matrix, N = 128   f32 forward 6.67 -> 5.67 ms, backward 14.6 -> 10.5
//                              (256-byte tiles and the staged value order in it)
// Widths that leave most of its lanes or of its last tile idle run elsewhere
// (default_tuning).
#pragma once

#include <type_traits>

#include "spmm_args.hpp"

namespace shiro {

constexpr int kWalkBatch = 8;  // rows gathered before the first of them is summed

// VEC elements of a dense row at any element alignment, as one access.
template <typename T, int VEC>
struct RowVec;
template <>
struct RowVec<float, 1> {
  typedef float V;
  __device__ __forceinline__ static void unpack(V v, float (&o)[1]) { o[0] = v; }
  __device__ __forceinline__ static V pack(const float (&a)[1]) { return a[0]; }
};
template <>
struct RowVec<float, 2> {
  typedef float V __attribute__((ext_vector_type(2), aligned(4)));
  __device__ __forceinline__ static void unpack(V v, float (&o)[2]) { o[0] = v.x; o[1] = v.y; }
  __device__ __forceinline__ static V pack(const float (&a)[2]) { return V{a[0], a[1]}; }
};
template <>
struct RowVec<float, 4> {
  typedef float V __attribute__((ext_vector_type(4), aligned(4)));
  __device__ __forceinline__ static void unpack(V v, float (&o)[4]) { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
  __device__ __forceinline__ static V pack(const float (&a)[4]) { return V{a[0], a[1], a[2], a[3]}; }
};
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
  return (uint32_t)f32_to_bf16(a) | ((uint32_t)f32_to_bf16(b) << 16);
}
template <>
struct RowVec<bf16_t, 1> {
  typedef bf16_t V;
  __device__ __forceinline__ static void unpack(V v, float (&o)[1]) { o[0] = bf16_to_f32(v); }
  __device__ __forceinline__ static V pack(const float (&a)[1]) { return f32_to_bf16(a[0]); }
};
template <>
struct RowVec<bf16_t, 2> {
  typedef uint32_t V __attribute__((aligned(2)));
  __device__ __forceinline__ static void unpack(V v, float (&o)[2]) { o[0] = bf16_lo(v); o[1] = bf16_hi(v); }
  __device__ __forceinline__ static V pack(const float (&a)[2]) { return bf16_pair(a[0], a[1]); }
};
template <>
struct RowVec<bf16_t, 4> {
  typedef uint32_t V __attribute__((ext_vector_type(2), aligned(2)));
  __device__ __forceinline__ static void unpack(V v, float (&o)[4]) {
    o[0] = bf16_lo(v.x); o[1] = bf16_hi(v.x); o[2] = bf16_lo(v.y); o[3] = bf16_hi(v.y);
  }
  __device__ __forceinline__ static V pack(const float (&a)[4]) { return V{bf16_pair(a[0], a[1]), bf16_pair(a[2], a[3])}; }
};
// Base of row r (wave-uniform), rows ldb bytes apart (below 2^32, checked by
// the launch).  The row offset passes through readfirstlane so that it
// stays two scalar multiplies, whatever address arithmetic it meets.
template <typename T>
__device__ __forceinline__ T* row_base(T* __restrict__ X, int32_t r, uint32_t ldb) {
  const uint64_t off = (uint64_t)uniform64((int64_t)((uint64_t)(uint32_t)r * ldb));
  typedef typename std::conditional<std::is_const<T>::value, const char, char>::type C;
  return reinterpret_cast<T*>(reinterpret_cast<C*>(X) + off);
}

// Sums over the wavefront of eight per-lane values: lane l returns the sum of
// q[l >> 3].  Each step halves the values in flight instead of reducing every
// value by itself: 18 instructions for eight sums instead of 48.
__device__ __forceinline__ float wave_sum8(float (&q)[8], int lane) {
  float a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // lanes 0-31: q[i], lanes 32-63: q[i + 4]
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(q[i]), __float_as_int(q[i + 4]), false, false);
    a[i] = __int_as_float(r[0]) + __int_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // rows of 16 lanes: q[i], q[i + 2], q[i + 4], q[i + 6]
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a[i]), __float_as_int(a[i + 2]), false, false);
    b[i] = __int_as_float(r[0]) + __int_as_float(r[1]);
  }
  const bool hi = lane & 8;
  const float keep = hi ? b[1] : b[0], give = hi ? b[0] : b[1];
  float s = keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0x128, 0xF, 0xF, false));
  s = dpp_add<0x141, 0xF>(s);  // row_half_mirror
  s = dpp_add<0xB1, 0xF>(s);   // quad_perm [1,0,3,2]
  s = dpp_add<0x4E, 0xF>(s);   // quad_perm [2,3,0,1]
  return s;
}

// VEC columns per lane; DOT: also the dot of each gathered row with the
// pattern row's own dense row D (value gradients); SCAT: 0 rows into out,
// 1 also added to scat, 2 also written to scat, -1 no sums at all (the sampled
// product: dots only).
// EDGE: N is no whole number of tiles, so there are idle lanes, and where N is
// no multiple of VEC the last active lane starts at N - VEC and shares columns
// with its neighbour (both compute and store the same sums; its shared columns
// are left out of the dots).  N >= VEC.
// WIDE: the gathered matrix spans 4 GB or more, or its rows are not whole
// dwords; otherwise a gather is a buffer load of a 32-bit row offset, which
// saves five of the instructions that bound the walk of cached rows.
// PERM: nonzero k's value is vals[vperm[k]] and its dot goes to
// dot_out[vperm[k]] (an instance of its own: carried as a runtime case it cost
// the other patterns 4%, 2^18 R-MAT training step 360 -> 375 us).
// A launch with several column tiles leaves one set of dots per tile, dot_ld
// apart.
template <typename TIN, typename TOUT, int VEC, bool DOT, int SCAT, bool EDGE, bool WIDE, bool PERM>
__global__ __launch_bounds__(kBlock) void k_walk(SHIRO_SPMM_PARAMS(TIN, TOUT)) {
  typedef RowVec<TIN, VEC> RI;
  typedef RowVec<TOUT, VEC> RO;
  typedef RowVec<float, VEC> RC;
  typedef typename RI::V VI;
  typedef typename RO::V VO;
  constexpr int UB = kWalkBatch;
  constexpr bool SUM = SCAT >= 0;
  const int lane = lane_id();
  const int32_t c0 = (int32_t)blockIdx.y * (kWave * VEC) + lane * VEC;
  const bool active = !EDGE || c0 < N;
  const int32_t c = !EDGE || c0 + VEC <= N ? c0 : N - VEC;  // idle lanes read the last columns
  const uint32_t cb = (uint32_t)c * sizeof(TIN);
  const uint32_t co = (uint32_t)c * sizeof(TOUT);
  const int32_t dup = EDGE ? c0 - c : 0;  // leading columns shared with the lane below
  const uint32_t xb = (uint32_t)ldx * sizeof(TIN), db = (uint32_t)ldd * sizeof(TIN);
  const uint32_t ob = (uint32_t)ldo * sizeof(TOUT), sb = (uint32_t)lds * sizeof(TOUT);

  auto at = [](auto* base, uint32_t off) {
    typedef typename std::remove_pointer<decltype(base)>::type T;
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type C;
    return reinterpret_cast<T*>(reinterpret_cast<C*>(base) + off);
  };
  auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<TIN*>(X), 0, 0xFFFFFFFFu, 0x00027000);
  // row of X: its index, or (not WIDE) its byte offset
  auto gather = [&](int32_t i) -> VI {
    if constexpr (WIDE) {
      return *reinterpret_cast<const VI*>(at(row_base(X, i, xb), cb));
    } else if constexpr (sizeof(VI) == 4) {
      return __builtin_bit_cast(VI, __builtin_amdgcn_raw_buffer_load_b32(rsrc, cb, i, 0));
    } else {
      return __builtin_bit_cast(VI, __builtin_amdgcn_raw_buffer_load_b64(rsrc, cb, i, 0));
    }
  };
  auto put = [&](int32_t r, int32_t sidx, const float(&a)[VEC], bool zero) {
    if (!active) return;
    if (out) __builtin_nontemporal_store(RO::pack(a), reinterpret_cast<VO*>(at(row_base(out, r, ob), co)));
    if constexpr (SCAT == 1) {
      if (!zero) {
        VO* o = reinterpret_cast<VO*>(at(row_base(scat, sidx, sb), co));
        float pre[VEC];
        RO::unpack(*o, pre);
#pragma unroll
        for (int e = 0; e < VEC; ++e) pre[e] += a[e];
        if (VEC > 1 && EDGE && dup > 0) {  // shared columns are added once, by the lane below
          float one[1];
#pragma unroll
          for (int e = 1; e < VEC; ++e) {
            one[0] = pre[e];
            if (e >= dup) reinterpret_cast<TOUT*>(o)[e] = RowVec<TOUT, 1>::pack(one);
          }
        } else {
          *o = RO::pack(pre);
        }
      }
    } else if constexpr (SCAT == 2) {
      __builtin_nontemporal_store(RO::pack(a), reinterpret_cast<VO*>(at(row_base(scat, sidx, sb), co)));
    }
  };

  const int32_t gw = uniform(logical_block(xcd_remap) * kWavesPerBlock + wave_id());
  const int32_t w_end = min((gw + 1) * cpw, W);
  for (int32_t w = gw * cpw; w < w_end; ++w) {
    const int32_t i0 = chunk_row[w], i1 = chunk_row[w + 1];
    const int32_t j0 = chunk_nz[w], j1 = chunk_nz[w + 1];
    if (i0 >= R) break;
    const bool has_head = j0 > (int32_t)ptr[i0];
    const int32_t row_end = i1 < R ? i1 : R;
    const int32_t first = has_head ? i0 + 1 : i0;  // rows [first, i1) end in this chunk
    int32_t next = first;                          // first of them not written yet
    auto to_slot = [&](int which, const float(&a)[VEC]) {
      if (!active) return;
      *reinterpret_cast<typename RC::V*>(carry + ((int64_t)w * 2 + which) * N + c) = RC::pack(a);
    };
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
    if (SUM && has_head && (int32_t)ptr[i0 + 1] <= j0) to_slot(0, acc);  // row i0 holds nothing here
    auto zero_rows = [&](int32_t lim) {  // complete rows [next, lim) hold no nonzeros
      float z[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) z[e] = 0.f;
      for (; next < lim; ++next) put(next, SCAT > 0 ? scat_idx[next] : 0, z, true);
    };
    const uint32_t span = i1 > first ? (uint32_t)(i1 - first) : 0u;
    int32_t cur = -1, scur = 0;
    auto flush = [&]() {
      if ((uint32_t)(cur - first) < span) put(cur, scur, acc, false);
      else if (cur >= 0) to_slot(cur >= first ? 1 : 0, acc);  // none open yet, or a piece
    };
    if (j0 < j1) {
      float dcur[DOT ? VEC : 1];
      // window of 64 nonzeros from kw: lane l holds nonzero kw + l (past the
      // chunk's end, its last nonzero again)
      struct Window {
        int32_t i, r, sc, p;
        float v;
      };
      auto place = [&](int32_t kw) { return lane < j1 - kw ? kw + lane : j1 - 1; };
      // where vals holds the window's values: loaded a window before the rest
      auto pload = [&](int32_t kw) { return PERM ? vperm[place(kw)] : 0; };
      auto wload = [&](int32_t kw, int32_t p) {
        Window o;
        const int32_t kk = place(kw);
        o.i = WIDE ? idx[kk] : (int32_t)((uint32_t)idx[kk] * xb);
        o.r = rid[kk];
        o.p = p;
        o.v = 0.f;
        o.sc = 0;
        if constexpr (SUM) o.v = vals[PERM ? p : kk];
        if constexpr (SCAT > 0) o.sc = scat_idx[o.r];
        return o;
      };
      Window cw = wload(j0, pload(j0));
      int32_t np = PERM && j1 - j0 > kWave ? pload(j0 + kWave) : 0;
      for (int32_t left = j1 - j0; left > 0; left -= kWave) {
        const int32_t kw = j1 - left;
        Window nw = cw;
        if (left > kWave) {
          nw = wload(kw + kWave, np);
          if (PERM && left > 2 * kWave) np = pload(kw + 2 * kWave);
        }
        // bit l: nonzero kw + l opens another row than the one before it
        const int32_t prev = __builtin_amdgcn_update_dpp(cur, cw.r, 0x138, 0xF, 0xF, false);  // wave_shr:1
        uint64_t opens = __ballot(cw.r != prev);
        const int32_t nn = min(kWave, left);
        for (int32_t b = 0; b < nn; b += UB, opens >>= UB) {
          const int32_t n = nn - b;  // nonzeros from here to the window's end
          const uint32_t m = (uint32_t)opens & ((1u << UB) - 1u);
          VI x[UB];
#pragma unroll
          for (int j = 0; j < UB; ++j) x[j] = gather(__builtin_amdgcn_readlane(cw.i, b + j));
          float q[UB];
          auto one = [&](int j) {
            float xf[VEC];
            RI::unpack(x[j], xf);
            if constexpr (SUM) {
              const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cw.v), b + j));
#pragma unroll
              for (int e = 0; e < VEC; ++e) acc[e] = fmaf(v, xf[e], acc[e]);
            }
            if constexpr (DOT) {
              float s = 0.f;
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                const float t = fmaf(dcur[e], xf[e], s);
                s = VEC > 1 && EDGE ? (e >= dup ? t : s) : t;
              }
              q[j] = active ? s : 0.f;
            }
          };
          if (m == 0 && n >= UB) {  // the whole batch belongs to the open row
#pragma unroll
            for (int j = 0; j < UB; ++j) one(j);
          } else {
            VI dn[DOT ? UB : 1];
            if constexpr (DOT) {
#pragma unroll
              for (int j = 0; j < UB; ++j)  // D rows of the rows that open here
                if (m >> j & 1)
                  dn[j] = __builtin_nontemporal_load(reinterpret_cast<const VI*>(
                      at(row_base(D, __builtin_amdgcn_readlane(cw.r, b + j), db), cb)));
            }
            // All loads at once: loads and stores retire in one order, so a
            // wait between the rows would be a wait for the stores of those
            // that ended before it.
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
#pragma unroll
            for (int j = 0; j < UB; ++j) {
              if constexpr (DOT) q[j] = 0.f;
              if (j < n) {
                if (m >> j & 1) {
                  const int32_t r = __builtin_amdgcn_readlane(cw.r, b + j);
                  if constexpr (SUM) {
                    flush();
                    if (next < r) zero_rows(r);
                    next = r + 1;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
                  }
                  cur = r;
                  if constexpr (SCAT > 0) scur = __builtin_amdgcn_readlane(cw.sc, b + j);
                  if constexpr (DOT) RI::unpack(dn[j], dcur);
                }
                one(j);
              }
            }
          }
          if constexpr (DOT) {
            const float s = wave_sum8(q, lane);
            const int j = lane >> 3;
            // lane 8 j holds the dot of nonzero b + j, lane b + j its place
            int32_t at_j = kw + b + j;
            if constexpr (PERM) at_j = __builtin_amdgcn_ds_bpermute((b + j) << 2, cw.p);
            if ((lane & 7) == 0 && j < n) dot_out[(int64_t)blockIdx.y * dot_ld + at_j] = s;
          }
        }
        cw = nw;
      }
      if constexpr (SUM) flush();
    }
    if constexpr (SUM) zero_rows(row_end);
  }
}

}  // namespace shiro
