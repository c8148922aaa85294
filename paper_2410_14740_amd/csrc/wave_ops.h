// Wave-wide scans and reductions on DPP moves (gfx950, 64 lanes): one VALU
// instruction per step instead of a trip through the LDS crossbar
// (ds_bpermute), which is what the one-workgroup kernels wait on.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace m2c {

constexpr int kDppRowShr = 0x110;     // + n: lane l of a row of 16 reads lane l - n
constexpr int kDppRowRor = 0x120;     // + n: rotation inside a row of 16
constexpr int kDppRowBcast15 = 0x142; // lane 15 of a row to the next row
constexpr int kDppRowBcast31 = 0x143; // lane 31 to rows 2 and 3

// v of the lane the DPP control names; 0 where there is none or the row is
// masked out.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum inside each row of 16 lanes.
__device__ __forceinline__ uint32_t row_incl_scan(uint32_t v) {
  v += dpp0<kDppRowShr + 1>(v);
  v += dpp0<kDppRowShr + 2>(v);
  v += dpp0<kDppRowShr + 4>(v);
  v += dpp0<kDppRowShr + 8>(v);
  return v;
}

// Inclusive prefix sum over the wave's 64 lanes (all lanes active).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v = row_incl_scan(v);
  v += dpp0<kDppRowBcast15, 0xa>(v);
  v += dpp0<kDppRowBcast31, 0xc>(v);
  return v;
}

// v of lane l ^ OFF of the row of 16 (OFF 1, 2, 4, 8).
template <int OFF>
__device__ __forceinline__ float row_xor(float v) {
  const int u = __float_as_int(v);
  if constexpr (OFF == 8) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, u, kDppRowRor + 8, 0xf, 0xf, false));
  } else if constexpr (OFF == 4) {  // l ^ 7 (mirror of 8 lanes), then ^ 3 (quad reversed)
    const int m = __builtin_amdgcn_update_dpp(0, u, 0x141, 0xf, 0xf, false);
    return __int_as_float(__builtin_amdgcn_update_dpp(0, m, 0x1b, 0xf, 0xf, false));
  } else if constexpr (OFF == 2) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, u, 0x4e, 0xf, 0xf, false));
  } else {
    static_assert(OFF == 1, "lane distances of a row of 16");
    return __int_as_float(__builtin_amdgcn_update_dpp(0, u, 0xb1, 0xf, 0xf, false));
  }
}

// One level of a cross-lane sum for two values at once: lanes without bit OFF
// get u[l] + u[l ^ OFF], lanes with it v[l] + v[l ^ OFF].
template <int OFF>
__device__ __forceinline__ float xor_fold(float u, float v) {
  if constexpr (OFF == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else if constexpr (OFF == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
  } else {
    const float a = u + row_xor<OFF>(u), b = v + row_xor<OFF>(v);
    return (threadIdx.x & OFF) ? b : a;
  }
}

// The xor-tree sums (p[l] + p[l ^ off] for off = OFF, OFF / 2, .. 1) of N
// values, N a power of two, every level on half the registers of the one
// before while there are two: afterwards v[i] holds value (i << F) + j in the
// lanes whose bits OFF, OFF / 2, .. (F of them) are the bits 0, 1, .. of j,
// F = min(log2 N, levels).
template <int OFF, int N>
__device__ __forceinline__ void xor_tree(float* v) {
  if constexpr (OFF >= 1) {
    if constexpr (N > 1) {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) v[i] = xor_fold<OFF>(v[2 * i], v[2 * i + 1]);
      xor_tree<OFF / 2, N / 2>(v);
    } else {
      v[0] = xor_fold<OFF>(v[0], v[0]);
      xor_tree<OFF / 2, 1>(v);
    }
  }
}

// Largest value of each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
  v = max(v, dpp0<kDppRowRor + 8>(v));
  v = max(v, dpp0<kDppRowRor + 4>(v));
  v = max(v, dpp0<kDppRowRor + 2>(v));
  v = max(v, dpp0<kDppRowRor + 1>(v));
  return v;
}

// Largest value of the wave, wave-uniform.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = row_max(v);
  const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
  const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
  return max(max(a, b), max(c, d));
}

// Exclusive prefix of v over a workgroup of 1024 threads, *total the sum.
// tmp: 16 words of LDS that nothing else uses until the next barrier after
// this call. One barrier; every wave scans the wave totals itself.
__device__ __forceinline__ uint32_t block_excl_scan_1024(uint32_t v, uint32_t* tmp,
                                                         uint32_t* total) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t incl = wave_incl_scan(v);
  if (lane == 63) tmp[wave] = incl;
  __syncthreads();
  const uint32_t wt = row_incl_scan(tmp[lane & 15]);  // every row scans all 16 totals
  *total = __builtin_amdgcn_readlane(wt, 15);
  const uint32_t before = wave > 0 ? __builtin_amdgcn_readlane(wt, wave - 1) : 0u;
  return before + incl - v;
}

}  // namespace m2c
