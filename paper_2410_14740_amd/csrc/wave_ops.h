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
