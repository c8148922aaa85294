// Top-k selection and score-rank precision tiers (Sec. 5.2: the top-k scored
// neurons are active, and the higher the score the higher the precision).
//
// One workgroup per token. Neurons are ranked by (score descending, id
// ascending) with scores compared as order-preserving u32 keys. Three rank
// boundaries are needed -- n_fp16, n_fp16 + n_int8 and k -- and a neuron's
// tier follows from how many of them its rank is below.
//
// What bounds it: one CU's instruction issue (a wave64 VALU instruction holds
// a 16-lane SIMD for four cycles, and every key is visited by the same four
// SIMDs) and the barriers between passes, not the 4 d_ff bytes read. So the
// keys are visited as few times as possible, with few instructions each:
//
//   1  load every score (registers), largest magnitude A of the row
//   2  histogram over 4096 bins of equal width on [-A, A]: bin = trunc(
//      fmaf(s, inv, 2047.5)), nondecreasing in s, so bins order the scores
//   3  a block scan from the top bin finds, for each boundary rank, its bin
//   4  bins above / below a boundary bin decide a neuron's tier at once; the
//      few neurons inside a boundary bin are listed in LDS
//   5  their exact ranks: the keys in higher bins plus the larger (key, id)
//      pairs of their own list
//
// Equal-width bins hold about 0.07% of a normal score distribution at a
// boundary (8 of 11008 neurons, 20 of 28672), where the top 12 bits of the
// key hold 2%, and spread the histogram's LDS atomics. When the distribution
// does not suit them (a boundary bin with more than kSelCand neurons, as with
// equal scores or a lone outlier; infinities, NaN, magnitudes near the ends
// of the fp32 range) an MSD radix select over the pairs (key, id) ranks the
// same keys. Measured (MI355X, rocprofv3 kernel time, the three-pass radix
// select it replaces -> this): d_ff 2752 9.0 -> 4.5 us, 11008 14.7 -> 6.0,
// 28672 29.1 -> 11.8, 40000 89.4 -> 15.5.
#include "m2c_internal.h"
#include "wave_ops.h"

namespace m2c {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelBins = 4096;
constexpr int kSelCand = 1024;       // most neurons of one boundary bin
constexpr int kSelIdBits = 18;       // d_ff <= 2^18
constexpr uint32_t kSelAmaxLo = 0x0d000000u;  // 3.9e-31: below, inv and the bins lose range
constexpr uint32_t kSelAmaxHi = 0x7e000000u;  // 4.3e37: from here, and for inf / NaN, radix

struct SelLds {
  union {
    struct {
      uint32_t hist[kSelBins];
      unsigned long long cand[3][kSelCand];
    } lin;
    uint32_t radix[3][kSelBins];
  };
  uint32_t red[kSelWaves];   // wave maxima, then wave totals
  uint32_t scan[kSelWaves];
  uint32_t bin[3], above[3], m[3];  // boundary bin, keys above it, keys in it
  uint32_t n[3];                    // candidates listed
  unsigned long long prefix[3];
  uint32_t remain[3];
};

// Scores of one row: J > 0 in registers, neuron tid + 1024 j at j; J == 0 (any
// d_ff) read from memory (the row stays in L2) by every pass.
template <int J>
struct SelKeys {
  float s[J > 0 ? J : 1];
  const float* sc;
  int d_ff;
  __device__ __forceinline__ void load(const float* scores, int n) {
    sc = scores;
    d_ff = n;
#pragma unroll
    for (int j = 0; j < J; ++j) s[j] = sc[min((int)threadIdx.x + kSelThreads * j, d_ff - 1)];
  }
  // f(id, score) over this thread's neurons
  template <typename F>
  __device__ __forceinline__ void each(F f) const {
    int n = d_ff;
    asm volatile("" : "+s"(n));  // one pass's id < d_ff masks are not kept for the next (they spill)
    if constexpr (J > 0) {
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int id = threadIdx.x + kSelThreads * j;
        if (id < n) f(id, s[j]);
      }
    } else {
      for (int i0 = threadIdx.x; i0 < n; i0 += 8 * kSelThreads) {
        float v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = sc[min(i0 + kSelThreads * q, n - 1)];
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (i0 + kSelThreads * q < n) f(i0 + kSelThreads * q, v[q]);
      }
    }
  }
};

__device__ __forceinline__ uint8_t tier_of_rank(uint32_t rank, const uint32_t (&R)[3]) {
  return (uint8_t)((rank < R[0]) + (rank < R[1]) + (rank < R[2]));
}

// MSD radix select over the 50-bit pairs key << 18 | (2^18 - 1 - id), which
// are distinct: digits of 12, 12, 8 bits of the key and twice 9 of the id,
// all three targets in the same passes. A neuron is within target t when its
// pair is not below the R[t]-th largest.
// The scores are read again by each pass: kept in registers as well, they
// and their pairs would spill in the kernels of wide rows.
__device__ void select_radix(const float* __restrict__ sc, int d_ff, const uint32_t (&R)[3],
                             SelLds& sm, uint8_t* __restrict__ out) {
  const int tid = threadIdx.x;
  SelKeys<0> K;
  K.load(sc, d_ff);
  auto pair = [](int id, float s) {
    return ((unsigned long long)score_key(s) << kSelIdBits) |
           (unsigned long long)((1 << kSelIdBits) - 1 - id);
  };
  if (tid < 3) {
    sm.prefix[tid] = 0;
    sm.remain[tid] = R[tid];
  }
  for (int pass = 0; pass < 5; ++pass) {
    const int width = pass < 2 ? 12 : pass == 2 ? 8 : 9;
    const int shift = pass == 0 ? 38 : pass == 1 ? 26 : pass == 2 ? 18 : pass == 3 ? 9 : 0;
    const int nbins = 1 << width, top = shift + width;
    __syncthreads();
    for (int t = 0; t < 3; ++t)
      for (int b = tid; b < nbins; b += kSelThreads) sm.radix[t][b] = 0;
    __syncthreads();
    const unsigned long long pre[3] = {sm.prefix[0] >> top, sm.prefix[1] >> top,
                                       sm.prefix[2] >> top};
    K.each([&](int id, float s) {
      const unsigned long long p = pair(id, s);
      const uint32_t dig = (uint32_t)(p >> shift) & (uint32_t)(nbins - 1);
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (R[t] > 0 && (p >> top) == pre[t]) atomicAdd(&sm.radix[t][dig], 1u);
    });
    __syncthreads();
    const int bpt = nbins >= kSelThreads ? nbins / kSelThreads : 1;
    const int hi_bin = nbins - tid * bpt;  // this thread owns bins [hi_bin - bpt, hi_bin)
    for (int t = 0; t < 3; ++t) {
      uint32_t c = 0;
      if (hi_bin > 0)
        for (int b = hi_bin - 1; b >= hi_bin - bpt; --b) c += sm.radix[t][b];
      const uint32_t rem = sm.remain[t];
      uint32_t tot;
      const uint32_t above = block_excl_scan_1024(c, sm.scan, &tot);
      __syncthreads();  // every thread has its rem, and the scan's words are free again
      if (hi_bin > 0 && R[t] > 0 && above < rem && above + c >= rem) {
        uint32_t cum = above;
        for (int b = hi_bin - 1; b >= hi_bin - bpt; --b) {
          if (cum + sm.radix[t][b] >= rem) {
            sm.prefix[t] |= (unsigned long long)b << shift;
            sm.remain[t] = rem - cum;
            break;
          }
          cum += sm.radix[t][b];
        }
      }
    }
  }
  __syncthreads();
  const unsigned long long T[3] = {sm.prefix[0], sm.prefix[1], sm.prefix[2]};
  K.each([&](int id, float s) {
    const unsigned long long p = pair(id, s);
    out[id] = (uint8_t)((R[0] > 0 && p >= T[0]) + (R[1] > 0 && p >= T[1]) + (R[2] > 0 && p >= T[2]));
  });
}

template <int J>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const float* __restrict__ scores,
                                                             int d_ff, int k, int n16, int n8,
                                                             uint8_t* __restrict__ tier_map) {
  __shared__ SelLds sm;
  const float* sc = scores + (int64_t)blockIdx.x * d_ff;
  uint8_t* out = tier_map + (int64_t)blockIdx.x * d_ff;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t R[3] = {(uint32_t)n16, (uint32_t)(n16 + n8), (uint32_t)k};
  SelKeys<J> K;
  K.load(sc, d_ff);
  reinterpret_cast<uint4*>(sm.lin.hist)[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < 3) {
    sm.n[tid] = 0;
    sm.m[tid] = 0;
    sm.bin[tid] = 0xffffffffu;  // a boundary of rank 0: above every bin
    sm.above[tid] = 0;
  }
  // 1: largest magnitude (as bits: inf and NaN compare above every number)
  uint32_t amax = 0;
  K.each([&](int, float s) { amax = max(amax, __float_as_uint(s) & 0x7fffffffu); });
  amax = wave_max(amax);
  if (lane == 0) sm.red[wave] = amax;
  __syncthreads();
  amax = __builtin_amdgcn_readfirstlane(row_max(sm.red[lane & 15]));
  if (amax < kSelAmaxLo || amax >= kSelAmaxHi) {  // workgroup-uniform
    select_radix(sc, d_ff, R, sm, out);
    return;
  }
  // 2: bins. fmaf rounds once, so the bin is nondecreasing in s; -A and A
  // land within half an ulp of 0 and 4095 (a negative float converts to 0)
  const float inv = 0.5f * (kSelBins - 1) / __uint_as_float(amax);
  auto bin_of = [&](float s) {
    return (uint32_t)max((int)__builtin_fmaf(s, inv, 0.5f * (kSelBins - 1)), 0);
  };
  K.each([&](int, float s) { atomicAdd(&sm.lin.hist[bin_of(s)], 1u); });
  __syncthreads();
  // 3: thread tid owns bins [4092 - 4 tid, 4096 - 4 tid), highest first
  static_assert(kSelBins == 4 * kSelThreads, "four bins per thread");
  const uint4 h = reinterpret_cast<const uint4*>(sm.lin.hist)[kSelThreads - 1 - tid];
  const uint32_t c = h.x + h.y + h.z + h.w;
  uint32_t tot;
  const uint32_t above = block_excl_scan_1024(c, sm.scan, &tot);
#pragma unroll
  for (int t = 0; t < 3; ++t)
    if (above < R[t] && above + c >= R[t]) {
      const uint32_t hv[4] = {h.w, h.z, h.y, h.x};
      uint32_t cum = above;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (cum < R[t] && cum + hv[q] >= R[t]) {
          sm.bin[t] = (uint32_t)(kSelBins - 1 - 4 * tid - q);
          sm.above[t] = cum;
          sm.m[t] = hv[q];
        }
        cum += hv[q];
      }
    }
  __syncthreads();
  const uint32_t b0 = sm.bin[0], b1 = sm.bin[1], b2 = sm.bin[2];
  if (max(max(sm.m[0], sm.m[1]), sm.m[2]) > (uint32_t)kSelCand) {  // workgroup-uniform
    select_radix(sc, d_ff, R, sm, out);
    return;
  }
  // 4: tiers by bin; neurons of a boundary bin go to its list (targets that
  // share a bin share the first one's list)
  K.each([&](int id, float s) {
    const uint32_t b = bin_of(s);
    if (b == b0 || b == b1 || b == b2) {
      const int u = b == b0 ? 0 : b == b1 ? 1 : 2;
      const uint32_t at = atomicAdd(&sm.n[u], 1u);
      sm.lin.cand[u][at] = ((unsigned long long)score_key(s) << kSelIdBits) |
                           (unsigned long long)((1 << kSelIdBits) - 1 - id);
    } else {
      out[id] = (uint8_t)((b > b0) + (b > b1) + (b > b2));
    }
  });
  __syncthreads();
  // 5: exact ranks of the listed neurons
  const uint32_t m0 = sm.n[0], m1 = sm.n[1], m2 = sm.n[2];
  for (uint32_t e = tid; e < m0 + m1 + m2; e += kSelThreads) {
    const int u = e < m0 ? 0 : e < m0 + m1 ? 1 : 2;
    const uint32_t p = e - (u > 0 ? m0 : 0) - (u > 1 ? m1 : 0);
    const uint32_t m = u == 0 ? m0 : u == 1 ? m1 : m2;
    const unsigned long long mine = sm.lin.cand[u][p];
    uint32_t rank = sm.above[u];
    for (uint32_t q = 0; q < m; ++q) rank += sm.lin.cand[u][q] > mine;
    const int id = (1 << kSelIdBits) - 1 - (int)(mine & ((1u << kSelIdBits) - 1u));
    out[id] = tier_of_rank(rank, R);
  }
}

// J: scores per thread, the next instance above ceil(d_ff / 1024). Past 40 the
// registers of a 16-wave workgroup (128) no longer hold them without spills:
// wider rows are read again by each pass.
hipError_t launch_select(const float* scores, int batch, int d_ff, int k, int n16, int n8,
                         uint8_t* tier_map, hipStream_t stream) {
  const int J = (d_ff + kSelThreads - 1) / kSelThreads;
#define M2C_SEL(JJ)                                                                        \
  hipLaunchKernelGGL(select_kernel<JJ>, dim3(batch), dim3(kSelThreads), 0, stream, scores, \
                     d_ff, k, n16, n8, tier_map)
  if (J <= 1)
    M2C_SEL(1);
  else if (J <= 2)
    M2C_SEL(2);
  else if (J <= 4)
    M2C_SEL(4);
  else if (J <= 8)
    M2C_SEL(8);
  else if (J <= 12)
    M2C_SEL(12);
  else if (J <= 16)
    M2C_SEL(16);
  else if (J <= 20)
    M2C_SEL(20);
  else if (J <= 24)
    M2C_SEL(24);
  else if (J <= 28)
    M2C_SEL(28);
  else if (J <= 32)
    M2C_SEL(32);
  else if (J <= 40)
    M2C_SEL(40);
  else
    M2C_SEL(0);
#undef M2C_SEL
  return hipGetLastError();
}

}  // namespace m2c
