// Low-rank neuron predictor (Sec. 1 "Active Neuron Identification"; Sec. 5.2:
// the predictor gives every FFN neuron a score): z = A x, s = B z + bias.
//
// Every dot product follows one fixed fp32 order so the scores -- and the
// top-k ids chosen from them -- are reproducible bit for bit: chunks of 8
// consecutive elements, chunk c feeds partial c % L with
// L = min(64, largest power of two <= n/8); each partial is an fmaf chain in
// ascending order from +0; then p[l] += p[l ^ off] for off = L/2 .. 1. On the
// GPU partial l is lane l of a group of L lanes, so a wave serves 64/L rows.
//
// What bounds it: with one token the bytes of A and B, after a launch and a
// memory round trip each; with several, instructions. So a wave issues every
// load of its rows at once (no LDS staging and no barrier: its lanes read x or
// z chunks of their own from L2), keeps the z chunk of its lanes in registers
// for all its rows, and the cross-lane sums of its (row, token) values share
// registers: a level of the tree on two values at a time costs one swap and
// one add, where a shuffle and an add per value and level went through the LDS
// crossbar. Measured (MI355X, rocprofv3 kernel time, z + s, before -> now):
// d 1024, r 128, d_ff 2752 7.9 -> 4.5 us; 7B 9.6 -> 5.4, batch 8 33.3 -> 8.5;
// 70B 23.0 -> 10.5.
#include "m2c_internal.h"
#include "wave_ops.h"

namespace m2c {

constexpr int kPredThreads = 256;
constexpr int kPredWaves = kPredThreads / 64;

__host__ __device__ inline int canon_lanes(int n) {
  int chunks = n / 8, L = 1;
  while (L * 2 <= chunks && L < 64) L *= 2;
  return L;
}

__device__ __forceinline__ void unpack8(const uint4 v, float* f) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f[2 * q] = h2f((uint16_t)(w[q] & 0xffffu));
    f[2 * q + 1] = h2f((uint16_t)(w[q] >> 16));
  }
}

constexpr int log2c(int v) { return v <= 1 ? 0 : 1 + log2c(v / 2); }

// After xor_tree<L / 2, N>: the value's index in register 0 of its group for
// this lane, and whether the lane is the one to store it.
template <int L, int N>
struct TreeOut {
  static constexpr int kLevels = log2c(L), kVals = log2c(N);
  static constexpr int kFolds = kLevels < kVals ? kLevels : kVals;
  static constexpr int kRegs = N >> kFolds;
  __device__ __forceinline__ static int index(int lane) {
    int j = 0;
#pragma unroll
    for (int f = 0; f < kFolds; ++f) j |= ((lane >> (kLevels - 1 - f)) & 1) << f;
    return j;
  }
  __device__ __forceinline__ static bool stores(int lane) {
    return (lane & ((1 << (kLevels - kFolds)) - 1)) == 0;
  }
};

// Chunks of a row whose x is in flight together: the most that divide its NCH
// with at most 16 loads for the NB tokens.
constexpr int x_chunks(int nch, int nb) {
  int q = nch;
  while (q > 1 && (q * nb > 16 || nch % q)) --q;
  return q;
}

// z[b][j], tokens NB blockIdx.y .. of the batch (the last group re-reads the
// last token). A lane's partial takes chunks sl, sl + L, ... of its row: all
// of them are loaded before the first fmaf (NCH >= chunks / L per lane).
template <int L, int NCH, int NB>
__global__ __launch_bounds__(kPredThreads) void pred_z_kernel(const uint16_t* __restrict__ A,
                                                              const uint16_t* __restrict__ x,
                                                              int d, int r, int batch,
                                                              float* __restrict__ z) {
  const int lane = threadIdx.x & 63;
  const int gw = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int sl = lane & (L - 1);
  const int j = gw * (64 / L) + lane / L;
  const int b0 = blockIdx.y * NB;
  const int chunks = d >> 3;
  const uint4* arow = reinterpret_cast<const uint4*>(A + (int64_t)min(j, r - 1) * d);
  uint4 av[NCH];
#pragma unroll
  for (int q = 0; q < NCH; ++q) av[q] = arow[min(sl + q * L, chunks - 1)];
  float acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = 0.0f;
  constexpr int QB = x_chunks(NCH, NB);
  static_assert(NCH % QB == 0, "a pass has no chunks past the row's");
#pragma unroll
  for (int q0 = 0; q0 < NCH; q0 += QB) {
    uint4 xv[QB][NB];
#pragma unroll
    for (int q = 0; q < QB; ++q)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        xv[q][b] = reinterpret_cast<const uint4*>(x + (int64_t)min(b0 + b, batch - 1) *
                                                          d)[min(sl + (q0 + q) * L, chunks - 1)];
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      if (sl + (q0 + q) * L < chunks) {
        float af[8];
        unpack8(av[q0 + q], af);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          float xf[8];
          unpack8(xv[q][b], xf);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[b] = __builtin_fmaf(af[e], xf[e], acc[b]);
        }
      }
    }
  }
  xor_tree<L / 2, NB>(acc);
  typedef TreeOut<L, NB> Out;
  const int jb = Out::index(lane);
#pragma unroll
  for (int i = 0; i < Out::kRegs; ++i) {
    const int b = b0 + (i << Out::kFolds) + jb;
    if (j < r && b < batch && Out::stores(lane)) z[(int64_t)b * r + j] = acc[i];
  }
}

// s[b][i] = dot(B[i], z[b]) (+ bias[i]), tokens NB blockIdx.y .. of the batch.
// A wave takes R row groups of 64 / L rows. A row has at most 2 L chunks
// (r <= 1024): a lane's chunks are sl and, when TWO, sl + L where it exists,
// in that order (the canonical order of its partial).
template <int L, bool TWO, int R, int NB>
__global__ __launch_bounds__(kPredThreads) void pred_s_kernel(const uint16_t* __restrict__ Bm,
                                                              const float* __restrict__ z,
                                                              const float* __restrict__ bias,
                                                              int d_ff, int r, int batch,
                                                              float* __restrict__ s) {
  constexpr int NH = TWO ? 2 : 1, rpw = 64 / L;
  const int lane = threadIdx.x & 63;
  const int sl = lane & (L - 1);
  const int gw = __builtin_amdgcn_readfirstlane((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const int row0 = gw * R * rpw + lane / L;  // the lane's row of group 0
  const int b0 = blockIdx.y * NB;
  const int chunks = r >> 3;
  const bool two = TWO && sl + L < chunks;
  uint4 bv[R][NH];
#pragma unroll
  for (int g = 0; g < R; ++g) {
    const uint4* brow =
        reinterpret_cast<const uint4*>(Bm + (int64_t)min(row0 + g * rpw, d_ff - 1) * r);
    bv[g][0] = brow[sl];
    if (TWO) bv[g][NH - 1] = brow[two ? sl + L : sl];
  }
  float acc[R * NB];  // value g NB + b
#pragma unroll
  for (int v = 0; v < R * NB; ++v) acc[v] = 0.0f;
  float4 zv[NB][NH][2];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const float* zb = z + (int64_t)min(b0 + b, batch - 1) * r + 8 * (h && two ? sl + L : sl);
      zv[b][h][0] = reinterpret_cast<const float4*>(zb)[0];
      zv[b][h][1] = reinterpret_cast<const float4*>(zb)[1];
    }
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    if (h == 1 && !two) break;
#pragma unroll
    for (int g = 0; g < R; ++g) {
      float bf[8];
      unpack8(bv[g][h], bf);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float4 z0 = zv[b][h][0], z1 = zv[b][h][1];
        const float zf[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g * NB + b] = __builtin_fmaf(bf[e], zf[e], acc[g * NB + b]);
      }
    }
  }
  xor_tree<L / 2, R * NB>(acc);
  typedef TreeOut<L, R * NB> Out;
  const int jv = Out::index(lane);
#pragma unroll
  for (int i = 0; i < Out::kRegs; ++i) {
    const int val = (i << Out::kFolds) + jv;
    const int row = row0 + (val / NB) * rpw, b = b0 + val % NB;
    if (row < d_ff && b < batch && Out::stores(lane)) {
      float v = acc[i];
      if (bias) v = v + bias[row];
      s[(int64_t)b * d_ff + row] = v;
    }
  }
}

struct PredArgs {
  const uint16_t* A;
  const uint16_t* B;
  const float* bias;
  const uint16_t* x;
  int d, r, d_ff, batch;
  float* z;
  float* s;
  hipStream_t stream;
};

template <int L, int NCH, int NB>
static void launch_z(const PredArgs& p) {
  const int waves = (p.r + 64 / L - 1) / (64 / L);
  // few waves (256 at 7B, 512 at 70B): one per workgroup, so that they spread
  // over the CUs (70B 4.4 us against 5.0 with four)
  const int threads = waves * ((p.batch + NB - 1) / NB) < 2048 ? 64 : kPredThreads;
  const int per = threads / 64;
  hipLaunchKernelGGL((pred_z_kernel<L, NCH, NB>), dim3((waves + per - 1) / per, (p.batch + NB - 1) / NB),
                     dim3(threads), 0, p.stream, p.A, p.x, p.d, p.r, p.batch, p.z);
}

template <int L, int NCH>
static void launch_z_nb(const PredArgs& p) {
  if (p.batch == 1)
    launch_z<L, NCH, 1>(p);
  else if (p.batch == 2)
    launch_z<L, NCH, 2>(p);
  else
    launch_z<L, NCH, 4>(p);
}

template <int L, bool TWO, int R, int NB>
static void launch_s(const PredArgs& p) {
  const int rows = R * (64 / L) * kPredWaves;
  hipLaunchKernelGGL((pred_s_kernel<L, TWO, R, NB>),
                     dim3((p.d_ff + rows - 1) / rows, (p.batch + NB - 1) / NB), dim3(kPredThreads),
                     0, p.stream, p.B, p.z, p.bias, p.d_ff, p.r, p.batch, p.s);
}

// Four row groups per wave at every size: with one token 1 / 4 / 8 groups take
// 8.2 / 6.1 / 6.5 us at d_ff 28672, r 512 and 3.0 / 2.8 / 2.9 at 11008, r 256.
constexpr int kPredGroups = 4;

template <int L, bool TWO>
static void launch_s_nb(const PredArgs& p) {
  if (p.batch == 1)
    launch_s<L, TWO, kPredGroups, 1>(p);
  else if (p.batch == 2)
    launch_s<L, TWO, kPredGroups, 2>(p);
  else if (p.batch <= 4)
    launch_s<L, TWO, kPredGroups, 4>(p);
  else
    launch_s<L, TWO, kPredGroups, 8>(p);
}

template <int L>
static void launch_s_two(const PredArgs& p) {
  if ((p.r >> 3) > L)
    launch_s_nb<L, true>(p);
  else
    launch_s_nb<L, false>(p);
}

hipError_t launch_predict(const m2c_layer* L, const uint16_t* x, int batch, float* z,
                          float* scores, hipStream_t stream) {
  const PredArgs p = {L->pred_a, L->pred_b, L->bias, x, (int)L->desc.d_model, (int)L->desc.pred_rank,
                      (int)L->desc.d_ff, batch, z, scores, stream};
  // d is a multiple of 128: 16 lanes (128, 1 chunk each; 256 and up have 32 or
  // 64), chunks per lane rounded up to an instance
  const int Lz = canon_lanes(p.d), nch = ((p.d >> 3) + Lz - 1) / Lz;
  if (Lz == 16)
    launch_z_nb<16, 1>(p);
  else if (Lz == 32)
    nch <= 1 ? launch_z_nb<32, 1>(p) : launch_z_nb<32, 2>(p);
  else if (nch <= 1)
    launch_z_nb<64, 1>(p);
  else if (nch <= 2)
    launch_z_nb<64, 2>(p);
  else if (nch <= 4)
    launch_z_nb<64, 4>(p);
  else if (nch <= 8)
    launch_z_nb<64, 8>(p);
  else if (nch <= 12)
    launch_z_nb<64, 12>(p);
  else if (nch <= 16)
    launch_z_nb<64, 16>(p);
  else
    launch_z_nb<64, 32>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (canon_lanes(p.r)) {
    case 1: launch_s_two<1>(p); break;
    case 2: launch_s_two<2>(p); break;
    case 4: launch_s_two<4>(p); break;
    case 8: launch_s_two<8>(p); break;
    case 16: launch_s_two<16>(p); break;
    case 32: launch_s_two<32>(p); break;
    default: launch_s_two<64>(p); break;
  }
  return hipGetLastError();
}

}  // namespace m2c
