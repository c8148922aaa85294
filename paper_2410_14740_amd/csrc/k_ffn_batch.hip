// Sparse mixed-precision SwiGLU FFN for a batch of 2..32 tokens. The plan's
// required set is the union of the batch rows' active sets, each neuron at
// the highest tier any row asked for, with a row mask (the paper keeps batch
// 1, Sec. 5.5; this follows the union reading in include/m2c.h). Row b sums
// only the neurons whose mask has bit b:
//
//   y_b += sum_{i : mask_i bit b} silu(<g_i, x_b>) * <u_i, x_b> * d_i
//
// With several tokens the gate / up side is a real dense contraction, a
// gathered (2|R| x d) by (d x B) product, so it runs on the matrix cores:
//
//   ffn_bh_kernel   a workgroup takes a tile of 16 neurons of one tier (8 for
//                   FP16, padded with the zero slot; twice that above 16
//                   rows on large unions); its 8
//                   waves split d by quantization group (group g to wave
//                   g % 8). For each group a wave issues four
//                   v_mfma_f32_16x16x32_f16 steps per row kind over the 128
//                   elements: A = the 16 neurons' codes (INT8 / INT4 unpacked
//                   to exact fp16), B = x of 16 batch rows (rows past the
//                   batch are zeros), read from the wave's LDS copy of the
//                   group's x rows. Which columns a lane takes in a step is
//                   chosen per tier so that every 16-byte record load of a
//                   wave covers 64 contiguous bytes of each row; both
//                   operands follow the same order. Each group's product is
//                   scaled by its fp16 scales in fp32 and added up, so the
//                   dequantization stays exact. The waves' partials meet in
//                   LDS; h_{b,i} = silu(a) * u, zero where row b did not
//                   select neuron i.
//   ffn_bdn_kernel  the down projection, also on the matrix cores, by
//                   quantization group (below).
#include "ffn_device.h"
#include "wave_ops.h"

namespace m2c {

typedef _Float16 half4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kBHThreads = 512;
constexpr int kBHWaves = kBHThreads / 64;

__device__ __forceinline__ half4v h4(uint32_t lo, uint32_t hi) {
  half4v r;
  const half2v a = as_h2(lo), b = as_h2(hi);
  r[0] = a[0];
  r[1] = a[1];
  r[2] = b[0];
  r[3] = b[1];
  return r;
}

// Four INT4 codes (16 bits, element e in bits 4e..4e+3) -> exact fp16 values.
__device__ __forceinline__ half4v i4x4_to_h4(uint32_t w16) {
  const uint32_t ob = w16 ^ 0x8888u;  // q + 8 per nibble
  const uint32_t lo = (ob & 0xfu) | ((ob & 0xf0u) << 12) | 0x64006400u;
  const uint32_t hi = ((ob >> 8) & 0xfu) | ((ob & 0xf000u) << 4) | 0x64006400u;
  const half2v bias = {(_Float16)1032.0f, (_Float16)1032.0f};
  const half2v a = as_h2(lo) - bias, b = as_h2(hi) - bias;
  half4v r;
  r[0] = a[0];
  r[1] = a[1];
  r[2] = b[0];
  r[3] = b[1];
  return r;
}

// Four INT8 codes (one word) -> exact fp16 values.
__device__ __forceinline__ half4v i8x4_to_h4(uint32_t w) {
  half2v a, b;
  i8x4_to_h2(w, a, b);
  half4v r;
  r[0] = a[0];
  r[1] = a[1];
  r[2] = b[0];
  r[3] = b[1];
  return r;
}

// The h values, written by the gate/up kernel and read by the down kernel as
// matrix-core operands: 4 consecutive items of one tier, then the batch row,
// then the next 4 items, each tier's items from a multiple of 32 (h_base + the
// item's place in its tier). Up to 16 rows only the batch's are stored: every
// workgroup of the down kernel reads these bytes, and at 2 rows padding to 16
// makes them eight times as many. Above, there are 32, zeros past the batch (a
// stride that is no constant cost 1 to 2% at 32 rows).
template <int NT>
__device__ __forceinline__ int h_rows(int B) {
  return NT == 1 ? B : 16 * NT;
}
constexpr int kHAlign = 32;
__device__ __forceinline__ int h_base(int tier, int n3, int n2) {
  const int p3 = (n3 + kHAlign - 1) / kHAlign * kHAlign;
  const int p2 = (n2 + kHAlign - 1) / kHAlign * kHAlign;
  return tier == 3 ? 0 : tier == 2 ? p3 : p3 + p2;
}

// Tile b: up to 16 consecutive work items of one tier. An FP16 tile takes 8
// items (the MFMA rows past them read the zero slot), so that it carries about
// as many record bytes as an INT8 tile of 16 and the workgroups finish
// together instead of the FP16 tiles trailing. Wide tiles are twice that.
__device__ __forceinline__ void bh_tile(int b, int n3, int n2, int n1, int wide, int& tier,
                                        int& item0, int& nitems) {
  const int l3 = 3 + wide, l = 4 + wide;  // log2 of the tile's items
  const int t3 = (n3 + (1 << l3) - 1) >> l3;
  const int t2 = (n2 + (1 << l) - 1) >> l, t1 = (n1 + (1 << l) - 1) >> l;
  if (b < t3) {
    tier = 3;
    item0 = b << l3;
    nitems = min(1 << l3, n3 - item0);
  } else if (b < t3 + t2) {
    tier = 2;
    item0 = (b - t3) << l;
    nitems = min(1 << l, n2 - item0);
    item0 += n3;
  } else if (b < t3 + t2 + t1) {
    tier = 1;
    item0 = (b - t3 - t2) << l;
    nitems = min(1 << l, n1 - item0);
    item0 += n3 + n2;
  } else {
    tier = 0;
    item0 = nitems = 0;
  }
}

// Above 16 rows a workgroup holds a CU alone (its registers), and each reads
// all of x (32 rows: as many bytes as 2 to 4 tiles' INT8 or INT4 codes). Wide
// tiles halve those reads and the rounds of workgroups; they are taken when the
// tiles of 16 are more than one per CU (256 CUs). Measured (MI355X, both launches
// of a call, tiles of 16 -> wide): 70B shape at 32 rows (935 tiles of 16) 121.5 ->
// 105.2 us, 13B (640) 67.3 -> 64.6, d 12288 (269) 68.7 -> 64.3, d 1024 (2000) 58.0 ->
// 47.0; with 260 to 1200 tiles and d 256 to 8192, at 17 and 32 rows, all between 0
// and 17% faster but one (d 8192 at 17 rows with 600, where the wide ones just miss
// one round: 82.1, 83.1).
constexpr int kBHWideTiles = 256;

// One group (128 columns) of a tile on the matrix cores, as four
// v_mfma_f32_16x16x32_f16 steps per row kind (gate, up). Lane (row r, lane
// group j) supplies 8 codes of neuron row r per step; which 8 of the group's
// 128 columns a (j, step) pair takes is chosen per tier so that every 16-byte
// record load of a wave covers 64 contiguous bytes of each of its rows:
//
//   FP16  load e = step e:            columns 32 s + 8 j .. + 8
//   INT8  load e = steps 2e, 2e + 1:  columns 64 (s >> 1) + 16 j + 8 (s & 1) .. + 8
//   INT4  one load, word s = step s:  columns 32 j + 8 s .. + 8
//
// The B operand (x of the lane's batch column, same 8 columns) is read from
// the wave's copy of the group's x rows in LDS, so both operands pair the
// same columns whatever the mapping.
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
constexpr int kBXRow = 136;  // halves per staged x row: 128 and a pad against bank conflicts
// halves per row of the staged gate and up scales (2 G, padded to 16 bytes)
__host__ __device__ constexpr int bh_scale_row(int G) { return 8 * ((G + 3) / 4); }

__device__ __forceinline__ half8v h8(half4v lo, half4v hi) {
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int TIER>
__host__ __device__ constexpr int bh_xcol(int j, int s) {
  return TIER == 3 ? 32 * s + 8 * j : TIER == 2 ? 64 * (s >> 1) + 16 * j + 8 * (s & 1) : 32 * j + 8 * s;
}

template <int TIER>
struct GroupA {
  static constexpr int NV = TIER == 3 ? 4 : TIER == 2 ? 2 : 1;  // 16-byte loads per row
  uint4 g[NV], u[NV];
  __device__ __forceinline__ void load(const uint8_t* rec, int d, int grp, int j) {
    const int64_t row = TIER == 3 ? 2 * (int64_t)d : TIER == 2 ? d : (d >> 1);
#pragma unroll
    for (int e = 0; e < NV; ++e) {
      const int64_t off = TIER == 3   ? 256 * (int64_t)grp + 64 * e + 16 * j
                          : TIER == 2 ? 128 * (int64_t)grp + 64 * e + 16 * j
                                      : 64 * (int64_t)grp + 16 * j;
      g[e] = *reinterpret_cast<const uint4*>(rec + off);
      u[e] = *reinterpret_cast<const uint4*>(rec + row + off);
    }
  }
  // the 8 codes of step s, as exact fp16 values
  __device__ __forceinline__ static half8v step(const uint4 (&v)[NV], int s) {
    if (TIER == 3) {
      return __builtin_bit_cast(half8v, v[s]);
    } else if (TIER == 2) {
      const uint4 c = v[s >> 1];
      return (s & 1) ? h8(i8x4_to_h4(c.z), i8x4_to_h4(c.w)) : h8(i8x4_to_h4(c.x), i8x4_to_h4(c.y));
    } else {
      const uint4 c = v[0];
      const uint32_t w = s == 0 ? c.x : s == 1 ? c.y : s == 2 ? c.z : c.w;
      return h8(i4x4_to_h4(w & 0xffffu), i4x4_to_h4(w >> 16));
    }
  }
};

// The global loads of one group: x rows 4 q + j (q < NXQ; 16-byte chunk
// col; rows past the batch re-read the last row, and are stored as zeros)
// and the records. Every load is unconditional.
template <int TIER, int MT, int NXQ>
struct BhLoads {
  GroupA<TIER> A[MT];
  uint4 xr[NXQ];
  __device__ __forceinline__ void issue_x(const uint16_t* x, int d, int B, int grp, int lane) {
    const int j = lane >> 4, col = lane & 15;
#pragma unroll
    for (int q = 0; q < NXQ; ++q) {
      const int row = min(4 * q + j, B - 1);
      xr[q] = *reinterpret_cast<const uint4*>(x + (int64_t)row * d + 128 * grp + 8 * col);
    }
  }
  __device__ __forceinline__ void issue_a(const uint8_t* const* rec, int d, int grp, int lane) {
#pragma unroll
    for (int m = 0; m < MT; ++m) A[m].load(rec[m], d, grp, lane >> 4);
  }
  // the x rows into the wave's LDS copy (the asm makes the values used
  // whatever the row, so that no load of a row past the batch moves under
  // a branch)
  __device__ __forceinline__ void stage(uint16_t* s_xw, int B, int lane) {
    const int j = lane >> 4, col = lane & 15;
#pragma unroll
    for (int q = 0; q < NXQ; ++q)
      asm volatile("" : "+v"(xr[q].x), "+v"(xr[q].y), "+v"(xr[q].z), "+v"(xr[q].w));
#pragma unroll
    for (int q = 0; q < NXQ; ++q) {
      const int row = 4 * q + j;
      *reinterpret_cast<uint4*>(s_xw + row * kBXRow + 8 * col) =
          row < B ? xr[q] : make_uint4(0u, 0u, 0u, 0u);
    }
  }
};

// The arithmetic of one group, x staged in s_xw: MT tiles of 16 neurons.
template <int TIER, int MT, int NT, int MA>
__device__ __forceinline__ void bh_compute(const GroupA<TIER> (&A)[MT], const uint16_t* s_xw,
                                           const uint16_t* s_sc, int G, int grp, int lane,
                                           float4v (&acc_g)[MA][NT], float4v (&acc_u)[MA][NT]) {
  const int j = lane >> 4, col = lane & 15;
  // one tile of neurons after the other: both at once read x from LDS once, but
  // their products do not fit the registers
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    float4v tg[NT], tu[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      tg[t] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
      tu[t] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const half8v ag = GroupA<TIER>::step(A[m].g, s), au = GroupA<TIER>::step(A[m].u, s);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const half8v bx = *reinterpret_cast<const half8v*>(s_xw + (16 * t + col) * kBXRow +
                                                            bh_xcol<TIER>(j, s));
        tg[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ag, bx, tg[t], 0, 0, 0);
        tu[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(au, bx, tu[t], 0, 0, 0);
      }
    }
    // rows 4j + i of the tile's result: scale each by its neuron's group scale
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float sg = 1.0f, su = 1.0f;
      if (TIER != 3) {
        sg = h2f(s_sc[(16 * m + 4 * j + i) * bh_scale_row(G) + grp]);
        su = h2f(s_sc[(16 * m + 4 * j + i) * bh_scale_row(G) + G + grp]);
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        acc_g[m][t][i] = fmaf(sg, tg[t][i], acc_g[m][t][i]);
        acc_u[m][t][i] = fmaf(su, tu[t][i], acc_u[m][t][i]);
      }
    }
    if (m + 1 < MT) __builtin_amdgcn_sched_barrier(0);
  }
}

// The loads of the next group, and the current one's x rows into LDS. With
// wide tiles, and for 9 to 16 rows, the next x rows are loaded only when the
// current ones have left their registers: both sets do not fit, or (9 to 16
// rows) take 138 registers, one workgroup per CU, where one set takes 122 and
// two fit. Both launches of a call (MI355X, before -> now): 16 rows 7B 39.9 ->
// 36.4 us, 13B 43.1 -> 39.8, 70B 67.7 -> 65.2, d 1024 23.4 -> 20.7; where the
// tiles are fewer than the CUs alike (d_ff 2752 at 12 rows 12.5, 12.7). At 8 rows
// and below both sets fit twice.
template <int TIER, int MT, int NXQ>
__device__ __forceinline__ void bh_next(BhLoads<TIER, MT, NXQ>& next, BhLoads<TIER, MT, NXQ>& cur,
                                        const uint16_t* x, const uint8_t* const* rec, int d, int B,
                                        int grp, uint16_t* s_xw, int lane) {
  constexpr bool late = MT > 1 || NXQ == 4;
  if (!late) next.issue_x(x, d, B, grp, lane);
  next.issue_a(rec, d, grp, lane);
  cur.stage(s_xw, B, lane);
  if (late) {
    __builtin_amdgcn_sched_barrier(0);
    next.issue_x(x, d, B, grp, lane);
  }
}

// NT: 16-column tiles of the batch (1 for B <= 16, 2 for B <= 32); NXQ: x
// loads per lane and group (4 NXQ >= B); MT: 16-row tiles of neurons. s_xw: this wave's x rows (16 NT of
// kBXRow halves; rows from 4 NXQ on are zero from the start). s_sc: the
// tile's gate and up group scales, [16 MT][bh_scale_row(G)] halves. The wave's
// groups are w, w + 8, ...; the loads of the next one go out before the
// current one's arithmetic (past the last group the prefetch re-reads the
// current one, which keeps every load unconditional).
template <int TIER, int MT, int NT, int NXQ, int MA>
__device__ __forceinline__ void bh_tier(int lane, int w, int d, int G, int B, const uint16_t* x,
                                        const uint8_t* const (&rec)[MA], uint16_t* s_xw,
                                        const uint16_t* s_sc, float4v (&acc_g)[MA][NT],
                                        float4v (&acc_u)[MA][NT]) {
  int grp = w;
  if (grp >= G) return;  // wave-uniform
  BhLoads<TIER, MT, NXQ> L0, L1;
  L0.issue_x(x, d, B, grp, lane);
  L0.issue_a(rec, d, grp, lane);
  for (;;) {
    const int g1 = grp + kBHWaves;
    bh_next(L1, L0, x, rec, d, B, g1 < G ? g1 : grp, s_xw, lane);
    bh_compute<TIER, MT, NT>(L0.A, s_xw, s_sc, G, grp, lane, acc_g, acc_u);
    if (g1 >= G) break;
    const int g2 = g1 + kBHWaves;
    bh_next(L0, L1, x, rec, d, B, g2 < G ? g2 : g1, s_xw, lane);
    bh_compute<TIER, MT, NT>(L1.A, s_xw, s_sc, G, g1, lane, acc_g, acc_u);
    if (g2 >= G) break;
    grp = g2;
  }
}

// LDS of ffn_bh_kernel: the waves' x rows, then (after the main loop, over
// the same bytes) the waves' partial results; the tile's gate and up scales
// follow, [16 MA][bh_scale_row(G)] halves (rows padded to 16 bytes; G <= 128).
// MA: the most 16-row tiles of neurons of a workgroup (wide tiles from 17 rows).
template <int NT>
__host__ __device__ constexpr int bh_lds_words() {
  return (kBHWaves * 16 * NT * kBXRow * 2 + 16 * NT * bh_scale_row(128) * 2) / 16;
}
static_assert(kBHWaves * 2 * 16 * 16 * 4 <= kBHWaves * 16 * kBXRow * 2, "partials fit over the x rows");
static_assert(kBHWaves * 2 * 32 * 32 * 4 <= kBHWaves * 32 * kBXRow * 2, "partials fit over the x rows");

template <int NT, int NXQ>
__global__ __launch_bounds__(kBHThreads) void ffn_bh_kernel(
    const uint16_t* __restrict__ x, int d, int B, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ work_slot, const uint32_t* __restrict__ work_mask,
    const uint8_t* __restrict__ slots, int64_t slot_bytes, int cap, int n_slots,
    float* __restrict__ hB) {
  __shared__ uint4 bh_lds[bh_lds_words<NT>()];
  constexpr int MA = NT;
  __shared__ uint32_t s_mask[16 * MA];
  int n3, n2, n1;
  work_counts(counts, cap, n3, n2, n1);
  int tier, item0, nitems;
  const int wide = MA == 2 && ((n3 + 7) >> 3) + ((n2 + 15) >> 4) + ((n1 + 15) >> 4) > kBHWideTiles;
  bh_tile(blockIdx.x, n3, n2, n1, wide, tier, item0, nitems);
  if (nitems <= 0) return;  // workgroup-uniform
  const int G = d >> 7;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint16_t* s_x = reinterpret_cast<uint16_t*>(bh_lds);
  uint16_t* s_xw = s_x + w * 16 * NT * kBXRow;
  uint16_t* s_sc = s_x + kBHWaves * 16 * NT * kBXRow;
  // The tile's slot ids by scalar loads (a wave-uniform range, inside the
  // plan's spare work_slot entries past the list), which do not queue behind
  // other workgroups' vector loads; each lane then picks the ids it needs with
  // branch-free masks.
  int u[16 * MA];
#pragma unroll
  for (int m = 0; m < MA; ++m) {
#pragma unroll
    for (int k = 16 * m; k < 16 * m + 16; ++k) u[k] = n_slots;  // zero slot for padding
    if (m == 0 || wide) {  // workgroup-uniform: tiles of 16 skip the second half's work
#pragma unroll
      for (int k = 16 * m; k < 16 * m + 16; ++k) {
        const int s = __builtin_amdgcn_readfirstlane(work_slot[item0 + k]);
        u[k] = k < nitems && s >= 0 && s < n_slots ? s : n_slots;
      }
    }
  }
  int my_slot[MA];
  uint32_t my_mask[MA];  // stored after the main loop
  const uint8_t* rec[MA];
#pragma unroll
  for (int m = 0; m < MA; ++m) {
    my_slot[m] = n_slots;
    my_mask[m] = 0;
    if (m == 0 || wide) {
      my_slot[m] = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) my_slot[m] |= u[16 * m + k] & -((lane & 15) == k);
      my_mask[m] = work_mask[min(item0 + 16 * m + (lane & 15), cap - 1)];
    }
    rec[m] = slots + (int64_t)my_slot[m] * slot_bytes;
  }
  // the tile's gate and up scales (4 G contiguous bytes per record) into LDS
  if (tier != 3) {
    const int cpr = bh_scale_row(G) / 8;  // 16-byte chunks per row (the last may pass 4 G bytes)
    for (int e = threadIdx.x; e < (16 << wide) * cpr; e += kBHThreads) {
      const int r = e / cpr, c = e - r * cpr;
      int sr = 0;
#pragma unroll
      for (int k = 0; k < 16 * MA; ++k) sr |= u[k] & -(r == k);
      const int64_t sbase = tier == 1 ? 3 * (int64_t)(d >> 1) : 3 * (int64_t)d;
      reinterpret_cast<uint4*>(s_sc)[r * cpr + c] =
          *reinterpret_cast<const uint4*>(slots + (int64_t)sr * slot_bytes + sbase + 16 * c);
    }
  }
  // rows of the wave's x copy that the group loads never write stay zero
  for (int e = lane; e < (16 * NT - 4 * NXQ) * (kBXRow / 8); e += 64)
    reinterpret_cast<uint4*>(s_xw + 4 * NXQ * kBXRow)[e] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  float4v acc_g[MA][NT], acc_u[MA][NT];
#pragma unroll
  for (int m = 0; m < MA; ++m)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      acc_g[m][t] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
      acc_u[m][t] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    }
  // an FP16 tile, also a wide one, is one 16-row tile
  if (tier == 3)
    bh_tier<3, 1, NT, NXQ>(lane, w, d, G, B, x, rec, s_xw, s_sc, acc_g, acc_u);
  else if (tier == 2 && wide)
    bh_tier<2, MA, NT, NXQ>(lane, w, d, G, B, x, rec, s_xw, s_sc, acc_g, acc_u);
  else if (tier == 2)
    bh_tier<2, 1, NT, NXQ>(lane, w, d, G, B, x, rec, s_xw, s_sc, acc_g, acc_u);
  else if (wide)
    bh_tier<1, MA, NT, NXQ>(lane, w, d, G, B, x, rec, s_xw, s_sc, acc_g, acc_u);
  else
    bh_tier<1, 1, NT, NXQ>(lane, w, d, G, B, x, rec, s_xw, s_sc, acc_g, acc_u);
  if (threadIdx.x < 16) {
#pragma unroll
    for (int m = 0; m < MA; ++m)
      s_mask[16 * m + threadIdx.x] = my_slot[m] < n_slots && 16 * m + (int)threadIdx.x < nitems
                                         ? my_mask[m] & (0xffffffffu >> (32 - B))
                                         : 0u;
  }
  __syncthreads();  // every wave is done with its x rows: the partials take their bytes
  // partials of the waves -> LDS: [w][gate/up][row][col]
  float* s_part = reinterpret_cast<float*>(bh_lds);
  const int j = lane >> 4, col = lane & 15;
  constexpr int NC = 16 * NT;
  constexpr int NR = 16 * MA;
#pragma unroll
  for (int m = 0; m < MA; ++m)
    if (m == 0 || wide) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s_part[((w * 2 + 0) * NR + 16 * m + 4 * j + i) * NC + 16 * t + col] = acc_g[m][t][i];
          s_part[((w * 2 + 1) * NR + 16 * m + 4 * j + i) * NC + 16 * t + col] = acc_u[m][t][i];
        }
    }
  __syncthreads();
  // h in the down kernel's layout: 4 items, batch row, next 4 items; zero past
  // the tile's items and the batch
  const int per = (tier == 3 ? 8 : 16) << wide;
  const int local = item0 - (tier == 3 ? 0 : tier == 2 ? n3 : n3 + n2);
  float* hT = hB + (int64_t)(h_base(tier, n3, n2) + local) * h_rows<NT>(B);
  for (int e = threadIdx.x; e < per * NC; e += kBHThreads) {
    const int m = e & 3, b = (e >> 2) % NC, q4 = e / (4 * NC), r = 4 * q4 + m;  // item, batch row
    if (b >= h_rows<NT>(B)) continue;
    float a = 0.0f, u = 0.0f;
    for (int q = 0; q < kBHWaves; ++q) {  // waves in a fixed order
      a += s_part[((q * 2 + 0) * NR + r) * NC + b];
      u += s_part[((q * 2 + 1) * NR + r) * NC + b];
    }
    // zero where row b did not select neuron r (or its slot is invalid); the
    // masks of padding items and the bits past the batch are zero
    hT[(q4 * h_rows<NT>(B) + b) * 4 + m] = (s_mask[r] >> b) & 1u ? silu_mul(a, u) : 0.0f;
  }
}

// ---------------------------------------------------------------------------
// Batched down projection on the matrix cores. The contraction runs over the
// neurons: for one quantization group of 128 columns,
//   y[b][c] += sum_n (h[b][n] s[n]) q[n][c],
// so each neuron's scale folds into the h side and the codes q enter the
// matrix cores exactly, as fp16. The h side is split into an fp16 high and low
// part (two MFMAs per tile) after a power-of-two normalisation per wave and
// batch row, which keeps the products at fp32-level precision whatever the
// magnitudes.
//
// A group's items are cut into steps of 32 of one tier (FP16, INT8, INT4); each
// wave of the group's workgroups takes a run of them, so that most
// waves see one tier (steps dealt in turn, a share of every tier per wave,
// cost a load round trip per tier: 13.2 instead of 12.1 us at batch 8). In a
// step lane (x, j) (x = lane % 16, j = lane / 16) loads the 8
// codes at columns 8x .. 8x + 7 of the group from items 4j .. 4j + 3 and
// 16 + 4j .. 16 + 4j + 3; MFMA e (e = 0..7) takes code e of each, so that its
// 16 result columns are 8x + e, and the lane's A operand is h s of batch row x
// for the same eight items. The next step's loads are in flight while one is
// computed.
//
// What bounds it: with 32 rows the unpacking and the split of h (VALU), with 8
// latency. A wave keeps its sums in registers over all its steps: one
// workgroup per run of 128 .. 512 items, as before, spent most of its time on
// atomics (B x 128 per run and group; 12 M of them at 32 rows of the 70B
// shape) and on empty workgroups of a grid sized for the plan's capacity.
// Measured (MI355X, rocprofv3 kernel time, before -> now): 70B shape at 32 rows
// 105 -> 41.9 us, 7B at 8 / 17 / 32 rows 11.8 / 28.9 / 36.0 -> 10.7 / 17.0 / 20.8.
// What it costs: a wave's second step waits for a memory round trip of its own,
// where the runs before had all of a run in flight. With 2 to 8 rows and two or more
// steps per wave that shows: a call at d 1536 of d_ff 20000 with 4 rows 20.2 -> 21.2
// us, d 1024 of 30000 18.9 -> 19.7, d 2048 of 11008 17.4 -> 18.2. One step per wave
// needs three waves per SIMD and twice the workgroups' atomics: 21.4 us for the 21.2
// (both parts of h in one matrix tile, 168 registers); without that tile 168
// registers spill 222 values.

constexpr int kDMThreads = 256;
constexpr int kDMWaves = kDMThreads / 64;
constexpr int kDMRegions = kDMWaves / 2;  // LDS partial results per workgroup
constexpr int kDMStep = 32;               // items per step
// a wave reads the slot ids of whole steps, two steps ahead
static_assert(2 * kDMStep <= kWorkSlotPad, "steps longer than the plan's spare work_slot entries");
static_assert(kDMStep == kHAlign, "a step's h starts at a multiple of its length");

// The 8 codes of one neuron at the lane's columns: 16 bytes of FP16, 8 of
// INT8, 4 of INT4.
template <int TIER>
struct DmWord {
  typedef uint32_t T;
};
template <>
struct DmWord<3> {
  typedef uint4 T;
};
template <>
struct DmWord<2> {
  typedef uint2 T;
};

__device__ __forceinline__ uint32_t dm_dword(const uint4& v, int q) {
  return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w;
}
__device__ __forceinline__ uint32_t dm_dword(const uint2& v, int q) { return q == 0 ? v.x : v.y; }

// B operands of the 8 MFMAs of a step from the codes of the lane's neurons
// 4j + m (m = 0..3): element m of operand e is code e of neuron m, exact.
// INT8 / INT4 words arrive in offset binary (code + 128 per byte, code + 8
// per nibble); ORing the offset code under fp16 exponent 10 gives 1024 +
// offset code, and one packed subtraction restores the code.
template <int TIER>
__device__ __forceinline__ void dm_operands(const typename DmWord<TIER>::T (&c)[4],
                                            half4v (&bop)[8]) {
  if constexpr (TIER == 3) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;  // halves e & 1 of two words
      const int q = e >> 1;
      bop[e] = h4(__builtin_amdgcn_perm(dm_dword(c[1], q), dm_dword(c[0], q), sel),
                  __builtin_amdgcn_perm(dm_dword(c[3], q), dm_dword(c[2], q), sel));
    }
  } else if constexpr (TIER == 2) {
    const half4v bias = {(_Float16)1152.0f, (_Float16)1152.0f, (_Float16)1152.0f,
                         (_Float16)1152.0f};
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const int q = e >> 2;
      const uint32_t p = e & 3;
      // bytes (neuron 0 code e, neuron 1 code e, neuron 0 code e + 1, neuron 1 code e + 1)
      const uint32_t sel = p | ((4 + p) << 8) | ((p + 1) << 16) | ((5 + p) << 24);
      const uint32_t t01 = __builtin_amdgcn_perm(dm_dword(c[1], q), dm_dword(c[0], q), sel);
      const uint32_t t23 = __builtin_amdgcn_perm(dm_dword(c[3], q), dm_dword(c[2], q), sel);
      bop[e] = h4(__builtin_amdgcn_perm(0x64646464u, t01, 0x04010400u),
                  __builtin_amdgcn_perm(0x64646464u, t23, 0x04010400u)) -
               bias;
      bop[e + 1] = h4(__builtin_amdgcn_perm(0x64646464u, t01, 0x04030402u),
                      __builtin_amdgcn_perm(0x64646464u, t23, 0x04030402u)) -
                   bias;
    }
  } else {
    const half4v bias = {(_Float16)1032.0f, (_Float16)1032.0f, (_Float16)1032.0f,
                         (_Float16)1032.0f};
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t p = e >> 1;
      // bytes (neuron 0 byte p, 0, neuron 1 byte p, 0): codes e (low nibbles) and e + 1 (high)
      const uint32_t sel = p | (0x0cu << 8) | ((4 + p) << 16) | (0x0cu << 24);
      const uint32_t t01 = __builtin_amdgcn_perm(c[1], c[0], sel);
      const uint32_t t23 = __builtin_amdgcn_perm(c[3], c[2], sel);
      bop[e] = h4((t01 & 0x000f000fu) | 0x64006400u, (t23 & 0x000f000fu) | 0x64006400u) - bias;
      bop[e + 1] = h4(((t01 >> 4) & 0x000f000fu) | 0x64006400u,
                      ((t23 >> 4) & 0x000f000fu) | 0x64006400u) -
                   bias;
    }
  }
}

__device__ __forceinline__ uint4 dm_offset(uint4 v) { return v; }
__device__ __forceinline__ uint2 dm_offset(uint2 v) {
  return make_uint2(v.x ^ 0x80808080u, v.y ^ 0x80808080u);
}
__device__ __forceinline__ uint32_t dm_offset(uint32_t v) { return v ^ 0x88888888u; }

// The loads of one step; the slot ids come first (their own struct, one step
// further ahead). Every load is unconditional: items past the tier's last
// read the zero slot and whatever h words follow, and are masked; rows past
// the batch that are not stored repeat its last one (their sums are dropped).
typedef int int4u __attribute__((ext_vector_type(4), aligned(4)));
struct DmSlots {
  int4u s[2];
  __device__ __forceinline__ void issue(const int32_t* __restrict__ ids, int i0, int j) {
    s[0] = *reinterpret_cast<const int4u*>(ids + i0 + 4 * j);
    s[1] = *reinterpret_cast<const int4u*>(ids + i0 + 16 + 4 * j);
  }
};

template <int TIER, int NT>
struct DmLoads {
  typedef typename DmWord<TIER>::T Word;
  Word cw[2][4];
  half2v sc[2][2];  // two fp16 scales per register
  float4v h[2][NT];
  __device__ __forceinline__ void issue(const DmSlots& sl, int i0, int n, const float* __restrict__ hT,
                                        int B, const uint8_t* __restrict__ slots, int64_t slot_bytes,
                                        int n_slots, int64_t doff, int64_t soff, int x, int j) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int s = sl.s[a][m];
        const bool ok = i0 + 16 * a + 4 * j + m < n && s >= 0 && s < n_slots;
        const uint8_t* rec = slots + (int64_t)(ok ? s : n_slots) * slot_bytes;
        cw[a][m] = *reinterpret_cast<const Word*>(rec + doff);
        if (TIER != 3) sc[a][m >> 1][m & 1] = *reinterpret_cast<const _Float16*>(rec + soff);
      }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        h[a][t] = *reinterpret_cast<const float4v*>(
            hT + ((int64_t)((i0 + 16 * a) / 4 + j) * h_rows<NT>(B) +
                  (NT == 1 ? min(x, B - 1) : 16 * t + x)) * 4);
  }
};

// Largest value over the four lanes x, 16 + x, 32 + x, 48 + x, in all of them.
__device__ __forceinline__ uint32_t rows_max(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = max((uint32_t)r[0], (uint32_t)r[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max((uint32_t)q[0], (uint32_t)q[1]);
}

// One step's arithmetic. E: the running exponent of the lane's batch rows (row
// 16 t + x), whose sums are held times 2^E. It only falls, when a step brings a
// row values above 2^15, to put the largest one at 2^11 .. 2^12 (room for larger
// ones later, so that few steps rescale): values 2^-36 of the row's largest and
// below lose bits, which the fp32 sums lose anyway. A step adds to the running
// sums once per part: with one row tile the low parts have sums of their own,
// with two (no registers for that) a step's products are summed first. Adding
// both parts to one sum in turn was 2 us faster at 32 rows of the 70B shape,
// but its error against 64 bits was 7% larger (2.41e-7 instead of 2.26e-7).
template <int TIER, int NT>
__device__ __forceinline__ void dm_step(const DmLoads<TIER, NT>& L, int i0, int n, int j, int (&E)[NT],
                                        float4v (&acc)[2][8]) {
  float a[2][NT][4];
  uint32_t mx[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) mx[t] = 0;
  const bool whole = i0 + kDMStep <= n;  // wave-uniform
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        float v = L.h[q][t][m];
        if (TIER != 3) v *= (float)L.sc[q][m >> 1][m & 1];
        if (!whole && i0 + 16 * q + 4 * j + m >= n) v = 0.0f;
        a[q][t][m] = v;
        mx[t] = max(mx[t], __float_as_uint(v) & 0x7fffffffu);
      }
  int dE[NT];
  bool move = false;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const uint32_t m = rows_max(mx[t]);
    const int e = __builtin_amdgcn_frexp_expf(__uint_as_float(m));
    dE[t] = m > 0 && e + E[t] > 15 ? 12 - e - E[t] : 0;
    move |= dE[t] != 0;
  }
  if (__any(move)) {  // the sums of row 4 j + i are in lane group j, its exponent in lane 4 j + i
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      E[t] += dE[t];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int de = __shfl(dE[t], 4 * j + i);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          acc[t][c][i] = ldexpf(acc[t][c][i], de);
          if (NT == 1) acc[1][c][i] = ldexpf(acc[1][c][i], de);
        }
      }
    }
  }
  half8v ahi[NT], alo[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const float v = ldexpf(a[q][t][m], E[t]);
        const _Float16 hi = (_Float16)v;
        ahi[t][4 * q + m] = hi;
        alo[t][4 * q + m] = (_Float16)(v - (float)hi);
      }
  half4v b0[8], b1[8];
  typename DmWord<TIER>::T c0[4], c1[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    c0[m] = dm_offset(L.cw[0][m]);
    c1[m] = dm_offset(L.cw[1][m]);
  }
  dm_operands<TIER>(c0, b0);
  dm_operands<TIER>(c1, b1);
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const half8v b = h8(b0[c], b1[c]);
    if constexpr (NT == 1) {
      acc[0][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi[0], b, acc[0][c], 0, 0, 0);
      acc[1][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(alo[0], b, acc[1][c], 0, 0, 0);
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float4v p = {0.0f, 0.0f, 0.0f, 0.0f};
        p = __builtin_amdgcn_mfma_f32_16x16x32_f16(alo[t], b, p, 0, 0, 0);
        p = __builtin_amdgcn_mfma_f32_16x16x32_f16(ahi[t], b, p, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[t][c][i] += p[i];
      }
    }
  }
}

// A wave's steps [first, end) of one tier's n items (ids: their slots, hT:
// their h; sl: the first step's slots). Past the last step the prefetches
// re-read the first.
template <int TIER, int NT>
__device__ __forceinline__ void dm_tier(DmSlots sl, int first, int end, int n,
                                        const int32_t* __restrict__ ids,
                                        const float* __restrict__ hT, int B, int grp, int d, int G,
                                        const uint8_t* __restrict__ slots, int64_t slot_bytes,
                                        int n_slots, int (&E)[NT], float4v (&acc)[2][8]) {
  if (first >= end) return;  // wave-uniform
  const int lane = threadIdx.x & 63, x = lane & 15, j = lane >> 4;
  // byte offsets in a record: the lane's 8 down codes of group grp, and the group's down scale
  const int64_t doff = TIER == 3   ? 4 * (int64_t)d + 2 * (128 * grp + 8 * x)
                       : TIER == 2 ? 2 * (int64_t)d + 128 * grp + 8 * x
                                   : (int64_t)d + 64 * grp + 4 * x;
  const int64_t soff = (TIER == 1 ? 3 * (int64_t)(d >> 1) : 3 * (int64_t)d) + 4 * G + 2 * grp;
  auto at = [&](int st) { return kDMStep * (st < end ? st : first); };
  DmLoads<TIER, NT> L0, L1;
  auto load = [&](DmLoads<TIER, NT>& L, int i0) {
    L.issue(sl, i0, n, hT, B, slots, slot_bytes, n_slots, doff, soff, x, j);
  };
  load(L0, at(first));
  sl.issue(ids, at(first + 1), j);
  for (int st = first;;) {
    load(L1, at(st + 1));
    sl.issue(ids, at(st + 2), j);
    __builtin_amdgcn_sched_barrier(0);  // the loads go out before the arithmetic
    dm_step<TIER, NT>(L0, at(st), n, j, E, acc);
    if (++st >= end) break;
    load(L0, at(st + 1));
    sl.issue(ids, at(st + 2), j);
    __builtin_amdgcn_sched_barrier(0);
    dm_step<TIER, NT>(L1, at(st), n, j, E, acc);
    if (++st >= end) break;
  }
}

// NT: 16-row tiles of the batch (1 for B <= 16, 2 for B <= 32).
// blockIdx.x = group + G * (workgroup of the group).
template <int NT>
__global__ __launch_bounds__(kDMThreads, 2) void ffn_bdn_kernel(
    int d, int B, const int32_t* __restrict__ counts, const int32_t* __restrict__ work_slot,
    const float* __restrict__ hB, const uint8_t* __restrict__ slots, int64_t slot_bytes, int cap,
    int n_slots, float* __restrict__ y) {
  constexpr int kRow = 132;  // 128 columns (in the order 16 e + x) and a pad against bank conflicts
  // [region][batch row][column]: the first half of the waves store their partial
  // rows, then the others add theirs to them, so that every LDS word has one
  // writer at a time (LDS float atomics are slow)
  __shared__ float s_y[kDMRegions][16 * NT][kRow];
  const int G = d >> 7;
  int grp = blockIdx.x % G;
  // Groups 2i and 2i + 1 of a workgroup go to ids 8 apart: one XCD (ids are
  // dealt to the 8 XCDs in turn) and about the same start, so that a 128-byte
  // line of INT4 codes, which holds both groups of a neuron, is fetched into
  // that XCD's L2 once.
  if ((G & 15) == 0) {
    const int p = grp & 15;
    grp = (grp & ~15) + 2 * (p & 7) + (p >> 3);
  }
  int n3, n2, n1;
  work_counts(counts, cap, n3, n2, n1);
  const int S3 = (n3 + kDMStep - 1) / kDMStep, S2 = (n2 + kDMStep - 1) / kDMStep;
  const int S1 = (n1 + kDMStep - 1) / kDMStep;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // All the group's waves share its steps equally, or, where that is at most two
  // steps each, as few of them as have one (two) each: the workgroups left over
  // have none, and no atomics. Both launches of a call (MI355X, shared equally ->
  // this): d 2048 of d_ff 5632 at 2 / 32 rows 13.2 / 27.6 -> 12.5 / 25.3 us, d 1024
  // of 11008 at 32 rows 32.2 -> 30.1, d 4096 of 4000 28.4 -> 27.1. Longer equal runs
  // on fewer waves leave SIMDs idle (d 2048, 24 rows, 2.06 steps each or 3 on 88 of
  // 128 waves: 35.8, 36.7; the 70B shape at 32 rows, 14.4 or 15: 102.3, 104.9).
  const int wg = blockIdx.x / G, ST = S3 + S2 + S1;
  int W = (gridDim.x / G) * kDMWaves;
  if (ST <= 2 * W) W = ST <= W ? ST : (ST + 1) / 2;
  if (wg * kDMWaves >= W) return;  // no steps (workgroup-uniform)
  const int gw = min(wg * kDMWaves + w, W);  // W: no steps
  const int lo = (int)((uint32_t)(ST * gw) / (uint32_t)W);
  const int hi = (int)((uint32_t)(ST * min(gw + 1, W)) / (uint32_t)W);
  const int lane = threadIdx.x & 63, x = lane & 15, j = lane >> 4;
  // the wave's run of the group's steps, by tier
  const int st3 = lo, st2 = max(lo - S3, 0), st1 = max(lo - S3 - S2, 0);
  const int en3 = min(hi, S3), en2 = min(hi - S3, S2), en1 = hi - S3 - S2;
  const int32_t *ids2 = work_slot + n3, *ids1 = ids2 + n2;
  DmSlots sl3, sl2, sl1;
  sl3.issue(work_slot, kDMStep * min(st3, S3), j);
  sl2.issue(ids2, kDMStep * min(st2, S2), j);
  sl1.issue(ids1, kDMStep * min(st1, S1), j);
  float4v acc[2][8];  // sums of the row tiles; of the high and low parts when there is one tile
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[t][e] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
  int E[NT];  // above every exponent until a row's first value sets it
#pragma unroll
  for (int t = 0; t < NT; ++t) E[t] = 1 << 10;
  dm_tier<3, NT>(sl3, st3, en3, n3, work_slot, hB, B, grp, d, G, slots, slot_bytes, n_slots, E, acc);
  const int64_t rows = h_rows<NT>(B);
  dm_tier<2, NT>(sl2, st2, en2, n2, ids2, hB + h_base(2, n3, n2) * rows, B, grp, d, G, slots,
                 slot_bytes, n_slots, E, acc);
  dm_tier<1, NT>(sl1, st1, en1, n1, ids1, hB + h_base(1, n3, n2) * rows, B, grp, d, G, slots,
                 slot_bytes, n_slots, E, acc);
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int er = -__shfl(E[t], 4 * j + i);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        acc[t][e][i] = ldexpf(NT == 1 ? acc[0][e][i] + acc[1][e][i] : acc[t][e][i], er);
    }
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    if (w / kDMRegions == pass) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = 16 * t + 4 * j + i;
          if (row < B) {
            float* dst = &s_y[w % kDMRegions][row][x];
#pragma unroll
            for (int e = 0; e < 8; ++e) dst[16 * e] = pass ? dst[16 * e] + acc[t][e][i] : acc[t][e][i];
          }
        }
    }
    __syncthreads();
  }
  for (int q = threadIdx.x; q < B * 128; q += kDMThreads) {
    const int b = q >> 7, c = q & 127;
    float v = 0.0f;
#pragma unroll
    for (int r = 0; r < kDMRegions; ++r) v += s_y[r][b][16 * (c & 7) + (c >> 3)];
    atomicAdd(y + (int64_t)b * d + 128 * grp + c, v);
  }
}

// One round of workgroups, two per CU (the registers' limit), and so one set of
// atomics per two waves of a SIMD: 512 on the 256 CUs, or fewer where the plan's
// capacity has no step for them. 256 / 512 / 1024 workgroups, both launches of a
// call (MI355X): 7B at 8 rows 26.9 / 26.3 / 30.7 us, 70B shape at 32 rows 107.1 /
// 104.4 / 109.6. With at most 8 groups 512 are 64 or more that add into the same
// columns, and 256 are faster: d 1024 of d_ff 30000 at 8 / 32 rows 23.3 / 46.5 ->
// 22.9 / 42.7 us, d 256 of 60000 at 8 rows 34.1 -> 30.9 (at 12 groups, d 1536 of
// 20000 at 4 rows, fewer are slower: 21.3 -> 22.0).
constexpr int kDMGrid = 512;
constexpr int kDMFewGroups = 8;
static void launch_bdn(int d, int batch, int cap, hipStream_t stream, const int32_t* counts,
                       const int32_t* work_slot, const float* hB, const uint8_t* slots,
                       int64_t sb, int n_slots, float* y) {
  const int G = d >> 7;
  const int most = (cap / kDMStep + 3 + kDMWaves - 1) / kDMWaves;
  const int grid = G <= kDMFewGroups ? kDMGrid / 2 : kDMGrid;
  int per = grid > G ? grid / G : 1;
  if (per > most) per = most;
  if (batch <= 16)
    hipLaunchKernelGGL(ffn_bdn_kernel<1>, dim3(G * per), dim3(kDMThreads), 0, stream, d, batch,
                       counts, work_slot, hB, slots, sb, cap, n_slots, y);
  else
    hipLaunchKernelGGL(ffn_bdn_kernel<2>, dim3(G * per), dim3(kDMThreads), 0, stream, d, batch,
                       counts, work_slot, hB, slots, sb, cap, n_slots, y);
}

hipError_t launch_ffn_batch(m2c_layer* L, const uint16_t* x, int batch, const uint8_t* plan,
                            float* y, hipStream_t stream) {
  const int d = L->desc.d_model;
  const m2c_plan_layout& lay = L->layout;
  const int32_t* counts = reinterpret_cast<const int32_t*>(plan + lay.counts);
  const int32_t* work_slot = reinterpret_cast<const int32_t*>(plan + lay.work_slot);
  const uint32_t* work_mask = reinterpret_cast<const uint32_t*>(plan + lay.work_mask);
  const int64_t sb = L->info.slot_bytes;
  const int n_slots = L->desc.cache_slots + L->S;
  const int cap = L->cap;
  if (cap <= 0) return hipSuccess;
  float* hB = reinterpret_cast<float*>(L->ab);  // h_base() says how it is laid out
  // tiles of 8 (FP16) and 16 items: at most ceil(cap/8) + 2 for any split into tiers
  const int tiles = (cap + 7) / 8 + 2;
  if (batch <= 8) {
    hipLaunchKernelGGL((ffn_bh_kernel<1, 2>), dim3(tiles), dim3(kBHThreads), 0, stream, x, d,
                       batch, counts, work_slot, work_mask, L->slots, sb, cap, n_slots, hB);
  } else if (batch <= 16) {
    hipLaunchKernelGGL((ffn_bh_kernel<1, 4>), dim3(tiles), dim3(kBHThreads), 0, stream, x, d,
                       batch, counts, work_slot, work_mask, L->slots, sb, cap, n_slots, hB);
  } else {
    // at most kBHWideTiles tiles, or wide ones
    const int some = tiles < kBHWideTiles ? tiles : kBHWideTiles;
    const int most = some > cap / 16 + 3 ? some : cap / 16 + 3;
    hipLaunchKernelGGL((ffn_bh_kernel<2, 8>), dim3(most), dim3(kBHThreads), 0, stream, x, d,
                       batch, counts, work_slot, work_mask, L->slots, sb, cap, n_slots, hB);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_bdn(d, batch, cap, stream, counts, work_slot, hB, L->slots, sb, n_slots, y);
  return hipGetLastError();
}

}  // namespace m2c
