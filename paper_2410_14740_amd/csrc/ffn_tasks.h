// Task geometry of the one-launch batch-1 FFN (k_ffn_fused.hip): the task
// sizes, the launch order of the six task regions, the task of a workgroup
// id, and the task table the cache plan writes for it. Shared by the FFN
// kernel and the plan kernel that writes the table.
#pragma once

#include "ffn_device.h"

namespace m2c {

#ifndef M2C_FFN_THREADS
#define M2C_FFN_THREADS 256
#endif
constexpr int kFT = M2C_FFN_THREADS;     // threads per workgroup
constexpr int kFWaves = kFT / 64;
constexpr int kFL = 8;                   // 16-byte data loads per lane and task
constexpr int kFSW = 512;                // down tasks: output columns per slice
constexpr int kFLPN = kFSW / 32;         // lanes per neuron row of a slice
constexpr int kFNPR = kFT / kFLPN;       // neurons per round of a down task
constexpr int kFMaxItems = kFL * kFNPR;  // most work items of one task (INT4 down)
// Rounds of kFNPR neurons per down task by tier (INT4, INT8, FP16): one
// load per lane and round for INT4, two for INT8, four for FP16.
constexpr int kDnRounds1 = kFL, kDnRounds2 = kFL / 2, kDnRounds3 = kFL / 4;
constexpr int kFSpin = 1 << 16;          // polls of one h word before giving up
constexpr float kTwo24 = 16777216.0f;
static_assert(kFMaxItems <= kFT, "one slot id / h word per thread");
// The task table in a plan: task count and zero slot (16 bytes), one 32-byte
// header per workgroup, then kTaskIds slot ids per workgroup from a 256-byte
// boundary.
constexpr int kTaskIds = kFL * kFNPR;
inline int64_t task_ids_offset(int grid) { return (16 + 32 * (int64_t)grid + 255) / 256 * 256; }
static_assert(kFLPN == 16, "the fold pairs lanes 16 and 32 apart");
static_assert(kFSW % kFT == 0, "the cross-wave fold gives each thread whole columns of the slice");

struct FMap {
  int n3, n2, n1;  // work items by tier
  int w1, w2, w3;  // h tasks by tier (INT4, INT8, FP16)
  int n_slices;
  int e[6];        // ends of the six task regions in launch order
};

struct FTask {
  int kind;  // 0 none, 1 h, 2 down
  int tier;
  int lo, hi;
  int slice;
};

// The task table of a plan as the plan kernel writes it; grid 0: none.
// upt: units per h task, kFWaves * kFL / K for K 16-byte loads per lane and
// unit (a unit is d bytes of a neuron's gate and up rows).
struct TaskTable {
  int32_t* tasks;
  int32_t* task_ids;
  int d, grid, upt;
};

// Launch order of the six task regions: (kind, tier) per region.
constexpr int kOrderKind[6] = {1, 1, 1, 2, 2, 2};
constexpr int kOrderTier[6] = {1, 2, 3, 1, 2, 3};

constexpr int kLogFWaves = 2, kLogDn3 = 5;
static_assert(kFWaves == 1 << kLogFWaves && kDnRounds3 * kFNPR == 1 << kLogDn3 &&
                  kDnRounds2 == 2 * kDnRounds3 && kDnRounds1 == 2 * kDnRounds2,
              "the table writer shifts");

// Neurons per down task.
__device__ __forceinline__ int dn_items(int tier) {
  return (tier == 1 ? kDnRounds1 : tier == 2 ? kDnRounds2 : kDnRounds3) * kFNPR;
}

__device__ __forceinline__ FMap make_map(int n3, int n2, int n1, int d, int upt) {
  FMap m;
  m.n3 = n3;
  m.n2 = n2;
  m.n1 = n1;
  m.w1 = (n1 + upt - 1) / upt;
  m.w2 = (n2 + upt / 2 - 1) / (upt / 2);
  m.w3 = (n3 + upt / 4 - 1) / (upt / 4);
  m.n_slices = (d + kFSW - 1) / kFSW;
  const int u1 = (n1 + dn_items(1) - 1) / dn_items(1);
  const int u2 = (n2 + dn_items(2) - 1) / dn_items(2);
  const int u3 = (n3 + dn_items(3) - 1) / dn_items(3);
  int end = 0;
#pragma unroll
  for (int r = 0; r < 6; ++r) {
    const int tr = kOrderTier[r];
    end += kOrderKind[r] == 1 ? (tr == 1 ? m.w1 : tr == 2 ? m.w2 : m.w3)
                              : (tr == 1 ? u1 : tr == 2 ? u2 : u3) * m.n_slices;
    m.e[r] = end;
  }
  return m;
}

// First task of the region of a kind and tier.
template <int KIND>
__device__ __forceinline__ int region_start(const FMap& m, int tier) {
  int start = 0;
#pragma unroll
  for (int r = 1; r < 6; ++r)
    if (kOrderKind[r] == KIND && kOrderTier[r] == tier) start = m.e[r - 1];
  return start;
}

// Down tasks: runs of a tier in blocks of 8, slice-major within a block:
// workgroup b runs on XCD b % 8, so all slices of a run (which read the same
// scale lines of the run's records) land on one XCD and its L2.
// Task t in launch order. Work items are tier-major in the plan: FP16, INT8,
// INT4.
__device__ __forceinline__ FTask decode(const FMap& m, int t, int upt) {
  FTask k;
  k.kind = 0;
  k.tier = 1;
  k.lo = k.hi = 0;
  k.slice = 0;
  // region by comparisons (no indexed array: it would live in scratch memory)
  int kind = 0, tier = 1, start = 0;
#pragma unroll
  for (int r = 5; r >= 0; --r) {
    const int lo_r = r ? m.e[r - 1] : 0;
    if (t >= lo_r && t < m.e[r]) {
      kind = kOrderKind[r];
      tier = kOrderTier[r];
      start = lo_r;
    }
  }
  if (kind == 0) return k;
  const int q = t - start;
  k.tier = tier;
  // by value (a select between fields would index a stack copy of the map)
  const int i1 = tier == 1, i2 = tier == 2, i3 = tier == 3;
  const int base = i1 * (m.n3 + m.n2) + i2 * m.n3;
  const int n = i1 * m.n1 + i2 * m.n2 + i3 * m.n3;
  if (kind == 1) {
    k.kind = 1;
    const int per = tier == 1 ? upt : tier == 2 ? upt / 2 : upt / 4;
    k.lo = base + per * q;
    k.hi = base + min(per * (q + 1), n);
  } else {
    k.kind = 2;
    const int per = dn_items(tier);
    const int nr = (n + per - 1) / per;
    const int blk = q / (8 * m.n_slices);
    const int within = q - blk * 8 * m.n_slices;
    const int nb = min(8, nr - 8 * blk);
    k.slice = within / nb;
    const int run = 8 * blk + (within - k.slice * nb);
    k.lo = base + per * run;
    k.hi = base + min(per * (run + 1), n);
  }
  return k;
}

// The table: the task count and the zero slot's byte offset; per task t a
// 32-byte header {kind | tier << 8, first work item, items, slice, then the
// tier pool's byte offset, first slot id, slot count, record stride}; and the
// slot ids in the order the FFN's waves read them (a down task's items in
// work order; an h task's units at entry (uw / 4) kFNPR + 4 w + uw % 4 for
// unit w UW + uw, UW units per wave).
__device__ __forceinline__ void write_task_count(const TaskTable& tt, const SlotMap& map, int n) {
  tt.tasks[0] = n;
  tt.tasks[1] = (int32_t)map.zero;
}

__device__ __forceinline__ void write_task_header(const TaskTable& tt, const FMap& m,
                                                  const SlotMap& map, int t) {
  const FTask k = decode(m, t, tt.upt);
  const int tr = k.tier;
  int4* h = reinterpret_cast<int4*>(tt.tasks + 4) + 2 * t;
  h[0] = make_int4(k.kind | (tr << 8), k.lo, k.hi - k.lo, k.slice);
  h[1] = make_int4((int)(tr == 3   ? map.base[3]
                         : tr == 2 ? map.base[2]
                                   : map.base[1]),
                   tr == 3   ? map.first[3]
                   : tr == 2 ? map.first[2]
                             : map.first[1],
                   tr == 3   ? map.count[3]
                   : tr == 2 ? map.count[2]
                             : map.count[1],
                   (int)(tr == 3   ? map.stride[3]
                         : tr == 2 ? map.stride[2]
                                   : map.stride[1]));
}

// Every entry of one work item, the i-th of its tier, in slot `slot`: its
// units in its h task, and its place in the down task of every slice.
__device__ __forceinline__ void write_task_items(const TaskTable& tt, const FMap& m, int tier,
                                                 int i, int slot) {
  // every size is a power of two: shifts
  const int lupi = tier == 3 ? 2 : tier == 2 ? 1 : 0;
  const int lupt = 31 - __builtin_clz(tt.upt), luw = lupt - kLogFWaves;  // units per wave
  const int lper = lupt - lupi;                                          // items per h task
  const int th = region_start<1>(m, tier) + (i >> lper);
  if (th < tt.grid) {
    int32_t* out = tt.task_ids + (int64_t)th * kTaskIds;
    const int unit0 = (i & ((1 << lper) - 1)) << lupi;
    for (int v = 0; v < (1 << lupi); ++v) {
      const int w = (unit0 + v) >> luw, uw = (unit0 + v) & ((1 << luw) - 1);
      out[(uw >> 2) * kFNPR + 4 * w + (uw & 3)] = slot;
    }
  }
  const int n = tier == 3 ? m.n3 : tier == 2 ? m.n2 : m.n1;
  const int ld = tier == 3 ? kLogDn3 : tier == 2 ? kLogDn3 + 1 : kLogDn3 + 2;  // items per down task
  const int run = i >> ld, blk = run >> 3;
  const int nb = min(8, ((n + (1 << ld) - 1) >> ld) - 8 * blk);
  int t = region_start<2>(m, tier) + blk * 8 * m.n_slices + (run & 7);
  int32_t* out = tt.task_ids + (i & ((1 << ld) - 1));
  for (int s = 0; s < m.n_slices && t < tt.grid; ++s, t += nb) out[(int64_t)t * kTaskIds] = slot;
}

// The task table of a layer's plan buffer (k_ffn_fused.hip).
TaskTable plan_task_table(const m2c_layer* L, uint8_t* plan);

}  // namespace m2c
