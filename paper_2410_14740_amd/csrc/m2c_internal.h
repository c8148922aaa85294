// Internal definitions of the m2c HIP library (gfx950). Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "m2c.h"

namespace m2c {

// Bits of the per-layer device status word, reported (and cleared) by
// m2c_layer_stats.
constexpr int M2C_STATUS_PLAN_OVERFLOW = 2;  // a tier map had more active neurons than cap
constexpr int M2C_STATUS_FFN_WAIT = 4;      // a sparse FFN gave up waiting for an h value
// Spare entries after the plan's work_slot array: the batched FFN reads slot
// ids past the last item, in whole tiles (up to 32 items) and whole steps of 32,
// one step ahead. The number is part of the plan's layout in m2c.h.
constexpr int kWorkSlotPad = 512;

// ---------------------------------------------------------------------------
// Host-side layer object

// Pinned host-DRAM neuron store: every neuron at all three tiers, record
// stores back to back per tier. Shared (refcounted) between layers created
// with m2c_layer_create_shared.
struct Store {
  int refs = 1;
  int device = 0;
  int d_model = 0, d_ff = 0;
  uint8_t* host[4] = {nullptr, nullptr, nullptr, nullptr};  // by tier, [1..3]
  int64_t stride[4] = {0, 0, 0, 0};
  int64_t bytes = 0;
};

// Words of the plan's device state: a serial number per plan (the stamp of the
// slots it touches; kept on the device, so a replayed graph advances it), which
// of the two LRU orders is current, and the slots of each pool that were ever
// filled.
enum { kPlanSerial, kPlanCur, kPlanFilled, kPlanWords = kPlanFilled + 3 };

// Per-layer device state of the plan, the fill and the FFN. With tier pools
// the tables of the pools lie back to back (FP16, INT8, INT4) over the C
// resident slots; LRU orders and places hold such concatenated slot ids.
struct DeviceState {
  int32_t* slot_of = nullptr;    // [d_ff] slot in its pool or -1 (tier pools: one table per pool)
  int32_t* slot_key = nullptr;   // [C]
  uint8_t* slot_tier = nullptr;  // [C]
  int32_t* slot_last = nullptr;  // [C]
  int32_t* lru = nullptr;        // [2][C] slots by (last use, slot), current and next
  int32_t* lru_pos = nullptr;    // [2][C] place of each slot in that order
  int32_t* touch_slot = nullptr; // [C] serial of the last plan that touched the slot
  int32_t* touch_pos = nullptr;  // [C] the same by place in the order that plan read
  int32_t* plan_state = nullptr; // [kPlanWords]
  int32_t* plan_copy = nullptr;  // [kPlanWords] plan_state as the running plan found it
  uint32_t* info = nullptr;      // [d_ff] plan scratch: the neuron's word
  uint32_t* masks = nullptr;     // [d_ff] plan scratch: row masks (max_batch > 1)
  int32_t* chunk_counts = nullptr;  // plan scratch: counts per field and chunk of neurons
  int32_t* slot_rec = nullptr;   // [C + S] record a slot's bytes hold, 4 * neuron + tier (-1: none), kept by the fill
  unsigned long long* stats = nullptr;  // [16] cumulative counters
  int32_t* status = nullptr;           // [1] M2C_STATUS_* bits set by kernels
  unsigned long long* ffn_gen = nullptr;  // [ffn_grid] per-workgroup call counters of the one-launch FFN
  unsigned long long* ffn_hw = nullptr;   // [cap] (call tag, h) words of the one-launch FFN
};

// Where the record in a slot starts: a slot of tier t's pool at global id s,
// first[t] <= s < first[t] + count[t], holds its record at byte
// base[t] + (s - first[t]) * stride[t] of the arena; `zero` is the all-zero
// padding slot (where every id outside the tier's pool points). Without tier
// pools every tier maps with base 0, first 0, count C + S, stride slot_bytes.
struct SlotMap {
  uint32_t base[4];
  int32_t first[4];
  int32_t count[4];
  uint32_t stride[4];
  uint32_t zero;
};

}  // namespace m2c

struct m2c_layer {
  m2c_layer_desc desc;
  int S = 0;    // staging slots
  int cap = 0;  // plan capacity
  int num_cus = 0;
  m2c::Store* store = nullptr;
  m2c_layer_info info;
  m2c_plan_layout layout;
  // device memory (one allocation, carved)
  uint8_t* dev_base = nullptr;
  int64_t dev_bytes = 0;
  uint16_t* pred_a = nullptr;  // [r][d]
  uint16_t* pred_b = nullptr;  // [d_ff][r]
  float* bias = nullptr;       // [d_ff] or null
  float* z = nullptr;          // [max_batch][r]
  float* scores = nullptr;     // [max_batch][d_ff]
  uint8_t* slots = nullptr;    // [C+S][slot_bytes]
  float2* ab = nullptr;        // [4 * cap] partial gate/up dot products per FFN unit
  float* y_part = nullptr;     // [ffn_groups][d] down-projection partial rows
  int ffn_groups = 1;
  int ffn_grid = 0;  // workgroups of the one-launch FFN
  m2c::DeviceState st;
  int64_t last_step = -1;
  int ffn_withhold = 0;  // test support: > 0 = h words withheld, polls before giving up
  m2c_dram* dram = nullptr;  // records come from this DRAM cache (store is null)
  int dram_index = -1;
  // per-tier record arena (M2C_FLAG_TIER_POOLS)
  bool pools = false;
  int pool_C[4] = {0, 0, 0, 0};   // resident slots per tier
  int pool_S[4] = {0, 0, 0, 0};   // staging slots per tier
  int pool_rf[4] = {0, 0, 0, 0};  // first resident table index of the pool
  m2c::SlotMap map;               // slot id -> byte offset, by tier
  int64_t arena_bytes = 0;        // pools + zero slot
};

namespace m2c {

// ---------------------------------------------------------------------------
// Host-side helpers of the entry points (m2c_api.hip)

// Sets the thread's error message (m2c_last_error) and returns `code`.
m2c_status api_fail(m2c_status code, const char* fmt, ...);
// The host-side argument checks of m2c_predict_rank.
m2c_status check_predict_args(const m2c_layer* L, const uint16_t* x, int batch, int k, int n_fp16,
                              int n_int8, const uint8_t* tier_map);

// SSD -> DRAM tier (dram_cache.hip)
m2c_status dram_acquire(m2c_dram* D, int layer, const uint8_t** data, int* slot);
void dram_release(m2c_dram* D, int slot, hipEvent_t reader);
hipEvent_t dram_event(m2c_dram* D);
int64_t dram_layer_bytes(const m2c_dram* D);
int dram_layers(const m2c_dram* D);
int dram_device(const m2c_dram* D);
bool dram_pinned(const m2c_dram* D);
void dram_ref(m2c_dram* D, int delta);

// ---------------------------------------------------------------------------
// Launchers (one per kernel file). All enqueue on `stream` and return the
// hipError_t of the launch.

hipError_t launch_transpose_u16(const uint16_t* in, uint16_t* out, int rows, int cols,
                                hipStream_t stream);
hipError_t launch_quantize_records(const uint16_t* wg, const uint16_t* wu, const uint16_t* wdT,
                                   int d, int i0, int n, uint8_t* r16, int64_t st16, uint8_t* r8,
                                   int64_t st8, uint8_t* r4, int64_t st4, hipStream_t stream);
hipError_t launch_predict(const m2c_layer* L, const uint16_t* x, int batch, float* z,
                          float* scores, hipStream_t stream);
hipError_t launch_select(const float* scores, int batch, int d_ff, int k, int n16, int n8,
                         uint8_t* tier_map, hipStream_t stream);
hipError_t launch_plan(m2c_layer* L, const uint8_t* tier_map, int batch, int step, uint8_t* plan,
                       hipStream_t stream);
hipError_t launch_reset(m2c_layer* L, hipStream_t stream);
hipError_t launch_fill(const m2c_layer* L, const uint8_t* plan, const uint8_t* const host[4],
                       hipStream_t stream);
hipError_t launch_poison_fill_slots(const m2c_layer* L, const uint8_t* plan, hipStream_t stream);
// The state with the slot tables of tier t's pool (M2C_FLAG_TIER_POOLS).
DeviceState pool_state(const m2c_layer* L, int t);
hipError_t launch_ffn(m2c_layer* L, const uint16_t* x, int batch, const uint8_t* plan, float* y,
                      hipStream_t stream);
hipError_t launch_ffn_batch(m2c_layer* L, const uint16_t* x, int batch, const uint8_t* plan,
                            float* y, hipStream_t stream);
hipError_t launch_ffn_split(m2c_layer* L, const uint16_t* x, const uint8_t* plan, float* y,
                            hipStream_t stream);
bool ffn_fused_supported(const m2c_layer* L);
int ffn_fused_grid(int d_model, int cap);  // workgroups (and gen counters) of the one-launch FFN
// The one-launch FFN's task table in a plan: whether the layer's plans carry
// one (batch-1 FFN calls use that kernel) and its bytes for a grid.
bool ffn_tasks_used(const m2c_layer* L);
int ffn_loads_per_unit(int d);  // K of the one-launch FFN: 16-byte loads per lane and unit
int64_t ffn_task_table_bytes(int grid);
hipError_t launch_ffn_fused(m2c_layer* L, const uint16_t* x, const uint8_t* plan, float* y,
                            hipStream_t stream);

// ---------------------------------------------------------------------------
// Device helpers shared by the kernels

__device__ __forceinline__ float h2f(uint16_t b) {
  return (float)__builtin_bit_cast(_Float16, b);
}

__device__ __forceinline__ uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace m2c
