// Cache plan: resolves one step's active neurons against the layer's
// isolated HBM cache unit (Sec. 5.3) with LRU replacement of neurons
// (Sec. 1, Sec. 6.4): the single arena or the per-tier pools, any d_ff, one
// or more batch rows.
//
// Two launches, each over chunks of 256 neurons:
//
//   plan_classify_kernel  step tier and row mask of every neuron, the pool
//       that serves it and its slot there: HIT, REFILL (another tier in its
//       slot) or NEW. Writes one word per neuron, the chunk's counts, and
//       stamps the slots it touches, by slot and by place in the LRU order.
//   plan_place_kernel  every output, at its final place. Ranks in id order
//       are the counts of the chunks before plus wave ballots. The victims of
//       the NEW neurons are the unstamped slots in LRU order: every workgroup
//       ranks the order for itself (a few coalesced loads and ballots per
//       thread, cheaper than a launch to share it; of a long order only what
//       it needs) and keeps those its own NEW neurons take. The workgroups past the neuron chunks write the
//       new LRU order: the unstamped slots beyond the victims in their old
//       order, then every slot used this step in slot order (they share the
//       largest last use), which keeps it sorted by (last use, slot).
//
// With pools, the three pools are planned as one: their slots and LRU orders
// lie back to back (FP16, INT8, INT4), and ranks count from each pool's start.
//
// What bounds it: latency -- two launches, two dependent memory round trips
// in each, and block-wide ranks -- not bytes: about 13 d_ff + 30 C + 60 |R| from
// HBM, and from L2 12 C more of the LRU order for each of the d_ff / 256 + C / 1024
// workgroups (10 MB at d_ff 28672 with 7000 slots). Of more than 8192 slots that
// read is a sweep at a time, and grows with d_ff C: see plan_long.
// One workgroup doing the whole step was bound by one CU's instruction issue
// and a dozen dependent round trips, and the pools took two launches more.
// Measured (MI355X, rocprofv3 kernel time, all plan launches and the FFN's
// task table, before -> now): d_ff 2752 29.4 -> 10.9 us, 11008 40.1 -> 11.4 (batch
// 8: 62.5 -> 10.9), 40000 99.5 -> 12.6, 28672 with pools 39.0 -> 15.9.
#include "ffn_tasks.h"
#include "m2c_internal.h"
#include "wave_ops.h"

namespace m2c {

// A chunk has 256 neurons, one wave per SIMD, because a CU issues an
// instruction of 16 waves in the time of 16 (with chunks of 1024, one neuron
// per thread, the place kernel took 9.7 instead of 8.0 us at 7B and 13.7
// instead of 12.5 for the 70B pools); the place kernel's other waves help to
// rank the LRU order and write the task headers.
constexpr int kPC = 256;        // neurons per chunk, threads of the classify kernel
constexpr int kPCW = kPC / 64;
constexpr int kPT = 1024;       // threads of the place kernel
constexpr int kPW = kPT / 64;
constexpr int kPRounds = 8;    // LRU entries a thread ranks per sweep

// Counts of a chunk: required neurons and fills by tier, NEW neurons, fills
// made from the slot's FP16 record by tier.
enum PlanField { kR3, kR2, kR1, kF3, kF2, kF1, kNew, kD2, kD1, kPFields };
static_assert(kPFields <= kPW, "one wave sums each field");
static_assert(kPCW == 4, "the chunk's counts by wave are a uint4");

// A neuron's word: step tier | code << 2 (0 NEW, 1 HIT, 2 REFILL) | tier its
// slot held << 4 | slot in its pool << 8.
__device__ __forceinline__ uint32_t pack_info(int t, int code, int old, int slot) {
  return (uint32_t)t | ((uint32_t)code << 2) | ((uint32_t)old << 4) | ((uint32_t)slot << 8);
}

struct PlanPtrs {
  int32_t* counts;
  int32_t* req_ids;
  uint8_t* req_tier;
  uint8_t* req_hit;
  int32_t* req_slot;
  uint32_t* req_mask;
  int32_t* fill_ids;
  uint8_t* fill_tier;
  int32_t* fill_slot;
  uint8_t* fill_from;
  int32_t* evicted_ids;
  int32_t* work_slot;
  uint32_t* work_mask;
};

// The pools by index (0 FP16, 1 INT8, 2 INT4; without tier pools only 0, the
// whole unit): resident slots, first of them in the concatenated tables,
// first global slot id.
struct PoolGeom {
  int C[3];
  int rf[3];
  int first[3];
  int total;  // resident slots of every pool
};

// Step tier (max over rows, codes above FP16 read as FP16) and row mask of
// neuron i. ONE_ROW: B is 1 (a separate instantiation, so that no branch
// join forces a wait for the load).
template <bool ONE_ROW>
__device__ __forceinline__ void neuron_tiers(const uint8_t* __restrict__ tm, int d_ff, int i,
                                             int B, int& t, uint32_t& m) {
  t = 0;
  m = 0;
  if (ONE_ROW) {
    const int v = tm[i];
    t = v;
    m = v ? 1u : 0u;
  } else {
    for (int b0 = 0; b0 < B; b0 += 8) {
      uint8_t v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = tm[(int64_t)min(b0 + q, B - 1) * d_ff + i];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (b0 + q < B) {
          t = v[q] > t ? v[q] : t;
          m |= v[q] ? 1u << (b0 + q) : 0u;
        }
      }
    }
  }
  t = t > 3 ? 3 : t;
}

__device__ __forceinline__ uint32_t popc(unsigned long long v) { return (uint32_t)__popcll(v); }

// With pools and dominance hits (dom), a neuron required at tier t that is
// not resident in pool t but is resident in a pool of higher precision is
// served by the lowest such pool, as a hit at that pool's tier. Residency is
// that of the step's start: nothing is changed before plan_place_kernel.
template <bool POOLS, bool ONE_ROW>
__global__ __launch_bounds__(kPC) void plan_classify_kernel(const uint8_t* __restrict__ tier_map,
                                                            int B, int d_ff, int dom,
                                                            PoolGeom g, DeviceState st) {
  __shared__ uint32_t s_w[kPFields][kPCW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = blockIdx.x * kPC + tid, nc = min(n, d_ff - 1);
  const int serial = st.plan_state[kPlanSerial], cur = st.plan_state[kPlanCur];
  // every load of a neuron at once
  int r0 = st.slot_of[nc], r1 = -1, r2 = -1;
  if (POOLS) {
    r1 = st.slot_of[(int64_t)d_ff + nc];
    r2 = st.slot_of[2 * (int64_t)d_ff + nc];
  }
  int t;
  uint32_t m;
  neuron_tiers<ONE_ROW>(tier_map, d_ff, nc, B, t, m);
  if (n >= d_ff) t = 0;
  int q = 0, sl = r0;
  if (POOLS) {
    if (dom && t > 0) {
      const bool own = (t == 3 ? r0 : t == 2 ? r1 : r2) >= 0;
      if (!own) t = (t < 2 && r1 >= 0) ? 2 : r0 >= 0 ? 3 : t;
    }
    q = t == 3 ? 0 : t == 2 ? 1 : 2;
    sl = q == 0 ? r0 : q == 1 ? r1 : r2;
  }
  const bool req = t > 0, res = req && sl >= 0;
  int old = 0, at = 0;
  const int cs = (POOLS ? (q == 0 ? g.rf[0] : q == 1 ? g.rf[1] : g.rf[2]) : 0) + sl;
  if (res) {
    old = POOLS ? t : st.slot_tier[cs];  // a pool's slots hold records of its own tier only
    at = st.lru_pos[(int64_t)cur * g.total + cs];
  }
  const bool hit = res && (old == t || (!POOLS && dom && old > t));
  if (hit) t = old;  // the step tier of a hit is the resident tier
  if (res) {
    st.touch_slot[cs] = serial;
    st.touch_pos[at] = serial;
  }
  if (n < d_ff) {
    st.info[n] = req ? pack_info(t, hit ? 1 : res ? 2 : 0, old, res ? sl : 0) : 0u;
    if (!ONE_ROW) st.masks[n] = m;
  }
  const bool fill = req && !hit;
  const unsigned long long b[kPFields] = {
      __ballot(t == 3),         __ballot(t == 2),         __ballot(t == 1),
      __ballot(fill && t == 3), __ballot(fill && t == 2), __ballot(fill && t == 1),
      __ballot(req && !res),    __ballot(fill && old == 3 && t == 2),
      __ballot(fill && old == 3 && t == 1)};
  if (lane == 0) {
#pragma unroll
    for (int f = 0; f < kPFields; ++f) s_w[f][wave] = popc(b[f]);
  }
  __syncthreads();
  if (tid < kPFields) {
    uint32_t v = 0;
#pragma unroll
    for (int w = 0; w < kPCW; ++w) v += s_w[tid][w];
    st.chunk_counts[tid * (int)gridDim.x + (int)blockIdx.x] = (int32_t)v;
  }
  // what the place kernel reads while it changes the originals
  if (blockIdx.x == 0 && tid < kPlanWords) st.plan_copy[tid] = st.plan_state[tid];
}

// Ranks of the set flags among kPRounds per thread, entry order (round, wave,
// lane): rank[r] is base plus the set ones before the caller's entry r (every
// rank[r] is written; flags of rounds past `rounds` count as not set), and base
// ends as base plus all of them. cnt: kPRounds * kPW words, written here before
// the caller's barrier (store) and read after it (read).
struct BlockRanks {
  unsigned long long bal[kPRounds];
  __device__ __forceinline__ void store(const bool (&f)[kPRounds], int rounds, uint32_t* cnt,
                                        int wave, int lane) {
#pragma unroll
    for (int r = 0; r < kPRounds; ++r) {
      bal[r] = __ballot(r < rounds && f[r]);
      if (lane == 0) cnt[r * kPW + wave] = popc(bal[r]);
    }
  }
  __device__ __forceinline__ void read(uint32_t (&rank)[kPRounds], const uint32_t* cnt, int wave,
                                       int lane, uint32_t& base) const {
    static_assert(kPRounds * kPW == 128, "two counts per lane");
    const uint2 c = reinterpret_cast<const uint2*>(cnt)[lane];
    const uint32_t incl = wave_incl_scan(c.x + c.y);
    const uint32_t ex = incl - c.x - c.y;  // set flags before count 2 lane
    const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < kPRounds; ++r) {
      const int e = r * kPW + wave;  // the wave's count of round r
      uint32_t pre = __builtin_amdgcn_readlane(ex, e >> 1);
      if (e & 1) pre += __builtin_amdgcn_readlane(c.x, e >> 1);
      rank[r] = base + pre + popc(bal[r] & lt);
    }
    base += __builtin_amdgcn_readlane(incl, 63);
  }
};

struct PlaceArgs {
  int d_ff, chunks, cap, step, one_row;
  PoolGeom g;
  DeviceState st;
  PlanPtrs P;
  SlotMap map;
  TaskTable tt;
};

// LONG: an order of several sweeps, of which a workgroup ranks only the part it
// needs (plan_long says when).
template <bool POOLS, bool LONG>
__global__ __launch_bounds__(kPT) void plan_place_kernel(const PlaceArgs a) {
  constexpr int NP = POOLS ? 3 : 1;
  __shared__ uint32_t s_tot[kPW], s_pre[kPW], s_own[kPW];  // fields: all chunks, those before, this one
  __shared__ uint4 s_cw[7];  // the chunk's counts by wave
  __shared__ __align__(8) uint32_t s_cnt[kPRounds * kPW];
  __shared__ uint32_t s_lo[3], s_hi[3];  // a pool's first rank and the one past its last
  __shared__ int s_cut[3];               // LRU place of a pool's first unstamped slot kept
  __shared__ int s_vict[kPC];            // victims of this chunk's NEW neurons
  const DeviceState& st = a.st;
  const PoolGeom& g = a.g;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool neurons = (int)blockIdx.x < a.chunks;
  const int chunk = neurons ? (int)blockIdx.x : 0;
  const int own_round = neurons ? -1 : (int)blockIdx.x - a.chunks;  // its 1024 LRU places and slots
  const int n = tid < kPC ? chunk * kPC + tid : a.d_ff;  // its neuron (the first kPCW waves)
  const unsigned long long lt = (1ull << lane) - 1ull;
  auto pool_of = [&](int e) { return POOLS ? (e >= g.rf[1]) + (e >= g.rf[2]) : 0; };
  // one of three values by a pool index (selects of registers)
  auto pick = [&](int q, auto v0, auto v1, auto v2) { return q == 0 ? v0 : q == 1 ? v1 : v2; };

  // ---- first loads: the neuron's word, the counts, the first LRU sweep
  const uint32_t info = neurons && n < a.d_ff ? st.info[n] : 0u;
  const uint32_t mask = a.one_row || !neurons ? 1u : st.masks[min(n, a.d_ff - 1)];
  const int serial = st.plan_copy[kPlanSerial], cur = st.plan_copy[kPlanCur];
  const int rounds_all = (g.total + kPT - 1) / kPT;
  // LONG: the pools whose order the workgroup ranks, and the round its first
  // sweep starts at. One that writes the new order ranks the pools of its own
  // places; a neuron workgroup learns below which ones its NEW neurons go to.
  bool need[3] = {!neurons, false, false};
  int r_first = 0;
  if (LONG && POOLS && !neurons) {
#pragma unroll
    for (int q = NP - 1; q >= 0; --q) {
      need[q] = g.C[q] > 0 && g.rf[q] < (own_round + 1) * kPT && g.rf[q] + g.C[q] > own_round * kPT;
      if (need[q]) r_first = g.rf[q] / kPT;
    }
  }
  int32_t* lru_out = st.lru + (int64_t)(1 - cur) * g.total;
  int32_t* pos_out = st.lru_pos + (int64_t)(1 - cur) * g.total;
  // the first sweep reads both orders, so that its loads do not wait for `cur`
  int tp[kPRounds], sv[kPRounds], sw[kPRounds];
  auto load_lru = [&](int r0) {
#pragma unroll
    for (int r = 0; r < kPRounds; ++r) {
      tp[r] = sv[r] = sw[r] = 0;
      if (r0 + r < rounds_all) {
        const int p = min((r0 + r) * kPT + tid, g.total - 1);
        tp[r] = st.touch_pos[p];
        sv[r] = st.lru[p];
        sw[r] = st.lru[g.total + p];
      }
    }
  };
  load_lru(r_first);
  if (wave < kPFields) {
    uint32_t tot = 0, pre = 0, own = 0;
    for (int c0 = 0; c0 < a.chunks; c0 += 64) {
      const uint32_t v = c0 + lane < a.chunks ? (uint32_t)st.chunk_counts[wave * a.chunks + c0 + lane] : 0u;
      const uint32_t incl = wave_incl_scan(v);
      if (chunk >= c0 && chunk < c0 + 64) {
        own = __builtin_amdgcn_readlane(v, chunk - c0);
        pre = tot + __builtin_amdgcn_readlane(incl, chunk - c0) - own;
      }
      tot += __builtin_amdgcn_readlane(incl, 63);
    }
    if (lane == 0) {
      s_tot[wave] = tot;
      s_pre[wave] = pre;
      s_own[wave] = own;
    }
  }
  if (tid < NP) {
    s_lo[tid] = s_hi[tid] = 0;
    s_cut[tid] = g.rf[tid] + g.C[tid];
  }
  int t = (int)(info & 3u);
  const int code = (int)(info >> 2) & 3;
  const bool req = t > 0, fill = req && code != 1, fresh = req && code == 0;
  const unsigned long long b3 = __ballot(t == 3), b2 = __ballot(t == 2), b1 = __ballot(t == 1);
  const unsigned long long f3 = __ballot(fill && t == 3), f2 = __ballot(fill && t == 2),
                           f1 = __ballot(fill && t == 1), bn = __ballot(fresh);
  if (lane == 0 && wave < kPCW) {
    const uint32_t c[7] = {popc(b3), popc(b2), popc(b1), popc(f3), popc(f2), popc(f1), popc(bn)};
#pragma unroll
    for (int f = 0; f < 7; ++f) reinterpret_cast<uint32_t*>(&s_cw[f])[wave] = c[f];
  }

  // ---- the LRU order: rank the unstamped places, hand out victims. LONG: a
  // neuron workgroup ranks, in the pools its NEW neurons go to, the places up to
  // its last victim; one that writes the new order those of its pools up to its
  // own places and up to the first place kept.
  uint32_t base = 0;
  int r0 = r_first;
  uint32_t nnew[3] = {0, 0, 0}, npre[3] = {0, 0, 0}, nown[3] = {0, 0, 0};
  // unstamped places of a pool: of its required neurons, all but the NEW ones stamped a slot
  auto unstamped = [&](int q, uint32_t n_new) {
    return (uint32_t)g.C[q] - (POOLS ? s_tot[kR3 + q] : s_tot[kR3] + s_tot[kR2] + s_tot[kR1]) + n_new;
  };
  uint32_t want[3] = {0, 0, 0};  // unstamped places of the pool that have to be ranked
  do {
    bool unt[kPRounds];
    const int rounds = min(rounds_all - r0, kPRounds);
#pragma unroll
    for (int r = 0; r < kPRounds; ++r)
      unt[r] = r < rounds && (r0 + r) * kPT + tid < g.total && tp[r] != serial;
    BlockRanks br;
    br.store(unt, rounds, s_cnt, wave, lane);
    __syncthreads();
    if (r0 == r_first) {
      if (s_tot[kR3] + s_tot[kR2] + s_tot[kR1] > (uint32_t)a.cap) break;  // workgroup-uniform
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        nnew[q] = s_tot[POOLS ? kF3 + q : kNew];
        npre[q] = s_pre[POOLS ? kF3 + q : kNew];
        nown[q] = s_own[POOLS ? kF3 + q : kNew];
        if (LONG) {
          const uint32_t n_unt = unstamped(q, nnew[q]);
          if (neurons) need[q] = nown[q] > 0 && npre[q] < n_unt;
          want[q] = min(neurons ? npre[q] + nown[q] : nnew[q] + 1u, n_unt);
        }
      }
    }
    uint32_t rank[kPRounds];
    br.read(rank, s_cnt, wave, lane, base);
    if (POOLS) {
#pragma unroll
      for (int r = 0; r < kPRounds; ++r) {
        const int p = (r0 + r) * kPT + tid;
        if (r < rounds && p < g.total) {
          const int q = pool_of(p);
          const int q0 = pick(q, g.rf[0], g.rf[1], g.rf[2]), qc = pick(q, g.C[0], g.C[1], g.C[2]);
          if (p == q0) s_lo[q] = rank[r];
          if (!LONG && p == q0 + qc - 1) s_hi[q] = rank[r] + unt[r];
        }
      }
      __syncthreads();
    } else if (!LONG && tid == 0) {
      s_hi[0] = base;
    }
#pragma unroll
    for (int r = 0; r < kPRounds; ++r) {
      if (!unt[r]) continue;
      const int slot = cur ? sw[r] : sv[r];
      const int p = (r0 + r) * kPT + tid, q = pool_of(p);
      const uint32_t u = POOLS ? rank[r] - s_lo[q] : rank[r];
      const uint32_t nn = pick(q, nnew[0], nnew[1], nnew[2]);
      if (u < nn) {
        const uint32_t j = u - pick(q, npre[0], npre[1], npre[2]);
        if (neurons && j < pick(q, nown[0], nown[1], nown[2]))
          s_vict[j + (q > 0 ? nown[0] : 0u) + (q > 1 ? nown[1] : 0u)] = slot;
      } else {
        if (u == nn) s_cut[q] = p;
        if (r0 + r == own_round) {  // kept, in the old order
          const int np = pick(q, g.rf[0], g.rf[1], g.rf[2]) + (int)(u - nn);
          lru_out[np] = slot;
          pos_out[slot] = np;
        }
      }
    }
    if constexpr (LONG) {
      // the next sweep: behind this one, at the start of the next pool to rank, or none
      const int end = r0 + kPRounds;
      r0 = rounds_all;
#pragma unroll
      for (int q = 0; q < NP; ++q)
        if (need[q] && g.rf[q] + g.C[q] > end * kPT &&
            (g.rf[q] >= end * kPT || base - (POOLS ? s_lo[q] : 0u) < want[q] || own_round >= end))
          r0 = min(r0, max(end, g.rf[q] / kPT));
#pragma unroll
      for (int r = 0; r < kPRounds; ++r) {
        tp[r] = sv[r] = sw[r] = 0;
        if (r0 + r < rounds_all) {
          const int p = min((r0 + r) * kPT + tid, g.total - 1);
          tp[r] = st.touch_pos[p];
          sv[r] = sw[r] = st.lru[(int64_t)cur * g.total + p];
        }
      }
    } else {
      r0 += kPRounds;
      if (r0 < rounds_all) load_lru(r0);
    }
    __syncthreads();
  } while (r0 < rounds_all);

  const uint32_t N3 = s_tot[kR3], N2 = s_tot[kR2], N1 = s_tot[kR1], NREQ = N3 + N2 + N1;
  const bool tasks = a.tt.grid > 0;
  if (NREQ > (uint32_t)a.cap) {
    // More active neurons than the layer was sized for (a tier map that did
    // not come from m2c_predict_rank with k <= k_max): write an empty plan
    // with the overflow flagged and leave the cache untouched (the stamps
    // carry this plan's serial, which no other plan uses).
    if (blockIdx.x == 0) {
      if (tid < M2C_NCOUNTS) a.P.counts[tid] = tid == M2C_NCOUNTS - 1 ? (int32_t)NREQ : 0;
      if (tid == 0) {
        atomicOr(st.status, M2C_STATUS_PLAN_OVERFLOW);
        st.plan_state[kPlanSerial] = serial + 1;
        if (tasks) write_task_count(a.tt, a.map, 0);
      }
    }
    return;
  }
  int nunt[3] = {0, 0, 0}, nv[3] = {0, 0, 0}, ne[3] = {0, 0, 0}, filled[3] = {0, 0, 0};
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    filled[q] = st.plan_copy[kPlanFilled + q];
    nunt[q] = LONG ? (int)unstamped(q, nnew[q]) : (int)(s_hi[q] - s_lo[q]);
    nv[q] = min((int)nnew[q], nunt[q]);
    ne[q] = min(nv[q], g.C[q] - filled[q]);  // never-used slots come first in the order
  }

  if (!neurons) {
    // ---- slots used this step (stamped, or before the first kept place) go
    // to the end of their pool's order, in slot order
    const int32_t* pos_in = st.lru_pos + (int64_t)cur * g.total;
    base = 0;
    for (r0 = r_first; r0 <= own_round; r0 += kPRounds) {
      const int rounds = min(own_round + 1 - r0, kPRounds);
      int ts[kPRounds], ps[kPRounds];
#pragma unroll
      for (int r = 0; r < kPRounds; ++r) {
        ts[r] = ps[r] = 0;
        if (r < rounds) {
          const int s = min((r0 + r) * kPT + tid, g.total - 1);
          ts[r] = st.touch_slot[s];
          ps[r] = pos_in[s];
        }
      }
      bool used[kPRounds];
#pragma unroll
      for (int r = 0; r < kPRounds; ++r) {
        const int s = (r0 + r) * kPT + tid;
        used[r] = r < rounds && s < g.total && (ts[r] == serial || ps[r] < s_cut[pool_of(s)]);
      }
      BlockRanks br;
      br.store(used, rounds, s_cnt, wave, lane);
      __syncthreads();
      uint32_t rank[kPRounds];
      br.read(rank, s_cnt, wave, lane, base);
      if (POOLS) {
#pragma unroll
        for (int r = 0; r < kPRounds; ++r) {
          const int s = (r0 + r) * kPT + tid;
          if (r < rounds && s < g.total) {
            const int q = pool_of(s);
            if (s == pick(q, g.rf[0], g.rf[1], g.rf[2])) s_lo[q] = rank[r];
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kPRounds; ++r) {
        if (r0 + r != own_round || !used[r]) continue;
        const int s = (r0 + r) * kPT + tid, q = pool_of(s);
        const int np = pick(q, g.rf[0], g.rf[1], g.rf[2]) +
                       pick(q, nunt[0] - nv[0], nunt[1] - nv[1], nunt[2] - nv[2]) +
                       (int)(rank[r] - (POOLS ? s_lo[q] : 0u));
        lru_out[np] = s;
        pos_out[s] = np;
        st.slot_last[s] = a.step;
      }
    }
    return;
  }

  const FMap fm = make_map((int)N3, (int)N2, (int)N1, a.tt.d, a.tt.upt);
  if (wave >= 2 * kPCW) {
    if (blockIdx.x != 0 || wave != 2 * kPCW) return;
    // ---- counts, statistics, the next plan's state (one wave of workgroup 0)
    const uint32_t F3 = s_tot[kF3], F2 = s_tot[kF2], F1 = s_tot[kF1], NF = F3 + F2 + F1;
    const uint32_t D2 = s_tot[kD2], D1 = s_tot[kD1], NNEW = s_tot[kNew];
    const uint32_t V = (uint32_t)(nv[0] + nv[1] + nv[2]), E = (uint32_t)(ne[0] + ne[1] + ne[2]);
    const uint32_t c[M2C_NCOUNTS] = {NREQ, NREQ - NF, NF - NNEW, V,  NNEW - V, V - E,   NF, N3,
                                     N2,   N1,        F3,        F2, F1,       D2 + D1, 0u, 0u};
    // cumulative: plans, req, hit, refill, new, bypass, evict, fills INT4 /
    // INT8 / FP16, required INT4 / INT8 / FP16, derived INT8 / INT4
    const uint32_t s[16] = {1u, NREQ, NREQ - NF, NF - NNEW, V,  NNEW - V, V - E, F1,
                            F2, F3,   N1,        N2,        N3, D2,       D1,    0u};
    uint32_t cv = 0, sv_ = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {  // by value: an indexed array would live in scratch memory
      cv = lane == i ? c[i] : cv;
      sv_ = lane == i ? s[i] : sv_;
    }
    if (lane < M2C_NCOUNTS) a.P.counts[lane] = (int32_t)cv;
    if (lane < 15) st.stats[lane] += (unsigned long long)sv_;
    if (lane == 0) {
      st.plan_state[kPlanSerial] = serial + 1;
      st.plan_state[kPlanCur] = 1 - cur;
#pragma unroll
      for (int q = 0; q < NP; ++q) st.plan_state[kPlanFilled + q] = filled[q] + ne[q];
      if (tasks) write_task_count(a.tt, a.map, min(fm.e[5], a.tt.grid));
    }
    return;
  }
  if (wave >= kPCW) {  // ---- task headers
    if (!tasks) return;
    const int n_tasks = min(fm.e[5], a.tt.grid);
    for (int k = chunk * kPC + tid - kPC; k < n_tasks; k += a.chunks * kPC)
      write_task_header(a.tt, fm, a.map, k);
    return;
  }
  // ---- the neuron's outputs
  uint32_t before[7];  // in the chunk's waves before this one
#pragma unroll
  for (int f = 0; f < 7; ++f) {
    const uint4 v = s_cw[f];
    before[f] = (wave > 0 ? v.x : 0u) + (wave > 1 ? v.y : 0u) + (wave > 2 ? v.z : 0u);
  }
  if (req) {
    const unsigned long long bt = t == 3 ? b3 : t == 2 ? b2 : b1;
    const unsigned long long ft = t == 3 ? f3 : t == 2 ? f2 : f1;
    const int q = POOLS ? 3 - t : 0;
    const int pos = (int)(s_pre[kR3] + s_pre[kR2] + s_pre[kR1] + before[0] + before[1] + before[2] +
                          popc((b3 | b2 | b1) & lt));
    // place in its tier, and in the work list (FP16, INT8, INT4)
    const int it = (int)(pick(3 - t, s_pre[kR3], s_pre[kR2], s_pre[kR1]) +
                         pick(3 - t, before[0], before[1], before[2]) + popc(bt & lt));
    const int wp = it + (t < 3 ? (int)N3 : 0) + (t < 2 ? (int)N2 : 0);
    const int rf = pick(q, g.rf[0], g.rf[1], g.rf[2]), C = pick(q, g.C[0], g.C[1], g.C[2]);
    const int first = pick(q, g.first[0], g.first[1], g.first[2]);
    int sl = (int)(info >> 8), hit = code, from = 0;
    if (fresh) {
      const uint32_t lj = POOLS ? pick(q, before[3], before[4], before[5]) + popc(ft & lt)
                                : before[6] + popc(bn & lt);  // among the chunk's NEW of its pool
      const int j = (int)(pick(q, npre[0], npre[1], npre[2]) + lj);
      const int v = pick(q, nv[0], nv[1], nv[2]);
      if (j < v) {
        const int cs = s_vict[lj + (q > 0 ? nown[0] : 0u) + (q > 1 ? nown[1] : 0u)];
        const int old = st.slot_key[cs];
        int32_t* of = st.slot_of + (int64_t)q * a.d_ff;
        sl = cs - rf;
        if (old >= 0) {
          of[old] = -1;
          a.P.evicted_ids[j - pick(q, ne[0], ne[1], ne[2]) + (q > 0 ? nv[0] - ne[0] : 0) +
                          (q > 1 ? nv[1] - ne[1] : 0)] = old;
        }
        of[n] = sl;
        st.slot_key[cs] = n;
        st.slot_tier[cs] = (uint8_t)t;
      } else {  // no victim left: a staging slot, not retained
        sl = C + (j - v);
        hit = 3;
      }
    } else if (code == 2) {
      from = (int)(info >> 4) & 3;
      st.slot_tier[rf + sl] = (uint8_t)t;
    }
    const int gs = first + sl;
    a.P.req_ids[pos] = n;
    a.P.req_tier[pos] = (uint8_t)t;
    a.P.req_hit[pos] = (uint8_t)hit;
    a.P.req_slot[pos] = gs;
    a.P.req_mask[pos] = mask;
    a.P.work_slot[wp] = gs;
    a.P.work_mask[wp] = mask;
    if (fill) {
      const int fi = (int)(s_pre[kF3] + s_pre[kF2] + s_pre[kF1] + before[3] + before[4] + before[5] +
                           popc((f3 | f2 | f1) & lt));
      a.P.fill_ids[fi] = n;
      a.P.fill_tier[fi] = (uint8_t)t;
      a.P.fill_slot[fi] = gs;
      a.P.fill_from[fi] = (uint8_t)from;
    }
    if (tasks) write_task_items(a.tt, fm, t, it, gs);
  }
}

// Empties the cache unit (every pool of the per-tier arena), clears the
// fill's record table, the counters and the plan's state.
__global__ void reset_kernel(DeviceState st, int64_t n_slot_of, int C, int n_rec) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = gridDim.x * blockDim.x;
  for (int64_t i = idx; i < n_slot_of; i += n) st.slot_of[i] = -1;
  for (int s = idx; s < C; s += n) {
    st.slot_key[s] = -1;
    st.slot_tier[s] = 0;
    st.slot_last[s] = -1;
    st.lru[s] = st.lru[C + s] = s;
    st.lru_pos[s] = st.lru_pos[C + s] = s;
    st.touch_slot[s] = st.touch_pos[s] = -1;
  }
  for (int s = idx; s < n_rec; s += n) st.slot_rec[s] = -1;
  if (idx < kPlanWords) st.plan_state[idx] = 0;
  if (idx < 16) st.stats[idx] = 0;
}

DeviceState pool_state(const m2c_layer* L, int t) {
  DeviceState v = L->st;
  if (!L->pools) return v;
  const int rf = L->pool_rf[t];
  v.slot_of = L->st.slot_of + (int64_t)(3 - t) * L->desc.d_ff;
  v.slot_key = L->st.slot_key + rf;
  v.slot_tier = L->st.slot_tier + rf;
  v.slot_last = L->st.slot_last + rf;
  return v;
}

static PlanPtrs plan_ptrs(const m2c_layer* L, uint8_t* plan) {
  const m2c_plan_layout& lay = L->layout;
  PlanPtrs P;
  P.counts = reinterpret_cast<int32_t*>(plan + lay.counts);
  P.req_ids = reinterpret_cast<int32_t*>(plan + lay.req_ids);
  P.req_tier = plan + lay.req_tier;
  P.req_hit = plan + lay.req_hit;
  P.req_slot = reinterpret_cast<int32_t*>(plan + lay.req_slot);
  P.req_mask = reinterpret_cast<uint32_t*>(plan + lay.req_mask);
  P.fill_ids = reinterpret_cast<int32_t*>(plan + lay.fill_ids);
  P.fill_tier = plan + lay.fill_tier;
  P.fill_slot = reinterpret_cast<int32_t*>(plan + lay.fill_slot);
  P.fill_from = plan + lay.fill_from;
  P.evicted_ids = reinterpret_cast<int32_t*>(plan + lay.evicted_ids);
  P.work_slot = reinterpret_cast<int32_t*>(plan + lay.work_slot);
  P.work_mask = reinterpret_cast<uint32_t*>(plan + lay.work_mask);
  return P;
}

// Whether the place kernel ranks only the parts of the LRU order it needs. Asking
// which costs scalar registers: about 1 us of a plan with pools, 0.1 to 0.5 with one
// order. With one sweep (8192 slots) there is nothing to leave out. With pools the
// workgroups of the later ones skip the earlier pools' sweeps; a single order's last
// workgroup ranks nearly all of it, and only the reads of the others are saved.
// Measured (MI355X, whole plans back to back, all of the order -> the parts):
//   pools, d_ff 28672: 2867 slots 12.3 -> 13.4 us; d_ff 32768: 8192 slots 14.8 ->
//   14.6, 16384 23.2 -> 21.1, 32768 39.6 -> 30.1
//   single: 9000 slots 14.2 -> 14.7, 28672 25.3 -> 25.6, 41000 35.8 -> 35.1, 65536
//   71 -> 52, 262144 535 -> 199
static bool plan_long(bool pools, int slots) {
  return slots > (pools ? kPRounds * kPT : 5 * kPRounds * kPT);
}

hipError_t launch_plan(m2c_layer* L, const uint8_t* tier_map, int batch, int step, uint8_t* plan,
                       hipStream_t stream) {
  const int d_ff = L->desc.d_ff;
  PlaceArgs a;
  a.d_ff = d_ff;
  a.chunks = (d_ff + kPC - 1) / kPC;
  a.cap = L->cap;
  a.step = step;
  a.one_row = batch == 1;
  for (int q = 0; q < 3; ++q) {
    const int t = 3 - q;
    a.g.C[q] = L->pools ? L->pool_C[t] : q == 0 ? L->desc.cache_slots : 0;
    a.g.rf[q] = L->pools ? L->pool_rf[t] : q == 0 ? 0 : L->desc.cache_slots;
    a.g.first[q] = L->pools ? L->map.first[t] : 0;
  }
  a.g.total = L->desc.cache_slots;
  a.st = L->st;
  a.P = plan_ptrs(L, plan);
  a.map = L->map;
  a.tt = plan_task_table(L, plan);
  const int dom = (L->desc.flags & M2C_FLAG_DOMINANT_HITS) ? 1 : 0;
  const dim3 gc(a.chunks), bc(kPC), gp(a.chunks + (a.g.total + kPT - 1) / kPT), b(kPT);
#define M2C_CLASSIFY(P, ONE)                                                                    \
  hipLaunchKernelGGL((plan_classify_kernel<P, ONE>), gc, bc, 0, stream, tier_map, batch, d_ff,   \
                     dom, a.g, a.st)
  if (L->pools)  // a layer with pools takes one row (max_batch 1)
    M2C_CLASSIFY(true, true);
  else if (batch == 1)
    M2C_CLASSIFY(false, true);
  else
    M2C_CLASSIFY(false, false);
#undef M2C_CLASSIFY
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool many = plan_long(L->pools, a.g.total);
  if (L->pools && many)
    hipLaunchKernelGGL((plan_place_kernel<true, true>), gp, b, 0, stream, a);
  else if (L->pools)
    hipLaunchKernelGGL((plan_place_kernel<true, false>), gp, b, 0, stream, a);
  else if (many)
    hipLaunchKernelGGL((plan_place_kernel<false, true>), gp, b, 0, stream, a);
  else
    hipLaunchKernelGGL((plan_place_kernel<false, false>), gp, b, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_reset(m2c_layer* L, hipStream_t stream) {
  const int n_rec = L->desc.cache_slots + L->S;
  const int64_t n_of = (int64_t)(L->pools ? 3 : 1) * L->desc.d_ff;
  int64_t n = n_of > n_rec ? n_of : n_rec;
  int blocks = (int)((n + 255) / 256);
  if (blocks < 1) blocks = 1;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(reset_kernel, dim3(blocks), dim3(256), 0, stream, L->st, n_of,
                     L->desc.cache_slots, n_rec);
  return hipGetLastError();
}

}  // namespace m2c
