// The first BFS levels of an exploration on one workgroup, level after level,
// with no host round trip and no table probe between them (Sec. 5.2 traces the
// low rate on small instances to small search layers and per-layer overhead).
#pragma once

#include <algorithm>
#include <cstdint>

#include "gx_explore_kernel.hpp"
#include "gx_lds_plan.hpp"

namespace gx {

constexpr uint64_t kSmallMaxLevel = 4096;    // largest level the workgroup expands
constexpr uint64_t kSmallSuccBudget = 4096;  // and at most this many successors (worst case)

struct SmallArgs {
  TableDev t;
  const uint32_t* img;  // network image (global; copied to LDS)
  uint32_t img_words;
  uint32_t img_stride;
  uint32_t* f;          // frontier buffer 0, receives the current level at the end
  uint32_t* log;        // the states found, level after level, S words each
  uint64_t log_cap;
  uint32_t* dead;
  uint64_t dead_cap;
  uint64_t* ctr;        // the exploration's counters (see ctr_at)
  LevelCtl* out;
  uint64_t limit;       // largest level this launch expands
  const uint32_t* init_key;  // the level-0 state
  uint32_t set_mask;    // entries of the LDS visited set, minus one (a power of two)
  uint32_t ring;        // states of a level that LDS holds
  uint32_t max_succ;    // distinct successors a state can form at most
  uint32_t max_qs;      // log2 of the most lanes a state is worth
  uint64_t next_limit;  // largest level that level kernels take up right after it
  uint32_t number;      // the exploration's
  // report set: once the states are all placed, the counters and the control
  // block (they follow them), block_words words, are copied to host_block in
  // host memory and reported as launch 0's (see level_report)
  uint64_t* report;
  uint64_t* host_block;
  uint32_t block_words;
};

// A table that held states the launch did not put there (reported as
// GX_EINVAL: gx_explore needs an empty table).
constexpr uint32_t kFlagNotEmpty = 16;

// ------------------------------------------------ LDS-resident first levels
constexpr uint32_t kLocked = 0xFFFFFFFEu;  // an LDS set entry being written (packed
                                           // states never hold it: bit 31 is 0)

// Insert-if-absent of key into the workgroup's LDS set (open addressing,
// linear probing, set_mask + 1 entries of S words); true where this lane put
// it there.  A multi-word entry is claimed by a compare-and-swap of its first
// word to kLocked and published by writing the first word last; a lane that
// meets a locked entry looks at it again in the next step (its owner
// publishes within the step that claimed it).  Must be reached by the whole
// wavefront; act false: no key.
template <int S>
__device__ inline bool lds_set_insert(uint32_t* set, uint32_t mask, const uint32_t (&key)[S],
                                      bool act) {
  bool done = !act, fresh = false;
  uint32_t h = dedup_hash<S>(key) & mask;
  if constexpr (S == 1) {
    // one-word entries: the compare-and-swap is the look too
    while (!done) {
      uint32_t old = kEmpty;
      fresh = __hip_atomic_compare_exchange_strong(set + h, &old, key[0], __ATOMIC_RELAXED,
                                                   __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
      done = fresh || old == key[0];
      h = (h + 1) & mask;
    }
  } else {
    while (__ballot(!done)) {
      if (!done) {
        uint32_t* e = set + h * S;
        const uint32_t w0 = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (w0 == kEmpty) {
          uint32_t expect = kEmpty;
          if (__hip_atomic_compare_exchange_strong(e, &expect, kLocked, __ATOMIC_RELAXED,
                                                   __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP)) {
#pragma unroll
            for (int x = 1; x < S; ++x)
              __hip_atomic_store(e + x, key[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __hip_atomic_store(e, key[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            fresh = true;
            done = true;
          }
        } else if (w0 != kLocked) {
          bool same = w0 == key[0];
          if (same) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
            for (int x = 1; x < S; ++x)
              same &= __hip_atomic_load(e + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) ==
                      key[x];
          }
          if (same)
            done = true;
          else
            h = (h + 1) & mask;
        }
      }
    }
  }
  return fresh;
}

// Whether the launch places its states itself: the fill counts of the table's
// buckets fit the LDS of a visited set of n_set entries.
template <int S>
__host__ __device__ inline bool lds_places(uint64_t n_buckets, uint32_t n_set) {
  return n_buckets <= static_cast<uint64_t>(n_set) * S;
}

// The logged states into the table, by the workgroup that logged them, with
// no device-scope claim: the table held none of them and nothing else (the
// premise of an LDS-resident launch) and they are distinct (the visited set
// decided that), so each takes the next slot of the first bucket of its hash
// sequence that still has one, counted in LDS (fill, one word per bucket),
// and is written with a plain store.  That is the layout find-or-put builds:
// a bucket fills from its lowest slot, and a state lies in its j-th bucket
// only when buckets 1..j-1 of its sequence are full.  (Claimed one by one,
// the states of a small fresh table queue at a few memory channels: 29 us
// for 4096 of them.)  No slot left in any of the H buckets: FULL.  Log entry
// 0 is the initial state; its outcome goes to out->init_status.  Must be
// reached by the whole workgroup.
template <int S, int B>
__device__ inline void place_log(const SmallArgs& a, uint32_t* fill, const uint32_t* log,
                                 uint32_t log_n) {
  constexpr uint32_t kSlots = B / S;
  const uint32_t tid = threadIdx.x;
  const uint32_t nb = static_cast<uint32_t>(a.t.n_buckets);
  for (uint32_t k = tid; k < nb; k += small_threads<S>()) fill[k] = 0;
  __syncthreads();
  LaneStats st;
  uint32_t stored = 0, lookups = 0, full = 0;
  for (uint32_t i = tid; i < log_n; i += small_threads<S>()) {
    uint32_t key[S];
    load_slot<S>(log + static_cast<uint64_t>(i) * S, key);
    const uint64_t mix = key_mix<S>(key, a.t.seed);
    bool done = false;
    uint32_t j = 0;
    for (; j < a.t.H && !done; ++j) {
      const uint64_t ca = j == 0 ? a.t.a0 : a.t.hc[2 * j];
      const uint64_t cc = j == 0 ? a.t.c0 : a.t.hc[2 * j + 1];
      const uint64_t b = bucket_of(mix, ca, cc, a.t.n_buckets);
      const uint32_t slot = atomicAdd(&fill[b], 1u);
      ++st.probes;
      if (slot < kSlots) {
        store_slot<S>(a.t.words + b * B + slot * S, key);
        done = true;
        if (j > st.max_j) st.max_j = j;
      }
    }
    ++lookups;
    if (done) ++stored;
    else ++full;
    if (i == 0) a.out->init_status = done ? kNew : kFull;
  }
  st.stored = wave_sum(stored);
  st.lookups = wave_sum(lookups);
  st.full = wave_sum(full);
  if (st.full && __lane_id() == 0) atomicOr(ctr_at(a.ctr, kCtrFlags), kFlagTableFull);
  flush_stats(a.t, st, nullptr);
}

// Workgroup barrier that orders LDS accesses only: global stores stay in
// flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The first levels of an exploration, while the table holds nothing but what
// this launch puts there: an LDS set of every state reached so far decides
// NEW or SEEN exactly, with no table probe.  New states are appended to a log
// in global memory, level after level, so a level is a contiguous range of
// the log.  A level is expanded only while the set stays at most three
// quarters full even if every successor were new.  When the levels end (the
// exploration is complete, a level would not fit, or kChainLevels levels are
// done) the current level is copied to frontier buffer 0 for the host, and
// every logged state goes into the table: placed by this workgroup when the
// table's per-bucket fill counts fit in the LDS the visited set used (see
// place_log), else by log_insert_kernel, launched after it.
// Bound: the chain of dependent LDS reads and the barrier of a level.  The
// lanes share the states' items (walk_items), so that a level of a few
// hundred states has a few items a lane to walk instead of all of them.  No
// access to global memory is waited for within a level of up to `ring`
// states: its states are read from LDS, where two rings hold the last two
// levels beside the log, and every thread works out for itself, from one
// count, whether and how the levels go on.
template <int S, int B>
__global__ __launch_bounds__(small_threads<S>()) void lds_levels_kernel(SmallArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  constexpr uint32_t kWaves = small_threads<S>() / 64;
  // per level in turn: its new states, its deadlocks from bit kDeadShift on
  // (the next level's count is cleared while the one before last is read)
  constexpr uint32_t kDeadShift = 18;
  __shared__ uint32_t sh_lvl[3];
  __shared__ uint32_t sh_count[kChainLevels];
  __shared__ unsigned long long sh_trans;
  const uint32_t tid = threadIdx.x;
  const uint32_t wave = tid >> 6;
  const uint32_t lane = __lane_id();
  uint32_t* img = smem;
  uint32_t* set = smem + a.img_stride;
  const uint32_t n_set = a.set_mask + 1;
  uint32_t* stage = set + n_set * S + wave * kSmallStage * S;
  uint32_t* rings = set + n_set * S + kWaves * kSmallStage * S;
  uint32_t* log = a.log;
  const uint64_t set_cap = static_cast<uint64_t>(n_set) / 4 * 3;
  uint32_t init[S];
#pragma unroll
  for (int x = 0; x < S; ++x) init[x] = a.init_key[x];
  for (uint32_t k = tid; k < a.img_words; k += small_threads<S>()) img[k] = a.img[k];
  for (uint32_t k = tid; k < n_set * S / 4; k += small_threads<S>())
    reinterpret_cast<uint4*>(set)[k] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
  if (tid == 0) {
    store_slot<S>(log, init);
    store_slot<S>(rings, init);
    sh_lvl[0] = 0;
    sh_trans = 0;
  }
  __syncthreads();
  if (wave == 0) (void)lds_set_insert<S>(set, a.set_mask, init, lane == 0);
  __syncthreads();
  // the level: states [ls, le) of the log (the same in every thread, as all
  // that decides how the levels go on)
  uint32_t ls = 0, le = 1, levels = 0, dead = 0, turn = 0, parity = 0;
  bool go = a.limit >= 1 && 1 + static_cast<uint64_t>(a.max_succ) <= min(set_cap, a.log_cap);
  uint64_t trans = 0;  // this lane's
  while (go) {
    const uint32_t n_in = le - ls;
    const uint32_t* ring_in = rings + parity * a.ring * S;
    uint32_t* ring_out = rings + (parity ^ 1u) * a.ring * S;
    const uint32_t qs = lanes_per_state(n_in, kWaves, a.max_qs);
    const uint32_t q = 1u << qs, per = 64u >> qs;
    uint32_t cnt = 0;
    // the last 64 staged successors (or all that are left) into the set; the
    // new ones go to the log
    auto take = [&]() {
      wave_lds_sync();
      const uint32_t n = cnt < 64 ? cnt : 64u;
      cnt -= n;
      uint32_t key[S];
#pragma unroll
      for (int x = 0; x < S; ++x) key[x] = 0;
      if (lane < n) load_slot<S>(stage + (cnt + lane) * S, key);
      const bool fresh = lds_set_insert<S>(set, a.set_mask, key, lane < n);
      const uint64_t m = __ballot(fresh);
      if (m) {
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&sh_lvl[turn], static_cast<uint32_t>(__popcll(m)));
        const uint32_t k = (uniform32(base) & ((1u << kDeadShift) - 1u)) + lane_rank(m);
        if (fresh) {
          store_slot<S>(log + static_cast<uint64_t>(le + k) * S, key);
          if (k < a.ring) store_slot<S>(ring_out + k * S, key);
        }
      }
      wave_lds_sync();
    };
    for (uint32_t g0 = wave * per; g0 < n_in; g0 += kWaves * per) {
      const uint32_t i = g0 + (lane >> qs);
      const bool has = i < n_in;
      uint32_t sw[S];
#pragma unroll
      for (int x = 0; x < S; ++x) sw[x] = 0;
      if (n_in <= a.ring) {
        if (has) load_slot<S>(ring_in + i * S, sw);
      } else if (has) {
        load_slot<S>(log + static_cast<uint64_t>(ls + i) * S, sw);
      }
      const uint32_t own = walk_items<S>(img, sw, has, lane & (q - 1), q, stage, cnt, 63u, take);
      trans += own;
      const uint64_t m = __ballot(own != 0);
      const uint64_t mine = (m >> (lane & ~(q - 1))) & (q == 64 ? ~0ull : (1ull << q) - 1ull);
      if (has && (lane & (q - 1)) == 0 && mine == 0) {
        const uint64_t d = dead + (atomicAdd(&sh_lvl[turn], 1u << kDeadShift) >> kDeadShift);
        if (d < a.dead_cap) store_slot<S>(a.dead + d * S, sw);
      }
    }
    if (cnt) take();
    const uint32_t after = turn == 2 ? 0u : turn + 1;
    if (tid == 0) sh_lvl[after] = 0;
    lds_barrier();  // the level's new states are logged
    const uint32_t v = uniform32(sh_lvl[turn]);
    const uint32_t n_next = v & ((1u << kDeadShift) - 1u);
    dead += v >> kDeadShift;
    turn = after;
    parity ^= 1u;
    ls = le;
    le += n_next;
    if (n_next) {
      if (tid == 0) sh_count[levels] = n_next;
      ++levels;
    }
    // (n_next <= limit: the level after it fits the frontier buffer, which
    // receives the current level when the launch ends)
    go = n_next > 0 && n_next <= a.limit && levels < kChainLevels &&
         le + static_cast<uint64_t>(n_next) * a.max_succ <= min(set_cap, a.log_cap) &&
         n_next <= a.dead_cap - min(static_cast<uint64_t>(dead), a.dead_cap);
    if (n_next > a.ring) __syncthreads();  // (the next level is read from the log)
  }
  trans = wave_sum64(trans);
  if (lane == 0 && trans) atomicAdd(&sh_trans, static_cast<unsigned long long>(trans));
  __syncthreads();
  // the current level becomes frontier buffer 0 (when the levels go on)
  const uint32_t n_cur = le - ls;
  for (uint32_t k = tid; k < n_cur * S; k += small_threads<S>())
    a.f[k] = log[static_cast<uint64_t>(ls) * S + k];
  for (uint32_t k = tid; k < levels; k += small_threads<S>()) a.out->levels[k] = sh_count[k];
  // the visited set is done with: its LDS holds the bucket fill counts
  const bool placed = lds_places<S>(a.t.n_buckets, n_set);
  if (placed) place_log<S, B>(a, set, log, le);
  if (tid == 0) {
    a.out->n_levels = levels;
    a.out->n_in = n_cur;  // 0: the last level expanded found nothing new
    a.out->cur = 0;
    a.out->log_n = placed ? 0 : le;  // states left for log_insert_kernel
    LevelCtl::Entry& e = a.out->entry[0];
    e.n_in = n_cur;
    e.cur = 0;
    e.n_levels = 0;
    e.go = n_cur > 0 && n_cur <= a.next_limit &&
                   n_cur <= a.dead_cap - min(static_cast<uint64_t>(dead), a.dead_cap)
               ? a.number
               : 0u;
    e.fresh = 0;  // (the level's size is among those above)
    e.scan = 0;   // (no monitor)
    if (sh_trans) atomicAdd(ctr_at(a.ctr, kCtrTrans), sh_trans);
    if (dead) atomicAdd(ctr_at(a.ctr, kCtrDead), static_cast<unsigned long long>(dead));
  }
  if (placed && a.report != nullptr) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    copy_to_host(a.host_block, a.ctr, a.block_words);
    if (tid == 0) level_report(a.report, 0, 0, 0, n_cur);
  }
}

// The states an LDS-resident launch logged go into the table, spread over
// the device (launched right after it on the same stream).  They are
// distinct and the table held none of them (it was empty when the
// exploration started), so each must come back NEW: FULL raises the
// table-full flag, anything else kFlagNotEmpty.  The initial state (log
// entry 0) reports its status in out->init_status.
template <int S, int B>
__global__ __launch_bounds__(256) void log_insert_kernel(TableDev t, const uint32_t* log,
                                                         LevelCtl* out, uint64_t* ctr) {
  const uint64_t n = out->log_n;
  const int lane = __lane_id();
  const uint64_t wave = (static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x) >> 6;
  const uint64_t n_waves = (static_cast<uint64_t>(gridDim.x) * blockDim.x) >> 6;
  LaneStats st;
  bool full = false, seen = false;
  for (uint64_t base = wave * 64; base < n; base += n_waves * 64) {
    const uint64_t idx = base + lane;
    const bool act = idx < n;
    uint32_t key[S];
#pragma unroll
    for (int x = 0; x < S; ++x) key[x] = 0;
    if (act) load_slot<S>(log + idx * S, key);
    const uint8_t r = find_or_put_quads<S, B>(t, key, act, st);
    full |= act && r == kFull;
    seen |= act && r != kNew && r != kFull;
    if (idx == 0) out->init_status = r;
  }
  if (__ballot(full) && lane == 0) atomicOr(ctr_at(ctr, kCtrFlags), kFlagTableFull);
  if (__ballot(seen) && lane == 0) atomicOr(ctr_at(ctr, kCtrFlags), kFlagNotEmpty);
  flush_stats(t, st, nullptr);
}

template <int S, int B>
hipError_t launch_lds_b(const SmallArgs& a, size_t lds, hipStream_t s) {
  const void* k = reinterpret_cast<const void*>(&lds_levels_kernel<S, B>);
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((lds_levels_kernel<S, B>), dim3(1), dim3(small_threads<S>()), lds, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the launch places its log itself when the table's fill counts fit the
  // set's LDS (the test place_log's caller makes)
  if (lds_places<S>(a.t.n_buckets, a.set_mask + 1)) return hipSuccess;
  // else the logged states (at most three quarters of the set) into the table
  const uint32_t grid = static_cast<uint32_t>(
      std::min<uint64_t>(256, (static_cast<uint64_t>(a.set_mask) + 1) / 256 + 1));
  hipLaunchKernelGGL((log_insert_kernel<S, B>), dim3(grid), dim3(256), 0, s, a.t, a.log,
                     a.out, a.ctr);
  return hipGetLastError();
}

// Launch the LDS-resident first levels with the largest visited set that fits
// lds_limit bytes of LDS, then the insertion of the states they logged;
// returns hipErrorInvalidValue (nothing launched) when not even 2^10 entries
// fit.
template <int S>
hipError_t launch_lds_levels(uint32_t B, SmallArgs a, size_t lds_limit, hipStream_t s) {
  const LdsPlan plan = lds_plan<S>(a.img_stride, a.limit, lds_limit);
  if (plan.set_bits < 10) return hipErrorInvalidValue;
  a.set_mask = (1u << plan.set_bits) - 1u;
  a.ring = plan.ring;
  switch (B) {
    case 4: return launch_lds_b<S, 4>(a, plan.bytes, s);
    case 8: return launch_lds_b<S, 8>(a, plan.bytes, s);
    case 16: return launch_lds_b<S, 16>(a, plan.bytes, s);
    case 32: return launch_lds_b<S, 32>(a, plan.bytes, s);
    case 64: return launch_lds_b<S, 64>(a, plan.bytes, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gx
