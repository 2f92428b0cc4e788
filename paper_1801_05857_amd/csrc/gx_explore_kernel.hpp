// Expansion of BFS levels: successor generation from the network image and
// find-or-put of the successors in one kernel, for one slot width S; each
// slot width is instantiated in a translation unit of its own.
#pragma once

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "gx_internal.hpp"

namespace gx {

// ------------------------------------------------------------ network image
// 32-bit words, indices absolute within the image:
//   [0] items  [2] S  [3] words per state
//   [4 + 4 i .. 4 i + 7]  item i: one process's free transitions, or one rule
//       {outer, outer offsets, field, offsets}: the item's last participant
//       (its only one: outer = 0) by its field (word | shift << 8 | width <<
//       16) and the index of its offsets; outer: the field of the other
//       participant of a two-party rule and the index of its offsets, or
//       kItemGeneral and the index of a record (participants before the last,
//       then per participant field, index of its offsets)
//   offsets arrays: n_q + 1 entries each; entry l is the index of local state
//                   l's list, entry l+1 one past its end
//   lists:          distinct target local states, shifted to their field's
//                   position; where that leaves out transitions (several to
//                   one target; a process's own steps that change nothing,
//                   whose successor is the state itself) the entry has
//                   kListCounted set and the list begins with the number of
//                   transitions it stands for
// Items that no local state offers anything for are left out.
constexpr uint32_t kItemGeneral = 0xFFFFFFFFu;
constexpr uint32_t kListCounted = 0x80000000u;
// A network whose transition tables take more than kImgMaxWords words (46
// KiB) is read from global memory; an image that stays in LDS takes at most
// kImgStoreWords (its items take up to that many words more).
constexpr uint32_t kImgMaxWords = 11776;
constexpr uint32_t kImgStoreWords = kImgMaxWords + 2048;

enum : uint32_t { kFlagFrontierOverflow = 1, kFlagTableFull = 2 };

// Field access with mask arithmetic only: a select chain over the words is
// folded by the compiler into an indexed load from a private array, which
// would live in scratch memory.  (Bit-field instructions use the low five bits
// of a shift and a width.)
template <int S>
__device__ __forceinline__ uint32_t get_field(const uint32_t (&sw)[S], uint32_t f) {
  uint32_t x = sw[0];
  if constexpr (S == 2) {
    x ^= (sw[0] ^ sw[1]) & (0u - (f & 1u));
  } else if constexpr (S == 4) {
    const uint32_t lo = 0u - (f & 1u), hi = 0u - ((f >> 1) & 1u);
    const uint32_t a = sw[0] ^ ((sw[0] ^ sw[1]) & lo), b = sw[2] ^ ((sw[2] ^ sw[3]) & lo);
    x = a ^ ((a ^ b) & hi);
  }
  return __builtin_amdgcn_ubfe(x, f >> 8, f >> 16);
}

// Field f of the state set to v, which is shifted to the field's position.
template <int S>
__device__ __forceinline__ void put_field(uint32_t (&sw)[S], uint32_t f, uint32_t v) {
  const uint32_t m = ((1u << (f >> 16)) - 1u) << ((f >> 8) & 31u);
  if constexpr (S == 1) {
    sw[0] = (sw[0] & ~m) | v;
  } else {
    const uint32_t word = f & 0xFF;
#pragma unroll
    for (int t = 0; t < S; ++t) {
      const uint32_t sel = 0u - static_cast<uint32_t>(word == static_cast<uint32_t>(t));
      sw[t] = (sw[t] & ~(m & sel)) | (v & sel);
    }
  }
}

template <int S>
__device__ __forceinline__ void load_slot(const uint32_t* p, uint32_t (&k)[S]) {
  if constexpr (S == 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(p);
    k[0] = v.x;
    k[1] = v.y;
    k[2] = v.z;
    k[3] = v.w;
  } else if constexpr (S == 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    k[0] = v.x;
    k[1] = v.y;
  } else {
    k[0] = *p;
  }
}

template <int S>
__device__ __forceinline__ void store_slot(uint32_t* p, const uint32_t (&k)[S]) {
  if constexpr (S == 4) {
    *reinterpret_cast<uint4*>(p) = make_uint4(k[0], k[1], k[2], k[3]);
  } else if constexpr (S == 2) {
    *reinterpret_cast<uint2*>(p) = make_uint2(k[0], k[1]);
  } else {
    *p = k[0];
  }
}

// Orders the LDS accesses of one wavefront (its lanes exchange staged
// successors through LDS; no other wavefront touches that region).
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Rank of this lane among the lanes of m.
__device__ __forceinline__ uint32_t lane_rank(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// Local state l's list: its first target's index, its targets, the
// transitions they stand for.
struct TargetList {
  uint32_t first, n, total;
};
__device__ __forceinline__ TargetList target_list(const uint32_t* img, uint32_t offsets,
                                                  uint32_t l) {
  const uint32_t e0 = img[offsets + l], e1 = img[offsets + l + 1];
  TargetList t;
  t.first = (e0 & ~kListCounted) + (e0 >> 31);
  t.n = (e1 & ~kListCounted) - t.first;
  const uint32_t count = img[t.first - 1];  // (a list's index is never 0)
  t.total = e0 >> 31 ? count : t.n;
  return t;
}

// The outer participants of an item's combination c written into mid.
template <int S>
__device__ __forceinline__ void put_outer(const uint32_t* img, const uint4& it,
                                          const uint32_t (&sw)[S], uint32_t a0, uint32_t c,
                                          uint32_t (&mid)[S]) {
  if (it.x != kItemGeneral) {
    put_field<S>(mid, it.x, img[a0 + c]);
    return;
  }
  const uint32_t np = img[it.y];
  uint32_t rem = c;
  for (uint32_t i = 0; i < np; ++i) {
    const uint32_t f = img[it.y + 1 + 2 * i], ob = img[it.y + 2 + 2 * i];
    const TargetList t = target_list(img, ob, get_field<S>(sw, f));
    put_field<S>(mid, f, img[t.first + rem % t.n]);
    rem /= t.n;
  }
}

// The successors of the wavefront's states, appended to stage[cnt * S ..] (the
// wavefront's own LDS); sink() is called, by the whole wavefront, whenever
// more than `limit` are staged, and lowers cnt.  q lanes (a power of two)
// share a state, lane `sub` of them taking items sub, sub + q, ...: with few
// states the walk of a state's items, a chain of dependent LDS reads each,
// is spread over the lanes that would otherwise idle.  The lanes walk in
// step: every loop runs until no lane has work left in it (its exit test is a
// ballot, so the wavefront never splits), and at each step the lanes that
// form a successor take consecutive places.  Nothing is counted beforehand:
// the walk stops at any point to have the staged successors taken and goes
// on.  Several transitions to one successor form it once, and a step that
// changes nothing forms none: at random targets among 6 local states, 3
// transitions a state, that leaves 2.1 of 3 successors to look up.  Must be
// reached by the whole wavefront; a lane without a state passes has = false.
// Returns the number of this lane's transitions.
template <int S, typename Sink>
__device__ __forceinline__ uint32_t walk_items(const uint32_t* img, const uint32_t (&sw)[S],
                                               bool has, uint32_t sub, uint32_t q,
                                               uint32_t* stage, uint32_t& cnt, uint32_t limit,
                                               Sink&& sink) {
  const uint32_t n_items = uniform32(img[0]);
  uint32_t own = 0;
  for (uint32_t i0 = 0; i0 < n_items; i0 += q) {
    const uint32_t i = i0 + sub;
    const bool valid = has && i < n_items;
    const uint4 it = *reinterpret_cast<const uint4*>(img + 4 + 4 * (i < n_items ? i : 0));
    const TargetList in = target_list(img, it.w, get_field<S>(sw, it.z));
    const uint32_t b0 = in.first, bend = in.first + in.n;
    uint32_t outer = 1, a0 = 0, total = in.total;
    if (it.x) {
      if (it.x != kItemGeneral) {
        const TargetList t = target_list(img, it.y, get_field<S>(sw, it.x));
        a0 = t.first;
        outer = t.n;
        total *= t.total;
      } else {
        const uint32_t np = img[it.y];
        for (uint32_t k = 0; k < np; ++k) {
          const uint32_t f = img[it.y + 1 + 2 * k], ob = img[it.y + 2 + 2 * k];
          const TargetList t = target_list(img, ob, get_field<S>(sw, f));
          outer *= t.n;
          total *= t.total;
        }
      }
    }
    uint32_t left = valid ? in.n * outer : 0u;  // successors the item has yet to form
    own += valid ? total : 0u;
    uint32_t mid[S];
#pragma unroll
    for (int x = 0; x < S; ++x) mid[x] = sw[x];
    put_field<S>(mid, it.z, 0u);
    if (left && it.x) put_outer<S>(img, it, sw, a0, 0u, mid);
    uint32_t b = b0, c = 0;
    uint32_t tgt = img[left ? b : 0u];
    while (true) {
      const uint64_t m = __ballot(left != 0);
      if (!m) break;
      if (left) {
        uint32_t succ[S];
#pragma unroll
        for (int x = 0; x < S; ++x)
          succ[x] = mid[x] | (S == 1 || (it.z & 0xFF) == static_cast<uint32_t>(x) ? tgt : 0u);
        store_slot<S>(stage + (cnt + lane_rank(m)) * S, succ);
        ++b;
        --left;
        if (left && b == bend) {
          ++c;
          b = b0;
          put_outer<S>(img, it, sw, a0, c, mid);
        }
        tgt = img[left ? b : 0u];
      }
      cnt += static_cast<uint32_t>(__popcll(m));
      if (cnt > limit) sink();
    }
  }
  return own;
}

// An exploration's counters live kCtrSpread words apart, each on a cache
// line of its own: every workgroup of a level updates some of them, and
// counters sharing a line would serialise at one L2 atomic unit.
constexpr uint32_t kCtrSpread = 16;
enum : uint32_t { kCtrTail = 0, kCtrDead = 1, kCtrTrans = 2, kCtrFlags = 3, kCtrDups = 4,
                  kCtrTailAlt = 5, kCtrViol = 6, kCtrViolLevel = 7, kCtrCount = 8 };

__device__ __forceinline__ unsigned long long* ctr_at(uint64_t* ctr, uint32_t k) {
  return reinterpret_cast<unsigned long long*>(ctr + k * kCtrSpread);
}

// A tail's upper bits count the workgroups that have finished with a level
// (levels that the device strings together, see LevelArgs).
constexpr uint32_t kArriveShift = 48;
constexpr uint64_t kTailMask = (uint64_t(1) << kArriveShift) - 1;

// LDS of a wavefront: kWaveKeys keys.  Staged successors grow from the front
// (at most 127: probed 64 at a time), NEW states from the back (at most 127:
// they leave 64 at a time).
constexpr uint32_t kWaveKeys = 192;
// With the local duplicate filter: kFilterKeys staged successors, 128 NEW
// states and the filter's hash set, twice as many entries as staged keys, so
// it is never more than half full.
template <int S>
__host__ __device__ constexpr uint32_t filter_keys() {
  return 1024u / S;
}
template <int S, bool kFilter>
__host__ __device__ constexpr uint32_t wave_words() {
  return kFilter ? (filter_keys<S>() + 128u) * S + 2u * filter_keys<S>() : kWaveKeys * S;
}

// A BFS level of one exploration, as one wavefront sees it.
struct WaveJob {
  TableDev t;
  const uint32_t* img;  // network image
  const uint32_t* frontier_in;
  uint64_t n_in;
  uint32_t* frontier_out;
  uint64_t cap_out;
  uint32_t* dead;       // deadlock states (S words each)
  uint32_t* dead_tag;   // nullable: per deadlock record, the exploration's tag
  uint32_t tag;
  uint64_t dead_cap;
  uint64_t* dead_ctr;   // deadlock records used (may be shared by explorations)
  uint64_t* ctr;
  uint32_t tail;        // the level's tail: kCtrTail or kCtrTailAlt
};

// What a wavefront has not yet handed over.
struct WaveAcc {
  LaneStats st;
  uint32_t n_new = 0;       // NEW states at the back of its LDS
  uint32_t flags = 0;
  uint32_t dups = 0;        // this lane's
  uint64_t trans = 0;       // this lane's transitions
};

// Hash of a staged successor for the duplicate filter (any mix will do: it
// only spreads the chunk over the filter's entries).
template <int S>
__device__ __forceinline__ uint32_t dedup_hash(const uint32_t (&k)[S]) {
  uint32_t h = 0x9E3779B9u;
#pragma unroll
  for (int x = 0; x < S; ++x) h = (h ^ k[x]) * 0x85EBCA6Bu;
  return h ^ (h >> 15);
}

// Local duplicate filter (the block-local state cache of the tool, Sec. 3):
// the first occurrence of a successor among the n_st staged ones claims an
// entry of the wavefront's LDS set `dtab`; later occurrences find it and are
// marked in *dupmask (bit r: this lane's staged index of round r, 64 r +
// lane).  Must be reached by the whole wavefront; the stage is only read.
template <int S>
__device__ inline uint32_t dedup_stage(uint32_t* dtab, const uint32_t* stage, uint32_t n_st) {
  constexpr uint32_t D = 2u * filter_keys<S>();
  const uint32_t lane = __lane_id();
  for (uint32_t e = lane; e < D; e += 64) dtab[e] = kEmpty;
  wave_lds_sync();
  uint32_t mask = 0;
  for (uint32_t r0 = 0, r = 0; r0 < n_st; r0 += 64, ++r) {
    const uint32_t idx = r0 + lane;
    if (idx < n_st) {
      uint32_t key[S];
      load_slot<S>(stage + idx * S, key);
      uint32_t h = dedup_hash<S>(key) & (D - 1);
      while (true) {
        uint32_t prev = kEmpty;
        if (__hip_atomic_compare_exchange_strong(&dtab[h], &prev, idx, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT))
          break;  // first occurrence
        bool same = true;
#pragma unroll
        for (int x = 0; x < S; ++x) same &= stage[prev * S + x] == key[x];
        if (same) {
          mask |= 1u << r;
          break;
        }
        h = (h + 1) & (D - 1);
      }
    }
  }
  wave_lds_sync();
  return mask;
}

// This lane's state of a tile (zero where there is none).
template <int S>
__device__ __forceinline__ void load_tile(const WaveJob& j, uint64_t tile, uint32_t qs,
                                          uint32_t (&sw)[S]) {
  const uint64_t i = tile * (64u >> qs) + (static_cast<uint32_t>(__lane_id()) >> qs);
#pragma unroll
  for (int x = 0; x < S; ++x) sw[x] = 0;
  if (i < j.n_in) load_slot<S>(j.frontier_in + i * S, sw);
}

// Expands tiles tile0, tile0 + stride, ... below n_tiles of a level: 64 >>
// qs frontier states each, 2^qs lanes a state (see walk_items).  Generation
// and probes share the wavefront: the successors pass through its LDS only
// (a successor buffer in memory between two kernels cost a write and a read
// of every successor, a fifth of the probes' own traffic, and two launches
// and their latencies a level).  Bound by random 64-byte reads, as
// find_or_put_quads; the wavefronts of a SIMD overlap one's walk with the
// others' reads.  NEW states leave the LDS 64 at a time, with one atomic add
// and one coalesced store; what is left goes out with the workgroup's
// (finish_block).  sw: tile0's states (load_tile), read before the caller
// waited for the image.  Must be reached by the whole wavefront.
template <int S, int B, bool kFilter>
__device__ __forceinline__ void expand_tiles(const WaveJob& j, uint32_t* lds, uint64_t tile0,
                                             uint64_t n_tiles, uint64_t stride, uint32_t qs,
                                             uint32_t (&sw)[S], WaveAcc& acc) {
  constexpr uint32_t kStageKeys = kFilter ? filter_keys<S>() : kWaveKeys;
  constexpr uint32_t kTop = kFilter ? filter_keys<S>() + 128u : kWaveKeys;  // end of the NEW keys
  const uint32_t lane = __lane_id();
  uint32_t* stage = lds;
  uint32_t* dtab = lds + kTop * S;  // (with the filter)
  uint32_t cnt = 0;

  // the NEW states' last 64, or all that are left
  auto flush = [&]() {
    wave_lds_sync();
    acc.n_new -= 64;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(ctr_at(j.ctr, j.tail), 64ull);
    base = uniform64(base) & kTailMask;
    if (base + 64 > j.cap_out) acc.flags |= kFlagFrontierOverflow;
    if (base + lane < j.cap_out) {
      uint32_t key[S];
      load_slot<S>(lds + (kTop - 1 - acc.n_new - lane) * S, key);
      store_slot<S>(j.frontier_out + (base + lane) * S, key);
    }
    wave_lds_sync();
  };
  // find-or-put of staged keys [at, at + 64) (those where act)
  auto probe = [&](uint32_t at, bool act) {
    uint32_t key[S];
#pragma unroll
    for (int x = 0; x < S; ++x) key[x] = 0;
    if (act) load_slot<S>(stage + (at + lane) * S, key);
    const uint8_t r = find_or_put_quads<S, B>(j.t, key, act, acc.st);
    const bool is_new = act && r == kNew;
    if (__any(act && r == kFull)) acc.flags |= kFlagTableFull;
    const uint64_t m = __ballot(is_new);
    if (is_new) store_slot<S>(lds + (kTop - 1 - acc.n_new - lane_rank(m)) * S, key);
    acc.n_new += static_cast<uint32_t>(__popcll(m));
    if (acc.n_new >= 64) flush();
  };
  auto take = [&]() {
    wave_lds_sync();
    if constexpr (kFilter) {
      const uint32_t mask = dedup_stage<S>(dtab, stage, cnt);
      acc.dups += static_cast<uint32_t>(__popc(mask));
      for (uint32_t r0 = 0, r = 0; r0 < cnt; r0 += 64, ++r)
        probe(r0, r0 + lane < cnt && !((mask >> r) & 1u));
      cnt = 0;
    } else {
      const uint32_t n = cnt < 64 ? cnt : 64u;
      cnt -= n;
      probe(cnt, lane < n);
    }
    wave_lds_sync();  // read before the stage is written again
  };

  const uint32_t q = 1u << qs;
  const uint32_t sub = lane & (q - 1);
  const uint32_t per = 64u >> qs;  // states per tile
  for (uint64_t tile = tile0; tile < n_tiles; tile += stride) {
    const uint64_t i = tile * per + (lane >> qs);
    const bool has = i < j.n_in;
    const uint32_t own = walk_items<S>(j.img, sw, has, sub, q, stage, cnt,
                                       kFilter ? kStageKeys - 64u : 63u, take);
    acc.trans += own;
    // a state none of whose lanes found a successor is a deadlock
    const uint64_t m = __ballot(own != 0);
    const uint64_t mine = (m >> (lane & ~(q - 1))) & (q == 64 ? ~0ull : (1ull << q) - 1ull);
    if (has && sub == 0 && mine == 0) {
      const uint64_t d = atomicAdd(reinterpret_cast<unsigned long long*>(j.dead_ctr), 1ull);
      if (j.dead_ctr != reinterpret_cast<uint64_t*>(ctr_at(j.ctr, kCtrDead)))
        atomicAdd(ctr_at(j.ctr, kCtrDead), 1ull);
      if (d < j.dead_cap) {
        // read again: the walk's registers need not keep it
        uint32_t k[S];
        load_slot<S>(j.frontier_in + i * S, k);
        store_slot<S>(j.dead + d * S, k);
        if (j.dead_tag) j.dead_tag[d] = j.tag;
      }
    }
    if (tile + stride < n_tiles) load_tile<S>(j, tile + stride, qs, sw);
  }
  if (cnt) take();
}

// (values below 2^50)
__device__ inline uint64_t wave_sum64(uint64_t x) {
  return wave_sum(static_cast<uint32_t>(x) & 0xFFFFFFu) +
         (static_cast<uint64_t>(wave_sum(static_cast<uint32_t>(x >> 24))) << 24);
}

// The workgroup's wavefronts hand over what they hold: NEW states, transition
// and duplicate counts, flags and (kStats) the table's statistics.  One atomic
// of each kind per workgroup, all issued together: each takes about half a
// microsecond, which a small level would otherwise spend several times.
// `arrive` (0 or 1 << kArriveShift) is added to the tail with the NEW states;
// returns (to thread 0) the tail before and, in *n_new, what was added to it.
// Every thread of the workgroup must come here, its wavefront's expand_tiles
// done; lds: this wavefront's region.
template <int S, bool kFilter, bool kStats>
__device__ __forceinline__ uint64_t finish_block(const WaveJob& j, const uint32_t* lds,
                                                 WaveAcc& acc, uint64_t arrive, uint64_t* n_new) {
  constexpr uint32_t kTop = kFilter ? filter_keys<S>() + 128u : kWaveKeys;
  enum : uint32_t { kNewStates, kFlags, kDups, kProbes, kMaxJ, kStored, kFulls, kRows };
  __shared__ uint32_t sh[kRows][16];
  __shared__ uint64_t sh_trans[16];
  __shared__ unsigned long long sh_base;
  const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  const uint32_t lane = __lane_id();
  const uint64_t trans = wave_sum64(acc.trans);
  const uint32_t dups = kFilter ? wave_sum(acc.dups) : 0u;
  uint32_t probes = 0, max_j = 0;
  if constexpr (kStats) {
    probes = wave_sum(acc.st.probes);
    max_j = wave_max(acc.st.max_j);
  }
  if (lane == 0) {
    sh[kNewStates][wave] = acc.n_new;
    sh[kFlags][wave] = acc.flags;
    sh_trans[wave] = trans;
    if (kFilter) sh[kDups][wave] = dups;
    if constexpr (kStats) {
      sh[kProbes][wave] = probes;
      sh[kMaxJ][wave] = max_j;
      sh[kStored][wave] = acc.st.stored;
      sh[kFulls][wave] = acc.st.full;
    }
  }
  __syncthreads();
  uint64_t before = 0;
  if (threadIdx.x == 0) {
    uint64_t t = 0, n = 0, d = 0;
    uint32_t f = 0;
    for (uint32_t w = 0; w < waves; ++w) {
      n += sh[kNewStates][w];
      f |= sh[kFlags][w];
      t += sh_trans[w];
      if (kFilter) d += sh[kDups][w];
    }
    if (f) {
      // before the arrival: the last workgroup to arrive reads the flags
      const auto old = atomicOr(ctr_at(j.ctr, kCtrFlags), static_cast<unsigned long long>(f));
      asm volatile("s_waitcnt vmcnt(0)" ::"v"(static_cast<uint32_t>(old)) : "memory");
    }
    if (t) atomicAdd(ctr_at(j.ctr, kCtrTrans), static_cast<unsigned long long>(t));
    if (d) atomicAdd(ctr_at(j.ctr, kCtrDups), static_cast<unsigned long long>(d));
    if (n + arrive) before = atomicAdd(ctr_at(j.ctr, j.tail), n + arrive);
    sh_base = before & kTailMask;
    *n_new = n;
    if ((before & kTailMask) + n > j.cap_out)
      atomicOr(ctr_at(j.ctr, kCtrFlags), static_cast<unsigned long long>(kFlagFrontierOverflow));
  }
  if constexpr (kStats) {
    // (threads of the second wavefront, beside the first one's)
    const uint32_t k = threadIdx.x - 64u;
    if (k < 5 && j.t.counters != nullptr) {
      // (every transition counts as a lookup, the ones known to find their
      // state among them, but for what the filter dropped)
      const uint32_t row = k == 0 ? kStored : k == 2 ? kProbes : k == 3 ? kFulls : kMaxJ;
      const uint32_t to = k == 4 ? kCntMaxJ : k;
      uint64_t x = 0;
      for (uint32_t w = 0; w < waves; ++w) {
        const uint64_t y = k == 1 ? sh_trans[w] - (kFilter ? sh[kDups][w] : 0u) : sh[row][w];
        x = k == 4 ? (y > x ? y : x) : x + y;
      }
      auto* c = reinterpret_cast<unsigned long long*>(
          j.t.counters + static_cast<uint64_t>(blockIdx.x % j.t.ctr_slots) * kNumCounters + to);
      if (x) {
        if (k == 4) atomicMax(c, static_cast<unsigned long long>(x));
        else atomicAdd(c, static_cast<unsigned long long>(x));
      }
    }
  }
  __syncthreads();
  uint64_t base = sh_base;
  for (uint32_t w = 0; w < wave; ++w) base += sh[kNewStates][w];
  for (uint32_t k = lane; k < acc.n_new; k += 64) {
    if (base + k < j.cap_out) {
      uint32_t key[S];
      load_slot<S>(lds + (kTop - 1 - k) * S, key);
      store_slot<S>(j.frontier_out + (base + k) * S, key);
    }
  }
  acc.n_new = 0;
  return before;
}
static_assert(kCntStored == 0 && kCntLookups == 1 && kCntProbes == 2 && kCntFull == 3 &&
                  kCntMaxJ == 5,
              "counter order");

// ------------------------------------------------------- a level's kernel
constexpr uint32_t kLevelBlock = 512;  // threads per workgroup
constexpr uint32_t kChainLevels = 64;  // level sizes a control block holds

// A level yet to be searched for violations: by the scan that follows the
// launch, or (more states than the buffer has room for records) by the host.
constexpr uint32_t kScanHere = 1, kScanHost = 2;
constexpr uint32_t kNoMonitor = 0xFFFFFFFFu;

// What the device leaves for the host between read-backs (after the level
// counters).
struct LevelCtl {
  uint64_t n_levels;     // levels completed since the last read-back; their sizes follow
  uint64_t n_in;         // size of the current level (0: the exploration is over)
  uint64_t cur;          // the frontier buffer holding it
  uint64_t init_status;  // find-or-put status of the initial state (when inserted)
  uint64_t log_n;        // LDS-resident launch: states it logged (they go into the table)
  // levels strung together: launch k of a string reads entry k & 1 and leaves
  // the next level in the other one, so that a workgroup that starts late
  // still finds the entry of its own launch (read in one piece)
  struct alignas(64) Entry {
    uint64_t n_in, cur, n_levels;
    uint32_t go;     // the exploration's number if the device may expand it, else 0
    uint32_t fresh;  // found by the launch that wrote the entry
    uint32_t scan;   // with a monitor, who searches the level: kScanHere, kScanHost or 0
  } entry[2];
  uint64_t levels[kChainLevels];
};

struct LevelArgs {
  TableDev t;
  const uint32_t* img;    // global memory (copied to LDS unless the kernel reads it there)
  uint32_t img_words;
  uint32_t img_stride;    // LDS words of the image: img_words rounded up to 4, or 0
  uint32_t* f[2];         // the two frontier buffers
  uint64_t cap_out;       // states the next level's buffer takes
  uint32_t* dead;
  uint64_t dead_cap;
  uint64_t* ctr;          // kCtrCount counters, kCtrSpread words apart (see ctr_at)
  uint32_t tail;          // this level's tail, zero before its first launch
  uint32_t waves;         // wavefronts the device holds at once
  uint32_t max_qs;        // log2 of the most lanes a state is worth
  // states [first, first + n_in) of buffer cur
  uint32_t cur;
  uint64_t first, n_in;
  // ctl set: launch `link` of a string of levels (see LevelCtl); with `given`
  // it takes the level above, else the control block's.  A level of more than
  // `limit` states, or more than the deadlock buffer has room for, is left
  // to the host.
  LevelCtl* ctl;
  uint32_t link;
  uint32_t given;
  uint32_t number;  // the exploration's, not 0
  uint64_t limit;
  // set: kReports words of host memory; a launch that takes its level from
  // the control block says there, as it starts, which one that is (see
  // level_report), and the control block keeps no level sizes.  A launch that
  // has nothing to expand copies the counters and the control block (they
  // follow them) to host_block, block_words words of host memory.
  uint64_t* report;
  uint64_t* host_block;
  uint32_t block_words;
  uint32_t viol_cap;  // records the violation buffer takes; kNoMonitor: no monitor
};

// What a launch reports: its link plus one (16 bits), whether it expands the
// level, whether the launch before it found the level, the level's size.
constexpr uint32_t kReports = 64;
constexpr uint64_t kReportGo = uint64_t(1) << 47, kReportFresh = uint64_t(1) << 46;
__device__ __forceinline__ void level_report(uint64_t* report, uint32_t link, uint64_t go,
                                             uint32_t fresh, uint64_t n_in) {
  const uint64_t w = static_cast<uint64_t>((link + 1) & 0xFFFFu) << 48 | go |
                     (fresh ? kReportFresh : 0) | (n_in & (kReportFresh - 1));
  __hip_atomic_store(report + link % kReports, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The workgroup copies words of device memory to host memory that the host
// reads once a report of the same workgroup has told it to.
__device__ inline void copy_to_host(uint64_t* host, const uint64_t* words, uint32_t n) {
  for (uint32_t k = threadIdx.x; k < n; k += blockDim.x)
    __hip_atomic_store(host + k,
                       __hip_atomic_load(words + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  __syncthreads();
}

// log2 of the lanes per state: as many as keep the device's wavefronts busy.
__host__ __device__ inline uint32_t lanes_per_state(uint64_t n_in, uint32_t waves, uint32_t max_qs) {
  const uint32_t all = waves * 64u;
  if (n_in > all / 2) return 0;
  const uint32_t n = n_in ? static_cast<uint32_t>(n_in) : 1u;
  uint32_t qs = static_cast<uint32_t>(__builtin_clz(n) - __builtin_clz(all));
  if (n << qs > all) --qs;
  return qs < max_qs ? qs : max_qs;
}

// Tiles of n states, 2^qs lanes each.
__host__ __device__ inline uint64_t tiles_of(uint64_t n, uint32_t qs) {
  return (n + (64u >> qs) - 1) >> (6 - qs);
}

// One BFS level (or a slice of it).  Levels that need no decision of the host
// are strung together: launches that take the current level's size and buffer
// from the control block follow each other on the stream with no read-back
// between them, and the workgroup that finishes a level last writes the next
// one's entry (1.6 us from one launch to the next, about 20 for a read-back).
// A launch that finds nothing to do, because the exploration is over or the
// level needs the host, ends at once.
template <int S, int B, bool kFilter, bool kGlobalImg>
__global__ __launch_bounds__(kLevelBlock) void level_kernel(LevelArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  uint64_t n_in = a.n_in, first = a.first;
  uint32_t cur = a.cur;
  // (the image's first words are on their way while the level's entry is read)
  uint32_t head = 0;
  if constexpr (!kGlobalImg) {
    if (threadIdx.x < a.img_words) head = a.img[threadIdx.x];
  }
  if (a.ctl != nullptr) {
    if (!a.given) {
      const LevelCtl::Entry& e = a.ctl->entry[a.link & 1u];
      if (e.go != a.number) {
        // (The host may return on the report of a string's last launch: what
        // is left of it then are workgroups that read an entry and end.  An
        // entry written since has another exploration's number.)
        if (blockIdx.x == 0) {
          if (threadIdx.x == 0) {
            LevelCtl::Entry& next = a.ctl->entry[(a.link & 1u) ^ 1u];
            next = e;
            next.fresh = 0;
            if (e.scan == kScanHere) next.scan = 0;
          }
          if (a.report != nullptr) {
            copy_to_host(a.host_block, a.ctr, a.block_words);
            if (threadIdx.x == 0) level_report(a.report, a.link, 0, e.fresh, e.n_in);
          }
        }
        return;
      }
      if (a.report != nullptr && blockIdx.x == 0 && threadIdx.x == 0)
        level_report(a.report, a.link, kReportGo, e.fresh, e.n_in);
      n_in = uniform64(e.n_in);
      cur = uniform32(static_cast<uint32_t>(e.cur));
    }
  } else if (blockIdx.x == 0 && threadIdx.x == 0) {
    *ctr_at(a.ctr, a.tail == kCtrTail ? kCtrTailAlt : kCtrTail) = 0;  // the next level's
  }
  constexpr uint32_t kWaves = kLevelBlock / 64;
  const uint32_t qs = lanes_per_state(n_in, a.waves, a.max_qs);
  const uint64_t n_tiles = tiles_of(n_in, qs);
  const uint64_t groups = min(static_cast<uint64_t>(gridDim.x), (n_tiles + kWaves - 1) / kWaves);
  if (blockIdx.x >= groups) return;
  const uint32_t wave = threadIdx.x >> 6;
  uint32_t* lds = smem + a.img_stride + wave * wave_words<S, kFilter>();
  WaveJob j;
  j.t = a.t;
  j.img = kGlobalImg ? a.img : smem;
  j.frontier_in = a.f[cur] + first * S;
  j.n_in = n_in;
  j.frontier_out = a.f[cur ^ 1u];
  j.cap_out = a.cap_out;
  j.dead = a.dead;
  j.dead_tag = nullptr;
  j.tag = 0;
  j.dead_cap = a.dead_cap;
  j.dead_ctr = reinterpret_cast<uint64_t*>(ctr_at(a.ctr, kCtrDead));
  j.ctr = a.ctr;
  j.tail = a.tail;
  WaveAcc acc;
  // neighbouring workgroups take neighbouring tiles at the same time
  const uint64_t tile0 = static_cast<uint64_t>(blockIdx.x) + wave * groups;
  uint32_t sw[S];
  load_tile<S>(j, tile0, qs, sw);
  if constexpr (!kGlobalImg) {
    if (threadIdx.x < a.img_words) smem[threadIdx.x] = head;
    for (uint32_t k = threadIdx.x + kLevelBlock; k < a.img_words; k += kLevelBlock)
      smem[k] = a.img[k];
  }
  __syncthreads();
  expand_tiles<S, B, kFilter>(j, lds, tile0, n_tiles, groups * kWaves, qs, sw, acc);
  uint64_t n_new = 0;
  const uint64_t before = finish_block<S, kFilter, true>(
      j, lds, acc, a.ctl != nullptr ? uint64_t(1) << kArriveShift : 0, &n_new);
  if (a.ctl != nullptr && threadIdx.x == 0 && (before >> kArriveShift) + 1 == groups) {
    // every workgroup has arrived: the level's NEW states are all counted
    auto* tail = ctr_at(a.ctr, a.tail);
    const uint64_t n_next = (before & kTailMask) + n_new;
    __hip_atomic_store(tail, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    auto counter = [&](uint32_t k) {
      return __hip_atomic_load(ctr_at(a.ctr, k), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    uint64_t flags = counter(kCtrFlags);
    const uint64_t dead = counter(kCtrDead);
    const bool monitor = a.viol_cap != kNoMonitor;
    const uint64_t viol = monitor ? counter(kCtrViol) : 0;
    uint64_t n_levels = a.ctl->entry[a.link & 1u].n_levels;
    if (a.given) n_levels = 0;
    if (n_next > a.cap_out) {
      atomicOr(ctr_at(a.ctr, kCtrFlags), static_cast<unsigned long long>(kFlagFrontierOverflow));
      flags |= kFlagFrontierOverflow;
    }
    const bool recorded = !monitor || viol + n_next <= a.viol_cap;
    if (n_next) {
      if (a.report == nullptr) a.ctl->levels[n_levels] = n_next;
      ++n_levels;
    }
    LevelCtl::Entry& e = a.ctl->entry[(a.link & 1u) ^ 1u];
    e.n_in = n_next;
    e.cur = cur ^ 1u;
    e.n_levels = n_levels;
    e.fresh = flags == 0;
    e.scan = !monitor || flags != 0 || n_next == 0 ? 0u : recorded ? kScanHere : kScanHost;
    e.go = flags == 0 && n_next > 0 && n_next <= a.limit && recorded &&
                   (a.report != nullptr || n_levels < kChainLevels) && n_next <= a.dead_cap - min(dead, a.dead_cap)
               ? a.number
               : 0u;
  }
}

template <int S, int B, bool kFilter, bool kGlobalImg>
hipError_t launch_level_k(const LevelArgs& a, uint32_t grid, size_t lds, hipStream_t s) {
  if (lds > 65536) {  // more than the default per-workgroup LDS: ask for it
    const hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&level_kernel<S, B, kFilter, kGlobalImg>),
        hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((level_kernel<S, B, kFilter, kGlobalImg>), dim3(grid), dim3(kLevelBlock), lds,
                     s, a);
  return hipGetLastError();
}

// LDS bytes of a level's workgroup.
template <int S>
size_t level_lds(uint32_t img_stride, bool filter) {
  const uint32_t w = filter ? wave_words<S, true>() : wave_words<S, false>();
  return (static_cast<size_t>(img_stride) + w * (kLevelBlock / 64)) * sizeof(uint32_t);
}

// Workgroups of a level that a compute unit holds at once.
template <int S>
uint32_t level_blocks_per_cu(uint32_t B, size_t lds) {
  int b = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (B) {
#define GX_LEVEL_CASE(BB)                                                                  \
  case BB:                                                                                 \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, level_kernel<S, BB, false, false>, \
                                                     kLevelBlock, lds);                    \
    break;
    GX_LEVEL_CASE(4)
    GX_LEVEL_CASE(8)
    GX_LEVEL_CASE(16)
    GX_LEVEL_CASE(32)
    GX_LEVEL_CASE(64)
#undef GX_LEVEL_CASE
  }
  if (e != hipSuccess || b <= 0) {
    (void)hipGetLastError();
    return 1;
  }
  return static_cast<uint32_t>(b);
}

template <int S, int B>
hipError_t launch_level_b(const LevelArgs& a, bool filter, uint32_t grid, size_t lds,
                          hipStream_t s) {
  const bool global_img = a.img_stride == 0;
  if (filter)
    return global_img ? launch_level_k<S, B, true, true>(a, grid, lds, s)
                      : launch_level_k<S, B, true, false>(a, grid, lds, s);
  return global_img ? launch_level_k<S, B, false, true>(a, grid, lds, s)
                    : launch_level_k<S, B, false, false>(a, grid, lds, s);
}

// Level launch for slot width S, dispatched over the bucket size.  (The
// probes are those of 4-lane subgroups whatever the table's own width: the
// claim protocol does not depend on how many lanes read a bucket.  64-word
// buckets, read in up to four pieces, stay close to the others: buckets of 16,
// 32 and 64 words, 5.6 M three-word states 2.92, 2.95 and 3.04 ms; 1.3 M
// two-word ring states 1.09 ms and, at 64, 1.24.)
template <int S>
hipError_t launch_level(uint32_t B, const LevelArgs& a, bool filter, uint32_t grid, size_t lds,
                        hipStream_t s) {
  switch (B) {
    case 4: return launch_level_b<S, 4>(a, filter, grid, lds, s);
    case 8: return launch_level_b<S, 8>(a, filter, grid, lds, s);
    case 16: return launch_level_b<S, 16>(a, filter, grid, lds, s);
    case 32: return launch_level_b<S, 32>(a, filter, grid, lds, s);
    case 64: return launch_level_b<S, 64>(a, filter, grid, lds, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace gx
