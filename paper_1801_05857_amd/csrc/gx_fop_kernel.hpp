// Find-or-put kernel and its (B, G, U) dispatch for one slot width S; each
// slot width is instantiated in a translation unit of its own so the
// specialisations compile in parallel.
#pragma once

#include <algorithm>

#include "gx_internal.hpp"

namespace gx {

constexpr uint32_t kLanesPerCu = 2048;  // 8 wavefronts on each of 4 SIMDs
constexpr uint64_t kMeet = 8;           // keys in a bucket that claim at once

// Threads per workgroup, at most.  4-lane subgroups take wide workgroups in
// large launches (their number sets how many atomics meet on n_new).  The
// others hold up to eight keys' buckets in registers and keep to 256 threads:
// 1024 leave a lane 128 registers, and a compute unit whole workgroups of 16
// wavefronts only.  2^23 two-word keys found: buckets of 64 words, eight lanes
// and eight keys 4930 us at 1024 threads, spilling, and 807 at 256; buckets of
// 16 words, 16 lanes and two keys 285 and 218 us.
template <int G>
constexpr uint32_t fop_block() {
  return G == 4 ? 1024u : 256u;
}
// Wavefronts a SIMD must be able to hold: all eight where one key's bucket is
// kept in registers and it is not spread over few lanes.  The compiler counts
// 88 scalar registers as eight wavefronts; from 81 on there are fewer (2^24
// four-word keys found in 8-word buckets by 4 lanes: 459 us at 82, 412 at 78;
// in 16-word buckets by 16 lanes, 2^23 keys, 526 and 330).
template <int S, int B, int G, int U>
constexpr uint32_t fop_waves() {
  return G == 4 || (U == 1 && B / (G < B ? G : B) < 8) ? 8u : 1u;
}

template <int S>
__device__ inline void load_key(const uint32_t* keys, uint32_t w, uint64_t idx,
                                uint32_t (&k)[S]) {
  if constexpr (S == 1) {
    k[0] = keys[idx];
  } else if constexpr (S == 2) {
    uint2 t = reinterpret_cast<const uint2*>(keys)[idx];
    k[0] = t.x;
    k[1] = t.y;
  } else {
    if (w == 4) {
      uint4 t = reinterpret_cast<const uint4*>(keys)[idx];
      k[0] = t.x;
      k[1] = t.y;
      k[2] = t.z;
      k[3] = t.w;
    } else {
      const uint32_t* p = keys + idx * 3;
      k[0] = p[0];
      k[1] = p[1];
      k[2] = p[2];
      k[3] = 0;
    }
  }
}

// One key per lane: a wavefront handles 64 consecutive keys per round (one
// coalesced read of the keys, one coalesced write of the statuses), its
// subgroups probing them U at a time (kTurns: claims in turns, see
// find_or_put_quads).  Grid-stride over rounds.
template <int S, int B, int G, int U, bool kTurns>
__global__ __launch_bounds__(fop_block<G>(), (fop_waves<S, B, G, U>())) void fop_kernel(
    TableDev t, const uint32_t* keys, uint32_t w, uint64_t n, uint8_t* status, uint64_t* n_new,
    uint32_t turns) {
  const int lane = __lane_id();
  const uint32_t local = uniform32(threadIdx.x >> 6);
  const uint64_t wave = static_cast<uint64_t>(blockIdx.x) * (blockDim.x >> 6) + local;
  const uint64_t n_waves = (static_cast<uint64_t>(gridDim.x) * blockDim.x) >> 6;
  LaneStats st;
  for (uint64_t base = wave * 64; base < n; base += n_waves * 64) {
    const uint64_t idx = base + lane;
    const bool act = idx < n;
    uint32_t key[S];
#pragma unroll
    for (int x = 0; x < S; ++x) key[x] = 0;
    if (act) load_key<S>(keys, w, idx, key);
    const uint8_t r = find_or_put_lanes<S, B, G, U, kTurns>(t, key, act, st, turns);
    if (act) status[idx] = r;
  }
  flush_stats_block(t, st, n_new, local);
}


template <int S, int B, int G, int U>
hipError_t launch_fop(const FopArgs& a) {
  // as many workgroups as can be resident at once (grid-stride over rounds);
  // narrow ones while they are few, so that a small launch spreads out
  constexpr uint32_t kBlock = fop_block<G>();
  static int per_cu = 0;
  if (per_cu == 0) {
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, fop_kernel<S, B, G, U, false>, kBlock, 0) !=
            hipSuccess ||
        b <= 0)
      b = 1;
    per_cu = b;
  }
  const uint32_t block = a.n <= static_cast<uint64_t>(a.cus) * 512 ? 256 : kBlock;
  const uint64_t want = (a.n + block - 1) / block;  // one key per thread per round
  const uint64_t resident =
      static_cast<uint64_t>(a.cus) * static_cast<uint32_t>(per_cu) * (kBlock / block);
  // Long launches come as more workgroups than are resident, of 16 rounds or
  // more each, so that those done early make room for others: keys with long
  // hash chains hold up their wavefront.  2^26 two-word keys found in 32-word
  // buckets by 4 lanes, resident workgroups alone and 16 times as many: 1515
  // and 1447 us half full, 6.4 and 4.2 ms full; by 8 lanes 1537 and 1494 us, 9.6
  // and 7.5 ms.  2e6 keys gain nothing (192 us).
  const uint64_t over = std::max<uint64_t>(1, std::min<uint64_t>(16, a.n / (resident * block * 16)));
  uint32_t grid = static_cast<uint32_t>(std::min<uint64_t>(want, resident * over));
  if (grid == 0) grid = 1;
  // 4-lane subgroups, with every key of a round in flight, claim in turns
  // (see find_or_put_quads) once more than kMeet keys of a round meet in a
  // bucket.  2^19 one-word keys into 2^15 empty buckets of 32 words: 147 us
  // all at once, 100 so (146 at 16 keys a bucket, 104 at four); 2^19 two-word
  // keys, 1024 different ones, into 128 buckets: 487 and 160 us; found there
  // 8.6 either way.  (Fewer workgroups instead, as many as bring eight keys a
  // bucket, keep most of the device idle where keys are found: 1475 us.)
  const uint64_t flight = std::min<uint64_t>(a.n, resident * block);
  uint32_t turns = 1;
  while (G == 4 && turns < 64 && flight > turns * kMeet * a.t.n_buckets) turns *= 2;
  // (a kernel of its own: the test for the turn costs the others 1%)
  if (turns > 1)
    hipLaunchKernelGGL((fop_kernel<S, B, G, U, G == 4>), dim3(grid), dim3(block), 0, a.stream, a.t,
                       a.keys, a.w, a.n, a.status, a.n_new, turns - 1);
  else
    hipLaunchKernelGGL((fop_kernel<S, B, G, U, false>), dim3(grid), dim3(block), 0, a.stream, a.t,
                       a.keys, a.w, a.n, a.status, a.n_new, 0u);
  return hipGetLastError();
}

template <int S, int B, int G>
hipError_t dispatch_u(uint32_t U, const FopArgs& a) {
  // (a 4-lane subgroup has its four keys in flight whatever U says)
  if constexpr (G == 4) {
    return launch_fop<S, B, 4, 1>(a);
  } else {
    switch (U) {
      case 1: return launch_fop<S, B, G, 1>(a);
      case 2: return launch_fop<S, B, G, 2>(a);
      case 4: return launch_fop<S, B, G, 4>(a);
      case 8: return launch_fop<S, B, G, 8>(a);
    }
    return hipErrorInvalidValue;
  }
}

template <int S, int B>
hipError_t dispatch_g(uint32_t G, uint32_t U, const FopArgs& a) {
  // A launch that fits the device with one key per lane takes 4-lane
  // subgroups whatever the table's width: all its probes are then in flight
  // at once, where subgroups of 8 lanes take 8 dependent rounds a wavefront.
  // Two-word keys, 32-word buckets, load 0.25, tables of subgroup 8: 4096
  // new keys 21.8 -> 10.0 us (found: 4.4 -> 2.5), 2^19 keys 120 -> 54 (11.1
  // -> 10.2); at 2^20 keys the 8-lane subgroups are the faster, 58 against 71
  // (21.0 and 20.6).  Buckets of 64 words keep their subgroups: read 64 bytes
  // at a time, four dependent reads take longer than one wide one (found, at
  // load 0.5: 5.2 -> 9.8 us for 4096 keys).
  if (B <= 32 && a.n <= static_cast<uint64_t>(a.cus) * kLanesPerCu) G = 4;
  switch (G) {
    case 4: return dispatch_u<S, B, 4>(U, a);  // (64-word buckets: the autotuner only)
    case 8: return dispatch_u<S, B, 8>(U, a);
    case 16: return dispatch_u<S, B, 16>(U, a);
    case 32: return dispatch_u<S, B, 32>(U, a);
    case 64: return dispatch_u<S, B, 64>(U, a);
  }
  return hipErrorInvalidValue;
}

template <int S>
hipError_t dispatch_b(uint32_t B, uint32_t G, uint32_t U, const FopArgs& a) {
  switch (B) {
    case 4: return dispatch_g<S, 4>(G, U, a);
    case 8: return dispatch_g<S, 8>(G, U, a);
    case 16: return dispatch_g<S, 16>(G, U, a);
    case 32: return dispatch_g<S, 32>(G, U, a);
    case 64: return dispatch_g<S, 64>(G, U, a);
  }
  return hipErrorInvalidValue;
}

}  // namespace gx
