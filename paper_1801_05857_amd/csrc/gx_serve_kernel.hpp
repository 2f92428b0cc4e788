// Step kernel of the exploration server and of the stepped batch schedule:
// one launch expands the current BFS level of every active job (jobs of one
// slot width and bucket size).  The concatenation of all jobs' levels is cut
// into groups of 256 >> qs states; every workgroup takes groups in turn,
// finds the group's job among the jobs' first groups, loads that job's
// network image into LDS when it is another one than before, and expands the
// group with the same per-wavefront routine as the single exploration.  After
// it, an update kernel makes every job's NEW states its next level and counts
// the groups, so that steps follow each other with no read-back between them
// (a read-back, the new descriptors and the launches took about 85 us a
// step).  Jobs join and leave between strings of steps.
#pragma once

#include <algorithm>
#include <cstdint>

#include "gx_explore_kernel.hpp"

namespace gx {

struct ServeJob {
  TableDev t;
  uint32_t img_off, img_words;
  uint32_t* f[2];       // frontier buffers; the current level is in f[cur]
  uint64_t n_in;        // its states (0: the job is over)
  uint64_t cap_out;
  uint32_t* dead;
  uint64_t dead_cap;
  uint64_t* ctr;        // the job's counters (ctr_at)
  // a deadlock buffer shared by several jobs: records used (null: the job's
  // own kCtrDead counter) and, per record, the job's tag (nullable)
  uint64_t* dead_ctr;
  uint32_t* dead_tag;
  uint32_t tag;
  uint32_t cur;
  uint32_t levels_left; // levels the job may still find
  uint32_t pad;
};

// A class's steps: what the update kernel leaves for the next one.
struct StepHdr {
  uint32_t total;  // groups of the step
  uint32_t qs;     // log2 of the lanes per state (see walk_items)
  uint32_t steps;  // steps done in this string
  uint32_t halt;   // the string is over early: its levels have grown large
};

struct StepOut {  // per step and job
  uint64_t n_next, flags;
};

constexpr uint32_t kStepBlock = 256;  // threads per workgroup

// Workgroups of a level of n states.
__host__ __device__ inline uint64_t step_groups(uint64_t n, uint32_t qs) {
  static_assert(kStepBlock == 256, "four tiles a group");
  return (tiles_of(n, qs) + 3) >> 2;
}

// LDS bytes of a workgroup with room for an image of img_stride words.
inline size_t step_lds(uint32_t S, uint32_t img_stride) {
  return (img_stride + static_cast<size_t>(kStepBlock / 64) * kWaveKeys * S) * sizeof(uint32_t);
}

// log2 of the lanes per state for jobs of `states` states in all: as many as
// keep the wavefronts of the device busy (about 20 a compute unit at this
// kernel's registers and LDS).
__host__ __device__ inline uint32_t step_lanes(uint64_t states, uint32_t cus) {
  return lanes_per_state(states, cus * 20, 6);
}

struct ServeArgs {
  const ServeJob* jobs;
  const uint32_t* begin;  // per job its first group
  uint32_t n_jobs;
  const StepHdr* hdr;
  const uint32_t* img;    // all jobs' network images
  uint32_t img_stride;    // LDS words reserved for one image
};

template <int S, int B>
__global__ __launch_bounds__(kStepBlock) void serve_step_kernel(ServeArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  uint32_t* img = smem;
  uint32_t* lds = smem + a.img_stride + (threadIdx.x >> 6) * wave_words<S, false>();
  const uint32_t total = uniform32(a.hdr->total);
  const uint32_t qs = uniform32(a.hdr->qs);
  uint32_t cached = 0xFFFFFFFFu;
  for (uint32_t group = blockIdx.x; group < total; group += gridDim.x) {
    // last job whose first group is <= this one: of as many evenly spaced
    // jobs as the workgroup has threads, those that begin at or before it are
    // counted, then the same between two of them (30000 small networks in a
    // batch, 12.7 ms with all jobs counted for every group, 7.5 so)
    uint32_t lo = 0;
    for (uint32_t len = a.n_jobs; len > 1;) {
      const uint32_t stride = (len + kStepBlock - 1) / kStepBlock;
      const uint32_t k = threadIdx.x * stride;
      const uint32_t at = uniform32(static_cast<uint32_t>(
                              __syncthreads_count(k < len && a.begin[lo + k] <= group ? 1 : 0))) - 1;
      lo += at * stride;
      len = min(stride, len - at * stride);
    }
    const ServeJob& jb = a.jobs[lo];
    const uint32_t cur = uniform32(jb.cur);
    WaveJob j;
    j.t = uniform_table(jb.t);
    j.img = img;
    j.frontier_in = uniform_ptr(jb.f[cur]);
    j.n_in = uniform64(jb.n_in);
    j.frontier_out = uniform_ptr(jb.f[cur ^ 1u]);
    j.cap_out = uniform64(jb.cap_out);
    j.dead = jb.dead;
    j.dead_tag = jb.dead_tag;
    j.tag = jb.tag;
    j.dead_cap = jb.dead_cap;
    j.dead_ctr = jb.dead_ctr ? jb.dead_ctr : reinterpret_cast<uint64_t*>(ctr_at(jb.ctr, kCtrDead));
    j.ctr = uniform_ptr(jb.ctr);
    j.tail = kCtrTail;
    WaveAcc acc;
    const uint64_t n_tiles = tiles_of(j.n_in, qs);
    const uint64_t tile = uniform64(static_cast<uint64_t>(group - a.begin[lo]) * (kStepBlock / 64) +
                                    (threadIdx.x >> 6));
    uint32_t sw[S];
    load_tile<S>(j, tile, qs, sw);
    if (lo != cached) {
      for (uint32_t k = threadIdx.x; k < jb.img_words; k += kStepBlock)
        img[k] = a.img[jb.img_off + k];
      cached = lo;
    }
    __syncthreads();
    expand_tiles<S, B, false>(j, lds, tile, n_tiles, n_tiles, qs, sw, acc);
    uint64_t n_new;
    (void)finish_block<S, false, false>(j, lds, acc, 0, &n_new);
  }
}

// The jobs' first steps: the initial state (key: S words) into the job's
// frontier and, by find-or-put, into its table; its counters zeroed.
template <int S, int B>
__global__ __launch_bounds__(64) void admit_kernel(TableDev t, const uint32_t* key,
                                                   uint32_t* frontier, uint64_t* ctr,
                                                   uint32_t ctr_words) {
  for (uint32_t k = threadIdx.x; k < ctr_words; k += 64) ctr[k] = 0;
  uint32_t init[S];
  load_slot<S>(key, init);
  if (threadIdx.x == 0) store_slot<S>(frontier, init);
  LaneStats st;
  (void)find_or_put_quads<S, B>(t, init, threadIdx.x == 0, st);
}

// One workgroup, after a step: every job's next level, what the host learns
// of it, and the next step's groups.  A string whose levels hold more than
// `limit` states in all ends early.
__global__ __launch_bounds__(1024) inline void step_update_kernel(ServeJob* jobs, uint32_t* begin,
                                                                  uint32_t n_jobs, StepHdr* hdr,
                                                                  StepOut* out, uint32_t cus,
                                                                  uint64_t limit) {
  __shared__ uint64_t wave_states[16];
  __shared__ uint32_t wave_groups[16];
  if (hdr->halt) return;
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  uint64_t states = 0;
  for (uint32_t k = threadIdx.x; k < n_jobs; k += 1024) {
    ServeJob& jb = jobs[k];
    uint64_t* c = jb.ctr;
    uint64_t n = c[kCtrTail * kCtrSpread] & kTailMask;
    const uint64_t flags = c[kCtrFlags * kCtrSpread];
    c[kCtrTail * kCtrSpread] = 0;
    out[k].n_next = n;
    out[k].flags = flags;
    if (flags != 0 || jb.levels_left == 0) n = 0;
    else --jb.levels_left;
    jb.n_in = n;
    jb.cur ^= 1u;
    states += n;
  }
  states = wave_sum64(states);
  if (lane == 0) wave_states[wave] = states;
  __syncthreads();
  states = 0;
  for (uint32_t w = 0; w < 16; ++w) states += wave_states[w];
  const uint32_t qs = step_lanes(states, cus);
  uint32_t carry = 0;
  for (uint32_t k0 = 0; k0 < n_jobs; k0 += 1024) {
    const uint32_t k = k0 + threadIdx.x;
    const uint32_t g = k < n_jobs ? static_cast<uint32_t>(step_groups(jobs[k].n_in, qs)) : 0u;
    uint32_t inc = g;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= static_cast<uint32_t>(d)) inc += y;
    }
    if (lane == 63) wave_groups[wave] = inc;
    __syncthreads();
    uint32_t at = carry + inc - g;
    for (uint32_t w = 0; w < 16; ++w) {
      if (w < wave) at += wave_groups[w];
      carry += wave_groups[w];
    }
    if (k < n_jobs) begin[k] = at;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    hdr->total = states > limit ? 0u : carry;
    hdr->qs = qs;
    hdr->steps += 1;
    hdr->halt = states > limit ? 1u : 0u;
  }
}

// (The probes are those of 4-lane subgroups whatever the jobs' own width.)
template <int S>
hipError_t serve_launch(uint32_t B, const ServeArgs& a, uint32_t grid, size_t lds, hipStream_t s) {
  switch (B) {
#define GX_SERVE_CASE(BB)                                                                       \
  case BB:                                                                                      \
    if (lds > 65536) {                                                                          \
      const hipError_t e = hipFuncSetAttribute(                                                 \
          reinterpret_cast<const void*>(&serve_step_kernel<S, BB>),                             \
          hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));                   \
      if (e != hipSuccess) return e;                                                            \
    }                                                                                           \
    hipLaunchKernelGGL((serve_step_kernel<S, BB>), dim3(grid), dim3(kStepBlock), lds, s, a);    \
    return hipGetLastError();
    GX_SERVE_CASE(8)
    GX_SERVE_CASE(16)
    GX_SERVE_CASE(32)
    GX_SERVE_CASE(64)
#undef GX_SERVE_CASE
  }
  return hipErrorInvalidValue;
}

template <int S>
hipError_t admit_launch(uint32_t B, const TableDev& t, const uint32_t* key, uint32_t* frontier,
                        uint64_t* ctr, uint32_t ctr_words, hipStream_t s) {
  switch (B) {
#define GX_SERVE_CASE(BB)                                                                      \
  case BB:                                                                                     \
    hipLaunchKernelGGL((admit_kernel<S, BB>), dim3(1), dim3(64), 0, s, t, key, frontier, ctr,  \
                       ctr_words);                                                             \
    return hipGetLastError();
    GX_SERVE_CASE(8)
    GX_SERVE_CASE(16)
    GX_SERVE_CASE(32)
    GX_SERVE_CASE(64)
#undef GX_SERVE_CASE
  }
  return hipErrorInvalidValue;
}

// Step workgroups a compute unit holds at once.
template <int S>
uint32_t step_blocks_per_cu(uint32_t B, size_t lds) {
  int b = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (B) {
#define GX_SERVE_CASE(BB)                                                                     \
  case BB:                                                                                    \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, serve_step_kernel<S, BB>, kStepBlock, \
                                                     lds);                                    \
    break;
    GX_SERVE_CASE(8)
    GX_SERVE_CASE(16)
    GX_SERVE_CASE(32)
    GX_SERVE_CASE(64)
#undef GX_SERVE_CASE
  }
  if (e != hipSuccess || b <= 0) {
    (void)hipGetLastError();
    return 1;
  }
  return static_cast<uint32_t>(b);
}

}  // namespace gx
