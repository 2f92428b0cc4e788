// Step kernel of the exploration server and of the stepped batch schedule:
// one launch expands the current BFS level of every active job (jobs of one
// slot width and bucket size).  Workgroup b takes group b of the
// concatenation of all jobs' levels (256 >> qs states per group), finds its
// job by binary search over the jobs' first groups, loads that job's network
// image into LDS and expands the group with the same per-wavefront routine as
// the single exploration.  Jobs join and leave between launches.
#pragma once

#include <cstdint>

#include "gx_explore_kernel.hpp"

namespace gx {

struct ServeJob {
  TableDev t;
  uint32_t img_off, img_words;
  const uint32_t* frontier_in;
  uint64_t n_in;
  uint32_t* frontier_out;
  uint64_t cap_out;
  uint32_t* dead;
  uint64_t dead_cap;
  uint64_t* ctr;        // the job's counters (ctr_at)
  uint64_t tile_begin;  // first group of this job in the step
  // a deadlock buffer shared by several jobs: records used (null: the job's
  // own kCtrDead counter) and, per record, the job's tag (nullable)
  uint64_t* dead_ctr;
  uint32_t* dead_tag;
  uint32_t tag;
  uint32_t qs;          // log2 of the lanes per state (see walk_items)
};

constexpr uint32_t kStepBlock = 256;  // threads per workgroup

// Frontier states per workgroup, and workgroups of a level of n states.
inline uint64_t step_groups(uint64_t n, uint32_t qs) {
  const uint64_t per = kStepBlock >> qs;
  return (n + per - 1) / per;
}

// LDS bytes of a workgroup with room for an image of img_stride words.
inline size_t step_lds(uint32_t S, uint32_t img_stride) {
  return (img_stride + static_cast<size_t>(kStepBlock / 64) * kWaveKeys * S) * sizeof(uint32_t);
}

// log2 of the lanes per state for jobs of `states` states in all: as many as
// keep the wavefronts of the device busy (about 20 a compute unit at this
// kernel's registers and LDS).
inline uint32_t step_lanes(uint64_t states, uint32_t cus) {
  return lanes_per_state(states, cus * 20, 6);
}

struct ServeArgs {
  const ServeJob* jobs;
  uint32_t n_jobs;
  const uint32_t* img;  // all jobs' network images
  uint32_t img_stride;  // LDS words reserved for one image
};

template <int S, int B>
__global__ __launch_bounds__(kStepBlock) void serve_step_kernel(ServeArgs a) {
  extern __shared__ __align__(16) uint32_t smem[];
  uint32_t* img = smem;
  uint32_t* lds = smem + a.img_stride + (threadIdx.x >> 6) * wave_words<S, false>();
  const uint64_t group = blockIdx.x;
  // last job whose first group is <= this one
  uint32_t lo = 0, hi = a.n_jobs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (a.jobs[mid].tile_begin <= group) lo = mid;
    else hi = mid;
  }
  const ServeJob& jb = a.jobs[lo];
  WaveJob j;
  j.t = uniform_table(jb.t);
  j.img = img;
  j.frontier_in = uniform_ptr(jb.frontier_in);
  j.n_in = uniform64(jb.n_in);
  j.frontier_out = uniform_ptr(jb.frontier_out);
  j.cap_out = uniform64(jb.cap_out);
  j.dead = jb.dead;
  j.dead_tag = jb.dead_tag;
  j.tag = jb.tag;
  j.dead_cap = jb.dead_cap;
  j.dead_ctr = jb.dead_ctr ? jb.dead_ctr : reinterpret_cast<uint64_t*>(ctr_at(jb.ctr, kCtrDead));
  j.ctr = uniform_ptr(jb.ctr);
  j.tail = kCtrTail;
  WaveAcc acc;
  const uint32_t qs = uniform32(jb.qs);
  const uint32_t per = 64u >> qs;
  const uint64_t n_tiles = (j.n_in + per - 1) / per;
  const uint64_t tile =
      uniform64((group - jb.tile_begin) * (kStepBlock / 64) + (threadIdx.x >> 6));
  uint32_t sw[S];
  load_tile<S>(j, tile, qs, sw);
  for (uint32_t k = threadIdx.x; k < jb.img_words; k += kStepBlock) img[k] = a.img[jb.img_off + k];
  __syncthreads();
  expand_tiles<S, B, false>(j, lds, tile, n_tiles, n_tiles, qs, sw, acc);
  uint64_t n_new;
  (void)finish_block<S, false, false>(j, lds, acc, 0, &n_new);
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

}  // namespace gx
