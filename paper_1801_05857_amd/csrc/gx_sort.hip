// Sorted lists of states: the keys stored in bucket storage gathered on the
// device, and lists of state records sorted there (lexicographically by their
// words, the order of every list the library returns) before they are copied
// to the host.
//
// The sort is a stable least-significant-digit radix sort of S-word records by
// 8-bit digits, over the digits in which the records differ (every other one
// is the same in all of them and is skipped).  A pass is two kernels, counts per
// digit and chunk and the move, with a third between them, the counts' prefix
// sum by one workgroup, for lists of more than 512 chunks.  Bound
// by launches and the move's rounds at the sizes explorations return (258,720
// one-word states: 4 passes), by memory beyond (a record is read twice and
// written once per pass).  Copied out unsorted and sorted by one host thread,
// gathering from a host copy of the whole bucket storage, the same list took
// 24 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <vector>

#include "gx_explore_kernel.hpp"

namespace gx {
namespace {

constexpr uint32_t kSortBlock = 256;
constexpr uint32_t kSortRounds = 8;
constexpr uint32_t kSortChunk = kSortBlock * kSortRounds;  // records per workgroup
// Up to this many chunks every workgroup of a move sums up all chunks' counts
// for itself (a count a thread and chunk, from the L2); beyond, one workgroup
// forms the prefix sums in between (5 rounds of 4 us at 75 chunks, 20 us of a
// pass of 34).
constexpr uint32_t kSumChunks = 512;
constexpr uint32_t kGatherBlock = 1024;
constexpr uint32_t kGatherBlocks = 256;  // few: their atomics meet on a line

// Head of the workspace: records gathered, then per word the bits set in some
// record and those set in all.
struct SortHead {
  unsigned long long n;
  uint32_t any[4], all[4];
  uint32_t pad[6];
};
constexpr uint32_t kHeadWords = sizeof(SortHead) / sizeof(uint32_t);

__global__ void sort_head_kernel(SortHead* h) {
  h->n = 0;
  for (int k = 0; k < 4; ++k) {
    h->any[k] = 0;
    h->all[k] = 0xFFFFFFFFu;
  }
}

template <int S>
__device__ inline void reduce_bits(SortHead* h, uint32_t (&any)[S], uint32_t (&all)[S]) {
  __shared__ uint32_t sh[2 * S];
  if (threadIdx.x < 2 * S) sh[threadIdx.x] = threadIdx.x < S ? 0u : 0xFFFFFFFFu;
  __syncthreads();
#pragma unroll
  for (int x = 0; x < S; ++x) {
    for (int d = 32; d >= 1; d >>= 1) {
      any[x] |= __shfl_xor(any[x], d, 64);
      all[x] &= __shfl_xor(all[x], d, 64);
    }
    if (__lane_id() == 0) {
      atomicOr(&sh[x], any[x]);
      atomicAnd(&sh[S + x], all[x]);
    }
  }
  __syncthreads();
  if (threadIdx.x < S) atomicOr(&h->any[threadIdx.x], sh[threadIdx.x]);
  else if (threadIdx.x < 2 * S) atomicAnd(&h->all[threadIdx.x - S], sh[threadIdx.x]);
}

// The FINAL slots among slots[0, n_slots), in any order, to out (none when
// out is null: counted only; never more than cap).  One reservation per
// workgroup: its slots are counted first.
template <int S>
__global__ __launch_bounds__(kGatherBlock) void gather_kernel(const uint32_t* slots,
                                                              uint64_t n_slots, uint32_t* out,
                                                              uint64_t cap, SortHead* h) {
  __shared__ uint32_t wave_n[kGatherBlock / 64];
  __shared__ unsigned long long sh_base;
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  // this workgroup's slots, and in them this wavefront's
  const uint64_t per = (n_slots + gridDim.x - 1) / gridDim.x;
  const uint64_t g0 = min(n_slots, per * blockIdx.x), g1 = min(n_slots, g0 + per);
  const uint64_t wper = (g1 - g0 + kGatherBlock / 64 - 1) / (kGatherBlock / 64);
  const uint64_t w0 = min(g1, g0 + wper * wave), w1 = min(g1, w0 + wper);
  uint32_t n = 0;
  for (uint64_t i = w0; i < w1; i += 64)
    n += static_cast<uint32_t>(__popcll(__ballot(i + lane < w1 && slots[(i + lane) * S] != kEmpty)));
  if (lane == 0) wave_n[wave] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (uint32_t w = 0; w < kGatherBlock / 64; ++w) t += wave_n[w];
    sh_base = t ? atomicAdd(&h->n, t) : 0;
  }
  __syncthreads();
  if (out == nullptr) return;
  uint64_t pos = sh_base;
  for (uint32_t w = 0; w < wave; ++w) pos += wave_n[w];
  uint32_t any[S], all[S];
#pragma unroll
  for (int x = 0; x < S; ++x) {
    any[x] = 0;
    all[x] = 0xFFFFFFFFu;
  }
  for (uint64_t i = w0; i < w1; i += 64) {
    uint32_t k[S];
#pragma unroll
    for (int x = 0; x < S; ++x) k[x] = kEmpty;
    if (i + lane < w1) load_slot<S>(slots + (i + lane) * S, k);
    const bool has = k[0] != kEmpty;
    const uint64_t m = __ballot(has);
    const uint64_t p = pos + lane_rank(m);
    if (has && p < cap) {
      store_slot<S>(out + p * S, k);
#pragma unroll
      for (int x = 0; x < S; ++x) {
        any[x] |= k[x];
        all[x] &= k[x];
      }
    }
    pos += static_cast<uint64_t>(__popcll(m));
  }
  reduce_bits<S>(h, any, all);
}

template <int S>
__global__ __launch_bounds__(kGatherBlock) void bits_kernel(const uint32_t* rec, uint64_t n,
                                                            SortHead* h) {
  uint32_t any[S], all[S];
#pragma unroll
  for (int x = 0; x < S; ++x) {
    any[x] = 0;
    all[x] = 0xFFFFFFFFu;
  }
  for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kGatherBlock + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * kGatherBlock) {
    uint32_t k[S];
    load_slot<S>(rec + i * S, k);
#pragma unroll
    for (int x = 0; x < S; ++x) {
      any[x] |= k[x];
      all[x] &= k[x];
    }
  }
  reduce_bits<S>(h, any, all);
}

// Records per digit value of each chunk: hist[chunk * 256 + digit] where the
// move sums them up itself (kSums), else hist[digit * n_chunks + chunk].
template <int S, bool kSums>
__global__ __launch_bounds__(kSortBlock) void count_kernel(const uint32_t* in, uint64_t n,
                                                           uint32_t word, uint32_t shift,
                                                           uint32_t* hist, uint32_t n_chunks) {
  __shared__ uint32_t cnt[256];
  cnt[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kSortChunk;
#pragma unroll
  for (uint32_t r = 0; r < kSortRounds; ++r) {
    const uint64_t i = base + r * kSortBlock + threadIdx.x;
    if (i < n) atomicAdd(&cnt[(in[i * S + word] >> shift) & 255u], 1u);
  }
  __syncthreads();
  const uint64_t at = kSums ? static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x
                            : static_cast<uint64_t>(threadIdx.x) * n_chunks + blockIdx.x;
  hist[at] = cnt[threadIdx.x];
}

// Exclusive prefix sum of x[0, n) in place, by one workgroup.
__global__ __launch_bounds__(1024) void scan_kernel(uint32_t* x, uint32_t n) {
  __shared__ uint32_t wave_t[16];
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  uint32_t carry = 0;
  for (uint32_t b = 0; b < n; b += 4096) {
    const uint32_t i = b + threadIdx.x * 4;
    uint32_t v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = i + k < n ? x[i + k] : 0u;
      s += v[k];
    }
    uint32_t inc = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= static_cast<uint32_t>(d)) inc += y;
    }
    if (lane == 63) wave_t[wave] = inc;
    __syncthreads();
    uint32_t at = carry + inc - s, total = 0;
    for (uint32_t w = 0; w < 16; ++w) {
      if (w < wave) at += wave_t[w];
      total += wave_t[w];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < n) x[i + k] = at;
      at += v[k];
    }
    carry += total;
    __syncthreads();  // wave_t is rewritten by the next block
  }
}

// Every record to its place: the chunk's start for its digit, then the order
// of the input (rounds, wavefronts, lanes).
template <int S, bool kSums>
__global__ __launch_bounds__(kSortBlock) void move_kernel(const uint32_t* in, uint32_t* out,
                                                          uint64_t n, uint32_t word,
                                                          uint32_t shift, const uint32_t* hist,
                                                          uint32_t n_chunks) {
  constexpr uint32_t kWaves = kSortBlock / 64;
  __shared__ uint32_t start[256];
  __shared__ uint32_t wcnt[kWaves][256];
  const uint32_t wave = threadIdx.x >> 6, lane = __lane_id();
  if constexpr (kSums) {
    // this thread's digit: its records in the chunks before this one, and in
    // all; then those of the digits before it
    uint32_t before = 0, all = 0;
#pragma unroll 8
    for (uint32_t c = 0; c < n_chunks; ++c) {
      const uint32_t x = hist[static_cast<uint64_t>(c) * 256 + threadIdx.x];
      before += c < blockIdx.x ? x : 0u;
      all += x;
    }
    uint32_t inc = all;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= static_cast<uint32_t>(d)) inc += y;
    }
    if (lane == 63) wcnt[0][wave] = inc;
    __syncthreads();
    uint32_t at = before + inc - all;
    for (uint32_t w = 0; w < wave; ++w) at += wcnt[0][w];
    start[threadIdx.x] = at;
    __syncthreads();
  } else {
    start[threadIdx.x] = hist[static_cast<uint64_t>(threadIdx.x) * n_chunks + blockIdx.x];
  }
#pragma unroll
  for (uint32_t w = 0; w < kWaves; ++w) wcnt[w][threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kSortChunk;
  for (uint32_t r = 0; r < kSortRounds; ++r) {
    const uint64_t i = base + r * kSortBlock + threadIdx.x;
    const bool has = i < n;
    uint32_t k[S];
#pragma unroll
    for (int x = 0; x < S; ++x) k[x] = 0;
    if (has) load_slot<S>(in + i * S, k);
    const uint32_t d = (key_word<S>(k, static_cast<int>(word)) >> shift) & 255u;
    uint64_t same = __ballot(has);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint64_t m = __ballot((d >> b) & 1u);
      same &= ((d >> b) & 1u) ? m : ~m;
    }
    const uint32_t rank = lane_rank(same);
    if (has && rank == 0) wcnt[wave][d] = static_cast<uint32_t>(__popcll(same));
    __syncthreads();
    if (has) {
      uint32_t at = start[d] + rank;
      for (uint32_t w = 0; w < wave; ++w) at += wcnt[w][d];
      store_slot<S>(out + static_cast<uint64_t>(at) * S, k);
    }
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWaves; ++w) {
      t += wcnt[w][threadIdx.x];
      wcnt[w][threadIdx.x] = 0;
    }
    start[threadIdx.x] += t;
    __syncthreads();
  }
}

// Four-word records of three-word states as three words each.
__global__ __launch_bounds__(256) void cut_kernel(const uint32_t* in, uint32_t* out, uint64_t n3) {
  const uint64_t stride = static_cast<uint64_t>(gridDim.x) * 256;
  for (uint64_t k = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; k < n3; k += stride)
    out[k] = in[k / 3 * 4 + k % 3];
}

template <int S>
hipError_t sort_s(uint32_t* a, uint32_t* b, uint64_t n, uint32_t* hist, const SortHead& bits,
                  hipStream_t s, uint32_t** out) {
  const uint32_t n_chunks = static_cast<uint32_t>((n + kSortChunk - 1) / kSortChunk);
  for (int word = S - 1; word >= 0; --word) {
    const uint32_t vary = bits.any[word] & ~bits.all[word];
    for (uint32_t shift = 0; shift < 32; shift += 8) {
      if (((vary >> shift) & 255u) == 0) continue;
      const uint32_t w = static_cast<uint32_t>(word);
      const dim3 grid(n_chunks), block(kSortBlock);
      if (n_chunks <= kSumChunks) {
        hipLaunchKernelGGL((count_kernel<S, true>), grid, block, 0, s, a, n, w, shift, hist,
                           n_chunks);
        hipLaunchKernelGGL((move_kernel<S, true>), grid, block, 0, s, a, b, n, w, shift, hist,
                           n_chunks);
      } else {
        hipLaunchKernelGGL((count_kernel<S, false>), grid, block, 0, s, a, n, w, shift, hist,
                           n_chunks);
        hipLaunchKernelGGL(scan_kernel, dim3(1), dim3(1024), 0, s, hist, 256u * n_chunks);
        hipLaunchKernelGGL((move_kernel<S, false>), grid, block, 0, s, a, b, n, w, shift, hist,
                           n_chunks);
      }
      std::swap(a, b);
    }
  }
  *out = a;
  return hipGetLastError();
}

}  // namespace

SortSpace::~SortSpace() {
  if (words) (void)hipFree(words);
}

bool SortSpace::reserve(uint64_t n) {
  const uint64_t need = kHeadWords + 256 * ((n + kSortChunk - 1) / kSortChunk + 1);
  if (cap >= need) return true;
  if (words) (void)hipFree(words);
  words = nullptr;
  cap = 0;
  if (hipMalloc(&words, need * sizeof(uint32_t)) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  cap = need;
  return true;
}

// n < 2^32 records of S words in `a`, sorted and copied to host memory, w
// words each; b: as large.  bits_known: the workspace's head holds the
// records' bits (a gather has put them there).
static gx_status sort_out(uint32_t S, uint32_t w, uint32_t* a, uint32_t* b, uint64_t n,
                          SortSpace& ws, bool bits_known, uint32_t* host, hipStream_t stream) {
  if (n == 0) return GX_OK;
  SortHead* h = reinterpret_cast<SortHead*>(ws.words);
  if (!bits_known) {
    hipLaunchKernelGGL(sort_head_kernel, dim3(1), dim3(1), 0, stream, h);
    const uint32_t grid = static_cast<uint32_t>(
        std::min<uint64_t>(kGatherBlocks, (n + kGatherBlock - 1) / kGatherBlock));
    switch (S) {
      case 1: hipLaunchKernelGGL(bits_kernel<1>, dim3(grid), dim3(kGatherBlock), 0, stream, a, n, h); break;
      case 2: hipLaunchKernelGGL(bits_kernel<2>, dim3(grid), dim3(kGatherBlock), 0, stream, a, n, h); break;
      default: hipLaunchKernelGGL(bits_kernel<4>, dim3(grid), dim3(kGatherBlock), 0, stream, a, n, h); break;
    }
  }
  SortHead bits;
  if (hipMemcpyAsync(&bits, h, sizeof(bits), hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return GX_EDEVICE;
  uint32_t* sorted = nullptr;
  uint32_t* hist = ws.words + kHeadWords;
  hipError_t e;
  switch (S) {
    case 1: e = sort_s<1>(a, b, n, hist, bits, stream, &sorted); break;
    case 2: e = sort_s<2>(a, b, n, hist, bits, stream, &sorted); break;
    default: e = sort_s<4>(a, b, n, hist, bits, stream, &sorted); break;
  }
  if (e == hipSuccess && w != S) {
    uint32_t* other = sorted == a ? b : a;
    hipLaunchKernelGGL(cut_kernel, dim3(static_cast<uint32_t>(std::min<uint64_t>(4096, (n * 3 + 255) / 256))),
                       dim3(256), 0, stream, sorted, other, n * 3);
    e = hipGetLastError();
    sorted = other;
  }
  if (e != hipSuccess ||
      hipMemcpyAsync(host, sorted, n * w * sizeof(uint32_t), hipMemcpyDeviceToHost, stream) !=
          hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return GX_EDEVICE;
  return GX_OK;
}

gx_status sort_records(uint32_t S, uint32_t w, uint32_t* a, uint32_t* b, uint64_t n, SortSpace& ws,
                       uint32_t* host, hipStream_t stream) {
  if (!ws.reserve(n)) return GX_ENOMEM;
  return sort_out(S, w, a, b, n, ws, false, host, stream);
}

gx_status gather_keys(uint32_t S, const uint32_t* words, uint64_t n_slots, uint32_t* out,
                      uint64_t cap, SortSpace& ws, uint64_t* n, hipStream_t stream) {
  if (!ws.reserve(out ? cap : 0)) return GX_ENOMEM;
  SortHead* h = reinterpret_cast<SortHead*>(ws.words);
  hipLaunchKernelGGL(sort_head_kernel, dim3(1), dim3(1), 0, stream, h);
  const uint32_t grid = static_cast<uint32_t>(std::max<uint64_t>(
      1, std::min<uint64_t>(kGatherBlocks, (n_slots + kGatherBlock - 1) / kGatherBlock)));
  switch (S) {
    case 1: hipLaunchKernelGGL(gather_kernel<1>, dim3(grid), dim3(kGatherBlock), 0, stream, words, n_slots, out, cap, h); break;
    case 2: hipLaunchKernelGGL(gather_kernel<2>, dim3(grid), dim3(kGatherBlock), 0, stream, words, n_slots, out, cap, h); break;
    default: hipLaunchKernelGGL(gather_kernel<4>, dim3(grid), dim3(kGatherBlock), 0, stream, words, n_slots, out, cap, h); break;
  }
  SortHead head;
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(&head, h, sizeof(head), hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return GX_EDEVICE;
  *n = head.n;
  return GX_OK;
}

gx_status sort_gathered(uint32_t S, uint32_t w, uint32_t* a, uint32_t* b, uint64_t n,
                        SortSpace& ws, uint32_t* host, hipStream_t stream) {
  return sort_out(S, w, a, b, n, ws, true, host, stream);
}

}  // namespace gx
