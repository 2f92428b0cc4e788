// LDS layout of the launch that expands an exploration's first levels (see
// gx_small_kernel.hpp): the network image, the visited set, a stage per
// wavefront and two rings of level states, in this order.  Host arithmetic
// only, so that a test can check it without a GPU.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace gx {

// Threads of the workgroup: 16 wavefronts, 8 for four-word slots (a
// wavefront's stage then takes twice the LDS, and the visited set needs it).
template <int S>
constexpr uint32_t small_threads() {
  return S == 4 ? 512u : 1024u;
}
constexpr uint32_t kSmallStage = 128;  // staged successors per wavefront
// Fewest states of a ring, whatever the largest level is: the initial state is
// always put into the first one.
constexpr uint32_t kRingMin = 4;

struct LdsPlan {
  uint32_t set_bits;  // log2 of the visited set's entries; below 10: no launch
  uint32_t ring;      // states each of the two rings holds
  size_t bytes;       // of the whole
};

// LDS bytes with 2^set_bits set entries and rings of `ring` states.
template <int S>
constexpr size_t lds_levels_bytes(uint32_t img_stride, uint32_t set_bits, uint32_t ring) {
  return (static_cast<size_t>(img_stride) + (size_t(S) << set_bits) +
          small_threads<S>() / 64 * kSmallStage * S + size_t(2) * ring * S) * sizeof(uint32_t);
}

// log2 of the entries of the largest visited set that fits (below 10: none).
template <int S>
uint32_t lds_set_bits(uint32_t img_stride, size_t lds_limit) {
  uint32_t bits = 20;
  while (bits >= 10 && lds_levels_bytes<S>(img_stride, bits, kRingMin) > lds_limit) --bits;
  return bits;
}

// The largest visited set, and in what it leaves the rings, at most as large
// as the largest level expanded (`limit` states).
template <int S>
LdsPlan lds_plan(uint32_t img_stride, uint64_t limit, size_t lds_limit) {
  LdsPlan p{lds_set_bits<S>(img_stride, lds_limit), 0, 0};
  if (p.set_bits < 10) return p;
  const size_t rest = lds_limit - lds_levels_bytes<S>(img_stride, p.set_bits, 0);
  const uint64_t fit = rest / (2 * S * sizeof(uint32_t));  // at least kRingMin
  p.ring = std::max(kRingMin, static_cast<uint32_t>(std::min<uint64_t>(limit, fit) & ~3ull));
  p.bytes = lds_levels_bytes<S>(img_stride, p.set_bits, p.ring);
  return p;
}

}  // namespace gx
