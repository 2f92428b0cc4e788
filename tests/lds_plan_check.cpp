// Host check of the LDS layout of an exploration's first levels: for every
// image size, level limit and LDS budget in reach, what the launch writes (the
// image, the visited set, the wavefronts' stages, two rings that hold at least
// the initial state) lies inside the bytes it asks for, and those inside the
// budget.  Exit status 0 when every check holds.
#include <cstdio>

#include "gx_lds_plan.hpp"

template <int S>
static int check() {
  const uint64_t limits[] = {1, 2, 3, 4, 5, 6, 7, 63, 1023, 4096};
  for (size_t budget : {size_t(32768) - 1024, size_t(65536) - 1024, size_t(163840) - 1024})
    for (uint32_t stride = 4; stride <= 13824; stride += 4)
      for (uint64_t limit : limits) {
        const gx::LdsPlan p = gx::lds_plan<S>(stride, limit, budget);
        if (p.set_bits < 10) {
          if (p.set_bits < 9 || gx::lds_levels_bytes<S>(stride, 10, gx::kRingMin) <= budget) return 1;
          continue;
        }
        const size_t set = size_t(S) << p.set_bits;
        const size_t stage = size_t(gx::small_threads<S>() / 64) * gx::kSmallStage * S;
        // the initial state goes to the first ring's first place
        const size_t words = stride + set + stage + size_t(2) * p.ring * S;
        if (p.ring < 1 || words * 4 > p.bytes || p.bytes > budget) {
          std::printf("FAIL S %d stride %u limit %llu budget %zu ring %u bytes %zu\n", S, stride,
                      static_cast<unsigned long long>(limit), budget, p.ring, p.bytes);
          return 1;
        }
        // no smaller a set than fits, no larger rings than the levels need
        if (p.set_bits < 20 && gx::lds_levels_bytes<S>(stride, p.set_bits + 1, gx::kRingMin) <= budget)
          return 1;
        if (p.ring % 4 || (p.ring > gx::kRingMin && p.ring > limit)) return 1;
      }
  return 0;
}

int main() {
  if (check<1>() || check<2>() || check<4>()) return 1;
  std::printf("ok\n");
  return 0;
}
