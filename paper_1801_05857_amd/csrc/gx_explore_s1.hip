// Exploration kernels (levels, the first levels in LDS) with 1-word slots.
#include "gx_small_kernel.hpp"

namespace gx {
template hipError_t launch_level<1>(uint32_t B, const LevelArgs& a, bool filter, uint32_t grid,
                                    size_t lds, hipStream_t s);
template uint32_t level_blocks_per_cu<1>(uint32_t B, size_t lds);
template hipError_t launch_lds_levels<1>(uint32_t B, SmallArgs a, size_t lds_limit,
                                         hipStream_t s);
}  // namespace gx
