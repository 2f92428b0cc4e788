// Server step kernels with 1-word slots.
#include "gx_serve_kernel.hpp"

namespace gx {
template hipError_t serve_launch<1>(uint32_t, const ServeArgs&, uint32_t, size_t, hipStream_t);
template hipError_t admit_launch<1>(uint32_t, const TableDev&, const uint32_t*, uint32_t*,
                                     uint64_t*, uint32_t, hipStream_t);
template uint32_t step_blocks_per_cu<1>(uint32_t, size_t);
}  // namespace gx
