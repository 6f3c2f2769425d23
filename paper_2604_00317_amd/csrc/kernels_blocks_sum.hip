// Patch kernels over blocks for fabrics of several patches, path cost = the sum of the prices.
#include "patch_blocks.hpp"

namespace nimble {

namespace patch {

PatchKernel block_kernel_sum(const PatchShape &s) { return block_kernel_for<false>(s); }

}  // namespace patch

}  // namespace nimble
