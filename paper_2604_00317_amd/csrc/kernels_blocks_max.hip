// Patch kernels over blocks for fabrics of several patches, path cost = the largest price.
#include "patch_blocks.hpp"

namespace nimble {

namespace patch {

PatchKernel block_kernel_max(const PatchShape &s) { return block_kernel_for<true>(s); }

}  // namespace patch

}  // namespace nimble
