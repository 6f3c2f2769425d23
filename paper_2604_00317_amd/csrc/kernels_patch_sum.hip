// Patch kernels for fabrics of several patches, path cost = the sum of the prices (a file of their own:
// they take long to compile).
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel multi_kernel_sum(const PatchShape &s) { return kernel_for<false, true, false>(s); }

}  // namespace patch

}  // namespace nimble
