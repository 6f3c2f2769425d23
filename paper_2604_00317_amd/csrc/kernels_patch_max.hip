// Patch kernels for fabrics of several patches, path cost = the largest price (a file of their own:
// they take long to compile).
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel multi_kernel_max(const PatchShape &s) { return kernel_for<true, true, false>(s); }

}  // namespace patch

}  // namespace nimble
