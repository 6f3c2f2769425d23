// Patch kernels of the solve with variable step and certificate (path cost = the sum of the
// prices), for fabrics of one patch and of several.
//
// The launched form takes two or three kernels per iteration and reads the topology in each.  Here
// an iteration is the fixed step's (scan, scatter, exchange of the loads of shared links: 2.2 us on
// the 16-node fabric) plus one more trip from patch to patch for the largest normalised load, 4.8 us
// together, and a check of the bound takes another 12 us.  With a check every 25 iterations: 9.3 ->
// 5.3 us per iteration on 16 nodes (6.3 before the patches met through a leader per XCD), 14.5 -> 6.4
// on 24, 7.8 -> 2.1 on 2 (one patch, no trips).
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel adaptive_kernel(const PatchShape &s, bool multi)
{
    return multi ? kernel_for<false, true, true>(s) : kernel_for<false, false, true>(s);
}

}  // namespace patch

}  // namespace nimble
