// Patch kernels of the solve with variable step and certificate (path cost = the sum of the
// prices), for fabrics of one patch and of several.
//
// The launched form takes two kernels per iteration (9.3 us on the 16-node fabric) and reads the
// topology in each.  Here an iteration is the fixed step's (scan, scatter, exchange of the loads of
// shared links: 2.9 us there) plus one more trip from patch to patch for the largest normalised
// load (2.2 to 3 us), and a check of the bound, every 25 iterations, takes 11 us: 6.3 us per
// iteration in all.  The two trips, about 1.6 us each, bound it.
#include "patch_kernel.hpp"

namespace nimble {

namespace patch {

PatchKernel adaptive_kernel(const PatchShape &s, bool multi)
{
    return multi ? kernel_for<false, true, true>(s) : kernel_for<false, false, true>(s);
}

}  // namespace patch

}  // namespace nimble
