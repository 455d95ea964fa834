// Gather kernels for mechanisms that also hold SRI, chemically activated,
// P-Log or Chebyshev reactions.
#include "gather_body.h"

namespace pj {

hipError_t launch_gather_ext(const GatherCall& c) { return launch_gather_impl<true>(c); }

}  // namespace pj
