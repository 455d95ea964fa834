// Wide kernels for mechanisms that also hold SRI, chemically activated, P-Log
// or Chebyshev reactions.
#include "wide_body.h"

namespace pj {

hipError_t launch_wide_ext(const GatherCall& c) { return launch_wide_impl<true>(c); }

}  // namespace pj
