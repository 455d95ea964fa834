// Wide kernels for mechanisms of the default reaction types, their LDS sizing,
// and the dispatch to the further types' (wide_ext.hip).
#include "wide_body.h"

namespace pj {

int64_t wide_lds(const GatherMech& gm, int waves) {
    return wide_doubles(gm.ns, 2 * waves, wide_batches(gm, 2 * waves)) * 8;
}

bool wide_fits(const GatherMech& gm, int waves) {
    return waves >= 2 && waves <= 8 && gm.own[waves] > 0 && wide_lds(gm, waves) <= gm.lds_max;
}

hipError_t launch_wide(const GatherCall& c) { return c.ext ? launch_wide_ext(c) : launch_wide_impl<false>(c); }

}  // namespace pj
