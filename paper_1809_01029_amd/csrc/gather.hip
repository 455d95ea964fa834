// Gather kernels for mechanisms of the default reaction types, their LDS
// sizing, and the dispatch to the further types' (gather_ext.hip).
#include "gather_body.h"

namespace pj {

int64_t gather_lds(const GatherMech& gm, int gmode, int S) {
    int64_t d = gmode != GM_SRC ? gm.npool : ((gm.nr + 2) & ~1);
    d += 5 * (int64_t)(gm.ns + 1);
    if (gmode != GM_SRC) d += 3 * (int64_t)(gm.ns + 1) + gm.n_dense_rows + 1;
    d += 7 + SC_N + (gmode != GM_SRC ? 4 * (MAX_THREADS / 64) : 0);
    return (d * S + 5) * 8;
}

hipError_t launch_gather(const GatherCall& c) { return c.ext ? launch_gather_ext(c) : launch_gather_impl<false>(c); }

}  // namespace pj
