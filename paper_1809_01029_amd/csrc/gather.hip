// Gather kernels for mechanisms of the default reaction types, their LDS
// sizing, and the dispatch to the further types' (gather_ext.hip).
#include "gather_body.h"

namespace pj {

int64_t gather_lds(const GatherMech& gm, int gmode, int S) {
    const bool jac = gmode == GM_JAC || gmode == GM_DENSE;
    int64_t d = jac ? gm.npool : gmode == GM_ADJ ? gm.b3 : ((gm.nr + 2) & ~1);
    d += 5 * (int64_t)(gm.ns + 1);
    if (gmode != GM_SRC) d += 3 * (int64_t)(gm.ns + 1);
    if (jac) d += gm.n_dense_rows + 1;
    d += 7 + SC_N + (jac ? 4 : gmode == GM_ADJ ? 7 : 0) * (MAX_THREADS / 64);
    // flags of the waves; the adjoint's parameter sums
    return (d * S + 5 + (gmode == GM_ADJ ? 3 * (int64_t)gm.nr : 0)) * 8;
}

hipError_t launch_gather(const GatherCall& c) { return c.ext ? launch_gather_ext(c) : launch_gather_impl<false>(c); }

}  // namespace pj
