// Kernels of the Stokes block-triangular preconditioner Q_t (Sec. 5): the
// pressure block solves M_p y = r_p by diagonally preconditioned CG, run with
// its state in device memory (CgState: the step's alpha and beta are read
// from device memory, and every launch after the stop returns at once), so
// the host enqueues a run of iterations and checks the stop flag once.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace auxp {

// the vectors of a mass-matrix CG solve, and its partials: two sets, the
// second kMaxBlocks after the first, and one for p.q
struct MassBufs {
    double *x, *r, *z, *p, *p2, *q;
    const double *dinv;      // 1 / diag M
    double *partials, *pq_parts;
};
// x = 0, r = b, z = D^-1 b, the stop flag cleared; the workgroups' shares of
// b.b and r.z in the two sets of partials.  Returns their number.
int mass_start(hipStream_t s, int n, const double *b, const double *dinv, double *x, double *r, double *z,
               double *partials, const CgState &st);
// Step k (from 0): the stop test on ||r|| (against sqrt(tol2) ||b||), the
// direction, the product, x, r and z.  nparts: what the call before returned
// (mass_start's for k = 0).  Every launch after the stop returns at once.
int mass_step(hipStream_t s, const DevCsrView &M, int k, double tol2, const MassBufs &v, int nparts, const CgState &st);
// y = -x
void vec_negate(hipStream_t s, int n, const double *x, double *y);

}  // namespace auxp
