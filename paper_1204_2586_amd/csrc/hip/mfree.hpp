// Matrix-free P^k element operator (see mfree.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace auxp {

// Patches of tets (host side: build_patches); dofs in the internal order
template <typename T>
struct MfView {
    int n;               // dofs
    int nloc;            // nodes per tet: 10 (P2), 20 (P3) or 35 (P4)
    int tp;              // places per patch, a multiple of 16
    int npatch, max_dofs;
    int nshared;         // dofs of more than one patch
    const int4 *meta;    // per patch: first entry of dof, dofs, complete dofs, first entry of pos
    const int *dof;
    const unsigned *range;       // each one's slots: first, end << 16
    const unsigned *word;        // per place and node: position in the patch's dofs, slot << 16
    const int *pos;              // places of the patches' partial sums of shared dofs
    const int *sh_dof, *sh_ptr;  // shared dofs, ranges of their partial sums
    const T *w;          // [npatch tp][6] edge weights -kappa_e G^e_pq, pairs (01,02,03,12,13,23), 0 at empty places
    const T *S;          // reference tables in operand order (mf_tables)
    T *part;             // the partial sums
};

// the tables S^k (entry (a, b) at (6 a + k) nloc + b) in the order in which the
// matrix-core steps read them
template <typename T>
void mf_tables(int nloc, const double *S, T *out);
size_t mf_table_size(int nloc);
// LDS bytes of a workgroup
size_t mf_lds(int nloc, int tp, int max_dofs, size_t size);

// res = rhs - A x
template <typename T>
void mf_resid(hipStream_t s, const MfView<T> &op, const T *x, const T *rhs, T *res, const int *done);
// out = A x; with partials also x.out per workgroup (the number of partials is returned)
int mf_product(hipStream_t s, const MfView<double> &op, const double *x, double *out, double *partials, const int *done);
// out = x + dinv (rhs - A x); with partials also rhs.out per workgroup
template <typename T, typename TR, typename TZ>
int mf_sweep(hipStream_t s, const MfView<T> &op, const T *x, const T *dinv, const TR *rhs, TZ *out, double *partials,
             const int *done);

}  // namespace auxp
