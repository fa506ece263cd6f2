// Solve-phase kernels for gfx950 (CDNA4, wave64).
//
// The P^k operator A_h is stored as sliced ELLPACK with 64-row slices (one
// lane per row, four consecutive entries of a row adjacent: one load of a
// wavefront brings 1 or 2 KB of values and 512 bytes of 16-bit columns).  Its
// rows are numbered in an internal order, sorted by length so the padding of
// each slice stays small: either over the whole operator (a stable sort,
// which on structured meshes groups nodes of one kind and keeps a slice's
// gathers nearly contiguous) or within windows of consecutive dofs; the setup
// times both on the device and keeps the faster (the global sort wins on the
// benchmark meshes).  The AMG operators and the transfers are CSR with LPR
// lanes per row or row-split sliced ELL, whichever the setup times faster.
//
// Dot products are reduced deterministically without atomics: every
// workgroup writes one partial, and a one-workgroup "finish" kernel that
// follows in the stream sums them in a fixed order.  Kernels that belong to a
// CG iteration return at once when the device "done" flag is set, so
// iterations can be enqueued ahead of the convergence test.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace auxp {

constexpr int kBlock = 256;
constexpr int kMaxBlocks = 4096;       // partial sums per reduction at most
constexpr int kSlice = 64;             // rows per ELL slice (one wavefront)

struct DevCsrView {
    int n;
    const int *ptr;
    const int *col;
    const void *val;     // double or float
    int lpr;
    // Row-split sliced ELL copy of the same operator (ell_lanes > 0: the
    // products use it): slices of 64 / ell_lanes rows, one wavefront each,
    // entry k of the slice's row q in slot k / ell_lanes at lane
    // q * ell_lanes + k % ell_lanes; ell_off[s] is the first entry of slice s
    // (a multiple of 64), padding entries have column 0 and value 0.
    int ell_lanes;
    const int *ell_off;
    const int *ell_col;
    const void *ell_val;
};

struct DevSellView {
    int n;               // rows
    int nslices;
    int waves;           // single-vector kernels: wavefronts per slice (1, 2, 4 or 8)
    // per slice: first group (of 4 slots, 256 entries), groups, first group
    // in wide or -1 (16-bit columns), slots in use
    const int4 *meta;
    // 16-bit columns: entry e of slot t has column
    // (off[e] >> 15 ? base[t].y : base[t].x) + (off[e] & 0x7fff)
    const int2 *base;
    const unsigned short *off;
    const int *wide;     // 32-bit columns of the other slices
    const void *val;     // double or float, padding entries are 0
    // block kernels only: when set, die d (the workgroups b with b % 8 == d,
    // which the dispatcher places on die d) takes slices [die_off[d],
    // die_off[d + 1]) (9 entries); otherwise slices go round-robin
    const int *die_off = nullptr;
};

// Three values side by side: an element of an interleaved block of three
// vectors (the velocity components of a Stokes vector).  The kernels written
// for a scalar element run on it as they are: an operator is read once for
// the three, and a gathered entry is one load of 12 or 24 bytes.
template <typename T>
struct Vec3 {
    T a, b, c;
};
template <typename T>
__host__ __device__ __forceinline__ Vec3<T> operator+(const Vec3<T> &x, const Vec3<T> &y)
{
    return {x.a + y.a, x.b + y.b, x.c + y.c};
}
template <typename T>
__host__ __device__ __forceinline__ Vec3<T> operator-(const Vec3<T> &x, const Vec3<T> &y)
{
    return {x.a - y.a, x.b - y.b, x.c - y.c};
}
template <typename T>
__host__ __device__ __forceinline__ Vec3<T> operator*(T s, const Vec3<T> &y)
{
    return {s * y.a, s * y.b, s * y.c};
}
template <typename T>
__host__ __device__ __forceinline__ Vec3<T> &operator+=(Vec3<T> &x, const Vec3<T> &y)
{
    x.a += y.a;
    x.b += y.b;
    x.c += y.c;
    return x;
}

// State of a CG solve in device memory.
struct CgState {
    int *iter;           // completed iterations
    int *done;           // 0 running, 1 converged, 2 maxit, 3 breakdown, 4 non-finite
    double *rz;          // rz[k] = r_k . z_k
    double *pq;          // pq[k] = p_k . A p_k
    double *rr;          // rr[k] = r_k . r_k
    double *scal;        // [0] f.f, [1] r_0.r_0, [2] tol^2 f.f
    int maxit;
    struct CgReport *report = nullptr;   // host memory the kernels write to, or null
};

// What the host sees of a running solve without a copy or a wait: written by
// the kernels that finish r.r (and by those that stop a solve) into pinned
// host memory.  word: iterations, stop flag << 28, and in the low half the
// bits of the float r.r / (tol^2 f.f).
struct CgReport {
    unsigned long long word;
    double rr, ff;
};

// the r.r reduction of a CG update, finished by a later kernel
struct RrFinish {
    const double *partials = nullptr;
    int nparts = 0;
    CgState st = {};
};

enum FinishMode { FIN_PLAIN = 0, FIN_PQ = 1, FIN_RZ = 2, FIN_RR = 3 };

// ---- P^k level (SELL).  Kernels that reduce write one partial per
// workgroup to `partials` (if non-null) and return the grid size used.

// Vectors of the functions below are arrays of elements: T, or Vec3<T> (X, XR
// and XZ; the operators stay scalar of type T).

// z = D^{-1} r (one sweep from zero); rT = (T) r if rT
template <typename T, typename X, typename XR>
int vec_jacobi0(hipStream_t s, int n, const T *dinv, const XR *r, X *z, X *rT, const int *done);
// z = D^{-1} r for r in the working precision
template <typename T>
void vec_jacobi0_t(hipStream_t s, int n, const T *dinv, const T *r, T *z, const int *done);
// rint = r[perm], z = D^{-1} rint; rT = (T) rint if rT
template <typename T>
void vec_gather_jacobi0(hipStream_t s, int n, const int *perm, const T *dinv, const double *r, double *rint, T *z, T *rT);
// zout = zin + D^{-1} (rhs - A zin); with partials, also sum_i rdot_i zout_i;
// with operm, row r's result goes to zout[operm[r]]; with fin (and no
// partials) one more workgroup finishes that r.r reduction
// (inner products and fin for scalar elements only)
template <typename T, typename X, typename XR, typename XZ>
int sell_sweep(hipStream_t s, const DevSellView &A, const T *dinv, const XR *rhs, const X *zin, XZ *zout,
               const double *rdot, double *partials, const int *done, const int *operm = nullptr,
               const RrFinish *fin = nullptr);
// res = rhs - A z
template <typename T>
int sell_resid(hipStream_t s, const DevSellView &A, const T *rhs, const T *z, T *res, const int *done);
// y = A x (FP64); with partials also x.y; with operm, row r's result goes to y[operm[r]]
int sell_spmv64(hipStream_t s, const DevSellView &A, const double *x, double *y, double *partials, const int *done,
                const int *operm = nullptr);
// the same for three vectors
void sell_spmv64x3(hipStream_t s, const DevSellView &A, const Vec3<double> *x, Vec3<double> *y);
// workgroups (so partials) of a pass over A
int sell_parts(const DevSellView &A);
// p = z + beta p_old and q = A p in one pass, with the p.q partials; beta from
// the r.z partials (see k_cg_product)
int cg_product(hipStream_t s, const DevSellView &A, const double *z, const double *p_old, double *p, double *q,
               const double *rz_parts, int rz_n, double *pq_parts, const CgState &st);
// The start of a CG solve: f and u gathered into the internal order (fi, x),
// then r = fi - A x with the partials of r.r and f.f and the preconditioner's
// first sweep from zero (z0 = D^-1 r, and with rT non-null r in its type), and
// the solve's state from them.  partials: 2 kMaxBlocks / 2 words.
template <typename T>
void cg_start(hipStream_t s, const DevSellView &A, const int *perm, const double *f, const double *u, double *fi,
              double *x, double *r, const T *dinv, T *z0, T *rT, double *partials, const CgState &st, double tol2);
// r = f - A u (FP64)
int sell_residual64(hipStream_t s, const DevSellView &A, const double *f, const double *u, double *r);

// ---- CSR (AMG levels, transfers)
template <typename T, typename X>
void csr_matvec(hipStream_t s, const DevCsrView &M, const X *x, X *y, const int *done);
template <typename T, typename X>
void csr_matvec_add(hipStream_t s, const DevCsrView &M, const X *e, X *x, const int *done);
// z += M e for M with at most w (1..4) entries per row in w column-major
// slots (slot k of row i at k n + i, padding value 0 at column 0)
template <typename T, typename X>
void fixed_matvec_add(hipStream_t s, int n, int w, const int *col, const T *val, const X *e, X *z, const int *done);
// y = M [x1; x2] (columns below split index x1, the rest x2)
template <typename T, typename X>
void csr_matvec2(hipStream_t s, const DevCsrView &M, const X *x1, const X *x2, int split, X *y, const int *done);

// x = D^{-1} b, r = b - A x (V-cycle presmoothing from zero fused with the residual)
template <typename T>
void csr_vpre(hipStream_t s, const DevCsrView &A, const T *dinv, const T *b, T *x, T *r, const int *done);
// y = x + D^{-1} (b - A x)
template <typename T>
void csr_sweep(hipStream_t s, const DevCsrView &A, const T *dinv, const T *b, const T *x, T *y, const int *done);
// x = Ainv b, dense row-major n x n (one workgroup)
template <typename T, typename X>
void dense_gemv(hipStream_t s, int n, const T *Ainv, const X *b, X *x, const int *done);

// ---- vectors and CG bookkeeping (FP64)
int vec_dot(hipStream_t s, int n, const double *a, const double *b, double *partials);
// sum nparts partials; FIN_PLAIN writes out[0]; the others write the CG slot of
// the current iteration and update the state (see kernels.hip)
void finish(hipStream_t s, const double *partials, int nparts, FinishMode mode, double *out, const CgState &st);
// x += alpha p ; r -= alpha q ; partial r.r; also the preconditioner's first
// sweep from zero, z0 = D^-1 r, and (rT non-null) r in the preconditioner's
// type.  pq_n > 0: p.q is summed from its partials here, else read from st.
template <typename T>
int cg_update_prep(hipStream_t s, int n, double *x, double *r, const double *p, const double *q, const CgState &st,
                   double *partials, const T *dinv, T *z0, T *rT, const double *pq_parts, int pq_n);
// p = z + beta p, beta = rz[k]/rz[k-1] (p = z at k = 0)
void cg_direction(hipStream_t s, int n, const double *z, double *p, const CgState &st);
// three component blocks of n (stride n) to or from n interleaved elements:
// y[i].c = x[c n + idx[i]], and y[c n + idx[i]] = x[i].c (idx null: i)
void vec_interleave3(hipStream_t s, int n, const int *idx, const double *x, Vec3<double> *y);
void vec_split3(hipStream_t s, int n, const int *idx, const Vec3<double> *x, double *y);
// y[i] = x[idx[i]]
void vec_gather(hipStream_t s, int n, const int *idx, const double *x, double *y);
// y[idx[i]] = x[i]
void vec_scatter(hipStream_t s, int n, const int *idx, const double *x, double *y);

// g_t = -kappa_t sum_pq G_pq lam_t^T M^pq u_t per tet (FP64).  By column (entry
// a of tet t at a nt + t): dofs, the tets' dof numbers (-1 on the boundary);
// G6, the metrics of the vertex pairs (0,1) (0,2) (0,3) (1,2) (1,3) (2,3) (the
// first columns of those that the coefficient update reads).  S: the pairs' symmetric tables S^k = M^pp + M^qq - M^pq - M^qp: for each pair
// of rows (2 m, 2 m + 1) and column b >= 2 m the six entries of the first row,
// then of the second (zero below the diagonal and past the last row), the
// diagonal's halved.
void kappa_grad(hipStream_t s, int nt, int nloc, const int *dofs, const double *G6, const double *kappa,
                const double *S, const double *u, const double *lam, double *g);

int pick_lpr(double avg_row_nnz);

}  // namespace auxp
