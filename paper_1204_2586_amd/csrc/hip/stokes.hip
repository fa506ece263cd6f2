// Pressure mass-matrix CG of the Stokes preconditioner Q_t (Sec. 5, the
// Schur complement replaced by the pressure mass matrix, solved by
// diagonally preconditioned CG as in the paper's Stokes experiments).  FP64.
//
// The mass matrix is a few per cent of the velocity work of one Q_t
// application, but a solve takes 15 to 30 steps, so its launches count.  The
// reductions write one partial per workgroup, and every workgroup of the
// kernel that needs a sum adds the partials up itself, in the same order; the
// step number comes with the launch, so no kernel waits for a bookkeeping
// launch.  A step is three launches (direction, product, update), or two
// where the product forms the direction from both gathered vectors.
#include <hip/hip_runtime.h>

#include <cmath>

#include "stokes.hpp"

namespace auxp {

namespace {

// partial sums per reduction at most: every workgroup of the next kernel reads
// them all (16 KB from L2), and 2048 workgroups fill the chip
constexpr int kMassParts = 2048;
// rows up to which the product forms the direction itself: there a step is
// bound by its launches
constexpr int kMassGatherRows = 32768;

inline int mass_grid(int n)
{
    int g = (n + kBlock - 1) / kBlock;
    return g < 1 ? 1 : (g > kMassParts ? kMassParts : g);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// the workgroup's sums of a and b in every thread, in a fixed order
__device__ __forceinline__ void block_pair(double &a, double &b)
{
    __shared__ double red[2][kBlock / 64];
    a = wave_sum(a);
    b = wave_sum(b);
    const int w = threadIdx.x / 64;
    if (threadIdx.x % 64 == 0) {
        red[0][w] = a;
        red[1][w] = b;
    }
    __syncthreads();
    a = b = 0.0;
    for (int k = 0; k < kBlock / 64; k++) {
        a += red[0][k];
        b += red[1][k];
    }
    __syncthreads();
}
// partials[blockIdx.x] = the workgroup's sum of a, and of b kMaxBlocks further on
__device__ __forceinline__ void write_pair(double a, double b, double *partials, bool two)
{
    block_pair(a, b);
    if (threadIdx.x == 0) {
        partials[blockIdx.x] = a;
        if (two) partials[kMaxBlocks + blockIdx.x] = b;
    }
}
// The sums of n partials (and of the second set) in every thread; false if the
// solve has stopped.  The first workgroup may set the flag in the launch that
// tests it here, so a workgroup reads it once for all its wavefronts, which
// then leave together or all see the whole sums.
__device__ __forceinline__ bool sum_pair(const int *done, const double *__restrict__ partials, int n, bool two, double &a,
                                         double &b)
{
    __shared__ int halt;
    if (threadIdx.x == 0) halt = *done;
    a = b = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += kBlock) {
        a += partials[i];
        if (two) b += partials[kMaxBlocks + i];
    }
    block_pair(a, b);
    return halt == 0;
}

// The head of step k by every workgroup alike: r.r and r.z of the residual
// after k steps from the partials of the update (or the start), the stop test
// (tolerance, limit, a non-finite or non-positive sum) and beta.  The first
// workgroup records them.  True: go on.
__device__ __forceinline__ bool mass_head(const double *__restrict__ partials, int n, int k, double tol2,
                                          const CgState &st, double &beta)
{
    double rr, rz;
    if (!sum_pair(st.done, partials, n, true, rr, rz)) return false;
    const double target = k > 0 ? st.scal[2] : tol2 * rr;
    int d = 0;
    if (!std::isfinite(rr)) d = 4;
    else if (rr <= target) d = 1;              // includes b = 0
    else if (k >= st.maxit) d = 2;
    else if (!std::isfinite(rz)) d = 4;
    else if (!(rz > 0.0)) d = 3;
    beta = k > 0 && !d ? rz / st.rz[k - 1] : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (k == 0) st.scal[2] = target;
        st.rr[k] = rr;
        st.rz[k] = rz;
        *st.iter = k;
        if (d) *st.done = d;
    }
    return d == 0;
}

__global__ __launch_bounds__(kBlock) void k_mass_start(int n, const double *__restrict__ b,
                                                       const double *__restrict__ dinv, double *__restrict__ x,
                                                       double *__restrict__ r, double *__restrict__ z,
                                                       double *__restrict__ partials, CgState st)
{
    double bb = 0.0, rz = 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) *st.done = 0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const double bi = b[i], zi = dinv[i] * bi;
        x[i] = 0.0;
        r[i] = bi;
        z[i] = zi;
        bb += bi * bi;
        rz += bi * zi;
    }
    write_pair(bb, rz, partials, true);
}

// p = z + beta p
__global__ __launch_bounds__(kBlock) void k_mass_direction(int n, const double *__restrict__ z, double *__restrict__ p,
                                                           const double *__restrict__ partials, int nparts, int k,
                                                           double tol2, CgState st)
{
    double beta;
    if (!mass_head(partials, nparts, k, tol2, st, beta)) return;
    if (k == 0) {
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) p[i] = z[i];
        return;
    }
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) p[i] = z[i] + beta * p[i];
}

// q = M p with LPR lanes per row (rows of M_p hold 15 entries at P1 and
// about 40 at P2 on the benchmark meshes; one lane per row left each lane a
// chain of dependent loads over the whole row, 241 us per product at P2
// 32^3) and the partial sums of p.q.  DIR: the step's head comes first and
// p = z + beta p_old is formed for every gathered entry (p and p_old are
// different buffers).
template <int LPR, bool DIR>
__global__ __launch_bounds__(kBlock) void k_mass_product(int n, const int *__restrict__ ptr,
                                                         const int *__restrict__ col, const double *__restrict__ val,
                                                         const double *__restrict__ z, const double *__restrict__ p_old,
                                                         double *__restrict__ p, double *__restrict__ q,
                                                         const double *__restrict__ head_parts, int nparts, int k,
                                                         double tol2, double *__restrict__ pq_parts, CgState st)
{
    double beta = 0.0;
    if (DIR) {
        if (!mass_head(head_parts, nparts, k, tol2, st, beta)) return;
    } else if (*st.done) {
        return;
    }
    const double *__restrict__ po = k > 0 ? p_old : z;
    auto at = [&](int j) { return DIR ? z[j] + beta * po[j] : p_old[j]; };
    double pq = 0.0;
    const int sub = threadIdx.x % LPR;
    for (int base = blockIdx.x * (kBlock / LPR); base < n; base += gridDim.x * (kBlock / LPR)) {
        const int row = base + (int)(threadIdx.x / LPR);
        double s = 0.0;
        if (row < n) {
            const int e1 = ptr[row + 1];
#pragma unroll 4
            for (int e = ptr[row] + sub; e < e1; e += LPR) s += val[e] * at(col[e]);
        }
#pragma unroll
        for (int off = LPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, LPR);
        if (row < n && sub == 0) {
            const double pr = at(row);
            if (DIR) p[row] = pr;
            q[row] = s;
            pq += pr * s;
        }
    }
    write_pair(pq, 0.0, pq_parts, false);
}

// alpha = rz[k] / p.q: x += alpha p, r -= alpha q, z = D^-1 r, the partials of
// r.r and r.z
__global__ __launch_bounds__(kBlock) void k_mass_update(int n, double *__restrict__ x, double *__restrict__ r,
                                                        const double *__restrict__ p, const double *__restrict__ q,
                                                        const double *__restrict__ dinv, double *__restrict__ z,
                                                        const double *__restrict__ pq_parts, int nparts, int k,
                                                        double *__restrict__ partials, CgState st)
{
    double pq, none;
    if (!sum_pair(st.done, pq_parts, nparts, false, pq, none)) return;
    const int bad = !std::isfinite(pq) ? 4 : !(pq > 0.0) ? 3 : 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st.pq[k] = pq;
        if (bad) *st.done = bad;
    }
    if (bad) return;
    const double alpha = st.rz[k] / pq;
    double rr = 0.0, rz = 0.0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        x[i] += alpha * p[i];
        const double ri = r[i] - alpha * q[i], zi = dinv[i] * ri;
        r[i] = ri;
        z[i] = zi;
        rr += ri * ri;
        rz += ri * zi;
    }
    write_pair(rr, rz, partials, true);
}

__global__ __launch_bounds__(kBlock) void k_negate(int n, const double *__restrict__ x, double *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) y[i] = -x[i];
}

}  // namespace

int mass_start(hipStream_t s, int n, const double *b, const double *dinv, double *x, double *r, double *z,
               double *partials, const CgState &st)
{
    const int g = mass_grid(n);
    hipLaunchKernelGGL(k_mass_start, dim3(g), dim3(kBlock), 0, s, n, b, dinv, x, r, z, partials, st);
    return g;
}

int mass_step(hipStream_t s, const DevCsrView &M, int k, double tol2, const MassBufs &v, int nparts, const CgState &st)
{
    const int n = M.n, lpr = M.lpr >= 16 ? 16 : (M.lpr >= 8 ? 8 : 4);
    long long need = ((long long)n * lpr + kBlock - 1) / kBlock;
    const int g = (int)(need < 1 ? 1 : (need > kMassParts ? kMassParts : need)), gv = mass_grid(n);
    const bool dir = M.n <= kMassGatherRows;
    double *p = dir && k % 2 ? v.p2 : v.p;
    const double *po = !dir ? v.p : k % 2 ? v.p : v.p2;
    if (!dir)
        hipLaunchKernelGGL(k_mass_direction, dim3(gv), dim3(kBlock), 0, s, n, v.z, v.p, v.partials, nparts, k, tol2, st);
#define PRODUCT(L, D)                                                                                               \
    hipLaunchKernelGGL((k_mass_product<L, D>), dim3(g), dim3(kBlock), 0, s, n, M.ptr, M.col, (const double *)M.val, \
                       v.z, po, p, v.q, v.partials, nparts, k, tol2, v.pq_parts, st)
    if (dir) {
        if (lpr == 16) PRODUCT(16, true);
        else if (lpr == 8) PRODUCT(8, true);
        else PRODUCT(4, true);
    } else {
        if (lpr == 16) PRODUCT(16, false);
        else if (lpr == 8) PRODUCT(8, false);
        else PRODUCT(4, false);
    }
#undef PRODUCT
    hipLaunchKernelGGL(k_mass_update, dim3(gv), dim3(kBlock), 0, s, n, v.x, v.r, p, v.q, v.dinv, v.z, v.pq_parts, g, k,
                       v.partials, st);
    return gv;
}

void vec_negate(hipStream_t s, int n, const double *x, double *y)
{
    hipLaunchKernelGGL(k_negate, dim3(mass_grid(n)), dim3(kBlock), 0, s, n, x, y);
}

}  // namespace auxp
