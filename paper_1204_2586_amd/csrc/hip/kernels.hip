// Solve-phase kernels of the auxiliary-space preconditioned CG (gfx950).
//
// All of this work is memory-bound sparse algebra: every kernel streams its
// operator once, gathers the vector it multiplies, and fuses the elementwise
// smoother / residual / CG updates into the same pass (one l1-Jacobi sweep is
// one pass over A).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <stdexcept>
#include <type_traits>

#include "kernels.hpp"

namespace auxp {

namespace {

__device__ __forceinline__ bool stop(const int *done) { return done != nullptr && *done != 0; }

// the stop flag itself, for kernels that request other words before testing it
__device__ __forceinline__ int stop_word(const int *done)
{
    int d = 0;
    if (done != nullptr) d = *done;
    return d;
}

// Element j of a vector addressed by a 32-bit byte offset from its (uniform)
// base: the load takes the scalar-base form, one address register instead of
// two.  Vectors of the single-vector solve are far below 4 GiB (row numbers
// are 32-bit, and an operator's stored entries too).
template <typename T>
__device__ __forceinline__ T at32(const T *__restrict__ base, int j)
{
    return *(const T *)((const char *)base + (unsigned)j * (unsigned)sizeof(T));
}

template <int LPR, typename A>
__device__ __forceinline__ A group_sum(A v)
{
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, LPR);
    return v;
}
template <int LPR, typename T>
__device__ __forceinline__ Vec3<T> group_sum(Vec3<T> v)
{
    return {group_sum<LPR>(v.a), group_sum<LPR>(v.b), group_sum<LPR>(v.c)};
}

// an element in another precision
template <typename X, typename Y>
struct Cast {
    static __device__ __forceinline__ X of(const Y &y) { return (X)y; }
};
template <typename T, typename S>
struct Cast<Vec3<T>, Vec3<S>> {
    static __device__ __forceinline__ Vec3<T> of(const Vec3<S> &y) { return {(T)y.a, (T)y.b, (T)y.c}; }
};
template <typename X, typename Y>
__device__ __forceinline__ X cast(const Y &y)
{
    return Cast<X, Y>::of(y);
}

// sum over the block (BS threads) in a fixed order; valid in thread 0
template <int BS = kBlock>
__device__ double block_sum(double v)
{
    __shared__ double red[BS / 64];
    v = group_sum<64>(v);
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < BS / 64; i++) s += red[i];
    return s;
}

template <int BS = kBlock>
__device__ __forceinline__ void write_partial(double *partials, double v)
{
    double b = block_sum<BS>(v);
    if (threadIdx.x == 0) partials[blockIdx.x] = b;
}

inline int grid_cap(long long need)
{
    if (need < 1) need = 1;
    if (need > kMaxBlocks) need = kMaxBlocks;
    return (int)need;
}

// The sum of a reduction's partials by one workgroup of BS threads, in a fixed
// order (valid in thread 0): four accumulators, loads unrolled, so all of a
// thread's partials are in flight.
template <int BS>
__device__ __forceinline__ double partials_sum(const double *__restrict__ partials, int nparts)
{
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * BS < nparts; i += 4 * BS) {
        s0 += partials[i];
        s1 += partials[i + BS];
        s2 += partials[i + 2 * BS];
        s3 += partials[i + 3 * BS];
    }
    for (; i < nparts; i += BS) s0 += partials[i];
    return block_sum<BS>((s0 + s1) + (s2 + s3));
}
// The same, known to every thread; false if the solve has stopped.  The first
// workgroup of such a launch may set the flag (the sum is what it tests), so
// the others read it once for all their wavefronts: these leave together or
// not at all, and then all see the whole sum.
template <int BS>
__device__ __forceinline__ bool partials_sum_all(const int *done, const double *__restrict__ partials, int nparts,
                                                 double &sum)
{
    __shared__ double total;
    __shared__ int halt;
    int d = 0;
    if (threadIdx.x == 0) d = *done;
    const double s = partials_sum<BS>(partials, nparts);
    if (threadIdx.x == 0) {
        total = s;
        halt = d;
    }
    __syncthreads();
    sum = total;
    return halt == 0;
}

// the stop code an inner product (r.z or p.Ap) gives: 0 to go on
__device__ __forceinline__ int product_stop(double s) { return !std::isfinite(s) ? 4 : !(s > 0.0) ? 3 : 0; }

// (one thread) the state of the solve after k iterations with stop flag d, for the host
__device__ __forceinline__ void report(const CgState &st, int k, int d, double rr)
{
    if (!st.report) return;
    st.report->rr = rr;
    const double target = st.scal[2];
    const float ratio = (float)fmin(target > 0.0 ? rr / target : 3e38, 3e38);
    const unsigned long long w = (unsigned long long)((unsigned)k | (unsigned)d << 28) << 32 | __float_as_uint(ratio);
    __hip_atomic_store(&st.report->word, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// (one thread) a breakdown at iteration k: the last iterate stands
__device__ __forceinline__ void stop_solve(const CgState &st, int k, int d)
{
    *st.done = d;
    report(st, k, d, st.rr[k]);
}

// One workgroup: the sum of a reduction's partials into its CG slot, and what
// follows from it (the stop flag, the iteration count).
template <int BS>
__device__ __forceinline__ void finish_block(const double *__restrict__ partials, int nparts, int mode, double *out,
                                             const CgState &st)
{
    if (mode != FIN_PLAIN && *st.done) return;
    const double s = partials_sum<BS>(partials, nparts);
    if (threadIdx.x != 0) return;
    if (mode == FIN_PLAIN) {
        *out = s;
        return;
    }
    const int k = *st.iter;
    int d = 0;
    if (mode == FIN_RR) {
        st.rr[k + 1] = s;
        *st.iter = k + 1;
        if (!std::isfinite(s)) d = 4;
        else if (s <= st.scal[2]) d = 1;
        else if (k + 1 >= st.maxit) d = 2;
        if (d) *st.done = d;
        report(st, k + 1, d, s);
    } else {
        (mode == FIN_PQ ? st.pq : st.rz)[k] = s;
        d = product_stop(s);
        if (d) stop_solve(st, k, d);
    }
}

// ------------------------------------------------------------------ SELL

// W wavefronts per 64-row slice, one lane per row; consecutive slices go to
// consecutive workgroups, which the dispatcher spreads round-robin over the
// dies, so at any moment all dies gather from the same neighbourhood of the
// vector and share it through the last-level cache (giving each die its own
// contiguous range of slices measured twice as slow, and no faster when the
// ranges are balanced by entries).

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// four consecutive values of a lane: one 16-byte load, or two
__device__ __forceinline__ void load4(const float *p, float v[4])
{
    const f32x4 t = *(const f32x4 *)p;
    v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
}
__device__ __forceinline__ void load4(const double *p, double v[4])
{
    const f64x2 a = *(const f64x2 *)p, b = *(const f64x2 *)(p + 2);
    v[0] = a.x, v[1] = a.y, v[2] = b.x, v[3] = b.y;
}

// Groups h, h + W, ... of a slice (m its meta) for the row of this lane; four
// accumulators, one per entry of a group.
template <typename T, typename X, int W, typename XF>
__device__ __forceinline__ X sell_part(const DevSellView &A, const int4 m, int lane, int h, XF x)
{
    const T *__restrict__ val = (const T *)A.val + (size_t)m.x * (4 * kSlice) + 4 * lane;
    X s0{}, s1{}, s2{}, s3{};
    if (m.z < 0) {
        const unsigned short *__restrict__ off = A.off + (size_t)m.x * (4 * kSlice) + 4 * lane;
        const int2 *__restrict__ base = A.base + (size_t)m.x * 4;
#pragma unroll 2
        for (int g = h; g < m.y; g += W) {
            T v[4];
            load4(val + (size_t)g * (4 * kSlice), v);
            const u16x4 o = *(const u16x4 *)(off + (size_t)g * (4 * kSlice));
            const int2 *__restrict__ b = base + 4 * g;
            s0 += v[0] * x((o.x & 0x8000 ? b[0].y : b[0].x) + (o.x & 0x7fff));
            s1 += v[1] * x((o.y & 0x8000 ? b[1].y : b[1].x) + (o.y & 0x7fff));
            s2 += v[2] * x((o.z & 0x8000 ? b[2].y : b[2].x) + (o.z & 0x7fff));
            s3 += v[3] * x((o.w & 0x8000 ? b[3].y : b[3].x) + (o.w & 0x7fff));
        }
    } else {
        const int *__restrict__ col = A.wide + (size_t)m.z * (4 * kSlice) + 4 * lane;
#pragma unroll 2
        for (int g = h; g < m.y; g += W) {
            T v[4];
            load4(val + (size_t)g * (4 * kSlice), v);
            const i32x4 c = *(const i32x4 *)(col + (size_t)g * (4 * kSlice));
            s0 += v[0] * x(c.x);
            s1 += v[1] * x(c.y);
            s2 += v[2] * x(c.z);
            s3 += v[3] * x(c.w);
        }
    }
    return (s0 + s1) + (s2 + s3);
}

// threads of a workgroup with W wavefronts per slice, and its slices
template <int W>
constexpr int sell_block() { return W > 4 ? 64 * W : kBlock; }
template <int W>
constexpr int sell_per_block() { return sell_block<W>() / (64 * W); }

// Every row of A by `grid` workgroups: s = (A x)_row, then epi(row, s, in) with in = pre(row) the
// row's other inputs, requested before the row's entries; nothing when the
// stop flag `halt` is set (it is tested after the first slice's meta is
// requested, so the two loads overlap).  With W > 1 the other wavefronts' sums
// pass through LDS and are added in a fixed order; every thread of the block
// then runs the same number of steps, so the barriers are uniform.  SET: the
// flag may be set while the launch runs, so the wavefronts of a workgroup may
// read it differently; with W > 1 those that find it set pass the barriers
// without doing anything (rows that miss their share are not read again: the
// solve has stopped).
template <typename T, typename X, int W, bool SET = false, typename XF, typename PRE, typename EPI>
__device__ __forceinline__ void sell_rows(const DevSellView &A, int grid, int halt, XF x, PRE pre, EPI epi)
{
    constexpr int S = sell_per_block<W>();
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int q = w / W, h = w % W;
    int sl = (int)blockIdx.x * S + q;
    int4 m = make_int4(0, 0, -1, 0);
    if (sl < A.nslices) m = A.meta[sl];
    asm volatile("" ::"s"(m.x), "s"(halt));
    if (halt && (W == 1 || !SET)) return;
    const bool work = W == 1 || !SET || !halt;
    if constexpr (W == 1) {
        for (; sl < A.nslices; sl += grid * S) {
            if (sl != (int)blockIdx.x * S + q) m = A.meta[sl];
            const int row = sl * kSlice + lane;
            const auto in = pre(min(row, A.n - 1));
            const X s = sell_part<T, X, W>(A, m, lane, 0, x);
            if (row < A.n) epi(row, s, in);
        }
    } else {
        __shared__ X part[S][W - 1][64];
        const int per_step = S * grid;
        const int steps = (A.nslices + per_step - 1) / per_step;
        for (int it = 0; it < steps; it++, sl += per_step) {
            const int row = sl * kSlice + lane;
            decltype(pre(0)) in = {};
            X s{};
            if (sl < A.nslices && work) {
                if (it > 0) m = A.meta[sl];
                if (h == 0) in = pre(min(row, A.n - 1));
                s = sell_part<T, X, W>(A, m, lane, h, x);
            }
            if (it > 0) __syncthreads();           // the previous step's sums are consumed
            if (h > 0) part[q][h - 1][lane] = s;
            __syncthreads();
            if (h == 0 && sl < A.nslices && work) {
#pragma unroll
                for (int k = 0; k < W - 1; k++) s += part[q][k][lane];
                if (row < A.n) epi(row, s, in);
            }
        }
    }
}

#define WAVES_SWITCH(A, CALL)                                     \
    switch ((A).waves) {                                          \
    case 1: { constexpr int W = 1; CALL; } break;                 \
    case 2: { constexpr int W = 2; CALL; } break;                 \
    case 4: { constexpr int W = 4; CALL; } break;                 \
    default: { constexpr int W = 8; CALL; } break;                \
    }

template <int W>
inline int sell_grid(const DevSellView &A)
{
    return grid_cap(((long long)A.nslices + sell_per_block<W>() - 1) / sell_per_block<W>());
}

// FIN: the last workgroup is one more than the rows take and finishes the
// r.r reduction of the CG update before (nothing here waits for its result;
// a stop flag it sets is read by the kernels that follow).  operm: row r goes
// to zout[operm[r]].
template <typename T, typename X, typename XR, typename XZ, bool DOT, bool FIN, int W>
__global__ __launch_bounds__(sell_block<W>()) void k_sell_sweep(DevSellView A, const T *__restrict__ dinv,
                                                                const XR *__restrict__ rhs, const X *__restrict__ zin,
                                                                XZ *__restrict__ zout, const double *__restrict__ rdot,
                                                                double *partials, const int *done,
                                                                const int *__restrict__ operm, RrFinish fin)
{
    const int grid = (int)gridDim.x - (FIN ? 1 : 0);
    if (FIN && (int)blockIdx.x == grid) {
        finish_block<sell_block<W>()>(fin.partials, fin.nparts, FIN_RR, nullptr, fin.st);
        return;
    }
    const int halt = stop_word(done);
    double acc = 0.0;
    struct In {
        X z, b;
        T d;
        double r;
        int o;
    };
    sell_rows<T, X, W, FIN>(
        A, grid, halt, [&](int j) { return at32(zin, j); },
        [&](int row) {
            return In{zin[row], cast<X>(rhs[row]), dinv[row], DOT ? rdot[row] : 0.0, operm ? operm[row] : row};
        },
        [&](int row, const X &s, const In &in) {
            const XZ zi = cast<XZ>(in.z + in.d * (in.b - s));
            zout[in.o] = zi;
            if constexpr (DOT) acc += in.r * (double)zi;
        });
    if (DOT) write_partial<sell_block<W>()>(partials, acc);
}

template <typename T, int W>
__global__ __launch_bounds__(sell_block<W>()) void k_sell_resid(DevSellView A, const T *__restrict__ rhs,
                                                                const T *__restrict__ z, T *__restrict__ res,
                                                                const int *done)
{
    sell_rows<T, T, W>(A, (int)gridDim.x, stop_word(done), [&](int j) { return at32(z, j); },
                    [&](int row) { return rhs[row]; }, [&](int row, T s, T b) { res[row] = b - s; });
}

// operm: row r goes to y[operm[r]]
template <bool DOT, int W>
__global__ __launch_bounds__(sell_block<W>()) void k_sell_spmv64(DevSellView A, const double *__restrict__ x,
                                                                 double *__restrict__ y, double *partials,
                                                                 const int *done, const int *__restrict__ operm)
{
    const int halt = stop_word(done);
    double acc = 0.0;
    struct In {
        double x;
        int o;
    };
    sell_rows<double, double, W>(A, (int)gridDim.x, halt, [&](int j) { return at32(x, j); },
                         [&](int row) { return In{DOT ? x[row] : 0.0, operm ? operm[row] : row}; },
                         [&](int row, double s, const In &in) {
                             y[in.o] = s;
                             if (DOT) acc += in.x * s;
                         });
    if (DOT) write_partial<sell_block<W>()>(partials, acc);
}

// y = A x for three vectors
template <int W>
__global__ __launch_bounds__(sell_block<W>()) void k_sell_spmv64x3(DevSellView A, const Vec3<double> *__restrict__ x,
                                                                   Vec3<double> *__restrict__ y)
{
    sell_rows<double, Vec3<double>, W>(A, (int)gridDim.x, 0, [&](int j) { return at32(x, j); }, [&](int) { return 0; },
                                       [&](int row, const Vec3<double> &s, int) { y[row] = s; });
}

// The CG product with the direction formed on the way: p = z + beta p_old
// (p = z at k = 0), q = A p, partials of p.q, beta = r.z / (r.z)_{k-1} with r.z
// summed from its partials by every workgroup in the same order (the first
// one records it and its stop code).  p and p_old are different buffers.
template <int W>
__global__ __launch_bounds__(sell_block<W>()) void k_cg_product(DevSellView A, const double *__restrict__ z,
                                                                const double *__restrict__ p_old,
                                                                double *__restrict__ p, double *__restrict__ q,
                                                                const double *__restrict__ rz_parts, int rz_n,
                                                                double *__restrict__ pq_parts, CgState st)
{
    const int k = *st.iter;
    double rz;
    if (!partials_sum_all<sell_block<W>()>(st.done, rz_parts, rz_n, rz)) return;
    const int bad = product_stop(rz);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st.rz[k] = rz;
        if (bad) stop_solve(st, k, bad);
    }
    if (bad) return;
    const double beta = k > 0 ? rz / st.rz[k - 1] : 0.0;
    const double *__restrict__ po = k > 0 ? p_old : z;
    double acc = 0.0;
    sell_rows<double, double, W>(A, (int)gridDim.x, 0, [&](int j) { return at32(z, j) + beta * at32(po, j); },
                         [&](int row) { return z[row] + beta * po[row]; },
                         [&](int row, double s, double pr) {
                             p[row] = pr;
                             q[row] = s;
                             acc += pr * s;
                         });
    write_partial<sell_block<W>()>(pq_parts, acc);
}

template <int W>
__global__ __launch_bounds__(sell_block<W>()) void k_sell_residual64(DevSellView A, const double *__restrict__ f,
                                                                     const double *__restrict__ u,
                                                                     double *__restrict__ r)
{
    sell_rows<double, double, W>(A, (int)gridDim.x, 0, [&](int j) { return at32(u, j); }, [&](int row) { return f[row]; },
                         [&](int row, double s, double b) { r[row] = b - s; });
}

template <typename T, typename X, typename XR>
__global__ __launch_bounds__(kBlock) void k_jacobi0(int n, const T *__restrict__ dinv, const XR *__restrict__ r,
                                                    X *__restrict__ z, X *__restrict__ rT, const int *done)
{
    if (stop(done)) return;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const X ri = cast<X>(r[i]);
        z[i] = dinv[i] * ri;
        if (rT) rT[i] = ri;
    }
}

// r_int = r[perm], z = D^{-1} r_int (and r_int in the working precision)
template <typename T>
__global__ __launch_bounds__(kBlock) void k_gather_jacobi0(int n, const int *__restrict__ perm,
                                                           const T *__restrict__ dinv, const double *__restrict__ r,
                                                           double *__restrict__ rint, T *__restrict__ z,
                                                           T *__restrict__ rT)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const double v = r[perm[i]];
        const T ri = (T)v;
        rint[i] = v;
        z[i] = dinv[i] * ri;
        if (rT) rT[i] = ri;
    }
}

// ------------------------------------------------------------------- CSR

#define FOR_ROWS(LPR, n)                                                                                    \
    const int sub_ = threadIdx.x % (LPR);                                                                   \
    for (int base_ = blockIdx.x * (kBlock / (LPR)); base_ < (n); base_ += gridDim.x * (kBlock / (LPR)))     \
        for (int row = base_ + threadIdx.x / (LPR), once_ = 1; once_; once_ = 0)

template <int LPR, typename X, typename T, typename XF>
__device__ __forceinline__ X csr_row(const int *__restrict__ ptr, const int *__restrict__ col,
                                     const T *__restrict__ val, int row, int sub, XF x)
{
    X s{};
    const int e1 = ptr[row + 1];
#pragma unroll 8
    for (int e = ptr[row] + sub; e < e1; e += LPR) s += val[e] * x(col[e]);
    return group_sum<LPR>(s);
}

template <typename T, typename X, int LPR, bool ADD>
__global__ __launch_bounds__(kBlock) void k_csr_matvec(int n, const int *__restrict__ ptr, const int *__restrict__ col,
                                                       const T *__restrict__ val, const X *__restrict__ x,
                                                       X *__restrict__ y, const int *done)
{
    if (stop(done)) return;
    FOR_ROWS(LPR, n)
    {
        if (row < n) {
            const X s = csr_row<LPR, X>(ptr, col, val, row, sub_, [&](int j) { return x[j]; });
            if (sub_ == 0) y[row] = ADD ? y[row] + s : s;
        }
    }
}

// Row-split sliced ELL product, one wavefront per slice of 64 / L rows.
// MODE 0: y = M x1; 1: y += M x1; 2: y = M [x1; x2] (columns below split
// index x1).  Every slot is one coalesced load of 64 values and 64 columns;
// the slot count is uniform over the wavefront.
template <typename T, typename X, int L, int MODE>
__global__ __launch_bounds__(kBlock) void k_ell_matvec(int n, const int *__restrict__ off, const int *__restrict__ col,
                                                       const T *__restrict__ val, const X *__restrict__ x1,
                                                       const X *__restrict__ x2, int split, X *__restrict__ y,
                                                       const int *done)
{
    if (stop(done)) return;
    constexpr int C = 64 / L;
    const int lane = threadIdx.x % 64;
    const int nsl = (n + C - 1) / C;
    for (int sl = blockIdx.x * (kBlock / 64) + (int)(threadIdx.x / 64); sl < nsl; sl += gridDim.x * (kBlock / 64)) {
        const int e1 = off[sl + 1];
        X acc{};
#pragma unroll 8
        for (int e = off[sl] + lane; e < e1; e += 64) {
            const int j = col[e];
            acc += val[e] * (MODE == 2 ? (j < split ? x1[j] : x2[j - split]) : x1[j]);
        }
        acc = group_sum<L>(acc);
        const int row = sl * C + lane / L;
        if (lane % L == 0 && row < n) {
            if (MODE == 1) y[row] += acc;
            else y[row] = acc;
        }
    }
}

// y = M [x1; x2]: columns below `split` index x1, the others x2
template <typename T, typename X, int LPR>
__global__ __launch_bounds__(kBlock) void k_csr_matvec2(int n, const int *__restrict__ ptr, const int *__restrict__ col,
                                                        const T *__restrict__ val, const X *__restrict__ x1,
                                                        const X *__restrict__ x2, int split, X *__restrict__ y,
                                                        const int *done)
{
    if (stop(done)) return;
    FOR_ROWS(LPR, n)
    {
        if (row < n) {
            const X s = csr_row<LPR, X>(ptr, col, val, row, sub_, [&](int j) { return j < split ? x1[j] : x2[j - split]; });
            if (sub_ == 0) y[row] = s;
        }
    }
}

template <typename T, int LPR>
__global__ __launch_bounds__(kBlock) void k_csr_vpre(int n, const int *__restrict__ ptr, const int *__restrict__ col,
                                                     const T *__restrict__ val, const T *__restrict__ dinv,
                                                     const T *__restrict__ b, T *__restrict__ x, T *__restrict__ r,
                                                     const int *done)
{
    if (stop(done)) return;
    FOR_ROWS(LPR, n)
    {
        if (row < n) {
            const T s = csr_row<LPR, T>(ptr, col, val, row, sub_, [&](int j) { return dinv[j] * b[j]; });
            if (sub_ == 0) {
                x[row] = dinv[row] * b[row];
                r[row] = b[row] - s;
            }
        }
    }
}

template <typename T, int LPR>
__global__ __launch_bounds__(kBlock) void k_csr_sweep(int n, const int *__restrict__ ptr, const int *__restrict__ col,
                                                      const T *__restrict__ val, const T *__restrict__ dinv,
                                                      const T *__restrict__ b, const T *__restrict__ x,
                                                      T *__restrict__ y, const int *done)
{
    if (stop(done)) return;
    FOR_ROWS(LPR, n)
    {
        if (row < n) {
            const T s = csr_row<LPR, T>(ptr, col, val, row, sub_, [&](int j) { return x[j]; });
            if (sub_ == 0) y[row] = x[row] + dinv[row] * (b[row] - s);
        }
    }
}

// One workgroup per row: each lane's few loads of the row are all in flight
// at once (at most n / 256 per lane), then a workgroup sum; the rows of the
// dense cycle (at most 8192) are short enough that one wavefront per row
// leaves each lane a chain of dependent load rounds.
template <typename T, typename X>
__global__ __launch_bounds__(kBlock) void k_dense_gemv(int n, const T *__restrict__ Ainv, const X *__restrict__ b,
                                                       X *__restrict__ x, const int *done)
{
    if (stop(done)) return;
    __shared__ X red[kBlock / 64];
    const int w = threadIdx.x / 64, l = threadIdx.x % 64;
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const T *__restrict__ row = Ainv + (size_t)i * n;
        X s0{}, s1{};
        int j = threadIdx.x;
        for (; j + kBlock < n; j += 2 * kBlock) {
            s0 += row[j] * b[j];
            s1 += row[j + kBlock] * b[j + kBlock];
        }
        if (j < n) s0 += row[j] * b[j];
        const X s = group_sum<64>(s0 + s1);
        __syncthreads();                           // red of the previous row is consumed
        if (l == 0) red[w] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            X t{};
            for (int q = 0; q < kBlock / 64; q++) t += red[q];
            x[i] = t;
        }
    }
}

// ------------------------------------------------------------------ CG

__global__ __launch_bounds__(kBlock) void k_dot(int n, const double *__restrict__ a, const double *__restrict__ b,
                                                double *partials)
{
    double acc = 0.0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) acc += a[i] * b[i];
    write_partial(partials, acc);
}

__global__ __launch_bounds__(kBlock) void k_finish(const double *__restrict__ partials, int nparts, int mode,
                                                   double *out, CgState st)
{
    finish_block<kBlock>(partials, nparts, mode, out, st);
}

// the state of a solve from f.f and r_0.r_0
__device__ __forceinline__ void cg_state_init(const CgState &st, double f2, double r2, double tol2)
{
    *st.iter = 0;
    st.rr[0] = r2;
    st.scal[2] = tol2 * f2;
    int d = 0;
    if (!std::isfinite(f2) || !std::isfinite(r2)) d = 4;
    else if (r2 <= tol2 * f2) d = 1;     // includes f = 0 with u = 0
    else if (st.maxit <= 0) d = 2;
    *st.done = d;
    if (st.report) st.report->ff = f2;
    if (d) report(st, 0, d, r2);
    else if (st.report) st.report->rr = r2;
}

__global__ __launch_bounds__(kBlock) void k_cg_init_sums(const double *__restrict__ partials, int nparts, CgState st,
                                                         double tol2)
{
    const double r2 = partials_sum<kBlock>(partials, nparts), f2 = partials_sum<kBlock>(partials + nparts, nparts);
    if (threadIdx.x != 0) return;
    st.scal[0] = f2;
    st.scal[1] = r2;
    cg_state_init(st, f2, r2, tol2);
}

__global__ __launch_bounds__(kBlock) void k_gather_pair(int n, const int *__restrict__ idx,
                                                        const double *__restrict__ a, const double *__restrict__ b,
                                                        double *__restrict__ x, double *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const int j = idx[i];
        x[i] = a[j];
        y[i] = b[j];
    }
}

// r = f - A u with the partials of r.r, then of f.f, and the first sweep
template <typename T, int W>
__global__ __launch_bounds__(sell_block<W>()) void k_cg_first(DevSellView A, const double *__restrict__ f,
                                                              const double *__restrict__ u, double *__restrict__ r,
                                                              const T *__restrict__ dinv, T *__restrict__ z0,
                                                              T *__restrict__ rT, double *partials)
{
    double r2 = 0.0, f2 = 0.0;
    struct In {
        double f;
        T d;
    };
    sell_rows<double, double, W>(A, (int)gridDim.x, 0, [&](int j) { return at32(u, j); },
                         [&](int row) { return In{f[row], dinv[row]}; },
                         [&](int row, double s, const In &in) {
                             const double v = in.f - s;
                             const T t = (T)v;
                             r[row] = v;
                             z0[row] = in.d * t;
                             if (rT) rT[row] = t;
                             r2 += v * v;
                             f2 += in.f * in.f;
                         });
    write_partial<sell_block<W>()>(partials, r2);
    write_partial<sell_block<W>()>(partials + gridDim.x, f2);
}

// the update fused with the preconditioner's first sweep from zero:
// z0 = D^-1 r in the preconditioner's type (and its copy of r), with the
// expressions of k_jacobi0.  RESUM: p.q is summed from its pq_n partials by
// every workgroup in the same order (the first one records it).
template <typename T, bool RESUM>
__global__ __launch_bounds__(kBlock) void k_cg_update_prep(int n, double *__restrict__ x, double *__restrict__ r,
                                                           const double *__restrict__ p, const double *__restrict__ q,
                                                           CgState st, double *partials, const T *__restrict__ dinv,
                                                           T *__restrict__ z0, T *__restrict__ rT,
                                                           const double *__restrict__ pq_parts, int pq_n)
{
    const int k = *st.iter;
    double pq;
    if (RESUM) {
        if (!partials_sum_all<kBlock>(st.done, pq_parts, pq_n, pq)) return;
        const int bad = product_stop(pq);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st.pq[k] = pq;
            if (bad) stop_solve(st, k, bad);
        }
        if (bad) return;
    } else {
        if (*st.done) return;
        pq = st.pq[k];
    }
    const double alpha = st.rz[k] / pq;
    double acc = 0.0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        x[i] += alpha * p[i];
        double ri = r[i] - alpha * q[i];
        r[i] = ri;
        acc += ri * ri;
        T rt = (T)ri;
        z0[i] = dinv[i] * rt;
        if (rT) rT[i] = rt;
    }
    write_partial(partials, acc);
}

__global__ __launch_bounds__(kBlock) void k_cg_direction(int n, const double *__restrict__ z, double *__restrict__ p,
                                                         CgState st)
{
    if (*st.done) return;
    const int k = *st.iter;
    if (k == 0) {
        for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) p[i] = z[i];
        return;
    }
    const double beta = st.rz[k] / st.rz[k - 1];
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) p[i] = z[i] + beta * p[i];
}

__global__ __launch_bounds__(kBlock) void k_interleave3(int n, const int *__restrict__ idx,
                                                        const double *__restrict__ x, Vec3<double> *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const size_t j = idx ? idx[i] : i;
        y[i] = {x[j], x[j + n], x[j + 2 * (size_t)n]};
    }
}

__global__ __launch_bounds__(kBlock) void k_split3(int n, const int *__restrict__ idx,
                                                   const Vec3<double> *__restrict__ x, double *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
        const size_t j = idx ? idx[i] : i;
        const Vec3<double> v = x[i];
        y[j] = v.a;
        y[j + n] = v.b;
        y[j + 2 * (size_t)n] = v.c;
    }
}

__global__ __launch_bounds__(kBlock) void k_gather(int n, const int *__restrict__ idx, const double *__restrict__ x,
                                                   double *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) y[i] = x[idx[i]];
}

__global__ __launch_bounds__(kBlock) void k_scatter(int n, const int *__restrict__ idx, const double *__restrict__ x,
                                                    double *__restrict__ y)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) y[idx[i]] = x[i];
}

// ------------------------------------------------------------- adjoint

// 64 tets per workgroup, one lane each in every one of its NW wavefronts.
// The rows of G_t sum to zero, so
//     sum_pq G_pq lam^T M^pq u = -sum_k G_k lam^T S^k u
// over the six vertex pairs k = (p, q), S^k = M^pp + M^qq - M^pq - M^qp, and
// the S^k are symmetric: per node pair (a <= b) one entry sum_k G_k S^k_ab
// meets lam_a u_b + lam_b u_a (the diagonal's tables halved), nine FP64
// operations per pair and tet instead of 16 (nloc + 1) / nloc per entry of the
// sixteen tables.  The element vectors are staged in LDS, so the node loops
// are short loops (unrolled over the nodes they are 20 KB of code at P3, run
// once by each of a few waves, and the instruction fetch cost more than the
// arithmetic); a step takes the rows 2 m and 2 m + 1 at one column b: two LDS
// words per lane, twelve table words uniform over the wavefront (scalar
// loads), eighteen operations.  The steps of row pair m number nloc - 2 m;
// the wavefronts take the pairs in a zigzag, so their sums are nearly equal,
// and the partial sums meet in LDS in a fixed order.  Node numbers and
// metrics are stored by column (entry a of tet t at a nt + t), so every load
// but the gathers is coalesced.  Measured: P3 24^3 76.7 -> 12.4 us (19 MB and
// 0.31 GFLOP: 3 and 4 us at the card's rates), 32^3 23.1, P2 40^3 17.6 (1, 2
// and 4 wavefronts: 26.5, 19.6, 17.6), P4 18^3 16.0 (4 and 8: 18.6, 16.0).
template <int NLOC, int NW>
__global__ __launch_bounds__(64 * NW) void k_kappa_grad(int nt, const int *__restrict__ dofs,
                                                        const double *__restrict__ G6,
                                                        const double *__restrict__ kappa,
                                                        const double *__restrict__ S, const double *__restrict__ u,
                                                        const double *__restrict__ lam, double *__restrict__ g)
{
    constexpr int NP = (NLOC + 1) / 2, NA = (NLOC + NW - 1) / NW;
    __shared__ double us[2 * NP][64], ls[2 * NP][64], part[NW][64];
    const int lane = threadIdx.x & 63, h = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = blockIdx.x * 64 + lane, tc = min(t, nt - 1);
    double G[6];
    int at[NA];
#pragma unroll
    for (int i = 0; i < NA; i++) at[i] = dofs[(size_t)min(h + i * NW, NLOC - 1) * nt + tc];
#pragma unroll
    for (int k = 0; k < 6; k++) G[k] = G6[(size_t)k * nt + tc];
    const double kap = kappa[tc];
#pragma unroll
    for (int i = 0; i < NA; i++) {
        const int a = h + i * NW, j = max(at[i], 0);
        const double ua = u[j], la = lam[j];
        if (a < NLOC) {
            us[a][lane] = at[i] < 0 ? 0.0 : ua;
            ls[a][lane] = at[i] < 0 ? 0.0 : la;
        }
    }
    if (NLOC % 2 && h == 0) us[2 * NP - 1][lane] = ls[2 * NP - 1][lane] = 0.0;
    __syncthreads();
    double acc0 = 0.0, acc1 = 0.0;
    for (int r = 0; r * NW < NP; r++) {
        const int m = r * NW + (r % 2 ? NW - 1 - h : h);
        if (m >= NP) continue;
        // steps before row pair m: sum over m' < m of nloc - 2 m'
        const double *__restrict__ T = S + 12 * (m * NLOC - m * (m - 1));
        const double u0 = us[2 * m][lane], l0 = ls[2 * m][lane], u1 = us[2 * m + 1][lane], l1 = ls[2 * m + 1][lane];
#pragma unroll 2
        for (int b = 2 * m; b < NLOC; b++, T += 12) {
            const double ub = us[b][lane], lb = ls[b][lane];
            double e0 = G[0] * T[0], e1 = G[0] * T[6];
#pragma unroll
            for (int k = 1; k < 6; k++) {
                e0 += G[k] * T[k];
                e1 += G[k] * T[6 + k];
            }
            acc0 += e0 * (l0 * ub + u0 * lb);
            acc1 += e1 * (l1 * ub + u1 * lb);
        }
    }
    part[h][lane] = acc0 + acc1;
    __syncthreads();
    if (h == 0 && t < nt) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NW; w++) s += part[w][lane];
        g[t] = kap * s;
    }
}

}  // namespace

int pick_lpr(double avg)
{
    if (avg <= 1.5) return 1;
    if (avg <= 3.0) return 2;
    if (avg <= 8.0) return 4;
    if (avg <= 24.0) return 8;
    if (avg <= 64.0) return 16;
    return 32;
}

#define LPR_SWITCH(lpr, CALL)                         \
    switch (lpr) {                                    \
    case 1: { constexpr int L = 1; CALL; } break;     \
    case 2: { constexpr int L = 2; CALL; } break;     \
    case 4: { constexpr int L = 4; CALL; } break;     \
    case 8: { constexpr int L = 8; CALL; } break;     \
    case 16: { constexpr int L = 16; CALL; } break;   \
    default: { constexpr int L = 32; CALL; } break;   \
    }

static int vec_grid(long long n) { return grid_cap((n + kBlock - 1) / kBlock); }
static int rows_grid(int n, int lpr) { return grid_cap(((long long)n * lpr + kBlock - 1) / kBlock); }

template <typename T, typename X, typename XR>
int vec_jacobi0(hipStream_t s, int n, const T *dinv, const XR *r, X *z, X *rT, const int *done)
{
    int g = vec_grid(n);
    hipLaunchKernelGGL((k_jacobi0<T, X, XR>), dim3(g), dim3(kBlock), 0, s, n, dinv, r, z, rT, done);
    return g;
}

template <typename T>
void vec_gather_jacobi0(hipStream_t s, int n, const int *perm, const T *dinv, const double *r, double *rint, T *z, T *rT)
{
    hipLaunchKernelGGL(k_gather_jacobi0<T>, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, perm, dinv, r, rint, z, rT);
}

template <typename T>
void vec_jacobi0_t(hipStream_t s, int n, const T *dinv, const T *r, T *z, const int *done)
{
    hipLaunchKernelGGL((k_jacobi0<T, T, T>), dim3(vec_grid(n)), dim3(kBlock), 0, s, n, dinv, r, z, nullptr, done);
}

template <typename T, typename X, typename XR, typename XZ>
int sell_sweep(hipStream_t s, const DevSellView &A, const T *dinv, const XR *rhs, const X *zin, XZ *zout,
               const double *rdot, double *partials, const int *done, const int *operm, const RrFinish *fin)
{
    int g = 0;
#define SWEEP(DOT, FIN)                                                                                    \
    hipLaunchKernelGGL((k_sell_sweep<T, X, XR, XZ, DOT, FIN, W>), dim3(g + (FIN ? 1 : 0)),                 \
                       dim3(sell_block<W>()), 0, s, A, dinv, rhs, zin, zout, rdot, partials, done, operm, \
                       fin ? *fin : RrFinish())
    if constexpr (std::is_same<T, X>::value) {
        WAVES_SWITCH(A, g = sell_grid<W>(A);
                     if (partials) SWEEP(true, false);
                     else if (fin) SWEEP(false, true);
                     else SWEEP(false, false));
    } else {
        if (partials || fin) throw std::invalid_argument("sell_sweep: reductions of single vectors only");
        WAVES_SWITCH(A, g = sell_grid<W>(A); SWEEP(false, false));
    }
#undef SWEEP
    return g;
}

void sell_spmv64x3(hipStream_t s, const DevSellView &A, const Vec3<double> *x, Vec3<double> *y)
{
    WAVES_SWITCH(A, hipLaunchKernelGGL((k_sell_spmv64x3<W>), dim3(sell_grid<W>(A)), dim3(sell_block<W>()), 0, s, A, x, y));
}

template <typename T>
int sell_resid(hipStream_t s, const DevSellView &A, const T *rhs, const T *z, T *res, const int *done)
{
    int g = 0;
    WAVES_SWITCH(A, g = sell_grid<W>(A); hipLaunchKernelGGL((k_sell_resid<T, W>), dim3(g), dim3(sell_block<W>()), 0, s,
                                                            A, rhs, z, res, done));
    return g;
}

int sell_spmv64(hipStream_t s, const DevSellView &A, const double *x, double *y, double *partials, const int *done,
                const int *operm)
{
    int g = 0;
    WAVES_SWITCH(A, g = sell_grid<W>(A);
                 if (partials) hipLaunchKernelGGL((k_sell_spmv64<true, W>), dim3(g), dim3(sell_block<W>()), 0, s, A, x,
                                                  y, partials, done, operm);
                 else hipLaunchKernelGGL((k_sell_spmv64<false, W>), dim3(g), dim3(sell_block<W>()), 0, s, A, x, y,
                                         partials, done, operm));
    return g;
}

int sell_parts(const DevSellView &A)
{
    int g = 0;
    WAVES_SWITCH(A, g = sell_grid<W>(A));
    return g;
}

int cg_product(hipStream_t s, const DevSellView &A, const double *z, const double *p_old, double *p, double *q,
               const double *rz_parts, int rz_n, double *pq_parts, const CgState &st)
{
    int g = 0;
    WAVES_SWITCH(A, g = sell_grid<W>(A);
                 hipLaunchKernelGGL((k_cg_product<W>), dim3(g), dim3(sell_block<W>()), 0, s, A, z, p_old, p, q, rz_parts,
                                    rz_n, pq_parts, st));
    return g;
}

int sell_residual64(hipStream_t s, const DevSellView &A, const double *f, const double *u, double *r)
{
    int g = 0;
    WAVES_SWITCH(A, g = sell_grid<W>(A); hipLaunchKernelGGL((k_sell_residual64<W>), dim3(g), dim3(sell_block<W>()), 0, s,
                                                            A, f, u, r));
    return g;
}

static int ell_grid(int n, int lanes)
{
    const long long slices = ((long long)n * lanes + 63) / 64;
    return grid_cap((slices + kBlock / 64 - 1) / (kBlock / 64));
}

template <typename T, typename X, int MODE>
void ell_matvec(hipStream_t s, const DevCsrView &M, const X *x1, const X *x2, int split, X *y, const int *done)
{
    LPR_SWITCH(M.ell_lanes, hipLaunchKernelGGL((k_ell_matvec<T, X, L, MODE>), dim3(ell_grid(M.n, L)), dim3(kBlock), 0, s,
                                               M.n, M.ell_off, M.ell_col, (const T *)M.ell_val, x1, x2, split, y,
                                               done));
}

template <typename T, typename X>
void csr_matvec(hipStream_t s, const DevCsrView &M, const X *x, X *y, const int *done)
{
    if (M.ell_lanes > 0) return ell_matvec<T, X, 0>(s, M, x, nullptr, 0, y, done);
    LPR_SWITCH(M.lpr, hipLaunchKernelGGL((k_csr_matvec<T, X, L, false>), dim3(rows_grid(M.n, L)), dim3(kBlock), 0, s,
                                         M.n, M.ptr, M.col, (const T *)M.val, x, y, done));
}

template <typename T, typename X>
void csr_matvec_add(hipStream_t s, const DevCsrView &M, const X *e, X *x, const int *done)
{
    if (M.ell_lanes > 0) return ell_matvec<T, X, 1>(s, M, e, nullptr, 0, x, done);
    LPR_SWITCH(M.lpr, hipLaunchKernelGGL((k_csr_matvec<T, X, L, true>), dim3(rows_grid(M.n, L)), dim3(kBlock), 0, s,
                                         M.n, M.ptr, M.col, (const T *)M.val, e, x, done));
}

template <typename T, typename X>
void csr_matvec2(hipStream_t s, const DevCsrView &M, const X *x1, const X *x2, int split, X *y, const int *done)
{
    if (M.ell_lanes > 0) return ell_matvec<T, X, 2>(s, M, x1, x2, split, y, done);
    LPR_SWITCH(M.lpr, hipLaunchKernelGGL((k_csr_matvec2<T, X, L>), dim3(rows_grid(M.n, L)), dim3(kBlock), 0, s, M.n,
                                         M.ptr, M.col, (const T *)M.val, x1, x2, split, y, done));
}

template <typename T>
void csr_vpre(hipStream_t s, const DevCsrView &A, const T *dinv, const T *b, T *x, T *r, const int *done)
{
    LPR_SWITCH(A.lpr, hipLaunchKernelGGL((k_csr_vpre<T, L>), dim3(rows_grid(A.n, L)), dim3(kBlock), 0, s, A.n, A.ptr,
                                         A.col, (const T *)A.val, dinv, b, x, r, done));
}

template <typename T>
void csr_sweep(hipStream_t s, const DevCsrView &A, const T *dinv, const T *b, const T *x, T *y, const int *done)
{
    LPR_SWITCH(A.lpr, hipLaunchKernelGGL((k_csr_sweep<T, L>), dim3(rows_grid(A.n, L)), dim3(kBlock), 0, s, A.n,
                                         A.ptr, A.col, (const T *)A.val, dinv, b, x, y, done));
}

template <typename T, typename X>
void dense_gemv(hipStream_t s, int n, const T *Ainv, const X *b, X *x, const int *done)
{
    // one workgroup per row
    hipLaunchKernelGGL((k_dense_gemv<T, X>), dim3(grid_cap(n)), dim3(kBlock), 0, s, n, Ainv, b, x, done);
}

int vec_dot(hipStream_t s, int n, const double *a, const double *b, double *partials)
{
    int g = vec_grid(n);
    hipLaunchKernelGGL(k_dot, dim3(g), dim3(kBlock), 0, s, n, a, b, partials);
    return g;
}

void finish(hipStream_t s, const double *partials, int nparts, FinishMode mode, double *out, const CgState &st)
{
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kBlock), 0, s, partials, nparts, (int)mode, out, st);
}

template <typename T>
int cg_update_prep(hipStream_t s, int n, double *x, double *r, const double *p, const double *q, const CgState &st,
                   double *partials, const T *dinv, T *z0, T *rT, const double *pq_parts, int pq_n)
{
    int g = vec_grid(n);
    if (pq_n > 0)
        hipLaunchKernelGGL((k_cg_update_prep<T, true>), dim3(g), dim3(kBlock), 0, s, n, x, r, p, q, st, partials, dinv,
                           z0, rT, pq_parts, pq_n);
    else
        hipLaunchKernelGGL((k_cg_update_prep<T, false>), dim3(g), dim3(kBlock), 0, s, n, x, r, p, q, st, partials, dinv,
                           z0, rT, pq_parts, 0);
    return g;
}
template int cg_update_prep<float>(hipStream_t, int, double *, double *, const double *, const double *,
                                   const CgState &, double *, const float *, float *, float *, const double *, int);
template int cg_update_prep<double>(hipStream_t, int, double *, double *, const double *, const double *,
                                    const CgState &, double *, const double *, double *, double *, const double *,
                                    int);

void cg_direction(hipStream_t s, int n, const double *z, double *p, const CgState &st)
{
    hipLaunchKernelGGL(k_cg_direction, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, z, p, st);
}

template <typename T>
void cg_start(hipStream_t s, const DevSellView &A, const int *perm, const double *f, const double *u, double *fi,
              double *x, double *r, const T *dinv, T *z0, T *rT, double *partials, const CgState &st, double tol2)
{
    hipLaunchKernelGGL(k_gather_pair, dim3(vec_grid(A.n)), dim3(kBlock), 0, s, A.n, perm, f, u, fi, x);
    int g = 0;
    WAVES_SWITCH(A, g = std::min(sell_grid<W>(A), kMaxBlocks / 2);
                 hipLaunchKernelGGL((k_cg_first<T, W>), dim3(g), dim3(sell_block<W>()), 0, s, A, fi, x, r, dinv, z0, rT,
                                    partials));
    hipLaunchKernelGGL(k_cg_init_sums, dim3(1), dim3(kBlock), 0, s, partials, g, st, tol2);
}
template void cg_start<float>(hipStream_t, const DevSellView &, const int *, const double *, const double *, double *,
                              double *, double *, const float *, float *, float *, double *, const CgState &, double);
template void cg_start<double>(hipStream_t, const DevSellView &, const int *, const double *, const double *, double *,
                               double *, double *, const double *, double *, double *, double *, const CgState &,
                               double);

void vec_interleave3(hipStream_t s, int n, const int *idx, const double *x, Vec3<double> *y)
{
    hipLaunchKernelGGL(k_interleave3, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, idx, x, y);
}

void vec_split3(hipStream_t s, int n, const int *idx, const Vec3<double> *x, double *y)
{
    hipLaunchKernelGGL(k_split3, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, idx, x, y);
}

void vec_gather(hipStream_t s, int n, const int *idx, const double *x, double *y)
{
    hipLaunchKernelGGL(k_gather, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, idx, x, y);
}

void vec_scatter(hipStream_t s, int n, const int *idx, const double *x, double *y)
{
    hipLaunchKernelGGL(k_scatter, dim3(vec_grid(n)), dim3(kBlock), 0, s, n, idx, x, y);
}

void kappa_grad(hipStream_t s, int nt, int nloc, const int *dofs, const double *G6, const double *kappa,
                const double *S, const double *u, const double *lam, double *g)
{
    const int grid = (nt + 63) / 64;
    if (grid == 0) return;
#define GRAD(N, W)                                                                                              \
    hipLaunchKernelGGL((k_kappa_grad<N, W>), dim3(grid), dim3(64 * W), 0, s, nt, dofs, G6, kappa, S, u, lam, g)
    switch (nloc) {
    case 10: GRAD(10, 4); break;
    case 20: GRAD(20, 8); break;
    case 35: GRAD(35, 8); break;
    default: throw std::invalid_argument("kappa gradient: nodes per tet must be 10, 20 or 35");
    }
#undef GRAD
}

#define INST(T)                                                                                              \
    template void vec_jacobi0_t<T>(hipStream_t, int, const T *, const T *, T *, const int *);               \
    template int sell_resid<T>(hipStream_t, const DevSellView &, const T *, const T *, T *, const int *);    \
    template void vec_gather_jacobi0<T>(hipStream_t, int, const int *, const T *, const double *, double *, T *, \
                                        T *);                                                                \
    template void csr_vpre<T>(hipStream_t, const DevCsrView &, const T *, const T *, T *, T *, const int *); \
    template void csr_sweep<T>(hipStream_t, const DevCsrView &, const T *, const T *, const T *, T *,        \
                               const int *);
INST(double)
INST(float)
#define INSTX(T, X, XR)                                                                                        \
    template int vec_jacobi0<T, X, XR>(hipStream_t, int, const T *, const XR *, X *, X *, const int *);        \
    template int sell_sweep<T, X, X, X>(hipStream_t, const DevSellView &, const T *, const X *, const X *, X *, \
                                        const double *, double *, const int *, const int *, const RrFinish *); \
    template void csr_matvec<T, X>(hipStream_t, const DevCsrView &, const X *, X *, const int *);              \
    template void csr_matvec_add<T, X>(hipStream_t, const DevCsrView &, const X *, X *, const int *);          \
    template void csr_matvec2<T, X>(hipStream_t, const DevCsrView &, const X *, const X *, int, X *, const int *); \
    template void dense_gemv<T, X>(hipStream_t, int, const T *, const X *, X *, const int *);
INSTX(double, double, double)
INSTX(float, float, double)
INSTX(double, Vec3<double>, Vec3<double>)
INSTX(float, Vec3<float>, Vec3<double>)
#define INSTM(X, XZ)                                                                                            \
    template int sell_sweep<float, X, XZ, XZ>(hipStream_t, const DevSellView &, const float *, const XZ *,      \
                                              const X *, XZ *, const double *, double *, const int *,           \
                                              const int *, const RrFinish *);
INSTM(float, double)
INSTM(Vec3<float>, Vec3<double>)

}  // namespace auxp
