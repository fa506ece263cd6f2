// Matrix-free P^k element operator on the matrix cores (gfx950 MFMA).
//
// A_h x = sum_e P_e^T K_e P_e x with K_e = kappa_e sum_pq G^e_pq M^pq.  Since
// the barycentric gradients sum to zero, G^e has zero row sums and
//     K_e = sum_{p<q} w_e,pq S^pq,   w_e,pq = -kappa_e G^e_pq,
//     S^pq = M^pp + M^qq - M^pq - M^qp,
// six reference matrices shared by every tet.  For a tile of 16 tets the
// products of all six with the gathered element vectors form one dense
// contraction Y[a][t] = sum_{(k,b)} S[a][(k,b)] Z[(k,b)][t] with
// Z[(k,b)][t] = w_t,k x_t,b: an [nloc x 6 nloc] by [6 nloc x 16] product,
// evaluated with v_mfma_*_16x16x4 (A operand = the reference tables, staged
// once per workgroup in LDS in operand lane order and read back per step;
// B operand = Z formed in registers from the lane's gathered values and its
// tet's weights).
//
// A workgroup takes a patch of neighbouring tets: it reads the patch's values
// of x once into LDS, its wavefronts multiply tile by tile and put the element
// results into LDS, ordered by dof, and the sums of dofs whose tets are all in
// the patch are final: smoother, residual or product are written from there.
// Only dofs shared with other patches go through memory, one partial sum per
// patch, added in a fixed order by a second kernel -- no atomics, so the
// result is deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.hpp"
#include "mfree.hpp"

namespace auxp {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Operand layouts (16x16x4, both types): lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16].  Result register v of lane l holds D[row][l % 16] with
// row = 4 (l / 16) + v for FP32 and row = (l / 16) + 4 v for FP64.
// The last rows go through the four-row forms with the same B operand: FP64
// 4x4x4 (four blocks, A[l % 4][l / 16], D[l / 16][l % 16]); FP32 4x4x1 (sixteen
// blocks: A[l % 4] of lane group l / 16 and B as above, so the registers hold
// four partial sums over k, one per lane group, of rows v).
template <typename T>
struct Acc;
template <>
struct Acc<float> {
    using V = f32x4;
    using V4 = f32x4;
    static __device__ __forceinline__ V mfma(float a, float b, V c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ V4 mfma4(float a, float b, V4 c)
    {
        return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
    }
    // row grp of the four: the lane groups' partial sums added
    static __device__ __forceinline__ float result4(const V4 &c, int grp)
    {
        const bool hi = grp & 2, odd = grp & 1;
        const float k0 = (hi ? c[2] : c[0]) + __shfl_xor(hi ? c[0] : c[2], 32, 64);
        const float k1 = (hi ? c[3] : c[1]) + __shfl_xor(hi ? c[1] : c[3], 32, 64);
        return (odd ? k1 : k0) + __shfl_xor(odd ? k0 : k1, 16, 64);
    }
    static __host__ __device__ __forceinline__ int row(int grp, int v) { return 4 * grp + v; }
};
template <>
struct Acc<double> {
    using V = f64x4;
    using V4 = double;
    static __device__ __forceinline__ V mfma(double a, double b, V c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ V4 mfma4(double a, double b, V4 c)
    {
        return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ double result4(const V4 &c, int) { return c; }
    static __host__ __device__ __forceinline__ int row(int grp, int v) { return grp + 4 * v; }
};

__device__ __forceinline__ bool stop(const int *done) { return done != nullptr && *done != 0; }

constexpr int kDies = 8;

// 16-row tiles, and a four-row one if that holds the remaining nodes (P3, P4)
constexpr int tiles4(int nloc) { return nloc % 16 > 0 && nloc % 16 <= 4; }
constexpr int tiles16(int nloc) { return (nloc + 15) / 16 - tiles4(nloc); }
constexpr int table_size(int nloc) { return 6 * ((nloc + 3) / 4) * (64 * tiles16(nloc) + 16 * tiles4(nloc)); }

// MF_RESID: out = rhs - Ax;  MF_SWEEP: out = x + dinv (rhs - Ax);  MF_PRODUCT: out = Ax
enum { MF_RESID = 0, MF_SWEEP = 1, MF_PRODUCT = 2 };

template <typename T, typename TR, int MODE>
__device__ __forceinline__ T mf_result(T s, T x, T d, TR b)
{
    if constexpr (MODE == MF_RESID) return (T)b - s;
    else if constexpr (MODE == MF_SWEEP) return x + d * ((T)b - s);
    else return s;
}

template <int BS>
__device__ __forceinline__ void mf_partial(double acc, double *partials)
{
    __shared__ double red[BS / 64];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double b = 0.0;
        for (int w = 0; w < BS / 64; w++) b += red[w];
        *partials = b;
    }
}

// A patch's complete dofs, and its partial sums of the shared ones.
//
// Contraction order: the 6 nloc terms (k, b) are split into steps of four,
// step s covering k = s / NB and b = 4 (s % NB) + g for the four lane groups
// g = lane / 16 (NB = ceil(nloc / 4); b >= nloc is padding).  So lane (g, c)
// of a wave needs only the six weights of its tet c and its NB values b = g,
// g+4, ..., held in registers, from which it forms its B operand per step; the
// A operand (the reference tables) comes from LDS.  The tables' rows are
// ordered so that the lane's results are those same nodes' (result v of tile m
// is node 16 m + 4 v + g), and one word per node, read by the wave as one
// contiguous load, gives its place in the patch's x and among its results.
//
// What bounds it (P3, 196 608 tets, FP32 sweep: 23.4 us and 6.3 for the shared
// dofs; 26 and 9.4 with every element result through memory): 62 MB (85
// before), 13 us at the rate of a large copy; 6 us of matrix-core time (9.6 if
// the last 4 of the 20 rows took a 16-row tile); and the chain of a patch --
// list, values, products, sums, each behind a barrier -- which the four to nine
// workgroups of a compute unit hide only in part.  The FP64 product takes 32.2
// and 7.2 us (37 and 13.5 before), 12 us of them on the matrix cores.
// Requesting the sums' inputs before the products took 40 registers more and
// was slower (P2 48^3 solve 5.47 -> 5.64 ms).
template <typename T, typename TR, typename TZ, int NLOC, int BS, int MODE, bool DOT>
__global__ __launch_bounds__(BS) void k_mf_patch(MfView<T> op, const T *__restrict__ X, const T *__restrict__ dinv,
                                                 const TR *__restrict__ rhs, TZ *__restrict__ out, double *partials,
                                                 const int *done)
{
    if (stop(done)) return;
    constexpr int NB = (NLOC + 3) / 4;           // values per lane
    constexpr int KS = 6 * NB;                   // MFMA steps
    constexpr int MT = tiles16(NLOC), M4 = tiles4(NLOC);   // output tiles of 16 and of 4 rows
    constexpr int TBL = table_size(NLOC), PV = 16 / sizeof(T);
    extern __shared__ __align__(16) unsigned char lds_[];
    T *sA = (T *)lds_, *ys = sA + TBL, *xs = ys + op.tp * NLOC;
    const T *s4 = sA + MT * KS * 64 + (threadIdx.x >> 4 & 3) * 4 + (threadIdx.x & 3);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    typedef T tv __attribute__((ext_vector_type(PV)));
    for (int i = threadIdx.x; i < TBL / PV; i += BS) ((tv *)sA)[i] = ((const tv *)op.S)[i];

    // Each die (workgroups are dispatched round-robin over kDies dies, b to
    // b % kDies) takes a contiguous range of patches, so what neighbouring
    // patches share meets in one L2.  Any grid visits every patch exactly
    // once; placement affects only speed.
    int p = blockIdx.x, p_end = op.npatch, p_step = gridDim.x;
    if (p_step >= kDies) {
        const int d = p % kDies, per = (op.npatch + kDies - 1) / kDies;
        p_step = (p_step - d + kDies - 1) / kDies;
        p = d * per + p / kDies;
        p_end = min(op.npatch, (d + 1) * per);
    }
    constexpr int U = 4;
    const int tiles = op.tp / 16;
    double acc_dot = 0.0;
    for (; p < p_end; p += p_step) {
        const int4 m = op.meta[p];
        unsigned nw[NB];
        T nv[6];
        auto request = [&](int tile) {
            const size_t t = (size_t)p * tiles + tile;
#pragma unroll
            for (int j = 0; j < NB; j++) nw[j] = op.word[(t * NB + j) * 64 + lane];
#pragma unroll
            for (int k = 0; k < 6; k++) nv[k] = op.w[(t * 16 + (lane & 15)) * 6 + k];
        };
        if (w < tiles) request(w);
        __syncthreads();                         // the previous patch is done with xs and ys
        const unsigned *__restrict__ range = op.range + m.x;
        for (int i0 = threadIdx.x; i0 < m.y; i0 += U * BS) {
            int id[U];
            T x[U];
#pragma unroll
            for (int u = 0; u < U; u++) id[u] = op.dof[m.x + min(i0 + u * BS, m.y - 1)];
#pragma unroll
            for (int u = 0; u < U; u++) x[u] = X[id[u]];
#pragma unroll
            for (int u = 0; u < U; u++) xs[min(i0 + u * BS, m.y - 1)] = x[u];
        }
        if (threadIdx.x == 0) xs[m.y] = T(0);
        __syncthreads();
        for (int tile = w; tile < tiles; tile += BS / 64) {
            unsigned word[NB];
            T wv[6], xv[NB];
#pragma unroll
            for (int j = 0; j < NB; j++) word[j] = nw[j], xv[j] = xs[nw[j] & 0xffff];
#pragma unroll
            for (int k = 0; k < 6; k++) wv[k] = nv[k];
            if (tile + BS / 64 < tiles) request(tile + BS / 64);
            // B operand: lane (g, c) holds Z[(k, b)][c] = w_c,k x_c,b, formed step by step
            typename Acc<T>::V acc[MT];
            typename Acc<T>::V4 acc4[M4 > 0 ? M4 : 1];
#pragma unroll
            for (int i = 0; i < MT; i++) acc[i] = typename Acc<T>::V{0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < M4; i++) acc4[i] = typename Acc<T>::V4{};
#pragma unroll
            for (int s = 0; s < KS; s++) {
                const T bv = wv[s / NB] * xv[s % NB];
#pragma unroll
                for (int i = 0; i < MT; i++) acc[i] = Acc<T>::mfma(sA[(i * KS + s) * 64 + lane], bv, acc[i]);
#pragma unroll
                for (int i = 0; i < M4; i++) acc4[i] = Acc<T>::mfma4(s4[(i * KS + s) * 16], bv, acc4[i]);
            }
#pragma unroll
            for (int j = 0; j < NB; j++) {
                T y;
                if (j < 4 * MT) y = acc[j / 4 < MT ? j / 4 : 0][j % 4];
                else y = Acc<T>::result4(acc4[0], lane >> 4);
                if (word[j] < 0xffff0000u) ys[word[j] >> 16] = y;
            }
        }
        __syncthreads();
        // d: the dof, or the place of its partial sum
        auto finish = [&](int i, int d, unsigned r, TR rb, T rd) {
            const int b0 = r & 0xffff, b1 = r >> 16;
            // four results at a time (past the end into the words behind, unused)
            T s = T(0);
            for (int q = b0; q < b1; q += 4) {
                const T y0 = ys[q], y1 = ys[q + 1], y2 = ys[q + 2], y3 = ys[q + 3];
                s += y0;
                s += q + 1 < b1 ? y1 : T(0);
                s += q + 2 < b1 ? y2 : T(0);
                s += q + 3 < b1 ? y3 : T(0);
            }
            if (i < m.z) {
                const T xi = MODE == MF_SWEEP || DOT ? xs[i] : T(0);
                const TZ z = (TZ)mf_result<T, TR, MODE>(s, xi, rd, rb);
                out[d] = z;
                if (DOT) acc_dot += (MODE == MF_PRODUCT ? (double)xi : (double)rb) * (double)z;
            } else {
                op.part[d] = s;
            }
        };
        for (int i = threadIdx.x; i < m.y; i += BS) {
            const int d = i < m.z ? op.dof[m.x + i] : op.pos[m.w + i - m.z];
            TR rb{};
            T rd{};
            if (MODE != MF_PRODUCT && i < m.z) rb = rhs[d];
            if (MODE == MF_SWEEP && i < m.z) rd = dinv[d];
            finish(i, d, range[i], rb, rd);
        }
    }
    if (DOT) mf_partial<BS>(acc_dot, partials + blockIdx.x);
}

// the shared dofs: their partial sums, and the same results
template <typename T, typename TR, typename TZ, int MODE, bool DOT>
__global__ __launch_bounds__(kBlock) void k_mf_shared(MfView<T> op, const T *__restrict__ X, const T *__restrict__ dinv,
                                                      const TR *__restrict__ rhs, TZ *__restrict__ out,
                                                      double *partials, const int *done)
{
    if (stop(done)) return;
    double acc = 0.0;
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < op.nshared; i += gridDim.x * kBlock) {
        const int q0 = op.sh_ptr[i], q1 = op.sh_ptr[i + 1], d = op.sh_dof[i];
        TR b{};
        T dv{}, x{};
        if (MODE != MF_PRODUCT) b = rhs[d];
        if (MODE == MF_SWEEP) dv = dinv[d];
        if (MODE == MF_SWEEP || DOT) x = X[d];
        T s = T(0);
        for (int q = q0; q < q1; q++) s += op.part[q];
        const TZ z = (TZ)mf_result<T, TR, MODE>(s, x, dv, b);
        out[d] = z;
        if (DOT) acc += (MODE == MF_PRODUCT ? (double)x : (double)b) * (double)z;
    }
    if (DOT) mf_partial<kBlock>(acc, partials + blockIdx.x);
}

template <typename T, typename TR, typename TZ, int NLOC, int MODE, bool DOT>
int mf_launch(hipStream_t s, const MfView<T> &op, const T *x, const T *dinv, const TR *rhs, TZ *out, double *partials,
              const int *done)
{
    // P4's tables (31 and 62 KB) leave room for few workgroups: eight wavefronts
    // each instead of four (P4 24^3 solve, FP32 / FP64: 12.0 / 18.6 -> 10.5 / 14.0 ms)
    constexpr int BS = NLOC > 20 ? 512 : kBlock;
    const size_t lds = mf_lds(NLOC, op.tp, op.max_dofs, sizeof(T));
    // one patch per workgroup as far as the partial sums' places go
    const int g = std::max(1, std::min(op.npatch, kMaxBlocks / 4 * 3));
    const int h = std::max(1, std::min((op.nshared + kBlock - 1) / kBlock, kMaxBlocks / 4));
    hipLaunchKernelGGL((k_mf_patch<T, TR, TZ, NLOC, BS, MODE, DOT>), dim3(g), dim3(BS), lds, s, op, x, dinv, rhs, out,
                       partials, done);
    hipLaunchKernelGGL((k_mf_shared<T, TR, TZ, MODE, DOT>), dim3(h), dim3(kBlock), 0, s, op, x, dinv, rhs, out,
                       DOT ? partials + g : nullptr, done);
    return g + h;
}

template <typename T, typename TR, typename TZ, int MODE, bool DOT>
int mf_run(hipStream_t s, const MfView<T> &op, const T *x, const T *dinv, const TR *rhs, TZ *out, double *partials,
           const int *done)
{
    if (op.nloc == 10) return mf_launch<T, TR, TZ, 10, MODE, DOT>(s, op, x, dinv, rhs, out, partials, done);
    if (op.nloc == 20) return mf_launch<T, TR, TZ, 20, MODE, DOT>(s, op, x, dinv, rhs, out, partials, done);
    return mf_launch<T, TR, TZ, 35, MODE, DOT>(s, op, x, dinv, rhs, out, partials, done);
}

}  // namespace

size_t mf_table_size(int nloc) { return (size_t)table_size(nloc); }

size_t mf_lds(int nloc, int tp, int max_dofs, size_t size)
{
    return ((size_t)table_size(nloc) + (size_t)tp * nloc + std::max(max_dofs + 1, 4)) * size;
}

template <typename T>
void mf_tables(int nloc, const double *S, T *out)
{
    const int nb = (nloc + 3) / 4, ks = 6 * nb, mt = tiles16(nloc);
    auto entry = [&](int a, int s, int g) {
        const int b = 4 * (s % nb) + g;
        return a < nloc && b < nloc ? (T)S[((size_t)6 * a + s / nb) * nloc + b] : T(0);
    };
    for (int i = 0; i < mt; i++)
        for (int s = 0; s < ks; s++)
            for (int g = 0; g < 4; g++)
                // result v of group r is row Acc<T>::row(r, v): node 4 v + r of the tile
                for (int r = 0; r < 4; r++)
                    for (int v = 0; v < 4; v++)
                        out[(i * ks + s) * 64 + 16 * g + Acc<T>::row(r, v)] = entry(16 * i + 4 * v + r, s, g);
    T *o4 = out + (size_t)mt * ks * 64;
    for (int i = 0; i < tiles4(nloc); i++)
        for (int s = 0; s < ks; s++)
            for (int g = 0; g < 4; g++)
                for (int r = 0; r < 4; r++) o4[(i * ks + s) * 16 + 4 * g + r] = entry(16 * mt + 4 * i + r, s, g);
}

template <typename T>
void mf_resid(hipStream_t s, const MfView<T> &op, const T *x, const T *rhs, T *res, const int *done)
{
    mf_run<T, T, T, MF_RESID, false>(s, op, x, nullptr, rhs, res, nullptr, done);
}

int mf_product(hipStream_t s, const MfView<double> &op, const double *x, double *out, double *partials, const int *done)
{
    if (partials)
        return mf_run<double, double, double, MF_PRODUCT, true>(s, op, x, nullptr, nullptr, out, partials, done);
    return mf_run<double, double, double, MF_PRODUCT, false>(s, op, x, nullptr, nullptr, out, nullptr, done);
}

template <typename T, typename TR, typename TZ>
int mf_sweep(hipStream_t s, const MfView<T> &op, const T *x, const T *dinv, const TR *rhs, TZ *out, double *partials,
             const int *done)
{
    if (partials) return mf_run<T, TR, TZ, MF_SWEEP, true>(s, op, x, dinv, rhs, out, partials, done);
    return mf_run<T, TR, TZ, MF_SWEEP, false>(s, op, x, dinv, rhs, out, nullptr, done);
}

#define MFINST(T)                                                                                    \
    template void mf_tables<T>(int, const double *, T *);                                            \
    template void mf_resid<T>(hipStream_t, const MfView<T> &, const T *, const T *, T *, const int *); \
    template int mf_sweep<T, T, T>(hipStream_t, const MfView<T> &, const T *, const T *, const T *, T *, double *, \
                                   const int *);

MFINST(float)
MFINST(double)
template int mf_sweep<float, double, double>(hipStream_t, const MfView<float> &, const float *, const float *,
                                             const double *, double *, double *, const int *);

}  // namespace auxp
