// Batched solve phase: NR right-hand sides in lock-step.
//
// Block vectors are row-major [n][NR] (NR in {8, 16, 32, 64}); a row of a
// sparse operator is handled by NR consecutive lanes, one per right-hand
// side, so each matrix entry is read once per row and applied to all
// columns (sparse matrix times dense block).  The gathered rows of the block
// are NR contiguous words.  Every column follows the single right-hand-side
// CG exactly: its own alpha, beta and stopping test; converged columns are
// frozen while the others continue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "batched.hpp"

namespace auxp {

namespace {

__device__ __forceinline__ bool stop_all(const int *all_done) { return all_done != nullptr && *all_done != 0; }

inline int grid_cap(long long need)
{
    if (need < 1) need = 1;
    if (need > kMaxBlocks) need = kMaxBlocks;
    return (int)need;
}

// rows handled by a block: kBlock / NR
#define FOR_BROWS(NR, nrows)                                                                                 \
    const int c_ = threadIdx.x % (NR);                                                                       \
    for (int row = blockIdx.x * (kBlock / (NR)) + (int)threadIdx.x / (NR); row < (nrows);                    \
         row += gridDim.x * (kBlock / (NR)))

inline int brows_grid(int n, int NR) { return grid_cap(((long long)n * NR + kBlock - 1) / kBlock); }
// Workgroups of the vector passes that end in per-column sums: as many as are
// resident (8 per compute unit).  Their partials are summed by one workgroup,
// which reads 512 KB at 32 columns; from 4096 workgroups it took 18 us.
constexpr int kBatchParts = 2048;
inline int bsum_grid(int n, int NR) { return std::min(brows_grid(n, NR), kBatchParts); }

// Sums per column over a block of BS threads (thread t holds column t % NR):
// within the wavefronts by shuffles, then over the wavefronts in a fixed order.
// The result is valid in threads below NR.  (Summed from LDS by NR threads, the
// one-workgroup finish was 7.9 us at 8 columns, a chain of 128 reads.)
template <int NR, int BS>
__device__ __forceinline__ double col_sums(double v)
{
    __shared__ double red[BS / 64][NR];
#pragma unroll
    for (int off = 32; off >= NR; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63;
    if (lane < NR) red[threadIdx.x >> 6][lane] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x < NR)
#pragma unroll
        for (int w = 0; w < BS / 64; w++) s += red[w][threadIdx.x];
    return s;
}

// per-column partial sums of a block of BS threads: partials[blockIdx.x * NR + c]
template <int NR, int BS = kBlock>
__device__ void write_col_partials(double *partials, double v)
{
    const double s = col_sums<NR, BS>(v);
    if (threadIdx.x < NR) partials[(size_t)blockIdx.x * NR + threadIdx.x] = s;
}

// ------------------------------------------------------------------ SELL

// One block per 64-row slice.  The slice's values and decoded columns are
// staged in LDS in chunks of kChunk slots (coalesced, once per block), then
// every (row, column) pair of the slice is accumulated by the lane that owns
// it: kBlock / NR rows per pass, kSlice / (kBlock / NR) passes.  Blocks never
// share a slice, so no two XCDs fetch the same matrix lines.
constexpr int kChunk = 32;

// Element idx of a block vector addressed by a 32-bit byte offset from the
// (uniform) base: the load takes the scalar-base form, one address register
// per gather instead of two.  The caller guarantees blocks below 4 GiB.
template <typename T>
__device__ __forceinline__ T gather32(const T *__restrict__ base, unsigned idx)
{
    return *(const T *)((const char *)base + idx * (unsigned)sizeof(T));
}


// U: slots unrolled in the accumulation (more gathers in flight per lane;
// 4 for A_h and for level operators with long rows or few slices, 1 for the
// large prolongations)
template <typename T, int NR, int U, typename XL, typename BODY>
__device__ __forceinline__ void bsell_slices(const DevSellView &A, XL xload, BODY body)
{
    constexpr int RP = kBlock / NR, NP = kSlice / RP;
    __shared__ T vs[kChunk * kSlice];
    __shared__ int cs[kChunk * kSlice];
    const T *__restrict__ val = (const T *)A.val;
    const int c = threadIdx.x % NR, rl0 = threadIdx.x / NR;
    // Slices go round-robin over the workgroups (and so over the dies), or,
    // with die ranges (A_h in the spatially ordered batched layout), die d =
    // b % 8 walks its own contiguous range so its gathers stay in one region
    // (for operators in the length-sorted single-vector order, contiguous die
    // shares measured slower: the sweeps by 9%, I_P by 38%)
    int sl = blockIdx.x, sl_end = A.nslices, sl_step = gridDim.x;
    if (A.die_off) {
        const int d = blockIdx.x % 8;
        sl = A.die_off[d] + (int)blockIdx.x / 8;
        sl_end = A.die_off[d + 1];
        sl_step = ((int)gridDim.x - d + 7) / 8;
    }
    for (; sl < sl_end; sl += sl_step) {
        const int4 m = A.meta[sl];
        const int width = m.w;
        T acc[NP];
#pragma unroll
        for (int p = 0; p < NP; p++) acc[p] = T(0);
        for (int j0 = 0; j0 < width; j0 += kChunk) {
            const int jn = min(kChunk, width - j0);
            // four consecutive entries of a row per load; every load of the
            // chunk is issued before any is waited on (groups clamped into
            // the slice, stores predicated)
            constexpr int PER = kChunk / 4 * kSlice / kBlock, GW = kBlock / kSlice;
            const int gn = (jn + 3) / 4, lane = threadIdx.x % kSlice, g0 = threadIdx.x / kSlice;
            T vt[PER][4];
            int ct[PER][4];
#pragma unroll
            for (int i = 0; i < PER; i++) {
                const int g = j0 / 4 + min(g0 + i * GW, gn - 1);
                const size_t at = ((size_t)m.x + g) * (4 * kSlice) + 4 * lane;
#pragma unroll
                for (int k = 0; k < 4; k++) vt[i][k] = val[at + k];
                if (m.z < 0) {
                    const ushort4 o = *(const ushort4 *)(A.off + at);
                    const int2 *__restrict__ bs = A.base + ((size_t)m.x + g) * 4;
                    ct[i][0] = (o.x & 0x8000 ? bs[0].y : bs[0].x) + (o.x & 0x7fff);
                    ct[i][1] = (o.y & 0x8000 ? bs[1].y : bs[1].x) + (o.y & 0x7fff);
                    ct[i][2] = (o.z & 0x8000 ? bs[2].y : bs[2].x) + (o.z & 0x7fff);
                    ct[i][3] = (o.w & 0x8000 ? bs[3].y : bs[3].x) + (o.w & 0x7fff);
                } else {
                    const int4 cc = *(const int4 *)(A.wide + ((size_t)m.z + g) * (4 * kSlice) + 4 * lane);
                    ct[i][0] = cc.x, ct[i][1] = cc.y, ct[i][2] = cc.z, ct[i][3] = cc.w;
                }
            }
            __syncthreads();                           // the previous chunk is consumed
#pragma unroll
            for (int i = 0; i < PER; i++) {
                const int g = g0 + i * GW;
                if (g < gn)
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        vs[(4 * g + k) * kSlice + lane] = vt[i][k];
                        cs[(4 * g + k) * kSlice + lane] = ct[i][k];
                    }
            }
            __syncthreads();
            // the NP rows of a lane are independent: their gathers (for U
            // slots) are in flight together
#pragma unroll U
            for (int jj = 0; jj < jn; jj++) {
                T xv[NP], vv[NP];
#pragma unroll
                for (int p = 0; p < NP; p++) {
                    const int k = jj * kSlice + p * RP + rl0;
                    vv[p] = vs[k];
                    xv[p] = xload(cs[k], c);
                }
#pragma unroll
                for (int p = 0; p < NP; p++) acc[p] += vv[p] * xv[p];
            }
        }
#pragma unroll
        for (int p = 0; p < NP; p++) {
            const int row = sl * kSlice + p * RP + rl0;
            if (row < A.n) body(row, c, acc[p]);
        }
    }
}

// with die ranges every die needs a workgroup: at least 8
inline int bsell_grid(const DevSellView &A) { return A.die_off ? std::max(8, grid_cap(A.nslices)) : grid_cap(A.nslices); }

template <typename T, int NR>
__global__ __launch_bounds__(kBlock) void kb_jacobi0(int n, const T *__restrict__ dinv, const double *__restrict__ R,
                                                     T *__restrict__ Z, T *__restrict__ RT, const int *all_done)
{
    if (stop_all(all_done)) return;
    FOR_BROWS(NR, n)
    {
        size_t o = (size_t)row * NR + c_;
        T ri = (T)R[o];
        Z[o] = dinv[row] * ri;
        if (RT) RT[o] = ri;
    }
}

template <typename T, typename TR, typename TZ, int NR, bool DOT>
__global__ __launch_bounds__(kBlock) void kb_sweep(DevSellView A, const T *__restrict__ dinv,
                                                   const TR *__restrict__ RHS, const T *__restrict__ Zin,
                                                   TZ *__restrict__ Zout, const double *__restrict__ Rdot,
                                                   double *partials, const int *all_done)
{
    if (stop_all(all_done)) return;
    double acc = 0.0;
    bsell_slices<T, NR, 4>(A, [&](int j, int c) { return gather32(Zin, (unsigned)j * NR + c); }, [&](int row, int c, T s) {
        size_t o = (size_t)row * NR + c;
        T zi = Zin[o] + dinv[row] * ((T)RHS[o] - s);
        Zout[o] = (TZ)zi;
        if (DOT) acc += Rdot[o] * (double)(TZ)zi;
    });
    if (DOT) write_col_partials<NR>(partials, acc);
}

template <typename T, int NR>
__global__ __launch_bounds__(kBlock) void kb_resid(DevSellView A, const T *__restrict__ RHS, const T *__restrict__ Z,
                                                   T *__restrict__ Res, const int *all_done)
{
    if (stop_all(all_done)) return;
    bsell_slices<T, NR, 4>(A, [&](int j, int c) { return gather32(Z, (unsigned)j * NR + c); }, [&](int row, int c, T s) {
        size_t o = (size_t)row * NR + c;
        Res[o] = RHS[o] - s;
    });
}

template <int NR, bool DOT, bool RESID>
__global__ __launch_bounds__(kBlock) void kb_spmv64(DevSellView A, const double *__restrict__ X,
                                                    double *__restrict__ Y, const double *__restrict__ F,
                                                    double *partials, const int *all_done)
{
    if (stop_all(all_done)) return;
    double acc = 0.0;
    bsell_slices<double, NR, 4>(A, [&](int j, int c) { return gather32(X, (unsigned)j * NR + c); }, [&](int row, int c, double s) {
        size_t o = (size_t)row * NR + c;
        if (RESID) {
            Y[o] = F[o] - s;
        } else {
            Y[o] = s;
            if (DOT) acc += X[o] * s;
        }
    });
    if (DOT) write_col_partials<NR>(partials, acc);
}

// ------------------------------------------------------------------ tiles
// One workgroup per tile of rows along a space-filling curve.  Gathering a
// block row through L1 for every entry moves nnz * NR words per product (14.7
// GB in FP64 at P2 64^3 with 32 columns, for 1.7 GB of data); a tile of 64
// rows has about 270 distinct columns for 1800 entries (P2), so its block
// rows are staged in LDS once, in pieces of 128 bytes per row, and the
// entries read them there: LDS delivers 128 bytes per cycle and compute unit,
// one entry's piece.  Eight lanes take a row (16 bytes each; four lanes for
// pieces of at most 64 bytes, but in tiles of 32 rows, whose groups are then
// one per wavefront), a group of eight rows is one or half a
// wavefront, and a quad loads eight entries of its row at once (two a lane)
// and broadcasts them by DPP, so values and positions need no LDS.  Rows are
// sorted by length within a tile and the wavefronts take its groups in a
// zigzag, which evens their work.  Each die walks its own contiguous range of
// tiles: neighbouring tiles share most of their block rows in its L2.
// Measured at P2 64^3 with 32 columns (slices): FP32 sweep 350 us (635), FP64
// product 720 us (1230), 1.4 and 2.7 GB that cannot be left out, so 4.0 and
// 3.8 TB/s; the rest is the tiles' shared columns (each is read by four tiles
// on average) and the turn from one tile to the next.

template <typename T, int NR, int TS>
struct TileShape {
    static constexpr int RB = NR * (int)sizeof(T);            // bytes of a block row
    static constexpr int CB = RB < 128 ? RB : 128;            // staged at a time
    static constexpr int NCH = RB / CB;
    static constexpr int LPR = CB >= 128 || TS == 32 ? 8 : 4; // lanes per row
    static constexpr int VL = CB / LPR / (int)sizeof(T);      // columns per lane
    static constexpr int GP = 8 / LPR;                        // groups a wavefront takes at once
    // columns whose block rows are requested together (all of a tile up to 64 rows)
    static constexpr int COLS = TS == 32 ? 160 : 320;
};

template <int Q>
__device__ __forceinline__ int quad_get(int v)                // lane Q of the quad
{
    return __builtin_amdgcn_mov_dpp(v, Q * 0x55, 0xf, 0xf, true);
}
template <int Q>
__device__ __forceinline__ float quad_get(float v)
{
    return __int_as_float(quad_get<Q>(__float_as_int(v)));
}
template <int Q>
__device__ __forceinline__ double quad_get(double v)
{
    return __hiloint2double(quad_get<Q>(__double2hiint(v)), quad_get<Q>(__double2loint(v)));
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// VL values of a lane
template <typename T, int VL>
struct alignas(sizeof(T) * VL) Piece {
    T v[VL];
};

template <typename T, int VL, int Q>
__device__ __forceinline__ void quad_step(const T (&val)[2], const int (&at)[2], const unsigned char *xs, T (&acc)[VL])
{
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const T v = quad_get<Q>(val[k]);
        const Piece<T, VL> x = *(const Piece<T, VL> *)(xs + quad_get<Q>(at[k]));
#pragma unroll
        for (int c = 0; c < VL; c++) acc[c] += v * x.v[c];
    }
}


// epi(row, first column, chunk, sums, in) for every row and column piece of
// A X, with in = pre(row, first column) the piece's other inputs.  A tile is a
// chain of dependent loads (its column list, the block rows, then the row's
// own words), and few workgroups fit beside each other, so everything that
// can be is requested ahead: the next tile's column list while this one is
// computed; group offsets, rows, the first entries and the rows' other inputs
// before the block rows are waited for; AH blocks of values and positions
// while the AH before them are used.
template <typename T, int NR, int TS, int AH, typename PRE, typename EPI>
__device__ __forceinline__ void btile_rows(const DevTilesView &A, const T *__restrict__ X, PRE pre, EPI epi)
{
    using S = TileShape<T, NR, TS>;
    constexpr int VL = S::VL, SL = S::CB / 16, RS = kBlock / SL;     // staging: lanes per row, rows per step
    constexpr int U = (S::COLS + RS - 1) / RS;                       // rows in flight per thread
    constexpr int groups = TS / 8, P = groups / (4 * S::GP);         // passes of a wavefront
    extern __shared__ __align__(16) unsigned char lds_[];
    const T *__restrict__ val = (const T *)A.val;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int l = lane % S::LPR, r = (lane / S::LPR) % 8, half = lane / (8 * S::LPR), q = lane & 3;
    const int sl = threadIdx.x % SL, su = threadIdx.x / SL;
    // die d = b % 8 takes tiles [d per, (d + 1) per) (fewer workgroups than dies: all tiles)
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    int t = b, t_end = A.ntiles, t_step = nb;
    if (nb >= 8) {
        const int d = b % 8, per = (A.ntiles + 7) / 8;
        t = d * per + b / 8;
        t_end = min(A.ntiles, (d + 1) * per);
        t_step = (nb - d + 7) / 8;
    }
    if (t >= t_end) return;
    // the values and positions of AH blocks (of the last ones again past the end)
    struct Ahead {
        Piece<T, 2> v[AH];
        ushort2 i[AH];
    };
    const int last = A.grp_off[(size_t)A.ntiles * groups] - 1;
    auto ahead = [&](int blk) {
        Ahead a;
#pragma unroll
        for (int k = 0; k < AH; k++) {
            const size_t e = (size_t)min(blk + k, last) * 64 + 8 * r + 2 * q;
            a.v[k] = *(const Piece<T, 2> *)(val + e);
            a.i[k] = *(const ushort2 *)(A.lidx + e);
        }
        return a;
    };
    Ahead nx;
    int c0 = A.col_off[t], nc = A.col_off[t + 1] - c0, at[U];
#pragma unroll
    for (int k = 0; k < U; k++) at[k] = A.ucols[c0 + min(su + k * RS, nc - 1)];
    for (; t < t_end; t += t_step) {
        int b0[P], b1[P], row[P];
#pragma unroll
        for (int p = 0; p < P; p++) {
            const int gi = S::GP * (p * 4 + (p % 2 ? 3 - w : w)) + half;
            b0[p] = A.grp_off[(size_t)t * groups + gi];
            b1[p] = A.grp_off[(size_t)t * groups + gi + 1];
            row[p] = A.rows[(size_t)t * TS + 8 * gi + r];
        }
#pragma unroll
        for (int ch = 0; ch < S::NCH; ch++) {
            const unsigned char *__restrict__ src = (const unsigned char *)X + ch * S::CB + 16 * sl;
            u32x4 x[U];
#pragma unroll
            for (int k = 0; k < U; k++) x[k] = *(const u32x4 *)(src + (size_t)(unsigned)at[k] * S::RB);
            nx = ahead(b0[0]);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();                           // the previous pieces are consumed
            // past the end the last row again (the same words to the same
            // place), so nothing is conditional and the loads stay together
#pragma unroll
            for (int k = 0; k < U; k++) *(u32x4 *)(lds_ + min(su + k * RS, nc - 1) * S::CB + 16 * sl) = x[k];
            for (int u = su + U * RS; u < nc; u += RS)  // a tile of more columns
                *(u32x4 *)(lds_ + u * S::CB + 16 * sl) = *(const u32x4 *)(src + (size_t)(unsigned)A.ucols[c0 + u] * S::RB);
            // (not before: with the block rows' registers they would cost a
            // wavefront per SIMD in FP64)
            decltype(pre(0, 0)) in[P];
#pragma unroll
            for (int p = 0; p < P; p++) in[p] = pre(max(row[p], 0), ch * (S::CB / (int)sizeof(T)) + l * VL);
            __syncthreads();
            if (ch == S::NCH - 1 && t + t_step < t_end) {
                c0 = A.col_off[t + t_step];
                nc = A.col_off[t + t_step + 1] - c0;
#pragma unroll
                for (int k = 0; k < U; k++) at[k] = A.ucols[c0 + min(su + k * RS, nc - 1)];
            }
            const unsigned char *xs = lds_ + l * VL * (int)sizeof(T);
#pragma unroll
            for (int p = 0; p < P; p++) {
                T acc[VL];
#pragma unroll
                for (int c = 0; c < VL; c++) acc[c] = T(0);
                for (int blk = b0[p]; blk < b1[p]; blk += AH) {
                    const Ahead cur = nx;
                    nx = ahead(blk + AH < b1[p] ? blk + AH : b0[(p + 1) % P]);
#pragma unroll
                    for (int k = 0; k < AH; k++)
                        if (blk + k < b1[p]) {
                            const int pos[2] = {(int)cur.i[k].x * S::CB, (int)cur.i[k].y * S::CB};
                            quad_step<T, VL, 0>(cur.v[k].v, pos, xs, acc);
                            quad_step<T, VL, 1>(cur.v[k].v, pos, xs, acc);
                            quad_step<T, VL, 2>(cur.v[k].v, pos, xs, acc);
                            quad_step<T, VL, 3>(cur.v[k].v, pos, xs, acc);
                        }
                }
                if (b0[p] >= b1[p] && p + 1 < P) nx = ahead(b0[(p + 1) % P]);   // an empty group: the next pass's
                if (row[p] >= 0) epi(row[p], ch * (S::CB / (int)sizeof(T)) + l * VL, ch, acc, in[p]);
            }
        }
    }
}

// wavefronts per SIMD the tile kernels' registers leave room for: four FP32
// workgroups of 64-row tiles fill a compute unit's LDS (a register more than
// 128 costs one of them: 106 -> 133 us for the last sweep at P2 40^3 with 32
// columns); in FP64 the limit would only bring scratch memory
template <typename T, int NR, int TS>
constexpr int tile_waves() { return TS <= 64 && sizeof(T) == 4 && TileShape<T, NR, TS>::NCH == 1 ? 4 : 1; }

// per-column partial sums of a tile kernel: dot[chunk][column of the lane]
template <typename T, int NR, int TS>
__device__ __forceinline__ void btile_partials(double *partials, double (&dot)[TileShape<T, NR, TS>::NCH][TileShape<T, NR, TS>::VL])
{
    using S = TileShape<T, NR, TS>;
    __shared__ double red[kBlock / 64][NR];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l = lane % S::LPR;
#pragma unroll
    for (int ch = 0; ch < S::NCH; ch++)
#pragma unroll
        for (int c = 0; c < S::VL; c++) {
            double v = dot[ch][c];
#pragma unroll
            for (int off = 32; off >= S::LPR; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane < S::LPR) red[w][ch * (S::CB / (int)sizeof(T)) + l * S::VL + c] = v;
        }
    __syncthreads();
    if (threadIdx.x < NR) {
        double v = 0.0;
        for (int k = 0; k < kBlock / 64; k++) v += red[k][threadIdx.x];
        partials[(size_t)blockIdx.x * NR + threadIdx.x] = v;
    }
}

// DOT: the partials of RHS . Zout
template <typename T, typename TR, typename TZ, int NR, int TS, bool DOT>
__global__ __launch_bounds__(kBlock, (tile_waves<T, NR, TS>())) void kt_sweep(
    DevTilesView A, const T *__restrict__ dinv, const TR *__restrict__ RHS, const T *__restrict__ Zin,
    TZ *__restrict__ Zout, double *partials, const int *all_done)
{
    if (stop_all(all_done)) return;
    using S = TileShape<T, NR, TS>;
    constexpr int VL = S::VL;
    double dot[S::NCH][VL] = {};
    struct In {
        Piece<T, VL> z;
        Piece<TR, VL> b;
        T d;
    };
    btile_rows<T, NR, TS, DOT && sizeof(T) == 4 ? 3 : 4>(
        A, Zin,
        [&](int row, int col) {
            const size_t o = (size_t)row * NR + col;
            return In{*(const Piece<T, VL> *)(Zin + o), *(const Piece<TR, VL> *)(RHS + o), dinv[row]};
        },
        [&](int row, int col, int ch, const T (&s)[VL], const In &in) {
            const size_t o = (size_t)row * NR + col;
            Piece<TZ, VL> out;
#pragma unroll
            for (int c = 0; c < VL; c++) out.v[c] = (TZ)(in.z.v[c] + in.d * ((T)in.b.v[c] - s[c]));
            *(Piece<TZ, VL> *)(Zout + o) = out;
            if constexpr (DOT)
#pragma unroll
                for (int c = 0; c < VL; c++) dot[ch][c] += (double)in.b.v[c] * (double)out.v[c];
        });
    if constexpr (DOT) btile_partials<T, NR, TS>(partials, dot);
}

template <typename T, int NR, int TS>
__global__ __launch_bounds__(kBlock, (tile_waves<T, NR, TS>())) void kt_resid(
    DevTilesView A, const T *__restrict__ RHS, const T *__restrict__ Z, T *__restrict__ Res, const int *all_done)
{
    if (stop_all(all_done)) return;
    constexpr int VL = TileShape<T, NR, TS>::VL;
    btile_rows<T, NR, TS, 4>(
        A, Z, [&](int row, int col) { return *(const Piece<T, VL> *)(RHS + (size_t)row * NR + col); },
        [&](int row, int col, int, const T (&s)[VL], Piece<T, VL> out) {
#pragma unroll
            for (int c = 0; c < VL; c++) out.v[c] -= s[c];
            *(Piece<T, VL> *)(Res + (size_t)row * NR + col) = out;
        });
}

// RESID: Y = F - A X, else Y = A X (DOT: with the partials of X . Y)
template <int NR, int TS, bool DOT, bool RESID>
__global__ __launch_bounds__(kBlock) void kt_spmv64(DevTilesView A, const double *__restrict__ X,
                                                    double *__restrict__ Y, const double *__restrict__ F,
                                                    double *partials, const int *all_done)
{
    if (stop_all(all_done)) return;
    using S = TileShape<double, NR, TS>;
    constexpr int VL = S::VL;
    double dot[S::NCH][VL] = {};
    using In = Piece<double, VL>;
    btile_rows<double, NR, TS, 4>(
        A, X,
        [&](int row, int col) {
            In in = {};
            if (DOT || RESID) in = *(const In *)((RESID ? F : X) + (size_t)row * NR + col);
            return in;
        },
        [&](int row, int col, int ch, const double (&s)[VL], const In &in) {
            In out;
#pragma unroll
            for (int c = 0; c < VL; c++) out.v[c] = RESID ? in.v[c] - s[c] : s[c];
            *(In *)(Y + (size_t)row * NR + col) = out;
            if constexpr (DOT)
#pragma unroll
                for (int c = 0; c < VL; c++) dot[ch][c] += in.v[c] * s[c];
        });
    if constexpr (DOT) btile_partials<double, NR, TS>(partials, dot);
}

// The same products where slices are few: a workgroup takes RU rows of a slice
// and its KG lane groups share each row's entries, so a level of a few
// thousand long rows (the middle of the hierarchy) spreads over the chip
// instead of over one workgroup per 64 rows, and a row's chain is KG times
// shorter.  The groups' sums are added in LDS in a fixed order.
template <typename T, int NR, int U, typename XL, typename BODY>
__device__ __forceinline__ void bsell_rows(const DevSellView &A, XL xload, BODY body)
{
    constexpr int RU = NR >= 64 ? 4 : 8, KG = kBlock / (RU * NR), UNITS = kSlice / RU, CH = 64;
    __shared__ T vs[CH * RU];
    __shared__ int cs[CH * RU];
    __shared__ T red[kBlock];
    const T *__restrict__ val = (const T *)A.val;
    const int c = threadIdx.x % NR, rl = threadIdx.x / NR % RU, kg = threadIdx.x / (NR * RU);
    for (int u = blockIdx.x; u < A.nslices * UNITS; u += gridDim.x) {
        const int sl = u / UNITS, row0 = u % UNITS * RU;
        const int4 m = A.meta[sl];
        T acc = T(0);
        for (int j0 = 0; j0 < m.w; j0 += CH) {
            const int jn = min(CH, m.w - j0), g = threadIdx.x / RU, lane = row0 + (int)threadIdx.x % RU;
            T vt[4] = {};
            int ct[4] = {};
            const bool mine = threadIdx.x < CH / 4 * RU && 4 * g < jn;
            if (mine) {
                const size_t at = ((size_t)m.x + j0 / 4 + g) * (4 * kSlice) + 4 * lane;
#pragma unroll
                for (int k = 0; k < 4; k++) vt[k] = val[at + k];
                if (m.z < 0) {
                    const ushort4 o = *(const ushort4 *)(A.off + at);
                    const int2 *__restrict__ bs = A.base + ((size_t)m.x + j0 / 4 + g) * 4;
                    const unsigned short ok[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                    for (int k = 0; k < 4; k++) ct[k] = (ok[k] & 0x8000 ? bs[k].y : bs[k].x) + (ok[k] & 0x7fff);
                } else {
                    const int4 cc = *(const int4 *)(A.wide + ((size_t)m.z + j0 / 4 + g) * (4 * kSlice) + 4 * lane);
                    ct[0] = cc.x, ct[1] = cc.y, ct[2] = cc.z, ct[3] = cc.w;
                }
            }
            __syncthreads();                           // the previous chunk is consumed
            if (mine)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    vs[(4 * g + k) * RU + threadIdx.x % RU] = vt[k];
                    cs[(4 * g + k) * RU + threadIdx.x % RU] = ct[k];
                }
            __syncthreads();
#pragma unroll U
            for (int jj = kg; jj < jn; jj += KG) acc += vs[jj * RU + rl] * xload(cs[jj * RU + rl], c);
        }
        if (KG > 1) {
            __syncthreads();                           // the previous unit's sums are read
            red[threadIdx.x] = acc;
            __syncthreads();
            if (kg == 0)
#pragma unroll
                for (int k = 1; k < KG; k++) acc += red[threadIdx.x + k * NR * RU];
        }
        const int row = sl * kSlice + row0 + rl;
        if (kg == 0 && row < A.n) body(row, c, acc);
    }
}

// Rows of a level operator, shared out one way or the other: split where a
// workgroup per slice would not fill the 256 compute units four times (twice in
// FP32).  Measured with 32 columns, FP32 / FP64 us, whole slices -> split: 72
// slices 38 / 84 -> 18 / 25, 295 slices 27 / 63 -> 19 / 30, restriction of 927
// slices 60 / 131 -> 64 / 107; with 8 columns, restriction of 43 slices, FP64
// 39.7 -> 12.1.
template <typename T, int NR, int U, bool SPLIT, typename XL, typename BODY>
__device__ __forceinline__ void blevel_rows(const DevSellView &A, XL xload, BODY body)
{
    if constexpr (SPLIT) bsell_rows<T, NR, U>(A, xload, body);
    else bsell_slices<T, NR, U>(A, xload, body);
}
template <typename T>
constexpr int kSplitSlices = sizeof(T) == 8 ? 1024 : 512;

// ------------------------------------------------------- AMG levels, transfers
// Row-permuted sliced ELL: internal row r of M is row perm[r] of the
// operator; columns are not renumbered.

template <typename T, int NR, int MODE, int U, bool SPLIT>   // MODE 0: Y = M X, 1: Y += M X
__global__ __launch_bounds__(kBlock) void kb_lmatvec(DevSellView M, const int *__restrict__ perm,
                                                     const T *__restrict__ X, T *__restrict__ Y, const int *all_done)
{
    if (stop_all(all_done)) return;
    blevel_rows<T, NR, U, SPLIT>(M, [&](int j, int c) { return gather32(X, (unsigned)j * NR + c); }, [&](int r, int c, T s) {
        size_t o = (size_t)perm[r] * NR + c;
        if (MODE) Y[o] += s;
        else Y[o] = s;
    });
}

// Y = M [X1; X2] (columns below split index X1, the others X2)
template <typename T, int NR, int U, bool SPLIT>
__global__ __launch_bounds__(kBlock) void kb_lmatvec2(DevSellView M, const int *__restrict__ perm,
                                                      const T *__restrict__ X1, const T *__restrict__ X2, int split,
                                                      T *__restrict__ Y, const int *all_done)
{
    if (stop_all(all_done)) return;
    blevel_rows<T, NR, U, SPLIT>(
        M, [&](int j, int c) { return j < split ? gather32(X1, (unsigned)j * NR + c) : gather32(X2, (unsigned)(j - split) * NR + c); },
        [&](int r, int c, T s) { Y[(size_t)perm[r] * NR + c] = s; });
}

// X = D^-1 B, R = B - A X, with AD the values of A D^-1: the product
// gathers B alone (one load per slot keeps the unrolled gathers in flight)
template <typename T, int NR, int U, bool SPLIT>
__global__ __launch_bounds__(kBlock) void kb_lvpre(DevSellView AD, const int *__restrict__ perm,
                                                   const T *__restrict__ dinv, const T *__restrict__ B,
                                                   T *__restrict__ X, T *__restrict__ R, const int *all_done)
{
    if (stop_all(all_done)) return;
    blevel_rows<T, NR, U, SPLIT>(AD, [&](int j, int c) { return gather32(B, (unsigned)j * NR + c); }, [&](int r, int c, T s) {
        const int i = perm[r];
        size_t o = (size_t)i * NR + c;
        T b = B[o];
        X[o] = dinv[i] * b;
        R[o] = b - s;
    });
}

// Y = X + D^-1 (B - A X)
template <typename T, int NR, int U, bool SPLIT>
__global__ __launch_bounds__(kBlock) void kb_lsweep(DevSellView A, const int *__restrict__ perm,
                                                    const T *__restrict__ dinv, const T *__restrict__ B,
                                                    const T *__restrict__ X, T *__restrict__ Y, const int *all_done)
{
    if (stop_all(all_done)) return;
    blevel_rows<T, NR, U, SPLIT>(A, [&](int j, int c) { return gather32(X, (unsigned)j * NR + c); }, [&](int r, int c, T s) {
        const int i = perm[r];
        size_t o = (size_t)i * NR + c;
        Y[o] = X[o] + dinv[i] * (B[o] - s);
    });
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
// 16x16x4 forms: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and
// holds D[row][l % 16] in register v
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f64x4 mfma16(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
template <typename T>
__device__ __forceinline__ int mfma16_row(int grp, int v) { return sizeof(T) == 4 ? 4 * grp + v : grp + 4 * v; }

// X = M B for a dense row-major n x n matrix M (the coarsest inverse or the
// dense sub-cycle) on the matrix cores.  A workgroup takes 16 rows and (up to)
// 32 columns; its kDenseWaves wavefronts split the inner index in steps of 16,
// of which a lane reads four consecutive entries of its row of M (one load)
// and, for each, its columns' entries of B, and the partial products are added
// in LDS in a fixed order.  M is read once (twice with 64 columns): 14 MB in
// FP64 at n = 1340.  Steps past the end multiply zeros.  With 32 columns 154 ->
// 17.0 us (FP64) and 27.7 -> 18.1 (FP32) at n = 1340, with 8 columns 26.1 -> 8.2 at
// n = 960 (the vector units before, four rows per workgroup).
constexpr int kDenseWaves = 8;

template <typename T, int NR>
__global__ __launch_bounds__(64 * kDenseWaves) void kb_dense(int n, const T *__restrict__ M, const T *__restrict__ B,
                                                             T *__restrict__ X, const int *all_done)
{
    if (stop_all(all_done)) return;
    constexpr int NC = NR < 32 ? NR : 32, CT = (NC + 15) / 16;
    typedef T V __attribute__((ext_vector_type(4)));
    __shared__ T red[kDenseWaves][16 * 16 * CT];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = lane & 15, g = lane >> 4, r0 = (int)blockIdx.x * 16, col0 = (int)blockIdx.y * NC;
    const T *__restrict__ row = M + (size_t)min(r0 + i, n - 1) * n;          // clamped rows unused
    V acc[CT];
#pragma unroll
    for (int t = 0; t < CT; t++) acc[t] = V{0, 0, 0, 0};
#pragma unroll 2
    for (int k0 = 16 * w; k0 < n; k0 += 16 * kDenseWaves) {
        T a[4], b[4][CT];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int k = k0 + 4 * g + q, kc = min(k, n - 1);
            const T m = row[kc];
            a[q] = k < n ? m : T(0);
#pragma unroll
            for (int t = 0; t < CT; t++) b[q][t] = B[(size_t)kc * NR + col0 + min(16 * t + i, NC - 1)];
        }
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int t = 0; t < CT; t++) acc[t] = mfma16(a[q], b[q][t], acc[t]);
    }
#pragma unroll
    for (int t = 0; t < CT; t++)
#pragma unroll
        for (int v = 0; v < 4; v++) red[w][(mfma16_row<T>(g, v) * CT + t) * 16 + i] = acc[t][v];
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * 16 * CT; e += 64 * kDenseWaves) {
        const int r = r0 + e / (16 * CT), c = e % (16 * CT);
        T s = T(0);
#pragma unroll
        for (int k = 0; k < kDenseWaves; k++) s += red[k][e];
        if (r < n && c < NC) X[(size_t)r * NR + col0 + c] = s;
    }
}

// ------------------------------------------------------------------- CG

template <int NR>
__global__ __launch_bounds__(kBlock) void kb_dot(int n, const double *__restrict__ a, const double *__restrict__ b,
                                                 double *partials)
{
    double acc = 0.0;
    FOR_BROWS(NR, n)
    {
        size_t o = (size_t)row * NR + c_;
        acc += a[o] * b[o];
    }
    write_col_partials<NR>(partials, acc);
}

// sum the per-column partials and update the per-column CG state
constexpr int kFinishBlock = 1024;

template <int NR>
__global__ __launch_bounds__(kFinishBlock) void kb_finish(const double *__restrict__ partials, int nparts, int mode,
                                                          double *out, BCgState st)
{
    if (mode != FIN_PLAIN && *st.all_done) return;
    constexpr int G = kFinishBlock / NR;           // partial rows summed side by side
    const int c = threadIdx.x % NR, g = threadIdx.x / NR;
    // four independent accumulators keep several loads in flight
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int b = g;
    for (; b + 3 * G < nparts; b += 4 * G) {
        s0 += partials[(size_t)b * NR + c];
        s1 += partials[(size_t)(b + G) * NR + c];
        s2 += partials[(size_t)(b + 2 * G) * NR + c];
        s3 += partials[(size_t)(b + 3 * G) * NR + c];
    }
    for (; b < nparts; b += G) s0 += partials[(size_t)b * NR + c];
    __shared__ int active_left;
    if (threadIdx.x == 0) active_left = 0;
    const double t = col_sums<NR, kFinishBlock>((s0 + s1) + (s2 + s3));   // (a barrier: active_left is set)
    if (threadIdx.x < NR) {
        const int k = *st.k;
        if (mode == FIN_PLAIN) {
            out[c] = t;
        } else if (st.done[c] == 0) {
            int d = 0;
            if (mode == FIN_RR) {
                st.rr[(size_t)(k + 1) * NR + c] = t;
                st.iter[c] = k + 1;
                if (!std::isfinite(t)) d = 4;
                else if (t <= st.tol2ff[c]) d = 1;
                else if (k + 1 >= st.maxit) d = 2;
            } else {
                (mode == FIN_PQ ? st.pq : st.rz)[(size_t)k * NR + c] = t;
                if (!std::isfinite(t)) d = 4;
                else if (!(t > 0.0)) d = 3;
            }
            if (d) st.done[c] = d;
            else atomicAdd(&active_left, 1);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && mode != FIN_PLAIN) {
        if (mode == FIN_RR) *st.k += 1;
        if (active_left == 0) *st.all_done = 1;
    }
}

template <int NR>
__global__ void kb_cg_init(BCgState st, double tol2, const double *ff, const double *rr0)
{
    const int c = threadIdx.x;
    if (c >= NR) return;
    double f2 = ff[c], r2 = rr0[c];
    st.rr[c] = r2;
    st.tol2ff[c] = tol2 * f2;
    st.iter[c] = 0;
    int d = 0;
    if (!std::isfinite(f2) || !std::isfinite(r2)) d = 4;
    else if (r2 <= tol2 * f2) d = 1;
    else if (st.maxit <= 0) d = 2;
    st.done[c] = d;
    __shared__ int any;
    if (c == 0) any = 0;
    __syncthreads();
    if (d == 0) atomicAdd(&any, 1);
    __syncthreads();
    if (c == 0) {
        *st.k = 0;
        *st.all_done = any == 0;
    }
}

// X += alpha P, R -= alpha Q with the partials of R . R, and the
// preconditioner's first sweep from zero (the expressions of kb_jacobi0): Z0 = D^-1 R and RT = R in the type T
template <typename T, int NR>
__global__ __launch_bounds__(kBlock) void kb_cg_update_prep(int n, double *__restrict__ X, double *__restrict__ R,
                                                            const double *__restrict__ P,
                                                            const double *__restrict__ Q, BCgState st,
                                                            double *partials, const T *__restrict__ dinv,
                                                            T *__restrict__ Z0, T *__restrict__ RT)
{
    if (*st.all_done) return;
    const int k = *st.k;
    const int c = threadIdx.x % NR;
    const bool active = st.done[c] == 0;
    const double alpha = active ? st.rz[(size_t)k * NR + c] / st.pq[(size_t)k * NR + c] : 0.0;
    double acc = 0.0;
    FOR_BROWS(NR, n)
    {
        size_t o = (size_t)row * NR + c_;
        double ri = R[o];
        if (active) {
            X[o] += alpha * P[o];
            ri -= alpha * Q[o];
            R[o] = ri;
        }
        acc += ri * ri;
        T rt = (T)ri;
        Z0[o] = dinv[row] * rt;
        if (RT) RT[o] = rt;
    }
    write_col_partials<NR>(partials, acc);
}

template <int NR, typename TZ>
__global__ __launch_bounds__(kBlock) void kb_cg_direction(int n, const TZ *__restrict__ Z, double *__restrict__ P,
                                                          BCgState st)
{
    if (*st.all_done) return;
    const int k = *st.k;
    const int c = threadIdx.x % NR;
    if (st.done[c] != 0) return;
    const double beta = k == 0 ? 0.0 : st.rz[(size_t)k * NR + c] / st.rz[(size_t)(k - 1) * NR + c];
    FOR_BROWS(NR, n)
    {
        size_t o = (size_t)row * NR + c_;
        const double z = Z[o];
        P[o] = k == 0 ? z : z + beta * P[o];
    }
}

// internal block row i = external row perm[i]; external leading dimension ld
template <int NR>
__global__ __launch_bounds__(kBlock) void kb_gather(int n, int ld, const int *__restrict__ perm,
                                                    const double *__restrict__ x, double *__restrict__ y)
{
    FOR_BROWS(NR, n)
    {
        y[(size_t)row * NR + c_] = c_ < ld ? x[(size_t)perm[row] * ld + c_] : 0.0;
    }
}

template <int NR>
__global__ __launch_bounds__(kBlock) void kb_scatter(int n, int ld, const int *__restrict__ perm,
                                                     const double *__restrict__ x, double *__restrict__ y)
{
    FOR_BROWS(NR, n)
    {
        if (c_ < ld) y[(size_t)perm[row] * ld + c_] = x[(size_t)row * NR + c_];
    }
}

}  // namespace

#define NR_SWITCH(nr, CALL)                            \
    switch (nr) {                                      \
    case 8: { constexpr int NR = 8; CALL; } break;     \
    case 16: { constexpr int NR = 16; CALL; } break;   \
    case 32: { constexpr int NR = 32; CALL; } break;   \
    default: { constexpr int NR = 64; CALL; } break;   \
    }

// two workgroups per compute unit
constexpr size_t kTileLdsMax = 64 * 1024;

size_t btile_lds(const DevTilesView &A, int nr, int s)
{
    if (A.ntiles == 0) return 0;                        // not built for this operator
    const size_t b = (size_t)A.max_cols * std::min(128, nr * s);
    return b <= kTileLdsMax ? std::max<size_t>(b, 16) : 0;
}

// A tile kernel's workgroups walk several tiles each: at most 1024, as many
// as are resident with 40 KB of LDS each, so the per-column partial sums of a
// reduction stay few
inline int btile_grid(const DevTilesView &A) { return std::max(1, std::min(A.ntiles, 1024)); }

#define TILE_SWITCH(A, CALL)                              \
    if ((A).tile == 32) { constexpr int TS = 32; CALL; }        \
    else if ((A).tile == 64) { constexpr int TS = 64; CALL; }   \
    else { constexpr int TS = 128; CALL; }

template <typename T, typename TR, typename TZ>
int btile_sweep(hipStream_t s, int nr, const DevTilesView &A, const T *dinv, const TR *RHS, const T *Zin, TZ *Zout,
                double *partials, const int *all_done)
{
    const int g = btile_grid(A);
    const size_t lds = btile_lds(A, nr, sizeof(T));
    if (partials) {
        NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_sweep<T, TR, TZ, NR, TS, true>), dim3(g), dim3(kBlock), lds, s,
                                                        A, dinv, RHS, Zin, Zout, partials, all_done)));
    } else {
        NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_sweep<T, TR, TZ, NR, TS, false>), dim3(g), dim3(kBlock), lds,
                                                        s, A, dinv, RHS, Zin, Zout, partials, all_done)));
    }
    return g;
}

template <typename T>
int btile_resid(hipStream_t s, int nr, const DevTilesView &A, const T *RHS, const T *Z, T *Res, const int *all_done)
{
    const int g = btile_grid(A);
    const size_t lds = btile_lds(A, nr, sizeof(T));
    NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_resid<T, NR, TS>), dim3(g), dim3(kBlock), lds, s, A, RHS, Z, Res,
                                                    all_done)));
    return g;
}

int btile_spmv64(hipStream_t s, int nr, const DevTilesView &A, const double *X, double *Y, double *partials,
                 const int *all_done)
{
    const int g = btile_grid(A);
    const size_t lds = btile_lds(A, nr, 8);
    if (partials) {
        NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_spmv64<NR, TS, true, false>), dim3(g), dim3(kBlock), lds, s, A,
                                                        X, Y, (const double *)nullptr, partials, all_done)));
    } else {
        NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_spmv64<NR, TS, false, false>), dim3(g), dim3(kBlock), lds, s,
                                                        A, X, Y, (const double *)nullptr, partials, all_done)));
    }
    return g;
}

int btile_residual64(hipStream_t s, int nr, const DevTilesView &A, const double *F, const double *U, double *R)
{
    const int g = btile_grid(A);
    const size_t lds = btile_lds(A, nr, 8);
    NR_SWITCH(nr, TILE_SWITCH(A, hipLaunchKernelGGL((kt_spmv64<NR, TS, false, true>), dim3(g), dim3(kBlock), lds, s, A, U,
                                                    R, F, (double *)nullptr, (const int *)nullptr)));
    return g;
}

template <typename T>
void bjacobi0(hipStream_t s, int nr, int n, const T *dinv, const double *R, T *Z, T *RT, const int *all_done)
{
    int g = brows_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_jacobi0<T, NR>), dim3(g), dim3(kBlock), 0, s, n, dinv, R, Z, RT, all_done));
}

template <typename T, typename TR, typename TZ>
int bsell_sweep(hipStream_t s, int nr, const DevSellView &A, const T *dinv, const TR *RHS, const T *Zin, TZ *Zout,
                const double *Rdot, double *partials, const int *all_done)
{
    int g = bsell_grid(A);
    if (partials) {
        NR_SWITCH(nr, hipLaunchKernelGGL((kb_sweep<T, TR, TZ, NR, true>), dim3(g), dim3(kBlock), 0, s, A, dinv, RHS,
                                         Zin, Zout, Rdot, partials, all_done));
    } else {
        NR_SWITCH(nr, hipLaunchKernelGGL((kb_sweep<T, TR, TZ, NR, false>), dim3(g), dim3(kBlock), 0, s, A, dinv, RHS,
                                         Zin, Zout, Rdot, partials, all_done));
    }
    return g;
}

template <typename T>
int bsell_resid(hipStream_t s, int nr, const DevSellView &A, const T *RHS, const T *Z, T *Res, const int *all_done)
{
    int g = bsell_grid(A);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_resid<T, NR>), dim3(g), dim3(kBlock), 0, s, A, RHS, Z, Res, all_done));
    return g;
}

int bsell_spmv64(hipStream_t s, int nr, const DevSellView &A, const double *X, double *Y, double *partials,
                 const int *all_done)
{
    int g = bsell_grid(A);
    if (partials) {
        NR_SWITCH(nr, hipLaunchKernelGGL((kb_spmv64<NR, true, false>), dim3(g), dim3(kBlock), 0, s, A, X, Y,
                                         (const double *)nullptr, partials, all_done));
    } else {
        NR_SWITCH(nr, hipLaunchKernelGGL((kb_spmv64<NR, false, false>), dim3(g), dim3(kBlock), 0, s, A, X, Y,
                                         (const double *)nullptr, partials, all_done));
    }
    return g;
}

int bsell_residual64(hipStream_t s, int nr, const DevSellView &A, const double *F, const double *U, double *R)
{
    int g = bsell_grid(A);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_spmv64<NR, false, true>), dim3(g), dim3(kBlock), 0, s, A, U, R, F,
                                     (double *)nullptr, (const int *)nullptr));
    return g;
}

// unroll: slots per lane whose gathers are in flight together (1 or 4).
// Four pays off on operators with long rows (the level matrices, the
// restrictions); on the short rows of the prolongations the extra registers
// cost more occupancy than the overlap gains.
#define U_SWITCH(unroll, CALL)                                              \
    do {                                                                    \
        if ((unroll) >= 4 && blevel_split<T>(nslices_)) {                      \
            constexpr int U = 4;                                            \
            constexpr bool SPLIT = true;                                    \
            CALL;                                                           \
        } else if ((unroll) >= 4) {                                         \
            constexpr int U = 4;                                            \
            constexpr bool SPLIT = false;                                   \
            CALL;                                                           \
        } else {                                                            \
            constexpr int U = 1;                                            \
            constexpr bool SPLIT = false;                                   \
            CALL;                                                           \
        }                                                                   \
    } while (0)

template <typename T>
inline bool blevel_split(int nslices) { return nslices < kSplitSlices<T>; }
template <typename T>
inline int blevel_grid(const DevSellView &A, int unroll)
{
    return unroll >= 4 && blevel_split<T>(A.nslices) ? grid_cap(A.nslices * 8LL) : bsell_grid(A);
}

template <typename T>
void blevel_matvec(hipStream_t s, int nr, const DevSellView &M, int unroll, const int *perm, const T *X, T *Y,
                   bool add, const int *all_done)
{
    const int nslices_ = M.nslices, g = blevel_grid<T>(M, unroll);
    if (add) {
        U_SWITCH(unroll, NR_SWITCH(nr, hipLaunchKernelGGL((kb_lmatvec<T, NR, 1, U, SPLIT>), dim3(g), dim3(kBlock), 0, s, M, perm,
                                                     X, Y, all_done)));
    } else {
        U_SWITCH(unroll, NR_SWITCH(nr, hipLaunchKernelGGL((kb_lmatvec<T, NR, 0, U, SPLIT>), dim3(g), dim3(kBlock), 0, s, M, perm,
                                                     X, Y, all_done)));
    }
}

template <typename T>
void blevel_matvec2(hipStream_t s, int nr, const DevSellView &M, int unroll, const int *perm, const T *X1, const T *X2, int split,
                    T *Y, const int *all_done)
{
    const int nslices_ = M.nslices, g = blevel_grid<T>(M, unroll);
    U_SWITCH(unroll, NR_SWITCH(nr, hipLaunchKernelGGL((kb_lmatvec2<T, NR, U, SPLIT>), dim3(g), dim3(kBlock), 0, s, M, perm, X1,
                                                 X2, split, Y, all_done)));
}

template <typename T>
void blevel_vpre(hipStream_t s, int nr, const DevSellView &AD, int unroll, const int *perm, const T *dinv, const T *B, T *X, T *R,
                 const int *all_done)
{
    const int nslices_ = AD.nslices, g = blevel_grid<T>(AD, unroll);
    U_SWITCH(unroll, NR_SWITCH(nr, hipLaunchKernelGGL((kb_lvpre<T, NR, U, SPLIT>), dim3(g), dim3(kBlock), 0, s, AD, perm, dinv,
                                                 B, X, R, all_done)));
}

template <typename T>
void blevel_sweep(hipStream_t s, int nr, const DevSellView &A, int unroll, const int *perm, const T *dinv, const T *B, const T *X,
                  T *Y, const int *all_done)
{
    const int nslices_ = A.nslices, g = blevel_grid<T>(A, unroll);
    U_SWITCH(unroll, NR_SWITCH(nr, hipLaunchKernelGGL((kb_lsweep<T, NR, U, SPLIT>), dim3(g), dim3(kBlock), 0, s, A, perm, dinv,
                                                 B, X, Y, all_done)));
}

template <typename T>
void bdense(hipStream_t s, int nr, int n, const T *Ainv, const T *B, T *X, const int *all_done)
{
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_dense<T, NR>), dim3((n + 15) / 16, NR > 32 ? 2 : 1), dim3(64 * kDenseWaves), 0, s, n,
                                     Ainv, B, X, all_done));
}

int bvec_dot(hipStream_t s, int nr, int n, const double *a, const double *b, double *partials)
{
    int g = bsum_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_dot<NR>), dim3(g), dim3(kBlock), 0, s, n, a, b, partials));
    return g;
}

void bfinish(hipStream_t s, int nr, const double *partials, int nparts, FinishMode mode, double *out,
             const BCgState &st)
{
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_finish<NR>), dim3(1), dim3(kFinishBlock), 0, s, partials, nparts, (int)mode,
                                     out, st));
}

void bcg_init(hipStream_t s, int nr, const BCgState &st, double tol2, const double *ff, const double *rr0)
{
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_cg_init<NR>), dim3(1), dim3(64), 0, s, st, tol2, ff, rr0));
}

template <typename T>
int bcg_update_prep(hipStream_t s, int nr, int n, double *X, double *R, const double *P, const double *Q,
                    const BCgState &st, double *partials, const T *dinv, T *Z0, T *RT)
{
    int g = bsum_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_cg_update_prep<T, NR>), dim3(g), dim3(kBlock), 0, s, n, X, R, P, Q, st,
                                     partials, dinv, Z0, RT));
    return g;
}
template int bcg_update_prep<float>(hipStream_t, int, int, double *, double *, const double *, const double *,
                                    const BCgState &, double *, const float *, float *, float *);
template int bcg_update_prep<double>(hipStream_t, int, int, double *, double *, const double *, const double *,
                                     const BCgState &, double *, const double *, double *, double *);

template <typename TZ>
void bcg_direction(hipStream_t s, int nr, int n, const TZ *Z, double *P, const BCgState &st)
{
    int g = brows_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_cg_direction<NR, TZ>), dim3(g), dim3(kBlock), 0, s, n, Z, P, st));
}

void bgather(hipStream_t s, int nr, int n, int ld, const int *perm, const double *x, double *y)
{
    int g = brows_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_gather<NR>), dim3(g), dim3(kBlock), 0, s, n, ld, perm, x, y));
}

void bscatter(hipStream_t s, int nr, int n, int ld, const int *perm, const double *x, double *y)
{
    int g = brows_grid(n, nr);
    NR_SWITCH(nr, hipLaunchKernelGGL((kb_scatter<NR>), dim3(g), dim3(kBlock), 0, s, n, ld, perm, x, y));
}

#define BINST(T)                                                                                                   \
    template int btile_sweep<T, T, T>(hipStream_t, int, const DevTilesView &, const T *, const T *, const T *, T *, \
                                      double *, const int *);                                      \
    template int btile_resid<T>(hipStream_t, int, const DevTilesView &, const T *, const T *, T *, const int *);    \
    template void bjacobi0<T>(hipStream_t, int, int, const T *, const double *, T *, T *, const int *);            \
    template int bsell_sweep<T, T, T>(hipStream_t, int, const DevSellView &, const T *, const T *, const T *, T *, \
                                      const double *, double *, const int *);                                      \
    template int bsell_resid<T>(hipStream_t, int, const DevSellView &, const T *, const T *, T *, const int *);    \
    template void blevel_matvec<T>(hipStream_t, int, const DevSellView &, int, const int *, const T *, T *, bool,      \
                                   const int *);                                                                   \
    template void blevel_matvec2<T>(hipStream_t, int, const DevSellView &, int, const int *, const T *, const T *, int, \
                                    T *, const int *);                                                             \
    template void blevel_vpre<T>(hipStream_t, int, const DevSellView &, int, const int *, const T *, const T *, T *,     \
                                 T *, const int *);                                                                \
    template void blevel_sweep<T>(hipStream_t, int, const DevSellView &, int, const int *, const T *, const T *,         \
                                  const T *, T *, const int *);                                                    \
    template void bdense<T>(hipStream_t, int, int, const T *, const T *, T *, const int *);

BINST(double)
BINST(float)
template void bcg_direction<double>(hipStream_t, int, int, const double *, double *, const BCgState &);
template void bcg_direction<float>(hipStream_t, int, int, const float *, double *, const BCgState &);
template int bsell_sweep<float, double, float>(hipStream_t, int, const DevSellView &, const float *, const double *,
                                               const float *, float *, const double *, double *, const int *);
template int btile_sweep<float, double, float>(hipStream_t, int, const DevTilesView &, const float *, const double *,
                                                const float *, float *, double *, const int *);

}  // namespace auxp
