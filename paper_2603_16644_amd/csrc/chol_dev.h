// Steps of the FP64 Cholesky factorization (chol.hip, sketch_factor.hip).
//
// cholesky64, blocked by 64 columns, one launch per block column (CholStep
// k): every work-group takes one 64 x 64 tile (i, j) of the trailing lower
// triangle, forms X_i = C_ik L_kk^{-T} and X_j itself by substitution and
// subtracts X_i X_j^T; the work-group of tile (k + 1, k + 1) then factors its
// block at once, so that the next launch finds L_{k+1,k+1} ready.  Raw
// panels stay in C (other work-groups read them); L and L^T are written
// elsewhere.  The panel products and the diagonal factor that used to be
// launches of their own (a GEMM with the inverse block, a one-work-group
// factor-and-invert of 51 us per block) disappear; each work-group repeats
// the 64 x 64 substitution of its two panels, which costs less than a launch.
//
// Everything runs on the FP64 MFMA 16x16x4 in its accumulator layout: lane
// (r, g) (r = lane % 16, g = lane / 16) holds row r, register q of a
// 16-column block holds column g + 4 q, and that register is at once the
// MFMA's operand for the K values 4 q + g (on either side).  In the diagonal
// block wavefront w holds rows 16 w ..: for each block c of 16 columns
// wavefront c factors its 16 x 16 diagonal block, four columns a step (the 4 x
// 4 pivot block goes to every lane by readlane, each lane factors and inverts
// it, one MFMA applies the inverse and one updates the rest), and leaves the
// operands that it used in LDS (tab); after a barrier the wavefronts below
// substitute their block with them and leave it in LDS (xj), and after another
// they update what is right of it.  (One wavefront for all 64 rows, without
// LDS or barriers, took 30 us per block for 19.)  The operands are exactly the
// table that a panel substitution needs (tab in memory: per block column 16
// groups of the 4 x 4 inverse and its update, then the 6 blocks below the
// diagonal, negated).
//
// Bound: latency, 19 us per block column (launch 4, loads 2, panels and update
// 5, factor 8).  Measured with the block inverses, against the factor and
// inverse by one work-group, panel product and trailing product in launches
// of their own: n = 64 94 -> 41 us, 100 171 -> 60 us, 257 395 -> 129 us, 1000 1.25
// -> 0.37 ms, 2000 2.36 -> 0.80 ms.  (WPE 1: with 256 registers the kernel
// spills.)
//
// A non-positive or non-finite pivot at global column k sets *info to
// 2000 + k + 1 (first failure only) and the factor continues as NaN.  With
// tau > 0 (Gram matrix of a sketch) C + tau diag(C) is factored, and *info
// stays: *state gets 1 where a pivot is small (below CHOL_LOW tau C_kk, so
// that the shift counts), 2 or 3 where one is zero or not finite, else 0.  A
// shift of every pivot and not a floor under the small ones: raising single
// pivots that are rounding noise leaves the noise beside them to grow column
// by column, until the factor overflows.
#pragma once
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {

constexpr int CB = 64;

namespace {

typedef double v2d __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) double* gp64;
typedef __attribute__((address_space(1))) double* gw64;
typedef __attribute__((address_space(1))) v2d* gwv2;

__device__ __forceinline__ v4d mfma64(double a, double b, v4d c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Table of an upper triangular 64 x 64 block U (L_kk^T), in 16-byte entries:
// groups [c][q][lane] = (inverse operand, update operand), then the blocks
// (c, w), c < w, at tri_off: [p][lane] = (K step 2 p, K step 2 p + 1) of
// -U(16 c + 4 q + g, 16 w + r).
constexpr int TRI_DIAG = 16 * 64, TRI_OFF = 128, TRI_TAB = TRI_DIAG + 6 * TRI_OFF;   // v2d entries
__host__ __device__ constexpr int tri_off(int c, int w)
{
    return TRI_DIAG + TRI_OFF * (c * 3 - c * (c - 1) / 2 + (w - c - 1));
}
static_assert(TRI_TAB * 2 <= CB * CB, "a table fits the slot of a block inverse");

// (Everywhere below, what is taken from an entry is summed by itself and added
// once.  Taken from it product by product, each is rounded to the entry's last
// place: |L L^T - C| 5 to 7 times LAPACK's at n = 400 to 1000, for 1.1 to 1.3 times so.)
// t := t U^{-1} for one block of 16 columns and its groups.
__device__ __forceinline__ void tri_group(v4d& t, const v2d* tab, int lane)
{
    v4d u = (v4d){0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v2d f = tab[q * 64 + lane];
        const v4d y = mfma64(f[0], t[q] + u[q], (v4d){0, 0, 0, 0});
        t[q] = y[q];
        if (q < 3) u = mfma64(f[1], y[q], u);
    }
}
// x := x U^{-1} for 16 rows x 64 columns in accumulator layout.
__device__ __forceinline__ void tri_subst(v4d (&x)[4], const v2d* tab, int lane)
{
    v4d s[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = (v4d){0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        v4d t = x[c] + s[c];
        tri_group(t, tab + c * 256, lane);
        x[c] = t;
#pragma unroll
        for (int w = c + 1; w < 4; ++w)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const v2d f = tab[tri_off(c, w) + p * 64 + lane];
                s[w] = mfma64(f[0], t[2 * p], s[w]);
                s[w] = mfma64(f[1], t[2 * p + 1], s[w]);
            }
    }
}

// 1 / sqrt(d) to full precision from the hardware estimate (relative error
// below 2^-24, one step of third order).
__device__ __forceinline__ double rsqrt_full(double d)
{
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

}  // namespace

struct CholStepArgs {
    int64_t n, k;      // order; block column just factored (-1: none yet)
    double* C;         // lower triangle; trailing part updated in place
    int64_t ldc;
    double* L;         // null: not wanted
    int64_t ldl;
    double* Lt;        // upper triangle written
    int64_t ldt;
    double* tab;       // table of block column b at tab + b * CB * CB
    double* gd;        // tau > 0: copy of the diagonal of C
    double tau;
    int32_t* state;    // tau > 0 (null: not wanted)
    int32_t* zero2;    // two words set to zero by the first launch (null: none)
    int32_t* info;     // tau = 0
};
// PHASE: as a part of a longer loop (nothing that is made of the thread's index
// is kept in registers across the other parts).
template <bool SHIFT, bool PHASE = false>
struct CholStep {
    typedef CholStepArgs Args;
    static constexpr int NTH = 256, WPE = 1;
    static __device__ void run(const CholStepArgs& a, int bx, int by);
};

// Factor of a 16 x 16 diagonal block (one wavefront, accumulator layout), four
// columns a step; gt: the groups of its table (also put at lt in LDS).  Every
// lane factors the 4 x 4 pivot block, read by readlane; lane (r, g) then
// forms column g of its inverse.  Returns the columns whose pivot was bad, a
// bit each; or (SHIFT, with fl the shift of column r16) 1 for a small pivot, 2
// for a zero or non-finite one.
constexpr double CHOL_LOW = 256.0;
template <bool SHIFT>
__device__ __forceinline__ unsigned chol16(v4d& t, v2d* lt, gwv2 gt, double fl)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, g4 = lane >> 4;
    unsigned badm = 0;
    // the shift at once, for the whole diagonal: per pivot it would be part of
    // the serial chain, like the tests on the result
    const double lowest = 0.5 * fl;
    if (SHIFT)
#pragma unroll
        for (int q = 0; q < 4; ++q) t[q] += r16 == 4 * q + g4 ? fl : 0.0;
    double e[4];
    v4d u = (v4d){0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = g4 == j ? 1.0 : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // row 4 q + i of the pivot block in lanes r16 = 4 q + i, column j in g4 = j
        double l[4][4], r[4];
        t[q] += u[q];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) l[i][j] = lane_value(t[q], 4 * q + i + 16 * j);
        double ld = 0.0;   // L(j, j), j = g4
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double d = l[j][j];
            if (SHIFT) {
                const double f = lane_value(lowest, 4 * q + j);
                d = d < f ? f : d;   // (a NaN stays)
            }
            // d <= 0, NaN and infinity all give NaN
            r[j] = rsqrt_full(d);
            if (SHIFT) r[j] = d == 0.0 ? 0.0 : r[j];
            else if (__builtin_amdgcn_ballot_w64(r[j] != r[j]) != 0) badm |= 1u << (4 * q + j);
            ld = g4 == j ? d * r[j] : ld;
#pragma unroll
            for (int i = j + 1; i < 4; ++i) l[i][j] *= r[j];
#pragma unroll
            for (int i = j + 1; i < 4; ++i)
#pragma unroll
                for (int m = j + 1; m <= i; ++m) l[i][m] = fma(-l[i][j], l[m][j], l[i][m]);
        }
        // column g4 of the inverse of the factor; the lane keeps entry r16 % 4
        double op = 0.0;
        double y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = e[i];
#pragma unroll
            for (int m = 0; m < i; ++m) v = fma(-l[i][m], y[m], v);
            y[i] = v * r[i];
            op = (r16 & 3) == i ? y[i] : op;
        }
        op = (r16 >> 2) == q ? op : 0.0;
        const v4d z = mfma64(op, t[q], (v4d){0, 0, 0, 0});
        const double x = r16 == 4 * q + g4 ? ld : z[q];
        const double up = r16 >= 4 * q + 4 ? -x : 0.0;
        t[q] = x;
        if (q < 3) u = mfma64(up, x, u);
        lt[q * 64 + lane] = (v2d){op, up};
        gt[q * 64 + lane] = (v2d){op, up};
        if (SHIFT && r16 == 4 * q + g4) badm |= (x * x < CHOL_LOW * fl ? 1u : 0u) | (x > 0.0 ? 0u : 2u);
    }
    if (SHIFT)
        badm = (__builtin_amdgcn_ballot_w64(badm & 1u) != 0 ? 1u : 0u) | (__builtin_amdgcn_ballot_w64(badm & 2u) != 0 ? 2u : 0u);
    return badm;
}

template <bool SHIFT, bool PHASE>
__device__ __forceinline__ void CholStep<SHIFT, PHASE>::run(const CholStepArgs& a, int bx, int)
{
    __shared__ __attribute__((aligned(16))) v2d tab[TRI_TAB];
    __shared__ __attribute__((aligned(16))) v2d xj[4 * 4 * 2 * 64];   // [row block][c][p][lane]
    __shared__ unsigned small[4];                                     // (SHIFT) of each wavefront's 16 columns
    int tid = threadIdx.x;
    if (PHASE) asm volatile("" : "+v"(tid));
    const int lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n = a.n, k = a.k;
    int64_t ti = 0, tj = 0;
    if (k >= 0) {
        int64_t t = (int64_t)((sqrt(8.0 * (double)bx + 1.0) - 1.0) * 0.5);
        while (t * (t + 1) / 2 > bx) --t;
        while ((t + 1) * (t + 2) / 2 <= bx) ++t;
        ti = t;
        tj = bx - t * (t + 1) / 2;
    }
    const int64_t ib = k + 1 + ti, jb = k + 1 + tj;
    const gw64 C = (gw64)a.C;
    // 16 rows x 64 columns of C at (block row rb, block column cb); past the
    // matrix: the identity on the diagonal, else 0.  Above the diagonal
    // nothing has written C, and what lies there must not be read: chol16
    // multiplies it by the zeros of an inverse, which a NaN or an infinity
    // survives.
    auto load = [&](v4d (&x)[4], int64_t rb, int64_t cb) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (an entry that is written instead of none: a load under a
                // mask of its own is a branch, and the loads wait in line)
                const int64_t i = rb * CB + 16 * w + r16, j = cb * CB + 16 * c + 4 * q + g4;
                const int64_t ic = i < n ? i : n - 1, jc = j < ic ? j : ic;
                const double v = C[ic + jc * a.ldc];
                x[c][q] = (i < n && j <= i) ? v : (i == j ? 1.0 : 0.0);
            }
    };
    v4d acc[4], xx[4];   // the tile, and what is taken from it
    load(acc, ib, jb);
#pragma unroll
    for (int v = 0; v < 4; ++v) xx[v] = (v4d){0, 0, 0, 0};
    if (k >= 0) {
        v4d xi[4], xo[4];
        load(xi, ib, k);
        if (ti != tj) load(xo, jb, k);
        const gwv2 gt = (gwv2)((gw64)a.tab + k * CB * CB);
#pragma unroll
        for (int e = 0; e < TRI_TAB / 256; ++e) tab[tid + 256 * e] = gt[tid + 256 * e];
        __syncthreads();
        tri_subst(xi, tab, lane);
        if (ti != tj) {
            tri_subst(xo, tab, lane);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) xo[c] = xi[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int p = 0; p < 2; ++p) xj[((w * 4 + c) * 2 + p) * 64 + lane] = (v2d){-xo[c][2 * p], -xo[c][2 * p + 1]};
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c)       // K block
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int v = 0; v < 4; ++v) {   // column block of the tile = row block of X_j
                    const v2d f = xj[((v * 4 + c) * 2 + p) * 64 + lane];
                    xx[v] = mfma64(f[0], xi[c][2 * p], xx[v]);
                    xx[v] = mfma64(f[1], xi[c][2 * p + 1], xx[v]);
                }
        if (tj == 0) {
            // X_i is the part of L in block column k
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t i = ib * CB + 16 * w + r16, j = k * CB + 16 * c + 4 * q + g4;
                    if (i < n) {
                        ((gw64)a.Lt)[j + i * a.ldt] = xi[c][q];
                        if (a.L) ((gw64)a.L)[i + j * a.ldl] = xi[c][q];
                    }
                }
        }
    } else if (SHIFT) {
        for (int64_t i = tid; i < n; i += NTH) ((gw64)a.gd)[i] = C[i + i * a.ldc];
    }
    if (bx != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = ib * CB + 16 * w + r16, j = jb * CB + 16 * c + 4 * q + g4;
                if (i < n && j < n && j <= i) C[i + j * a.ldc] = acc[c][q] + xx[c][q];
            }
        return;
    }
    // tile (k + 1, k + 1), wavefront w holding its rows 16 w ..: for every
    // block of 16 columns c, wavefront c factors its diagonal block, the ones
    // below substitute theirs and update what is right of it
    __syncthreads();   // (xj and tab are free; the diagonal copy is written)
    const int64_t c0 = ib * CB;
    const gwv2 gt = (gwv2)((gw64)a.tab + ib * CB * CB);
    double fl = 0.0;
    if (SHIFT) {
        const int64_t col = c0 + 16 * w + r16;
        fl = col < n ? a.tau * ((gp64)a.gd)[col] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (w == c) {
            acc[c] += xx[c];
            const unsigned badm = chol16<SHIFT>(acc[c], tab + c * 256, gt + c * 256, fl);
            if (SHIFT) {
                if (lane == 0) small[c] = badm;
            } else if (badm != 0 && lane == 0 && *a.info == 0)
                *a.info = 2000 + (int32_t)(c0 + 16 * c + __builtin_ctz(badm)) + 1;
        }
        __syncthreads();
        if (w > c) {
            v4d t = acc[c] + xx[c];
            tri_group(t, tab + c * 256, lane);
            acc[c] = t;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const v2d f = (v2d){-t[2 * p], -t[2 * p + 1]};
                xj[(w * 2 + p) * 64 + lane] = f;
                gt[tri_off(c, 0) + w * TRI_OFF + p * 64 + lane] = f;
            }
        }
        if (c == 3) break;
        __syncthreads();
        if (w > c) {
#pragma unroll
            for (int v = c + 1; v < 4; ++v)
                if (v <= w)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const v2d f = xj[(v * 2 + p) * 64 + lane];
                        xx[v] = mfma64(f[0], acc[c][2 * p], xx[v]);
                        xx[v] = mfma64(f[1], acc[c][2 * p + 1], xx[v]);
                    }
        }
    }
    if (SHIFT && tid == 0 && k < 0 && a.zero2) a.zero2[0] = a.zero2[1] = 0;
    if (SHIFT && tid == 0 && a.state) *a.state = (k < 0 ? 0 : *a.state) | (int32_t)(small[0] | small[1] | small[2] | small[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c <= w)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = c0 + 16 * w + r16, j = c0 + 16 * c + 4 * q + g4;
                if (i < n && j <= i) {
                    ((gw64)a.Lt)[j + i * a.ldt] = acc[c][q];
                    if (a.L) ((gw64)a.L)[i + j * a.ldl] = acc[c][q];
                }
            }
}

}  // namespace pne
