// Cholesky factorization C = L L^T: of the n x n PNE matrix A_p^T A_p and of
// the Gram matrix of a sketch (both FP64, cholesky64), and of the FP32 Gram
// matrix of the condition estimate (cholesky_f32, further down).
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
// MFMA's operand for the K values 4 q + g (on either side).  The diagonal
// block is factored by one wavefront, four columns a step, with no LDS and no
// barrier: the 4 x 4 pivot block goes to every lane by readlane, each lane
// factors and inverts it, one MFMA per 16 rows applies the inverse, one MFMA
// per 16 x 16 block updates the rest.  The operands it used are exactly the
// table a panel substitution needs (tab: per block column 16 groups of the
// 4 x 4 inverse and its update, then the 6 blocks below the diagonal, negated).
//
// Bound: latency, 19 us per block column (launch 4, loads 2, panels and update
// 5, factor 8).  Measured with the block inverses, against the factor and
// inverse by one work-group, panel product and trailing product in launches
// of their own: n = 64 94 -> 41 us, 100 171 -> 60 us, 257 395 -> 129 us, 1000 1.25
// -> 0.37 ms, 2000 2.36 -> 0.80 ms.  (WPE 1: with 256 registers the kernel
// spills, and a spilled MFMA operand tuple came back wrong.)
//
// A non-positive or non-finite pivot at global column k sets *info to
// 2000 + k + 1 (first failure only) and the factor continues as NaN.  With
// tau > 0 (Gram matrix of a sketch) C + tau diag(C) is factored, and *info
// stays: *state gets 1 where a pivot is small (below CHOL_LOW tau C_kk, so
// that the shift counts), 2 or 3 where one is zero or not finite, else 0.  A
// shift of every pivot and not a floor under the small ones: raising single
// pivots that are rounding noise leaves the noise beside them to grow column
// by column, until the factor overflows.
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

// x := x U^{-1} for 16 rows x 64 columns in accumulator layout.
__device__ __forceinline__ void tri_subst(v4d (&x)[4], const v2d* tab, int lane)
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        v4d t = x[c];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v2d f = tab[(c * 4 + q) * 64 + lane];
            const v4d y = mfma64(f[0], t[q], (v4d){0, 0, 0, 0});
            t[q] = y[q];
            if (q < 3) {
                const v4d u = mfma64(f[1], y[q], t);
#pragma unroll
                for (int e = q + 1; e < 4; ++e) t[e] = u[e];
            }
        }
        x[c] = t;
#pragma unroll
        for (int w = c + 1; w < 4; ++w)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const v2d f = tab[tri_off(c, w) + p * 64 + lane];
                x[w] = mfma64(f[0], t[2 * p], x[w]);
                x[w] = mfma64(f[1], t[2 * p + 1], x[w]);
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
    int32_t* info;     // tau = 0
};
template <bool SHIFT>
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
    double e[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = g4 == j ? 1.0 : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        // row 4 q + i of the pivot block in lanes r16 = 4 q + i, column j in g4 = j
        double l[4][4], r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j <= i; ++j) l[i][j] = lane_value(t[q], 4 * q + i + 16 * j);
        double ld = 0.0;   // L(j, j), j = g4
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double d = l[j][j];
            if (SHIFT) {
                const double f = lane_value(fl, 4 * q + j);
                d += f;
                badm |= d < CHOL_LOW * f ? 1u : 0u;
                d = d < 0.5 * f ? 0.5 * f : d;   // (a NaN stays)
            }
            // d <= 0, NaN and infinity all give NaN
            r[j] = rsqrt_full(d);
            if (SHIFT) {
                badm |= d == 0.0 || r[j] != r[j] ? 2u : 0u;
                r[j] = d == 0.0 ? 0.0 : r[j];
            } else if (__builtin_amdgcn_ballot_w64(r[j] != r[j]) != 0) badm |= 1u << (4 * q + j);
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
        if (q < 3) {
            const v4d u = mfma64(up, x, t);
#pragma unroll
            for (int k = q + 1; k < 4; ++k) t[k] = u[k];
        }
        lt[q * 64 + lane] = (v2d){op, up};
        gt[q * 64 + lane] = (v2d){op, up};
    }
    return badm;
}

template <bool SHIFT>
__device__ __forceinline__ void CholStep<SHIFT>::run(const CholStepArgs& a, int bx, int)
{
    __shared__ __attribute__((aligned(16))) v2d tab[TRI_TAB];
    __shared__ __attribute__((aligned(16))) v2d xj[4 * 4 * 2 * 64];   // [row block][c][p][lane]
    __shared__ unsigned small[4];                                     // (SHIFT) of each wavefront's 16 columns
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
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
                const int64_t i = rb * CB + 16 * w + r16, j = cb * CB + 16 * c + 4 * q + g4;
                x[c][q] = (i < n && j <= i) ? C[i + j * a.ldc] : (i == j ? 1.0 : 0.0);
            }
    };
    v4d acc[4];
    load(acc, ib, jb);
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
                    acc[v] = mfma64(f[0], xi[c][2 * p], acc[v]);
                    acc[v] = mfma64(f[1], xi[c][2 * p + 1], acc[v]);
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
                if (i < n && j < n && j <= i) C[i + j * a.ldc] = acc[c][q];
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
            const unsigned badm = chol16<SHIFT>(acc[c], tab + c * 256, gt + c * 256, fl);
            if (SHIFT) {
                if (lane == 0) small[c] = badm;
            } else if (badm != 0 && lane == 0 && *a.info == 0)
                *a.info = 2000 + (int32_t)(c0 + 16 * c + __builtin_ctz(badm)) + 1;
        }
        __syncthreads();
        if (w > c) {
            v4d t = acc[c];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v2d f = tab[(c * 4 + q) * 64 + lane];
                const v4d y = mfma64(f[0], t[q], (v4d){0, 0, 0, 0});
                t[q] = y[q];
                if (q < 3) {
                    const v4d u = mfma64(f[1], y[q], t);
#pragma unroll
                    for (int e = q + 1; e < 4; ++e) t[e] = u[e];
                }
            }
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
                        acc[v] = mfma64(f[0], acc[c][2 * p], acc[v]);
                        acc[v] = mfma64(f[1], acc[c][2 * p + 1], acc[v]);
                    }
        }
    }
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

// L (optional) and L^T of C; C is destroyed.  tab: dinv_elems(n) values; info.
void cholesky64(Exec& ex, int64_t n, double* C, int64_t ldc, double* L, int64_t ldl, double* Lt, int64_t ldt,
                double* tab, int32_t* info)
{
    const int64_t nb = ceil_div(n, CB);
    for (int64_t k = -1; k + 1 < nb; ++k) {
        ex.iter((uint32_t)(k + 1));
        const int64_t r = nb - k - 1;
        const CholStepArgs a{n, k, C, ldc, L, ldl, Lt, ldt, tab, nullptr, 0.0, nullptr, info};
        launch<CholStep<false>>(ex, k < 0 ? 1 : r * (r + 1) / 2, 1, a);
    }
}
// L^T of C + tau diag(C); gd: n values (the diagonal of C, left there).  state:
// see above; only: where *only is 1 (null: always).
void cholesky64_shifted(Exec& ex, int64_t n, double* C, int64_t ldc, double* Lt, int64_t ldt, double* tab, double* gd,
                        double tau, int32_t* state, const int32_t* only)
{
    const int64_t nb = ceil_div(n, CB);
    for (int64_t k = -1; k + 1 < nb; ++k) {
        ex.iter((uint32_t)(k + 1));
        const int64_t r = nb - k - 1, wgs = k < 0 ? 1 : r * (r + 1) / 2;
        const CholStepArgs a{n, k, C, ldc, nullptr, 0, Lt, ldt, tab, gd, tau, state, nullptr};
        if (only) launch<When<CholStep<true>>>(ex, wgs, 1, When<CholStep<true>>::Args{a, only});
        else launch<CholStep<true>>(ex, wgs, 1, a);
    }
}

// ---------------------------------------------------------------- block inverses
// Inverses of the 64 x 64 diagonal blocks of a triangular FP64 matrix, one
// work-group per block: the block as an upper triangle U (of M, or of M^T for
// a lower M) becomes the table of tri_subst in LDS, and each of the four
// wavefronts substitutes 16 rows of the identity: X = U^{-1}.
// One launch takes the blocks of up to two matrices of the same order.
struct InvTri {
    struct Mat {
        const double* M;
        int64_t ld;
        int lower, unit;
        double* D;     // inverse of the block of M (64 x 64, column-major; null: not wanted)
        double* Dt;    // its transpose (null: not wanted)
    };
    struct Args {
        int64_t n;
        Mat m[2];
    };
    static constexpr int NTH = 256, WPE = 2;
    static __device__ void run(const Args& a, int bx, int by);
};
__device__ __forceinline__ void InvTri::run(const Args& g, int bx, int by)
{
    const Mat a = by == 0 ? g.m[0] : g.m[1];
    __shared__ double us[CB][CB + 1];   // us[j][k] = U(k, j)
    __shared__ __attribute__((aligned(16))) v2d tab[TRI_TAB];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g4 = lane >> 4, w = tid >> 6;
    const int64_t n = g.n, b0 = (int64_t)bx * CB;
    const gp64 M = (gp64)a.M;
#pragma unroll
    for (int e = 0; e < CB * CB / NTH; ++e) {
        // consecutive lanes read consecutive rows of M
        const int r = tid & 63, c = (tid >> 6) + 4 * e;
        const int kk = a.lower ? c : r, j = a.lower ? r : c;
        double v = 0.0;
        if (kk <= j) {
            v = (b0 + r < n && b0 + c < n) ? M[(b0 + r) + (b0 + c) * a.ld] : (kk == j ? 1.0 : 0.0);
            if (a.unit && kk == j) v = 1.0;
        }
        us[j][kk] = v;
    }
    __syncthreads();
    // groups: wavefront w builds those of block c = w
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int o = 16 * w + 4 * q, c = r16 - 4 * q;
        double inv = 0.0;
        if (c >= 0 && c < 4 && g4 <= c) {
            double y[4];
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                double s = k == c ? 1.0 : 0.0;
#pragma unroll
                for (int l = k + 1; l < 4; ++l)
                    if (l <= c) s -= us[o + l][o + k] * y[l];
                y[k] = k <= c ? s / us[o + k][o + k] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k == g4) inv = y[k];
        }
        tab[(w * 4 + q) * 64 + lane] = (v2d){inv, r16 >= 4 * q + 4 ? -us[16 * w + r16][o + g4] : 0.0};
    }
    for (int e = w; e < 12; e += 4) {
        // blocks (c, v) and their halves
        const int p = e & 1, t = e >> 1;
        const int c = t < 3 ? 0 : t < 5 ? 1 : 2, v = t < 3 ? t + 1 : t < 5 ? t - 1 : 3;
        tab[tri_off(c, v) + p * 64 + lane] =
            (v2d){-us[16 * v + r16][16 * c + 8 * p + g4], -us[16 * v + r16][16 * c + 8 * p + 4 + g4]};
    }
    __syncthreads();
    v4d x[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) x[c][q] = (16 * w + r16 == 16 * c + 4 * q + g4) ? 1.0 : 0.0;
    tri_subst(x, tab, lane);
    // X = U^{-1}: for a lower M its inverse is X^T
    const gw64 Du = (gw64)(a.lower ? a.Dt : a.D), Dl = (gw64)(a.lower ? a.D : a.Dt);
    const int64_t off = (int64_t)bx * CB * CB;
    const bool hu = (a.lower ? a.Dt : a.D) != nullptr, hl = (a.lower ? a.D : a.Dt) != nullptr;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 16 * w + r16, j = 16 * c + 4 * q + g4;
            const double v = i <= j ? x[c][q] : 0.0;
            if (hu) Du[off + i + j * CB] = v;
            if (hl) Dl[off + j + i * CB] = v;
        }
}

void inv_diag64(Exec& ex, int64_t n, const InvTriMat& a, const InvTriMat* b)
{
    auto mat = [](const InvTriMat& x) { return InvTri::Mat{x.M, x.ld, x.lower, x.unit, x.D, x.Dt}; };
    launch<InvTri>(ex, ceil_div(n, CB), b ? 2 : 1, InvTri::Args{n, {mat(a), mat(b ? *b : a)}});
}

// ---------------------------------------------------------------- FP32 (condition estimate)
// Right-looking with 64-column blocks, three launches per block column:
//   diagonal block: its factor L_JJ and the inverse L_JJ^{-1} by one
//     work-group (PotrfInv; the inverse serves the panel below and the
//     triangular solves);
//   panel below it: X := X L_JJ^{-T} (MFMA GEMM with the inverse);
//   trailing lower triangle: C -= X X^T (MFMA GEMM on lower tiles).
// (FP32 arithmetic throughout: the estimate's breakdown, which picks the
// precision, is FP32's.)
// Diagonal block with its inverse, by one work-group of 256 threads.  The
// w x w block (padded to 64 x 64 with the identity) is held in LDS and
// factored in four steps of 16 columns (right-looking):
//   the 16 x 16 diagonal block D by one wavefront, lane i holding row i:
//     column K of L_D is formed from the pivot C(K, K) and every lane
//     updates its row with the entries L(j, K) of the other rows, read by
//     readlane (no LDS round trip per column); the same wavefront then
//     forms L_D^{-1}, lane c solving L_D y = e_c by forward substitution;
//   the rows below: L21 = A21 L_D^{-T} (all threads);
//   the trailing lower triangle: A22 -= L21 L21^T (all threads).
// The inverse of the 64 x 64 factor is then assembled by block rows,
//   X_ii = L_ii^{-1},  X_ij = -X_ii sum_{k = j .. i-1} L_ik X_kj  (j < i).
// Sums run over whole blocks of 16 (the zeros of the triangles included), so
// that their LDS reads are in flight together: 44 -> 36 us.
// Outputs: L in the lower triangle of the block in C (zeros above), X in
// Dinv (64 x 64, column-major; the identity on padding).
constexpr int PD_LD = CB + 1;   // LDS leading dimension of the block

struct PotrfInvArgs {
    int w;
    void* C;          // diagonal block, ld ldc (lower triangle in, L out)
    int64_t ldc;
    int32_t* info;
    int64_t c0;       // global index of the block's first column
    void* Dinv;       // 64 x 64 inverse out
};
struct PotrfInv {
    typedef float T;
    typedef PotrfInvArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const PotrfInvArgs& p, int, int);
};
__device__ void PotrfInv::run(const PotrfInvArgs& p, int, int)
{
    __shared__ T L[CB * PD_LD];   // L[r + c * PD_LD]
    __shared__ T X[CB * PD_LD];   // inverse
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int w = p.w;
    const int64_t ldc = p.ldc;
    T* __restrict__ C = (T*)p.C;
    for (int e = tid; e < CB * CB; e += NTH) {
        const int r = e % CB, c = e / CB;
        T v = (T)0;
        if (r < w && c < w) v = (r >= c) ? C[r + c * ldc] : (T)0;
        else if (r == c) v = (T)1;
        L[r + c * PD_LD] = v;
    }
    __syncthreads();
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int o = 16 * kb;
        if (wid == 0) {
            T a[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) a[j] = (lane < 16 && j <= lane) ? L[(o + lane) + (o + j) * PD_LD] : (T)0;
#pragma unroll
            for (int K = 0; K < 16; ++K) {
                const T d = lane_value(a[K], K);
                const bool bad = !(d > (T)0) || !isfinite(d);
                if (bad && lane == 0 && o + K < w && *p.info == 0) *p.info = 2000 + (int32_t)(p.c0 + o + K) + 1;
                const T lkk = bad ? (T)NAN : (T)sqrt(d);
                const T rl = (T)1 / lkk;
                const T l = (lane > K) ? a[K] * rl : (lane == K ? lkk : (T)0);
                a[K] = l;
#pragma unroll
                for (int j = K + 1; j < 16; ++j) a[j] -= l * lane_value(l, j);
            }
            if (lane < 16) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (j <= lane) L[(o + lane) + (o + j) * PD_LD] = a[j];
            }
            // (the wavefront's own LDS writes are visible to its later reads)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // column `lane` of L_D^{-1}: y_r = (delta_{r, lane} - sum_{k<r}
            // L(r, k) y_k) / L(r, r), the entries of L_D read as LDS broadcasts
            T y[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                T s = (lane == r) ? (T)1 : (T)0;
#pragma unroll
                for (int k = 0; k < r; ++k) s -= L[(o + r) + (o + k) * PD_LD] * y[k];
                y[r] = s / L[(o + r) + (o + r) * PD_LD];
            }
            if (lane < 16) {
#pragma unroll
                for (int r = 0; r < 16; ++r) X[(o + r) + (o + lane) * PD_LD] = y[r];
            }
        }
        __syncthreads();
        const int nr = CB - o - 16;   // rows below the diagonal block
        if (nr > 0) {
            // L21 = A21 L_D^{-T}: element (r, c) = sum_{k <= c} A21(r, k) L_D^{-1}(c, k)
            T res[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int e = tid + NTH * t;
                T s = (T)0;
                if (e < nr * 16) {
                    const int r = o + 16 + e % nr, c = e / nr;
#pragma unroll
                    for (int k = 0; k < 16; ++k) s += L[r + (o + k) * PD_LD] * X[(o + c) + (o + k) * PD_LD];
                }
                res[t] = s;
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int e = tid + NTH * t;
                if (e < nr * 16) L[(o + 16 + e % nr) + (o + e / nr) * PD_LD] = res[t];
            }
            __syncthreads();
            // A22 -= L21 L21^T on the lower triangle
            for (int e = tid; e < nr * nr; e += NTH) {
                const int rr = e % nr, cc = e / nr;
                if (rr < cc) continue;
                T s = (T)0;
#pragma unroll
                for (int k = 0; k < 16; ++k) s += L[(o + 16 + rr) + (o + k) * PD_LD] * L[(o + 16 + cc) + (o + k) * PD_LD];
                L[(o + 16 + rr) + (o + 16 + cc) * PD_LD] -= s;
            }
            __syncthreads();
        }
    }
    // inverse by block rows
#pragma unroll 1
    for (int i = 1; i < 4; ++i) {
        const int cnt = 16 * 16 * i;   // block row i, columns 0 .. 16 i - 1
        T res[3];
        // S(r, col) = sum_{q = col .. 16 i - 1} L(16 i + r, q) X(q, col)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = tid + NTH * t;
            T s = (T)0;
            if (e < cnt) {
                const int r = e % 16, col = e / 16;
                for (int q0 = col & ~15; q0 < 16 * i; q0 += 16)
#pragma unroll
                    for (int q = 0; q < 16; ++q) s += L[(16 * i + r) + (q0 + q) * PD_LD] * X[q0 + q + col * PD_LD];
            }
            res[t] = s;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = tid + NTH * t;
            if (e < cnt) X[(16 * i + e % 16) + (e / 16) * PD_LD] = res[t];
        }
        __syncthreads();
        // X_ij = -X_ii S: element (r, col) = -sum_{u <= r} X(16 i + r, 16 i + u) S(u, col)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = tid + NTH * t;
            T s = (T)0;
            if (e < cnt) {
                const int r = e % 16, col = e / 16;
#pragma unroll
                for (int u = 0; u < 16; ++u) s += X[(16 * i + r) + (16 * i + u) * PD_LD] * X[(16 * i + u) + col * PD_LD];
            }
            res[t] = -s;
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int e = tid + NTH * t;
            if (e < cnt) X[(16 * i + e % 16) + (e / 16) * PD_LD] = res[t];
        }
        __syncthreads();
    }
    T* __restrict__ Dv = (T*)p.Dinv;
    for (int e = tid; e < CB * CB; e += NTH) {
        const int r = e % CB, c = e / CB;
        if (r < w && c < w) C[r + c * ldc] = (r >= c) ? L[r + c * PD_LD] : (T)0;
        Dv[r + c * CB] = (r >= c) ? X[r + c * PD_LD] : (T)0;
    }
}

void cholesky_f32(Exec& ex, int64_t n, float* C, int64_t ldc, int32_t* info, float* Dinv)
{
    typedef float T;
    for (int64_t c0 = 0; c0 < n; c0 += CB) {
        ex.iter((uint32_t)(c0 / CB));
        const int w = (int)((n - c0 < CB) ? n - c0 : CB);
        T* D = C + c0 + c0 * ldc;
        T* Db = Dinv + (c0 / CB) * CB * CB;
        launch<PotrfInv>(ex, 1, 1, PotrfInvArgs{w, D, ldc, info, c0, Db});
        const int64_t rem = n - c0 - w;
        if (rem <= 0) break;
        // X := X L_JJ^{-T}: in place (each work-group reads all of its rows
        // before it writes them)
        T* X = C + (c0 + w) + c0 * ldc;
        GemmArgs p{};
        p.M = rem; p.N = w; p.K = w;
        p.A = X; p.lda = ldc; p.transA = 0;
        p.B = Db; p.ldb = CB; p.transB = 1;
        p.alpha = 1.0; p.beta = 0.0;
        p.C = X; p.ldc = ldc;
        p.splits = 1;
        gemm_f32(ex, p);
        T* C22 = C + (c0 + w) + (c0 + w) * ldc;
        GemmArgs g{};
        g.M = rem; g.N = rem; g.K = w;
        g.A = X; g.lda = ldc; g.transA = 0;
        g.B = X; g.ldb = ldc; g.transB = 1;
        g.alpha = -1.0; g.beta = 1.0;
        g.Cin = C22; g.ldcin = ldc; g.C = C22; g.ldc = ldc;
        g.lower = 1; g.splits = 1;
        gemm_f32(ex, g);
    }
}

}  // namespace pne
