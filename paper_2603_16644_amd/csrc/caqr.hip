// FP64 Householder QR (R only) of a tall matrix, for the QR solver and the
// FP64 preconditioner: communication-avoiding QR (Demmel, Grigori, Hoemmen,
// Langou 2012), 16 columns at a time.
//
// The rows below the panel's first row are cut into chunks of 16, and up to
// 64 consecutive chunks (1024 rows) form a block:
//   panel   every block factors its 16 columns by Householder reflectors in
//           registers, one work-group each; its R is left in its first chunk
//   apply   the block's reflectors on the trailing columns: a work-group
//           holds 1024 rows of 16 columns in registers, so the columns are
//           read once and written once
// and then the first chunks of the blocks, which hold the R factors, are the
// chunks of the next level, until one block is left, whose R is the panel's
// rows of the result.  Chunk c of a level starts c * rstride rows down.
//
// A tree of Householder QRs of whole blocks (up to 6144 x n), which this
// replaces, runs three levels one after the other, each a chain of n / 8 or
// n / 16 panels in one work-group with two passes over the rest of the block.
// Here the chain is one of n / 16 panels whatever the height.  Measured:
// 60000 x 601 24.9 -> 5.55 ms (panel 33 us, first apply 87 us on average and
// 3 TB/s at its widest, upper levels 22 us, times 38; 5.43 with V Z added to W
// product by product, at 1.8 times the error); 3000 x 1000 5.6 -> 3.3
// ms (27 + 18 + 6 us, times 63).
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {
namespace {

constexpr int CW = 16;            // panel width, chunk height
// Chunks per block: 64 on the first level, 8 above it, where a panel of
// one chunk per wavefront then takes 13 us (of 64 chunks: 32) and runs beside
// the apply of the level below.
constexpr int CBLK = 64, CBLK_TOP = 8;
constexpr int CMAXLEV = 14;       // levels (8^13 blocks of 1024 rows)

typedef double v2d8 __attribute__((ext_vector_type(2), aligned(8)));

struct CaqrArgs {
    int64_t h, rem;      // rows from the panel's first row, trailing columns
    double* W;           // the panel's first entry
    int64_t ldw;
    double* V;           // 16 x 16 reflectors per chunk (first level: of the first chunk of every block,
                         // the others are in W)
    double* Tm;          // 16 x 16 triangular factor per block
    int64_t rstride;     // rows between two chunks of the level
    int32_t nch, cb;     // chunks of the level, chunks per block
    int32_t w, wr, top;  // columns of the panel, those of them that are factored; a level above the first
};

// DPP move within every row of 16 lanes
template <int CTRL>
__device__ __forceinline__ double row_move(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int K>
__device__ __forceinline__ double row_bcast(double v) { return row_move<0x150 + K>(v); }   // value of lane K
__device__ __forceinline__ double row_next4(double v) { return row_move<0x12C>(v); }       // value of lane l + 4 (mod 16)

struct CaqrShared {
    double red[2][8][CW];    // partial dot products per wavefront (two steps alternate)
    double rowk[2][CW];      // row k of the panel
    double G[CW][CW + 1];    // G[k][l] = V(:, l)^T v_k for l < k
    double tau[CW];
};

// Column k = 4 it + J of a block.  Lane (g, l) of a wavefront holds rows 4 g
// .. 4 g + 3 of column c = (l + 4 it) mod 16 of each of its chunks (the
// columns move on by four lanes after every four steps, so that the column at
// hand is in lane J).  The dot products of column k with all 16 columns are
// then one FMA per entry (the entry of column k comes from lane J of the row
// of lanes by DPP) and one value per lane is left to add up over 4 lanes and
// 8 wavefronts: one barrier per column.  LAPACK convention: beta =
// -sign(alpha) ||x||, tau = (beta - alpha) / beta, v = [1; x(r > k) / (alpha -
// beta)].  Column k is left unscaled; ivc is the scale of the lane's own
// column.
template <int J, int Q>
__device__ __forceinline__ void caqr_step(int it, int wv, int g, int c, int wr, double (&x)[Q][4], double& ivc,
                                          CaqrShared& sh)
{
    const int k = 4 * it + J;
    const bool w0 = wv == 0, owner = w0 && g == it;   // (owner: holds row k, as x[0][J])
    double xb[Q][4];   // column k below row k
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            double v = row_bcast<J>(x[q][t]);
            if (q == 0) v = (w0 && 4 * g + t <= k) ? 0.0 : v;
            xb[q][t] = v;
            if (t & 1) s1 += v * x[q][t];
            else s0 += v * x[q][t];
        }
    double s = s0 + s1;
    {
        double a = s, b = s;
        lane_swap<32>(a, b);
        s = a + b;
    }
    {
        double a = s, b = s;
        lane_swap<16>(a, b);
        s = a + b;
    }
    if (g == 0) sh.red[J & 1][wv][c] = s;
    if (owner) sh.rowk[J & 1][c] = x[0][J];
    __syncthreads();
    s = sh.red[J & 1][2 * g][c] + sh.red[J & 1][2 * g + 1][c];
    const double rk = sh.rowk[J & 1][c];
    {
        double a = s, b = s;
        lane_swap<32>(a, b);
        s = a + b;
    }
    {
        double a = s, b = s;
        lane_swap<16>(a, b);
        s = a + b;
    }
    const double alpha = row_bcast<J>(rk), sigma = row_bcast<J>(s);
    // with y = 1 / ||x||: tau = 1 + |alpha| y, 1 / (alpha - beta) =
    // sign(alpha) y / tau.  Reciprocal and reciprocal root by Newton steps
    // from the hardware's approximation (to about one unit in the last
    // place); outside the range where they stay normal, the divisions.
    const double nn = alpha * alpha + sigma;
    double beta, tau, inv;
    if (nn > 0x1p-960 && nn < 0x1p1000) {
        double y = __builtin_amdgcn_rsq(nn);
        double e = fma(-(nn * y), y, 1.0);
        y = fma(y * e, fma(0.375, e, 0.5), y);
        e = fma(-(nn * y), y, 1.0);
        y = fma(y * e, 0.5, y);
        double nrm = nn * y;
        nrm = fma(fma(-nrm, nrm, nn), 0.5 * y, nrm);
        tau = fma(fabs(alpha), y, 1.0);
        double r = __builtin_amdgcn_rcp(tau);
        r = fma(r, fma(-tau, r, 1.0), r);
        r = fma(r, fma(-tau, r, 1.0), r);
        beta = alpha >= 0.0 ? -nrm : nrm;
        inv = alpha >= 0.0 ? y * r : -(y * r);
    } else {
        const double nrm = sqrt(nn);
        beta = alpha >= 0.0 ? -nrm : nrm;
        tau = (beta - alpha) / beta;
        inv = 1.0 / (alpha - beta);
    }
    if (sigma == 0.0 || k >= wr) {
        beta = alpha; tau = 0.0; inv = 0.0;
    }
    const double dot = rk + s * inv;                // v^T x(:, c); for c < k without V's scale
    const double f = c > k ? tau * dot : 0.0;
    const double fi = f * inv;
    // (not c <= k with f = 0: a column k that is not finite would spread to the
    // finite ones before it)
    if (c > k)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) x[q][t] -= fi * xb[q][t];
    if (owner) x[0][J] = c == k ? beta : x[0][J] - f;
    if (w0 && g == 0) {
        if (c < k) sh.G[k][c] = ivc * dot;
        if (c == k) sh.tau[k] = tau;
    }
    if (c == k) ivc = inv;
}

// One block of a panel, at most 8 Q chunks, by 512 threads with 4 Q rows per
// lane.  Bound by the chain of a column: dot products, barrier, reciprocal
// root.
template <int Q>
__device__ __forceinline__ void caqr_panel(const CaqrArgs& a, int bx)
{
    __shared__ CaqrShared sh;
    const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b0 = bx * a.cb;
    const int nc = a.nch - b0 < a.cb ? a.nch - b0 : a.cb;
    const int64_t h = a.h, ldw = a.ldw;
    const int w = a.w;
    double* __restrict__ Wc = a.W + (c < w ? c : w - 1) * ldw;
    if (threadIdx.x < CW) sh.tau[threadIdx.x] = 0.0;
    double x[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int ch = wv + 8 * q;
        const int64_t row0 = (int64_t)(b0 + (ch < nc ? ch : 0)) * a.rstride + 4 * g;
#pragma unroll
        for (int t = 0; t < 4; ++t) x[q][t] = Wc[row0 + t < h ? row0 + t : h - 1];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (ch >= nc || row0 + t >= h || c >= w || (a.top && 4 * g + t > c)) x[q][t] = 0.0;
    }
    double ivc = 0.0;
    __syncthreads();
    // the loop stays rolled: sixteen steps in line are 30 to 60 KB of
    // code that every launch fetches anew
    int col = c;
#pragma unroll 1
    for (int it = 0; it < 4; ++it) {
        // (columns past w are zero, and so are their reflectors)
        caqr_step<0, Q>(it, wv, g, col, a.wr, x, ivc, sh);
        caqr_step<1, Q>(it, wv, g, col, a.wr, x, ivc, sh);
        caqr_step<2, Q>(it, wv, g, col, a.wr, x, ivc, sh);
        caqr_step<3, Q>(it, wv, g, col, a.wr, x, ivc, sh);
        col = (col + 4) & 15;
        ivc = row_next4(ivc);
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) x[q][t] = row_next4(x[q][t]);
    }
    __syncthreads();
    // T(i, k) = -tau_k sum_{l = i .. k-1} T(i, l) (V^T v_k)_l for i < k,
    // T(k, k) = tau_k: thread i builds row i
    if (threadIdx.x < CW) {
        const int i = threadIdx.x;
        double tr[CW];
#pragma unroll
        for (int k = 0; k < CW; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < k; ++l)
                if (l >= i) acc += tr[l] * sh.G[k][l];
            const double tau = sh.tau[k];
            tr[k] = i == k ? tau : (i < k ? -tau * acc : 0.0);
        }
        double* Tm = a.Tm + (int64_t)bx * (CW * CW);
#pragma unroll
        for (int k = 0; k < CW; ++k) Tm[i + k * CW] = tr[k];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int ch = wv + 8 * q;
        if (ch >= nc) continue;
        const int64_t row0 = (int64_t)(b0 + ch) * a.rstride + 4 * g;
        double* __restrict__ Vc = a.V + (int64_t)(a.top ? b0 + ch : bx) * (CW * CW) + c * CW + 4 * g;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int r = 4 * g + t;
            const bool up = ch == 0 && r <= c;       // R
            const double v = x[q][t] * ivc;
            if (row0 + t < h && c < w && (up || !a.top)) Wc[row0 + t] = up ? x[q][t] : v;
            if (a.top || ch == 0) Vc[t] = up ? (r == c ? 1.0 : 0.0) : v;
        }
    }
}

template <int Q>
struct CaqrPanel {
    typedef CaqrArgs Args;
    static constexpr int NTH = 512, WPE = 2;
    static __device__ __forceinline__ void run(const Args& a, int bx, int) { caqr_panel<Q>(a, bx); }
};

// The reflectors of a block on 16 trailing columns: Y = V^T W, Z = T^T Y,
// W -= V Z, all on the matrix cores, with the block's rows of W (at most
// 8 Q chunks) in the registers of eight wavefronts between the two products.
// Lane (g, c) loads rows 2 g, 2 g + 1, 2 g + 8, 2 g + 9 of column c of a chunk
// (64 bytes side by side per load): register t is then operand of K value g
// of product t, and also entry (g + 4 t, c) of an accumulator whose row i
// stands for the row of register i / 4 of lane group i % 4, so the update adds
// to W where it was loaded.  Bound by
// memory: the trailing columns once in and once out, V from L2.
// The first npan work-groups factor the next level's panel, which needs the R
// factors of this one only.
struct CaqrApplyArgs {
    CaqrArgs a, next;
    int32_t npan;        // blocks of the next level's panel (0: this is the last)
};
template <int Q>
struct CaqrApply {
    typedef CaqrApplyArgs Args;
    static constexpr int NTH = 512, WPE = 4;
    static __device__ __forceinline__ void body(const CaqrArgs& a, int b, int64_t j0, int nc)
    {
        __shared__ v4d ys[8][64];
        const int lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
        const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int64_t h = a.h, ldw = a.ldw;
        const bool top = a.top != 0;
        const int64_t j = j0 + c < a.rem ? j0 + c : a.rem - 1;
        double* __restrict__ Wj = a.W + (CW + j) * ldw + 2 * g;
        // Chunk of register set q; the sets are filled from the back, so that
        // a chunk that reaches past the last row is the last set of wavefront
        // 7.  Below zero: none (taken as zero; chunk 0 of the level is full,
        // as there are trailing columns).
        const int b0 = b * a.cb, ch0 = nc - 8 * Q + wv;
        auto chunk = [&](int q) { return (int64_t)(ch0 + 8 * q < 0 ? 0 : b0 + ch0 + 8 * q); };
        // rows of the last set that exist
        const int64_t lim = h - chunk(Q - 1) * a.rstride;
        auto rt = [&](int t) { return 2 * g + (t & 1) + 8 * (t >> 1); };   // row of the chunk in register t
        v4d x[Q];
#pragma unroll
        for (int q = 0; q < Q - 1; ++q) {
            const double* __restrict__ p = Wj + chunk(q) * a.rstride;
            const v2d8 lo = *(const v2d8*)p, hi = *(const v2d8*)(p + 8);
            x[q] = (v4d){lo[0], lo[1], hi[0], hi[1]};
            if (ch0 + 8 * q < 0) x[q] = (v4d){0, 0, 0, 0};
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) x[Q - 1][t] = Wj[chunk(Q - 1) * a.rstride + (rt(t) < lim ? rt(t) : lim - 1) - 2 * g];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (rt(t) >= lim || ch0 + 8 * (Q - 1) < 0) x[Q - 1][t] = 0.0;
        // V of set q: its first entry and leading dimension (on the first
        // level from W, but for the block's first chunk, which holds R there)
        // (selected by masks: branches would split the loads)
        auto vptr = [&](int q, int64_t& ldv) -> const double* {
            const int64_t inw = -(int64_t)(!top && ch0 + 8 * q > 0), tp = -(int64_t)top;
            const int64_t c8 = chunk(q);
            ldv = CW + ((ldw - CW) & inw);
            const uint64_t pw = (uint64_t)(a.W + c8 * a.rstride), pv = (uint64_t)(a.V + (b + ((c8 - b) & tp)) * (CW * CW));
            return (const double*)(pv + ((pw - pv) & (uint64_t)inw));
        };
        v4d y0 = (v4d){0, 0, 0, 0}, y1 = y0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int64_t ldv;
            const double* __restrict__ p = vptr(q, ldv);
            p += c * ldv + 2 * g;
            v4d v;
            if (q < Q - 1) {
                const v2d8 lo = *(const v2d8*)p, hi = *(const v2d8*)(p + 8);
                v = (v4d){lo[0], lo[1], hi[0], hi[1]};
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) v[t] = p[(rt(t) < lim ? rt(t) : lim - 1) - 2 * g];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (rt(t) >= lim) v[t] = 0.0;
            }
            y0 = __builtin_amdgcn_mfma_f64_16x16x4f64(v[0], x[q][0], y0, 0, 0, 0);
            y1 = __builtin_amdgcn_mfma_f64_16x16x4f64(v[1], x[q][1], y1, 0, 0, 0);
            y0 = __builtin_amdgcn_mfma_f64_16x16x4f64(v[2], x[q][2], y0, 0, 0, 0);
            y1 = __builtin_amdgcn_mfma_f64_16x16x4f64(v[3], x[q][3], y1, 0, 0, 0);
            if (q & 1) __builtin_amdgcn_sched_barrier(0);   // (V of two sets at a time: 128 registers)
        }
        const double* __restrict__ Tm = a.Tm + (int64_t)b * (CW * CW);
        double tk[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) tk[q] = -Tm[(4 * q + g) + c * CW];
        ys[wv][lane] = y0 + y1;
        __syncthreads();
        const v4d y = ((ys[0][lane] + ys[1][lane]) + (ys[2][lane] + ys[3][lane])) +
                      ((ys[4][lane] + ys[5][lane]) + (ys[6][lane] + ys[7][lane]));
        v4d z = (v4d){0, 0, 0, 0};   // -T^T Y
#pragma unroll
        for (int q = 0; q < 4; ++q) z = __builtin_amdgcn_mfma_f64_16x16x4f64(tk[q], y[q], z, 0, 0, 0);
        const int rp = 2 * (c & 3) + ((c >> 2) & 1) + 8 * (c >> 3);   // row of the chunk that accumulator row c stands for
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int64_t ldv;
            const double* __restrict__ p = vptr(q, ldv);
            p += g * ldv + (q < Q - 1 || rp < lim ? rp : lim - 1);
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = p[4 * k * ldv];
            // (V Z summed by itself: added to W product by product it would be
            // rounded to W's last place sixteen times instead of once)
            v4d vz = (v4d){0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < 4; ++k) vz = __builtin_amdgcn_mfma_f64_16x16x4f64(v[k], z[k], vz, 0, 0, 0);
            x[q] += vz;
            // (added here: moved down to the stores, as the compiler has it,
            // the sums keep both their terms in registers)
            asm volatile("" : "+v"(x[q]));
        }
        if (j0 + c >= a.rem) return;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (ch0 + 8 * q < 0) continue;
            double* __restrict__ p = Wj + chunk(q) * a.rstride;
            if (q < Q - 1) {
                *(v2d8*)p = (v2d8){x[q][0], x[q][1]};
                *(v2d8*)(p + 8) = (v2d8){x[q][2], x[q][3]};
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (rt(t) < lim) p[rt(t) - 2 * g] = x[q][t];
            }
        }
    }
    static __device__ __forceinline__ void run(const Args& p, int bx, int)
    {
        if (bx < p.npan) {
            caqr_panel<1>(p.next, bx);
            return;
        }
        bx -= p.npan;
        const CaqrArgs& a = p.a;
        // the tiles of a block on one XCD (work-groups go to the eight in
        // turn), whose L2 then holds the block's V (128 KB)
        const int tiles = (int)((a.rem + CW - 1) / CW);
        const int nblk = (a.nch + a.cb - 1) / a.cb;
        int b, tile;
        if (nblk >= 8) {
            const int slot = bx >> 3;
            b = (slot / tiles) * 8 + (bx & 7);
            tile = slot % tiles;
        } else {
            b = bx / tiles;
            tile = bx % tiles;
        }
        b = __builtin_amdgcn_readfirstlane(b);
        if (b >= nblk) return;
        const int nc = a.nch - b * a.cb < a.cb ? a.nch - b * a.cb : a.cb;
        body(a, b, (int64_t)tile * CW, nc);
    }
};

struct CaqrLevel {
    int64_t rstride;
    int64_t nch, cb, nblk;
};
int caqr_levels(int64_t h, CaqrLevel* lv)
{
    int n = 0;
    int64_t nch = ceil_div(h, CW), rs = CW;
    do {
        const int64_t cb = ceil_div(nch, ceil_div(nch, n == 0 ? CBLK : CBLK_TOP));
        const int64_t nblk = ceil_div(nch, cb);
        lv[n++] = CaqrLevel{rs, nch, cb, nblk};
        rs *= cb;
        nch = nblk;
    } while (nch > 1 && n < CMAXLEV);
    return n;
}

// 16 x 16 matrices of the workspace: T of every block, V of every block on
// the first level and of every chunk above it (bounds that grow with s, so
// they serve every panel)
int64_t caqr_mats(int64_t s)
{
    int64_t nch = ceil_div(ceil_div(s, CW), CBLK), mats = 2 * nch;
    while (nch > 1) {
        mats += nch;
        nch = ceil_div(nch, CBLK_TOP);
        mats += nch;
    }
    return mats;
}

}  // namespace

size_t caqr_workspace_bytes(int64_t s) { return (size_t)caqr_mats(s) * CW * CW * sizeof(double); }

// R of the s x n matrix W (s >= n), in place: its upper triangle is R, the
// rest is overwritten.  Only the first nr columns (n or n - 1) are factored: of a
// right-hand side in column n - 1 rows 0 .. n - 2 of the result are wanted, and
// its norm may overflow where they do not.
void caqr_factor(Exec& ex, int64_t s, int64_t n, int64_t nr, double* W, int64_t ldw, double* work)
{
    for (int64_t c0 = 0; c0 < nr; c0 += CW) {
        ex.iter((uint32_t)(c0 / CW));
        const int w = (int)(n - c0 < CW ? n - c0 : CW), wr = (int)(nr - c0 < CW ? nr - c0 : CW);
        CaqrLevel lv[CMAXLEV];
        const int nl = caqr_levels(s - c0, lv);
        CaqrArgs a[CMAXLEV];
        double* mem = work;
        for (int l = 0; l < nl; ++l) {
            const bool top = l > 0;
            double* Tm = mem;
            mem += lv[l].nblk * (CW * CW);
            a[l] = CaqrArgs{s - c0, n - c0 - w, W + c0 + c0 * ldw, ldw, mem, Tm, lv[l].rstride,
                            (int32_t)lv[l].nch, (int32_t)lv[l].cb, w, wr, top};
            mem += (top ? lv[l].nch : lv[l].nblk) * (CW * CW);
        }
        if (a[0].cb <= 8) launch<CaqrPanel<1>>(ex, lv[0].nblk, 1, a[0]);
        else launch<CaqrPanel<8>>(ex, lv[0].nblk, 1, a[0]);
        for (int l = 0; l < nl; ++l) {
            const bool last = l + 1 == nl;
            const CaqrApplyArgs p{a[l], a[last ? l : l + 1], last ? 0 : (int32_t)lv[l + 1].nblk};
            const int64_t nb = lv[l].nblk < 8 ? lv[l].nblk : ceil_div(lv[l].nblk, 8) * 8;
            const int64_t gx = nb * ceil_div(a[l].rem, CW);   // (none for the last columns)
            if (a[l].cb <= 8) launch<CaqrApply<1>>(ex, gx + p.npan, 1, p);
            else launch<CaqrApply<8>>(ex, gx + p.npan, 1, p);
        }
    }
}

}  // namespace pne
