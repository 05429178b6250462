// Kernels of A R^{-1} (trsm.hip, sketch_factor.hip).
#pragma once
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {

namespace {

constexpr int TB16 = 16;                 // columns per block
constexpr int PANEL = 8;                 // blocks per panel (at most)
constexpr int BLK = 256;                 // doubles of a packed 16 x 16 block
constexpr int DTAB = 512;                // doubles of a diagonal table

typedef double v2d __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) double* gp64;
typedef __attribute__((address_space(1))) double* gw64;
typedef const __attribute__((address_space(1))) char* gpc;
typedef __attribute__((address_space(1))) char* gwc;
typedef int v4i __attribute__((ext_vector_type(4)));

__host__ __device__ inline int64_t pack_block(int64_t nblk, int64_t kb, int64_t jb)
{
    return kb * nblk - kb * (kb - 1) / 2 + (jb - kb);
}

}  // namespace

// Packed R: block (kb, jb), jb >= kb, at pack_block(..) * BLK:
//   [p][lane][h] = -R(16 kb + 4 (2 p + h) + g, 16 jb + r)
// (K step 2 p + h, h = 0, 1: 16 bytes per lane); then the table of every
// diagonal block, [q][lane][2]: the operand of group q's inverse, entry
// (k = g, column r) of the 4 x 4 inverse in the rows 4 q .. 4 q + 3 of the
// result and 0 elsewhere, and the operand of its update,
// -R(16 b + 4 q + g, 16 b + r) for r >= 4 q + 4 and 0 elsewhere.  Rows and
// columns past n act as the identity.
struct TrsmPack {
    struct Args {
        int64_t n;
        const double* R;
        int64_t ldr;
        double* out;
    };
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const Args& a, int bx, int by)
    {
        const int64_t n = a.n, nblk = (n + TB16 - 1) / TB16;
        const int64_t kb = by, jb = kb + bx;
        if (jb >= nblk) return;
        const gp64 R = (gp64)a.R;
        const gw64 out = (gw64)a.out;
        auto rel = [&](int64_t i, int64_t j) -> double {
            return (i < n && j < n) ? R[i + j * a.ldr] : (i == j ? 1.0 : 0.0);
        };
        const int t = threadIdx.x;
        {
            const int h = t & 1, lane = (t >> 1) & 63, p = t >> 7;
            const int64_t i = TB16 * kb + 4 * (2 * p + h) + (lane >> 4), j = TB16 * jb + (lane & 15);
            out[pack_block(nblk, kb, jb) * BLK + t] = -rel(i, j);
        }
        if (jb != kb) return;
        const gw64 tab = out + nblk * (nblk + 1) / 2 * BLK + kb * DTAB;
        const int lane = t & 63, q = t >> 6, r = lane & 15, g = lane >> 4;
        const int64_t b0 = TB16 * kb + 4 * q;
        double inv = 0.0;
        const int c = r - 4 * q;
        if (c >= 0 && c < 4 && g <= c) {
            // column c of the inverse by back substitution, entry g
            double y[4];
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                double s = k == c ? 1.0 : 0.0;
#pragma unroll
                for (int l = k + 1; l < 4; ++l)
                    if (l <= c) s -= rel(b0 + k, b0 + l) * y[l];
                y[k] = k <= c ? s / rel(b0 + k, b0 + k) : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k == g) inv = y[k];
        }
        tab[t * 2] = inv;
        tab[t * 2 + 1] = r >= 4 * q + 4 ? -rel(b0 + g, TB16 * kb + r) : 0.0;
    }
};

struct TrsmArgs {
    int64_t m, n;
    const double* A;
    int64_t lda;
    const double* pack;
    double* X;         // 16-byte aligned, ldx even
    int64_t ldx;
};
// WIDE: leading dimensions of 2^26 or more (64-bit lane offsets)
template <bool WIDE>
struct TrsmRows {
    typedef TrsmArgs Args;
    static constexpr int NTH = 256, WPE = 3;
    static __device__ __forceinline__ void run(const TrsmArgs& a, int bx, int) { rows(a, bx, threadIdx.x); }
    static __device__ void rows(const TrsmArgs& a, int bx, int tid);   // (tid: the thread's index)
};

template <bool WIDE>
__device__ __forceinline__ void TrsmRows<WIDE>::rows(const TrsmArgs& a, int bx, int tid)
{
    __shared__ __attribute__((aligned(16))) v2d sr[2][PANEL * BLK / 2];
    __shared__ __attribute__((aligned(16))) v2d sd[2][DTAB / 2];
    const int lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
    const int w = tid >> 6;
    const int64_t m = a.m, n = a.n;
    const int nblk = (int)((n + TB16 - 1) / TB16);
    // uniform first row of the work-group and the lane's row below it (rows
    // past the matrix read its last row and are not stored)
    const int64_t i0 = (int64_t)bx * 64;
    const int row = w * 16 + r16;
    const bool in = i0 + row < m;
    const int ic = in ? row : (int)(m - 1 - i0);
    typedef typename std::conditional<WIDE, uint64_t, uint32_t>::type off_t;
    const off_t oi = (off_t)(ic * 8), lda8 = (off_t)(a.lda * 8), ldx8 = (off_t)(a.ldx * 8);
    const off_t ox = oi + g4 * ldx8;
    const gpc Ab = (gpc)((gp64)a.A + i0);
    const gwc Xb = (gwc)((gw64)a.X + i0);
    // X(row, 4 j4 + g)
    auto xat = [&](int64_t j4) { return (gw64)(Xb + j4 * (a.ldx * 32) + ox); };
    const gpc pk = (gpc)(gp64)a.pack;
    const gpc tabs = pk + (int64_t)nblk * (nblk + 1) / 2 * (BLK * 8);
    // panels of equal width (in a scalar register, like everything the buffer
    // descriptors below are made from)
    const int np = (nblk + PANEL - 1) / PANEL, pw = __builtin_amdgcn_readfirstlane((nblk + np - 1) / np);

    // strip of the work: panel (first block lp0, lnb blocks) and block row lkb
    // of R; strips lkb < lp0 come before the panel's own
    int lp0 = 0, lkb = 0;                // strip that is loaded next
    int lnb = pw < nblk ? pw : nblk;
    v4i vs[PANEL / 2], vd;               // a strip: up to 16 blocks of 128 16-byte entries, a diagonal table
    const int vo = tid * 16;
    // (buffer loads: the range check puts zeros past the strip's end without
    // a branch, so the loads stay in flight across the multiplications)
    auto fetch = [&]() {
        const bool live = lp0 < nblk;
        const int j0 = lkb < lp0 ? lp0 : lkb;   // (own strips start at the diagonal)
        const int first = __builtin_amdgcn_readfirstlane(live ? (int)pack_block(nblk, lkb, j0) : 0);
        const int bytes = __builtin_amdgcn_readfirstlane(live ? (lp0 + lnb - j0) * (BLK * 8) : 0);
        const gpc src = pk + (int64_t)first * (BLK * 8);
        const auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)src, 0, bytes, 0x00027000);
#pragma unroll
        for (int q = 0; q < PANEL / 2; ++q)
            vs[q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rs, vo + 4096 * q, 0, 0));
        const int dk = __builtin_amdgcn_readfirstlane(live ? lkb : 0);
        const gpc dsrc = tabs + (int64_t)dk * (DTAB * 8);
        const auto rd = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)dsrc, 0, DTAB * 8, 0x00027000);
        vd = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rd, vo, 0, 0));
    };
    auto advance = [&]() {
        if (++lkb == lp0 + lnb) {
            lp0 += lnb;
            lnb = nblk - lp0 < pw ? nblk - lp0 : pw;
            lkb = 0;
        }
    };
    int buf = 0;
    auto put = [&](int b) {
#pragma unroll
        for (int q = 0; q < PANEL / 2; ++q) sr[b][tid + 256 * q] = __builtin_bit_cast(v2d, vs[q]);
        sd[b][tid] = __builtin_bit_cast(v2d, vd);
    };
    // begin of a strip: its data is in LDS buffer `buf` after the barrier;
    // the next strip goes into the other one and the one after it is loaded
    auto turn = [&]() {
        __syncthreads();
        put(buf ^ 1);
        advance();
        fetch();
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch();
    put(0);
    advance();
    fetch();

    v4d acc[PANEL];
    for (int p0 = 0; p0 < nblk;) {
        const int nb = nblk - p0 < pw ? nblk - p0 : pw;
        // columns of A
#pragma unroll
        for (int c = 0; c < PANEL; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (columns past n read the last one and are not stored)
                const int64_t j = (int64_t)TB16 * (p0 + c) + 4 * q, jl = n - 1 - j;
                acc[c][q] = jl >= 0 ? *(gp64)(Ab + j * (a.lda * 8) + ((g4 < jl ? g4 : (int)jl) * lda8 + oi)) : 0.0;
            }
        // blocks C0 .. C1 - 1 of the panel minus X times a strip that starts at
        // block C0; the operands of the next block read
        // from LDS while one multiplies
        auto strip_mult = [&](const v2d* s, auto& x, auto c0c, auto c1c) {
            constexpr int C0 = decltype(c0c)::value, C1 = decltype(c1c)::value;
            v2d f[2][2];
#pragma unroll
            for (int e = 0; e < 2; ++e) f[0][e] = s[e * 64 + lane];
#pragma unroll
            for (int c = C0; c < C1; ++c) {
                const int b = (c - C0) & 1;
                if (c + 1 < C1)
#pragma unroll
                    for (int e = 0; e < 2; ++e) f[b ^ 1][e] = s[((c + 1 - C0) * 2 + e) * 64 + lane];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[b][p][h], x[2 * p + h], acc[c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // products with the earlier panels (with two panels or more each has
        // more than four blocks, but for the last)
        if (p0 > 0) {
            double xn[4], xc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) xn[q] = *xat(q);
            for (int kb = 0; kb < p0; ++kb) {
#pragma unroll
                for (int q = 0; q < 4; ++q) xc[q] = xn[q];
                const int kn = kb + 1 < p0 ? kb + 1 : kb;
#pragma unroll
                for (int q = 0; q < 4; ++q) xn[q] = *xat(4 * kn + q);
                turn();
                strip_mult(sr[buf], xc, std::integral_constant<int, 0>{}, std::integral_constant<int, PANEL>{});
                buf ^= 1;
            }
        }
        // the panel's own triangle
        auto own = [&](auto bc) {
            constexpr int B = decltype(bc)::value;
            if (B >= nb) return;
            turn();
            v4d t = acc[B];
            const v2d* d = sd[buf];
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!isfinite(t[0]) || !isfinite(t[1]) || !isfinite(t[2]) ||
                                                             !isfinite(t[3])) != 0, 0)) {
                // a non-finite entry: the zeros of the inverses must not
                // carry it into the columns left of it.  (The lane index is
                // made opaque so that nothing of this rare branch is kept in
                // registers outside it.)
                int ln = lane;
                asm volatile("" : "+v"(ln));
                const int r16 = ln & 15, g4 = ln >> 4;
#pragma unroll 1
                for (int q = 0; q < 4; ++q) {
                    const v2d f = d[q * 64 + ln];
                    const double tq = q == 0 ? t[0] : q == 1 ? t[1] : q == 2 ? t[2] : t[3];
                    double x = 0.0;
                    for (int k = 0; k < 4; ++k) {
                        const double tk = __shfl(tq, 16 * k + r16);
                        const double ik = __shfl(f[0], 16 * k + 4 * q + g4);
                        if (k <= g4) x += tk * ik;
                    }
                    const v4d u = __builtin_amdgcn_mfma_f64_16x16x4f64(f[1], x, t, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = e == q ? x : (e > q ? u[e] : t[e]);
                }
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v2d f = d[q * 64 + lane];
                    const v4d y = __builtin_amdgcn_mfma_f64_16x16x4f64(f[0], t[q], (v4d){0, 0, 0, 0}, 0, 0, 0);
                    t[q] = y[q];
                    if (q < 3) {
                        // (only the columns right of the group are taken)
                        const v4d u = __builtin_amdgcn_mfma_f64_16x16x4f64(f[1], y[q], t, 0, 0, 0);
#pragma unroll
                        for (int e = q + 1; e < 4; ++e) t[e] = u[e];
                    }
                }
            }
            acc[B] = t;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t j4 = 4 * (int64_t)(p0 + B) + q;
                if (in && 4 * j4 + g4 < n) *xat(j4) = t[q];
            }
            // the blocks right of it, up to the next multiple of four past nb
            // (the strip starts at its diagonal block, zeros past its end)
            const v2d* s = sr[buf] + BLK / 2;
            using C0 = std::integral_constant<int, B + 1>;
            if (nb > 4) strip_mult(s, t, C0{}, std::integral_constant<int, 8>{});
            else if (B < 3) strip_mult(s, t, C0{}, std::integral_constant<int, B < 3 ? 4 : B + 1>{});
            buf ^= 1;
        };
        own(std::integral_constant<int, 0>{});
        own(std::integral_constant<int, 1>{});
        own(std::integral_constant<int, 2>{});
        own(std::integral_constant<int, 3>{});
        own(std::integral_constant<int, 4>{});
        own(std::integral_constant<int, 5>{});
        own(std::integral_constant<int, 6>{});
        own(std::integral_constant<int, 7>{});
        p0 += nb;
    }
}

}  // namespace pne
