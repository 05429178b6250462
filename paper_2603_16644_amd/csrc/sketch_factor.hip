// Triangular factor of an FP32 sketch W (s x n) without the factorization of
// W: R^T R = W^T W with the Gram matrix and its Cholesky factor in FP64.
//
// The Householder QR of an s x n sketch is one panel of 8 or 16 columns after
// another, each with two barriers per column, and an update of the rest that
// reads W twice: 3.4 ms at 3000 x 1000 whatever the arithmetic.  The Gram
// matrix is one product.  R agrees with the Householder factor up to the signs
// of its rows, which cancel in A_p^T A_p, R_s x = y; where R itself is the
// result, the Householder QR runs.
//
// The products of FP32 entries are exact in FP64; what the Gram matrix and its
// factor lose is a perturbation of C = W^T W of norm up to about n 2^-53 |D|^2
// (D the columns' norms; the bound is some n^2 2^-53).  So the factor is
// taken of C + t D^2 with t = 8 n 2^-53, which no rounding makes indefinite,
// and R1 is the factor of W with each singular value (columns scaled to
// norm 1) raised by at most sqrt(t): nothing while they are well above it (1e-6
// at n = 1000).  A pivot below 256 t D^2 says that they may not be (the
// smallest pivot is 25 to 60 times the square of the smallest singular value
// for sketches of geometric spectra, n = 100 to 700).  Then W is factored once more
// where R1 has made it nearly orthogonal (Cholesky QR in two passes, Yamamoto
// et al. 2015, with the shift of Fukaya et al. 2020): X = [W; 2^-24.5 D] R1^{-1},
// in FP64, has singular values between 1 and 1 / sqrt(2^49 t) (0.03 at n =
// 1000), R2 is the factor of X^T X, and R = R2 R1 the factor of [W; 2^-24.5 D]
// to 1e-10 in every direction.  The rows 2^-24.5 D keep the directions that
// W does not have at the size that the rounding errors of an FP32 Householder
// factorization leave there: condition numbers of A R^-1 equal to or below that
// factorization's for kappa 1e4 to 1e14, for repeated columns and for sampled
// rows of a square matrix (emulated, n = 2 to 700).
//
// The second pass is part of the launch that writes R (SketchEnd), so that
// nothing is read back and solves that do not need it pay for no launch of it
// (as 3 + n / 64 launches that end at once it cost 5 us each: 2000 x 100 solves
// 212 -> 237 us, 100000 x 1000 6.11 -> 6.25 ms).
//
// Measured, 3000 x 1000: Householder QR 3.4 ms, this 0.45 ms (Gram and reduction
// 0.1, Cholesky 0.34, SketchEnd 0.014); 300 x 100 199 -> 57 us, 6000 x 2000 13.3 ->
// 1.3 ms.  The second pass adds 1.8 ms, 0.12 ms and 6.5 ms to these where it runs.
#include "chol_dev.h"
#include "common.h"
#include "convert.h"
#include "gemm_tn_dev.h"
#include "kernels.h"
#include "launch.h"
#include "trsm_dev.h"

namespace pne {

struct SketchEndArgs {
    int64_t s, n;
    const float* W;
    int64_t ldw;
    double* X;           // second pass: chunk rows of (s + n) x n at a time, ld chunk (even)
    int64_t chunk, nchunks;
    double* pack;        // packed R1
    const double* R1;    // ld n, like R2 and C
    double* R2;
    double* C;           // Gram matrix of X
    double* tab;
    double* gd;          // squared norms of the columns of W
    double t;            // shift of the Cholesky factors
    const int32_t* state;
    int32_t* work;       // next work item, items done (zero)
    double* R;
    int64_t ldr;
    int prec;
    const uint32_t* amax;
    int32_t wgs;
    int32_t* info;       // 1000 + first column whose diagonal entry is bad; 4001 where a wait gives up
};

// R = R1, or R2 R1 after a second pass (upper triangles), rounded to the
// precision of the factor (FP32, BF16, or FP16 with the input scale divided
// out), zero below, and its diagonal checked; 32 x 32 entries per tile, four per
// thread.
//
// The second pass runs where *state is 1.  Its work items are numbered in the
// order of its phases: pack R1; for every chunk of rows that X's memory holds form
// the chunk of [W; 2^-24.5 D], substitute, 64 rows an item, and add its part of the
// Gram matrix, a tile of 64 x 64 an item; the steps of the Cholesky
// factorization; tiles of R.  (The first chunk is formed while R1 is packed.)  A work-group takes the next number from a
// counter and waits until all items of the earlier phases are done.  Those
// have lower numbers, so other work-groups took them and are working on them
// or waiting for lower ones yet: whatever number of work-groups is on the
// machine, the lowest item not done is never waiting, and every wait ends.
struct SketchEnd {
    typedef SketchEndArgs Args;
    static constexpr int NTH = 256, WPE = 1;
    static constexpr int T = 32;
    static constexpr int FILL = 8;   // blocks of R1 or columns of X per item of the first phase

    static __host__ __device__ int64_t tiles(int64_t n) { return (n + T - 1) / T; }
    static __device__ __forceinline__ int64_t pack_items(int64_t n)
    {
        const int64_t nblk = (n + TB16 - 1) / TB16;
        return nblk * ((nblk + FILL - 1) / FILL);
    }
    // the thread's index, formed anew at every use: what is made of it is not
    // kept in registers across the phases
    static __device__ __forceinline__ int thread()
    {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    }
    static __device__ __forceinline__ void pack(const Args& a, int64_t e)
    {
        const int64_t n = a.n, nblk = (n + TB16 - 1) / TB16;
        const TrsmPack::Args p{n, a.R1, n, a.pack};
        for (int c = 0; c < FILL; ++c) TrsmPack::run(p, (int)(e / nblk) * FILL + c, (int)(e % nblk));
    }
    // rows r0 .. r0 + rows - 1 of [W; 2^-24.5 D]
    static __device__ __forceinline__ void fill(const Args& a, int64_t e, int64_t r0, int64_t rows)
    {
        const int64_t n = a.n, rt = (a.chunk + NTH - 1) / NTH;
        const int64_t l = e % rt * NTH + thread(), i = r0 + l, j0 = e / rt * FILL;
        if (l >= rows) return;
        for (int64_t j = j0; j < j0 + FILL && j < n; ++j)
            a.X[l + j * a.chunk] = i < a.s ? (double)a.W[i + j * a.ldw] : (i - a.s == j ? sqrt(0x1p-49 * a.gd[j]) : 0.0);
    }
    static __device__ __forceinline__ double upper(const double* M, int64_t n, int64_t r, int64_t c)
    {
        return r <= c && c < n ? M[r + c * n] : 0.0;
    }
    // (the lowest code stays, whichever comes first)
    static __device__ __forceinline__ void bad_column(int32_t* info, int32_t code)
    {
        int32_t old = __hip_atomic_load(info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while ((old == 0 || old > code) &&
               !__hip_atomic_compare_exchange_strong(info, &old, code, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT)) {}
    }
    // a tile of R2 R1
    static __device__ __forceinline__ void tile(const Args& a, int64_t e)
    {
        __shared__ double l[T][T + 1], u[T][T + 1];   // l[k][i] of R2, u[j][k] of R1
        const int64_t n = a.n, nt = tiles(n), ti = e % nt, tj = e / nt;
        const int i = thread() % T, q = thread() / T;
        double v[4] = {0, 0, 0, 0};
        for (int64_t k0 = T * ti; k0 <= T * tj; k0 += T) {
            __syncthreads();
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                l[q + 8 * x][i] = upper(a.R2, n, T * ti + i, k0 + q + 8 * x);
                u[q + 8 * x][i] = upper(a.R1, n, k0 + i, T * tj + q + 8 * x);
            }
            __syncthreads();
#pragma unroll 8
            for (int k = 0; k < T; ++k)
#pragma unroll
                for (int x = 0; x < 4; ++x) v[x] += l[k][i] * u[q + 8 * x][k];
        }
        store(a, ti, tj, v);
    }
    // R1 rounded, TILES tiles at a time (one work-group to a CU: with one
    // tile at a time its loads leave the memory idle: 64 members of a batch 102 us,
    // now 67)
    static constexpr int TILES = 4;
    static __device__ __forceinline__ void copy(const Args& a, int64_t e0, int64_t step)
    {
        const int64_t n = a.n, nt = tiles(n);
        const int i = thread() % T, q = thread() / T;
        double v[TILES][4];
#pragma unroll
        for (int y = 0; y < TILES; ++y) {
            const int64_t e = e0 + y * step, ti = e % nt, tj = e / nt;   // (columns past n: zero)
#pragma unroll
            for (int x = 0; x < 4; ++x) v[y][x] = upper(a.R1, n, T * ti + i, T * tj + q + 8 * x);
        }
#pragma unroll
        for (int y = 0; y < TILES; ++y) {
            const int64_t e = e0 + y * step;
            store(a, e % nt, e / nt, v[y]);
        }
    }
    static __device__ __forceinline__ void store(const Args& a, int64_t ti, int64_t tj, const double (&v)[4])
    {
        const int64_t n = a.n;
        const int i = thread() % T, q = thread() / T;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t r = T * ti + i, c = T * tj + q + 8 * x;
            if (r >= n || c >= n) continue;
            const float f = r <= c ? (float)v[x] : 0.0f;
            double w = (double)f;
            if (a.prec == PNE_PREC_BF16) w = (double)__uint_as_float((uint32_t)f32_to_bf16_bits(f) << 16);
            if (a.prec == PNE_PREC_FP16)
                w = (double)(float)__builtin_bit_cast(_Float16, f32_to_f16_bits(f)) / (double)qr_scale(a.amax, a.s);
            a.R[r + c * a.ldr] = w;
            if (r == c && (w == 0.0 || !isfinite(w))) bad_column(a.info, 1000 + (int32_t)r + 1);
        }
    }
    static __device__ __forceinline__ void wait(const Args& a, int64_t items)
    {
        for (uint32_t it = 0; it < (1u << 24); ++it) {
            if (__hip_atomic_load(a.work + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= items) return;
            __builtin_amdgcn_s_sleep(1);
        }
        int32_t expected = 0;
        __hip_atomic_compare_exchange_strong(a.info, &expected, 4001, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    }
    static __device__ __forceinline__ void second_pass(const Args& a)
    {
        __shared__ int32_t next;
        // (Thread 0 has one block of its own per turn, between two barriers.  With
        // one at each end of the turn the compiler joins the two into a path
        // for thread 0 alone, and the other lanes of its wavefront pass the
        // barriers without it.)
        if (threadIdx.x == 0) next = __hip_atomic_fetch_add(a.work, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (;;) {
            __syncthreads();
            const int32_t it = __builtin_amdgcn_readfirstlane(next);
            // (the sizes formed anew every turn, not kept in registers across
            // the phases)
            int32_t n = (int32_t)a.n, chunk = (int32_t)a.chunk;
            asm volatile("" : "+s"(n), "+s"(chunk));
            const int32_t rows = (int32_t)a.s + n, nb = (n + CB - 1) / CB, nt = (int32_t)tiles(n);
            const int32_t packs = (int32_t)pack_items(n), fills = (chunk + NTH - 1) / NTH * ((n + FILL - 1) / FILL);
            const int32_t subst = (chunk + 63) / 64, gram = nb * (nb + 1) / 2, per = fills + subst + gram;
            const int32_t gram_end = packs + (int32_t)a.nchunks * per;
            // (Cholesky step k = 0 .. nb - 2 has r (r + 1) / 2 tiles, r = nb - 1 - k)
            const int32_t chol = 1 + (nb - 1) * nb * (nb + 1) / 6;
            if (it >= gram_end + chol + nt * nt) break;
            // the item's phase: its first item, and its chunk's rows or (Cholesky)
            // its step
            int32_t first = 0, k = -1, r0 = 0;
            int phase = -1;
            if (it >= packs && it < gram_end) {
                // (in a scalar register, which the division leaves)
                const int32_t h = __builtin_amdgcn_readfirstlane((it - packs) / per), r = it - packs - h * per;
                r0 = h * chunk;
                phase = r < fills ? 0 : (r < fills + subst ? 1 : 2);
                first = packs + h * per + (phase > 0 ? fills : 0) + (phase > 1 ? subst : 0);
            } else if (it >= gram_end) {
                phase = 3;
                first = gram_end;
                for (int32_t c = 1; k + 1 < nb; ++k) {
                    if (it < first + c) break;
                    first += c;
                    const int32_t r = nb - 2 - k;   // of step k + 1
                    c = r * (r + 1) / 2;
                }
                if (k + 1 >= nb) phase = 4;
            }
            const int32_t crows = rows - r0 < chunk ? rows - r0 : chunk;
            if (threadIdx.x == 0 && first > packs) wait(a, first);   // (the first chunk waits for nothing)
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            const int e = it - first;
            if (phase < 0) {
                pack(a, e);
            } else if (phase == 0) {
                fill(a, e, r0, crows);
            } else if (phase == 1) {
                // (in place: a lane loads its entries of a panel's columns
                // before it stores there, and keeps nothing it loads of
                // another's row)
                const TrsmArgs p{crows, n, a.X, chunk, a.pack, a.X, chunk};
                if (64 * e < crows) TrsmRows<false>::rows(p, e, thread());
            } else if (phase == 2) {
                GemmArgs g{};
                g.M = n; g.N = n; g.K = crows;
                g.A = a.X; g.lda = chunk;
                g.B = a.X; g.ldb = chunk;
                g.lower = 1;
                g.splits = 1;
                g.kchunk = (crows + 15) / 16 * 16;
                g.P = a.C;
                g.accumulate_partials = r0 > 0;
                GemmTn<double, false>::tile(g, e, 0, thread());
            } else if (phase == 3) {
                const CholStepArgs p{n, k, a.C, n, nullptr, 0, a.R2, n, a.tab, a.gd, a.t, nullptr, nullptr, nullptr};
                CholStep<true, true>::run(p, e, 0);
            } else {
                tile(a, e);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            if (threadIdx.x == 0) {
                __hip_atomic_fetch_add(a.work + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                next = __hip_atomic_fetch_add(a.work, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    static __device__ __forceinline__ void run(const Args& a, int bx, int)
    {
        if (*a.state == 1) {
            second_pass(a);
            return;
        }
        const int64_t nt = tiles(a.n);
        for (int64_t e = bx; e < nt * nt; e += TILES * (int64_t)a.wgs) copy(a, e, a.wgs);
    }
};

static size_t own_doubles(int64_t n) { return trsm_pack_bytes(n) / sizeof(double) + (size_t)(n * n); }   // pack, R1

// Rows of [W; 2^-24.5 D] that the second pass takes at a time in a scratch of so
// many doubles: all, or a multiple of 64 that makes no more than eight chunks (each
// costs three waits of the whole launch, some 30 us); else none (0).
int64_t sketch_factor_chunk(int64_t s, int64_t n, size_t doubles)
{
    const size_t own = own_doubles(n);
    if (doubles <= own) return 0;
    const int64_t rows = s + n, fit = (int64_t)((doubles - own) / (size_t)n), even = (rows + 1) & ~(int64_t)1;
    if (fit >= even) return even;
    const int64_t chunk = fit / 64 * 64;
    return 8 * chunk >= rows ? chunk : 0;
}

// C: n x n scratch; P: scratch of pslots n x n FP64 matrices (at least one);
// tab: dinv_elems(n), gd: n, words: two (FP16: scale; state), work: two; X:
// scratch of xcap doubles, 16-byte aligned, in which sketch_factor_chunk is not 0.
int sketch_factor(Exec& ex, int64_t s, int64_t n, float* W, int64_t ldw, int prec, double* R, int64_t ldr, double* C,
                  double* P, int64_t pslots, double* tab, double* gd, uint32_t* words, int32_t* work, double* X,
                  size_t xcap, int32_t* info)
{
    uint32_t* amax = words;
    int32_t* state = (int32_t*)words + 1;
    const int64_t chunk = sketch_factor_chunk(s, n, xcap);
    double* pack = X + chunk * n;
    double* R1 = pack + trsm_pack_bytes(n) / sizeof(double);
    const double t = 8.0 * (double)n * 0x1p-53;
    ex.stage(ST_SKFACTOR);
    qr_round(ex, s, n, W, ldw, prec, amax);
    gram_f32(ex, s, n, W, ldw, C, P, pslots);
    ex.stage(ST_SKFACTOR_CHOL);
    cholesky64_shifted(ex, n, C, n, R1, n, tab, gd, t, state, work);
    ex.stage(ST_SKFACTOR_END);
    // one work-group per CU at most (LDS); in a batch as many as the copy of R1 needs
    const int64_t nt = SketchEnd::tiles(n), most = nt * nt > ceil_div(s, 64) ? nt * nt : ceil_div(s, 64);
    const int64_t want = ex.recording() ? ceil_div(nt * nt, SketchEnd::TILES) : most;
    const int32_t wgs = (int32_t)(want < 256 ? want : 256);
    launch<SketchEnd>(ex, wgs, 1, SketchEndArgs{s, n, W, ldw, X, chunk, ceil_div(s + n, chunk), pack, R1, P, C, tab, gd, t, state, work,
                                                R, ldr, prec, amax, wgs, info});
    return launch_status(ex);
}

}  // namespace pne
