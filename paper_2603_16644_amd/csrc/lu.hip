// LU factorization with partial pivoting P C = L U of the n x n HPNE matrix
// A_p^T A (Section 1, eq. e_hpne; the system is non-symmetric).  Blocked,
// right-looking:
//   panel (32 columns of up to 1024 rows, 16 of up to 2048, 8 above), one
//     work-group with the panel in registers: per column the pivot is the
//     first row of largest magnitude, the two rows are exchanged through LDS,
//     the column is scaled and the rest of the panel gets the rank-1 update;
//   the other columns, 16 to a work-group: the
//     panel's row exchanges (composed into one permutation of at most 2 PW
//     rows, so a column's loads are all in flight together instead of one
//     exchange after another) and, right of the panel, U12 := L11^{-1} C12
//     (unit lower forward substitution);
//   C22 -= L21 U12 (MFMA GEMM).
// A zero or non-finite pivot at global column k sets *info = 3000 + k + 1
// (first only); that column's elimination is skipped.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {

constexpr int LU_THREADS = 512;
constexpr int LU_WAVES = LU_THREADS / 64;

// Shared state of the panel kernel.  Rows k and p and the per-wavefront
// argmax candidates are double-buffered by the parity of the step, so step
// k + 1 never overwrites what a slower thread of step k still reads.
template <int PW>
struct LuShared {
    double rowK[2][PW], rowP[2][PW], rowPu[2][PW];
    double wv[2][LU_WAVES];
    int64_t wi[2][LU_WAVES];
    int32_t pivl[PW];              // pivot rows of the panel (relative to its first row)
};

// Panel of more than 2048 rows in one 512-thread work-group: the panel
// C(c0:n, c0:c0+w) factored in registers (partial pivoting), written back
// with its pivot rows.  LuTail then applies the exchanges to the other
// columns and forms U12; the trailing update C22 -= L21 U12 follows as an
// MFMA GEMM launch.
struct LuPanelArgs {
    int64_t n;
    int w;
    double* C;
    int64_t ldc;
    int32_t* piv;
    int64_t c0;
    int32_t* info;
};
template <int RPT, int PW>
struct LuPanel {
    typedef LuPanelArgs Args;
    static constexpr int NTH = LU_THREADS, WPE = 0;
    static __device__ void run(const LuPanelArgs& a, int bx, int by);
};
template <int RPT, int PW>
__device__ void LuPanel<RPT, PW>::run(const LuPanelArgs& a, int, int)
{
    const int64_t n = a.n, ldc = a.ldc, c0 = a.c0, h = n - c0;
    const int w = a.w;
    double* __restrict__ C = a.C;
    double* __restrict__ P = C + c0 + c0 * ldc;
    __shared__ LuShared<PW> sh;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wid = tid >> 6;
    int32_t* __restrict__ info = a.info;
    double x[RPT][PW];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t r = tid + LU_THREADS * q;
#pragma unroll
        for (int c = 0; c < PW; ++c) x[q][c] = (r < h && c < w) ? P[r + c * ldc] : 0.0;
    }
    // Column step k with the active column at register position J (a
    // compile-time constant).  The register row is rotated left after every
    // block of steps, so that every register index stays a compile-time
    // constant; after step k the columns already factored sit at the end
    // (positions PW - k .. PW - 1) or, inside a block, before J.  Two
    // barriers per step: after the wavefront argmax candidates are published
    // (every thread then forms the pivot row itself) and after the owners of
    // rows k and p publish them.  The owner of the pivot row also publishes
    // it with the factored columns zeroed (rowPu), which the rank-1 update
    // uses, so that no thread tests column positions.
    auto colstep = [&](auto jc, int k) {
        constexpr int J = decltype(jc)::value;
        const int B = k & 1;
        // argmax |x(r, k)| over r >= k, first index on ties; a NaN counts as
        // +inf, so a column holding one selects a non-finite pivot
        double best = -1.0;
        int64_t bidx = INT64_MAX;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t r = tid + LU_THREADS * q;
            double v = fabs(x[q][J]);
            if (v != v) v = INFINITY;
            if (r >= k && r < h && v > best) { best = v; bidx = r; }
        }
        wave_argmax(best, bidx);
        if (lane == 0) { sh.wv[B][wid] = best; sh.wi[B][wid] = bidx; }
        __syncthreads();
        double bb = sh.wv[B][0];
        int64_t p = sh.wi[B][0];
        for (int i = 1; i < LU_WAVES; ++i)
            if (sh.wv[B][i] > bb || (sh.wv[B][i] == bb && sh.wi[B][i] < p)) { bb = sh.wv[B][i]; p = sh.wi[B][i]; }
        if (p < k || p >= h) p = k;   // no candidate: keep the row in place
        if (tid == 0) sh.pivl[k] = (int32_t)p;
        const int live = PW - k + J;  // positions J .. live - 1 are not factored yet
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t r = tid + LU_THREADS * q;
            if (r == p)
#pragma unroll
                for (int c = 0; c < PW; ++c) {
                    sh.rowP[B][c] = x[q][c];
                    sh.rowPu[B][c] = c < live ? x[q][c] : 0.0;
                }
            if (r == k)
#pragma unroll
                for (int c = 0; c < PW; ++c) sh.rowK[B][c] = x[q][c];
        }
        __syncthreads();
        const double pv = sh.rowP[B][J];
        const bool ok = pv != 0.0 && isfinite(pv);
        if (!ok && tid == 0 && *info == 0) *info = 3000 + (int32_t)(c0 + k) + 1;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int64_t r = tid + LU_THREADS * q;
            // exchange rows k and p
            if (r == k && p != k)
#pragma unroll
                for (int c = 0; c < PW; ++c) x[q][c] = sh.rowP[B][c];
            if (r == p && p != k)
#pragma unroll
                for (int c = 0; c < PW; ++c) x[q][c] = sh.rowK[B][c];
            // multiplier and rank-1 update of the rows below k
            if (ok && r > k && r < h) {
                const double l = x[q][J] / pv;
                x[q][J] = l;
#pragma unroll
                for (int c = J + 1; c < PW; ++c) x[q][c] -= l * sh.rowPu[B][c];
            }
        }
    };
    // rotate the register row left by S positions
    auto rotate = [&](auto sc) {
        constexpr int S = decltype(sc)::value;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            double t[S];
#pragma unroll
            for (int c = 0; c < S; ++c) t[c] = x[q][c];
#pragma unroll
            for (int c = 0; c < PW - S; ++c) x[q][c] = x[q][c + S];
#pragma unroll
            for (int c = 0; c < S; ++c) x[q][PW - S + c] = t[c];
        }
    };
    // blocks of four steps (one rotation per block), then single steps
    int k = 0;
#pragma unroll 1
    for (; k + 4 <= w; k += 4) {
        colstep(std::integral_constant<int, 0>{}, k);
        colstep(std::integral_constant<int, 1>{}, k + 1);
        colstep(std::integral_constant<int, 2>{}, k + 2);
        colstep(std::integral_constant<int, 3>{}, k + 3);
        rotate(std::integral_constant<int, 4>{});
    }
#pragma unroll 1
    for (; k < w; ++k) {
        colstep(std::integral_constant<int, 0>{}, k);
        rotate(std::integral_constant<int, 1>{});
    }
    // position c now holds panel column (c + w) mod PW
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int64_t r = tid + LU_THREADS * q;
#pragma unroll
        for (int c = 0; c < PW; ++c) {
            int col = c + w;
            if (col >= PW) col -= PW;
            if (r < h && col < w) P[r + col * ldc] = x[q][c];
        }
    }
    if (tid < w) a.piv[c0 + tid] = (int32_t)(c0 + sh.pivl[tid]);
}

// Panels of 1024 rows or fewer (32 columns) and of 2048 or fewer (16): the same
// factorization with the columns over the lanes.
//
// Lane (g, l) of a wavefront holds rows 4 g .. 4 g + 3 of each of its 16-row
// chunks (chunk wv + NW q) in one column of each of NH groups of 16.  The
// columns of the group at hand move on by four lanes after every four steps
// (column (l + 4 it) mod 16), so that column k = 16 H + 4 it + J is in lane J.
// A multiplier is then formed in lane J and sent to the row of lanes by DPP,
// and the pivot row is one value per lane: the rank-1 update reads one entry
// of LDS per lane instead of a row.  One barrier per column: before it every
// wavefront publishes its largest entry of the column and that whole row, and
// the owner of row k that row.  Row k lies in chunk H, at a register known at
// compile time; the candidate's register is found by scalar branches.
// Multipliers are x (1 / pivot), formed again from the unscaled column at the
// end (as LAPACK does for pivots whose reciprocal is finite; a smaller one has
// its column scaled up first).
//
// Bound by the chain of a column (1 us) and, at 1024 rows, by instruction
// issue (1.6 us more: some 500 instructions in each of two wavefronts per
// SIMD).  All panels, against a row of the panel per thread with the pivot row
// read from LDS by every wavefront: n = 1000 2.89 -> 2.09 ms, n = 400 1.00 ->
// 0.61 ms.
template <int NW, int Q, int PW>
struct LuLaneShared {
    double mx[2][NW];
    int32_t row[2][NW];
    double cand[2][NW][PW];     // candidate rows
    double rowk[2][PW];
    double col[NW][16 * Q];     // the column at hand, per wavefront
    int32_t piv[PW];
    int32_t bad;                // first column with an entry that is not finite
};

template <int C>
__device__ __forceinline__ double lu_row_move(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, C, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), C, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int NW, int Q, int NH>
struct LuLanes {
    static constexpr int PW = 16 * NH;
    typedef LuPanelArgs Args;
    static constexpr int NTH = 64 * NW, WPE = NW / 4;
    typedef LuLaneShared<NW, Q, PW> Shared;

    struct State {
        double x[NH][Q][4];
        int g, l, wv, w, h, c0;
        int32_t* info;
    };

    template <int H, int J>
    static __device__ __forceinline__ void step(State& s, int it, double& ivc, Shared& sh)
    {
        const int kl = 4 * it + J, k = 16 * H + kl;      // column within the group, within the panel
        const int c = (s.l + 4 * it) & 15;               // own column of group H
        constexpr int B = J & 1;
        const int g = s.g, wv = s.wv;
        // the wavefront's part of the column over its 64 lanes, in row order
        double* __restrict__ cw = sh.col[wv];
        if (s.l == J) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) cw[16 * q + 4 * g + t] = s.x[H][q][t];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int lane = threadIdx.x & 63;
        constexpr int NV = Q > 4 ? Q / 4 : 1;
        double cv[NV], mx = -1.0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int e = lane + 64 * i, r = 16 * (wv + NW * (e >> 4)) + (e & 15);
            cv[i] = (e < 16 * Q && r >= k) ? fabs(cw[e < 16 * Q ? e : 0]) : -1.0;
            mx = fmax(mx, cv[i]);
        }
        {
            double a = mx, b = mx;
            lane_swap<32>(a, b);
            mx = fmax(a, b);
            a = b = mx;
            lane_swap<16>(a, b);
            mx = fmax(a, b);
        }
        mx = fmax(mx, dpp_partner<8>(mx));
        mx = fmax(mx, dpp_partner<4>(mx));
        mx = fmax(mx, dpp_partner<2>(mx));
        mx = fmax(mx, dpp_partner<1>(mx));
        int es = -1;
#pragma unroll
        for (int i = NV - 1; i >= 0; --i) {
            const uint64_t m = __ballot(cv[i] == mx && mx >= 0.0);
            if (m != 0) es = 64 * i + __builtin_ctzll(m);
        }
        const int qs = es >> 4, gs = es < 0 ? 0 : (es >> 2) & 3, ts = es & 3;   // (es < 0: qs < 0)
        double cand[NH];
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) cand[hh] = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (qs == q) {
#pragma unroll
                for (int hh = 0; hh < NH; ++hh) {
                    const double lo = (ts & 1) ? s.x[hh][q][1] : s.x[hh][q][0];
                    const double hi = (ts & 1) ? s.x[hh][q][3] : s.x[hh][q][2];
                    cand[hh] = (ts & 2) ? hi : lo;
                }
                asm volatile("" ::"n"(q));   // keeps the branches apart (merged, x goes to memory)
            }
        // (index of a column of group hh held by this lane)
        auto slot = [&](int hh) { return 16 * hh + (hh == H ? c : s.l); };
        if (s.g == gs) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) sh.cand[B][wv][slot(hh)] = cand[hh];
            if (s.l == J) {
                sh.mx[B][wv] = qs < 0 ? -1.0 : mx;
                sh.row[B][wv] = 16 * (wv + NW * qs) + 4 * gs + ts;
            }
        }
        if (wv == H && g == it) {
#pragma unroll
            for (int hh = 0; hh < NH; ++hh) sh.rowk[B][slot(hh)] = s.x[hh][0][J];
        }
        __syncthreads();
        // the wavefront with the largest, the smallest row among equals
        const double cm = sh.mx[B][s.l & (NW - 1)];
        const int cr = sh.row[B][s.l & (NW - 1)];
        double best = cm;
        best = fmax(best, dpp_partner<8>(best));
        best = fmax(best, dpp_partner<4>(best));
        best = fmax(best, dpp_partner<2>(best));
        best = fmax(best, dpp_partner<1>(best));
        uint64_t eq = __ballot(cm == best) & ((1ull << NW) - 1);
        int ws = 0, p = k;
        if (eq != 0) {
            ws = __builtin_ctzll(eq);
            p = __builtin_amdgcn_readlane(cr, ws);
            for (eq &= eq - 1; eq != 0; eq &= eq - 1) {
                const int w2 = __builtin_ctzll(eq), p2 = __builtin_amdgcn_readlane(cr, w2);
                if (p2 < p) { p = p2; ws = w2; }
            }
        }
        if (!(best >= 0.0) || p < k || p >= s.h) p = k;   // no candidate: the row stays
        p = __builtin_amdgcn_readfirstlane(p);
        ws = __builtin_amdgcn_readfirstlane(ws);
        double up[NH], rk[NH];
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) {
            rk[hh] = sh.rowk[B][slot(hh)];
            up[hh] = p == k ? rk[hh] : sh.cand[B][ws][slot(hh)];
        }
        const double pv = lane_value(up[H], J);
        const bool ok = pv != 0.0 && fabs(pv) < INFINITY && k < sh.bad;
        if (threadIdx.x == 0) {
            sh.piv[k] = p;
            if (!ok && *s.info == 0) *s.info = 3000 + s.c0 + k + 1;
        }
        // exchange rows k and p
        if (p != k) {
            const int ch = p >> 4, pq = ch / NW;
            if (ch % NW == wv) {
                const int pg = (p >> 2) & 3, pt = p & 3;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    if (pq == q) {
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const bool mine = g == pg && t == pt;
#pragma unroll
                            for (int hh = 0; hh < NH; ++hh) s.x[hh][q][t] = mine ? rk[hh] : s.x[hh][q][t];
                        }
                        asm volatile("" ::"n"(q));
                    }
            }
            if (wv == H && g == it) {
#pragma unroll
                for (int hh = 0; hh < NH; ++hh) s.x[hh][0][J] = up[hh];
            }
        }
        // reciprocal by Newton steps from the hardware's approximation
        double inv = __builtin_amdgcn_rcp(pv);
        inv = fma(inv, fma(-pv, inv, 1.0), inv);
        inv = fma(inv, fma(-pv, inv, 1.0), inv);
        if (ok && !(fabs(pv) > 0x1p-1000 && fabs(pv) < 0x1p1000)) {
            if (fabs(pv) < 1.0) {   // scale the column up
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (c == kl && !(q == 0 && 16 * wv + 4 * g + t <= k)) s.x[H][q][t] *= 0x1p300;
                inv = 1.0 / (pv * 0x1p300);
            } else {
                inv = 1.0 / pv;
            }
        }
        if (!ok) inv = 0.0;
        if (c == kl) ivc = ok ? inv : 1.0;
        double u[NH];
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) u[hh] = hh > H ? up[hh] : 0.0;
        u[H] = c > kl ? up[H] : 0.0;
        // (four entries side by side: moves, multipliers, updates)
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            double m[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) m[t] = lu_row_move<0x150 + J>(s.x[H][q][t]);
#pragma unroll
            for (int t = 0; t < 4; ++t) m[t] *= inv;
            if (q == 0) {
#pragma unroll
                for (int t = 0; t < 4; ++t) m[t] = 16 * wv + 4 * g + t <= k ? 0.0 : m[t];
            }
#pragma unroll
            for (int hh = H; hh < NH; ++hh)
#pragma unroll
                for (int t = 0; t < 4; ++t) s.x[hh][q][t] -= m[t] * u[hh];
        }
    }

    template <int H>
    static __device__ __forceinline__ void group(State& s, double& ivc, Shared& sh)
    {
#pragma unroll 1
        for (int it = 0; it < 4; ++it) {
            const int k = 16 * H + 4 * it;
            if (k < s.w) step<H, 0>(s, it, ivc, sh);
            if (k + 1 < s.w) step<H, 1>(s, it, ivc, sh);
            if (k + 2 < s.w) step<H, 2>(s, it, ivc, sh);
            if (k + 3 < s.w) step<H, 3>(s, it, ivc, sh);
            ivc = lu_row_move<0x12C>(ivc);
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int t = 0; t < 4; ++t) s.x[H][q][t] = lu_row_move<0x12C>(s.x[H][q][t]);
        }
    }

    static __device__ __forceinline__ void run(const Args& a, int, int)
    {
        __shared__ Shared sh;
        const int lane = threadIdx.x & 63;
        const int64_t ldc = a.ldc;
        const int h = (int)(a.n - a.c0);
        State s;
        s.g = lane >> 4;
        s.l = lane & 15;
        s.wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        s.w = a.w;
        s.h = h;
        s.c0 = (int)a.c0;
        s.info = a.info;
        double* __restrict__ P = a.C + a.c0 + a.c0 * ldc;
        if (threadIdx.x == 0) sh.bad = PW;
        __syncthreads();
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) {
            const int c = 16 * hh + s.l;
            const double* __restrict__ col = P + (c < s.w ? c : s.w - 1) * ldc;
            double z = 0.0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int r0 = 16 * (s.wv + NW * q) + 4 * s.g;
#pragma unroll
                for (int t = 0; t < 4; ++t) s.x[hh][q][t] = col[r0 + t < h ? r0 + t : h - 1];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (r0 + t >= h || c >= s.w) s.x[hh][q][t] = 0.0;
                    z += s.x[hh][q][t] * 0.0;
                }
            }
            if (z != 0.0 || z != z) atomicMin(&sh.bad, c);
        }
        __syncthreads();
        double iv[NH];
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) iv[hh] = 1.0;
        group<0>(s, iv[0], sh);
        if constexpr (NH > 1) group<1>(s, iv[1], sh);
#pragma unroll
        for (int hh = 0; hh < NH; ++hh) {
            const int c = 16 * hh + s.l;
            double* __restrict__ col = P + c * ldc;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int r0 = 16 * (s.wv + NW * q) + 4 * s.g;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (r0 + t < h && c < s.w) col[r0 + t] = r0 + t > c ? s.x[hh][q][t] * iv[hh] : s.x[hh][q][t];
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < s.w) a.piv[a.c0 + threadIdx.x] = (int32_t)(a.c0 + sh.piv[threadIdx.x]);
    }
};

// The row exchanges of a factored panel (pivots piv[c0 .. c0+w)) applied to
// every column outside it, and U12 := L11^{-1} C12 right of it.  The exchanges,
// applied in order k = 0 .. w-1 to the rows c0 + k and piv[c0 + k], move values
// among at most 2 w rows: they are composed into a table (row slot s receives
// the value that row slot src[s] held before the panel).  A wavefront takes 16
// columns, lane (g, c) the slots g, g + 4, ... of column c: 16 columns and not
// 64, as every row below the panel costs a cache line per column, which one CU
// takes in turn (n = 1000: 20.7 us per panel with 64 columns and a lane per
// column, 11.7 us so).
template <int PW>
struct LuTail {
    struct Args {
        int64_t n;
        int w;
        double* C;
        int64_t ldc;
        const int32_t* piv;
        int64_t c0;
    };
    static constexpr int NTH = 64, WPE = 0;
    static constexpr int COLS = 16;
    static __device__ void run(const Args& a, int bx, int by);
};
template <int PW>
__device__ void LuTail<PW>::run(const Args& a, int bx, int)
{
    __shared__ double L11[PW][PW + 1];     // L11[l][i], column l
    __shared__ double val[2 * PW][COLS];
    __shared__ int32_t srow[2 * PW], ssrc[2 * PW];
    constexpr int R = PW / 4;              // slots of a lane in each half
    const int64_t n = a.n, ldc = a.ldc, c0 = a.c0;
    const int w = a.w, tid = threadIdx.x, g = tid >> 4, c = tid & 15;
    double* __restrict__ C = a.C;
    // columns left of the panel, then right of it
    const int64_t jj = (int64_t)bx * COLS + c;
    const bool in = jj < n - w;
    const int64_t j = !in ? c0 : (jj < c0 ? jj : jj + w);
    double* __restrict__ col = C + j * ldc + c0;
    const int pv = tid < w ? a.piv[c0 + tid] - (int32_t)c0 : -1;
    double own[R], low[R];
#pragma unroll
    for (int q = 0; q < R; ++q) own[q] = col[4 * q + g < w ? 4 * q + g : 0];
    for (int e = tid; e < PW * PW; e += NTH) {
        const int i = e % PW, l = e / PW;
        L11[l][i] = (i < w && l < i) ? C[(c0 + i) + (c0 + l) * ldc] : 0.0;
    }
    // lane s: row slot s (the panel's rows, then the pivot rows below them) and
    // the slot its value comes from
    int row = tid, src = tid, ns = w;
    for (int k = 0; k < w; ++k) {
        const int pk = __builtin_amdgcn_readlane(pv, k);
        int sp = pk;
        if (pk >= w) {
            const uint64_t m = __ballot(tid >= w && tid < ns && row == pk);
            sp = ns;
            if (m != 0) sp = __builtin_ctzll(m);
            else {
                if (tid == ns) row = pk;
                ++ns;
            }
        }
        const int sk = __builtin_amdgcn_readlane(src, k), ss = __builtin_amdgcn_readlane(src, sp);
        src = tid == k ? ss : (tid == sp ? sk : src);
    }
    if (tid < 2 * PW) { srow[tid] = row; ssrc[tid] = src; }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int s = w + 4 * q + g;
        low[q] = s < ns ? col[srow[s]] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int s = w + 4 * q + g;
        if (4 * q + g < w) val[4 * q + g][c] = own[q];
        if (s < ns) val[s][c] = low[q];
    }
    __syncthreads();
    double u[R];
#pragma unroll
    for (int q = 0; q < R; ++q) u[q] = 4 * q + g < w ? val[ssrc[4 * q + g]][c] : 0.0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int s = w + 4 * q + g;
        if (in && s < ns) col[srow[s]] = val[ssrc[s]][c];
    }
    // (a group of columns may lie on both sides of the panel)
    const double right = in && j >= c0 + w ? 1.0 : 0.0;
    if (bx * (int64_t)COLS + COLS > c0) {
#pragma unroll
        for (int l = 0; l < PW - 1; ++l) {
            const double ul = __shfl(u[l / 4], 16 * (l % 4) + c) * right;
#pragma unroll
            for (int q = l / 4; q < R; ++q) u[q] -= L11[l][4 * q + g] * ul;   // (zero for rows up to l)
        }
    }
#pragma unroll
    for (int q = 0; q < R; ++q)
        if (in && 4 * q + g < w) col[4 * q + g] = u[q];
}

template <class Panel, int PW>
static void lu_steps(Exec& ex, int64_t n, double* C, int64_t ldc, int32_t* piv, int32_t* info, int64_t c0)
{
    ex.iter((uint32_t)c0);
    const int w = (int)((n - c0 < PW) ? n - c0 : PW);
    launch<Panel>(ex, 1, 1, LuPanelArgs{n, w, C, ldc, piv, c0, info});
    if (n > w)
        launch<LuTail<PW>>(ex, ceil_div(n - w, LuTail<PW>::COLS), 1, typename LuTail<PW>::Args{n, w, C, ldc, piv, c0});
    const int64_t rem = n - c0 - w;
    if (rem <= 0) return;
    GemmArgs g{};
    g.M = rem; g.N = rem; g.K = w;
    g.A = C + (c0 + w) + c0 * ldc; g.lda = ldc; g.transA = 0;
    g.B = C + c0 + (c0 + w) * ldc; g.ldb = ldc; g.transB = 0;
    g.alpha = -1.0; g.beta = 1.0;
    double* C22 = C + (c0 + w) + (c0 + w) * ldc;
    g.Cin = C22; g.ldcin = ldc; g.C = C22; g.ldc = ldc;
    g.splits = 1;
    gemm_f64(ex, g);
}

bool lu_supported(int64_t n) { return n <= 4096; }

void lu_factor(Exec& ex, int64_t n, double* C, int64_t ldc, int32_t* piv, int32_t* info)
{
    int64_t c0 = 0;
    while (c0 < n) {
        const int64_t h = n - c0;
        // 32 columns while the panel's 1024 rows fit the registers of 8
        // wavefronts, 16 to 2048 rows in 16, the row-per-thread panel above
        int pw = 32;
        if (h <= 128) lu_steps<LuLanes<8, 1, 2>, 32>(ex, n, C, ldc, piv, info, c0);
        else if (h <= 256) lu_steps<LuLanes<8, 2, 2>, 32>(ex, n, C, ldc, piv, info, c0);
        else if (h <= 512) lu_steps<LuLanes<8, 4, 2>, 32>(ex, n, C, ldc, piv, info, c0);
        else if (h <= 1024) lu_steps<LuLanes<8, 8, 2>, 32>(ex, n, C, ldc, piv, info, c0);
        else if (h <= 2048) { lu_steps<LuLanes<16, 8, 1>, 16>(ex, n, C, ldc, piv, info, c0); pw = 16; }
        else { lu_steps<LuPanel<8, 8>, 8>(ex, n, C, ldc, piv, info, c0); pw = 8; }
        c0 += pw;
    }
}

}  // namespace pne
