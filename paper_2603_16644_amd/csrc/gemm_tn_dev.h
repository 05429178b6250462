// Kernel of the 64 x 64 split-K products (gemm_tn.hip, sketch_factor.hip).
#pragma once
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {

namespace {

typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v2d8 __attribute__((ext_vector_type(2), aligned(8)));   // 16-byte load from an 8-byte boundary
// (explicitly global: in grouped launches the pointers come from a table,
// and the compiler would otherwise issue flat loads)
typedef const __attribute__((address_space(1))) char* gpc;
typedef const __attribute__((address_space(1))) double* gp64;
typedef const __attribute__((address_space(1))) v2d8* gpv2;

__device__ __forceinline__ void tn_lower_tile(int64_t id, int64_t& ti, int64_t& tj)
{
    int64_t t = (int64_t)((sqrt(8.0 * (double)id + 1.0) - 1.0) * 0.5);
    while (t * (t + 1) / 2 > id) --t;
    while ((t + 1) * (t + 2) / 2 <= id) ++t;
    ti = t;
    tj = id - t * (t + 1) / 2;
}

}  // namespace

// WIDE: leading dimensions of 2^23 or more (64-bit addresses).  Otherwise a
// lane's offset from the first column of its 64-column block fits 32 bits
// and the loads are buffer loads (uniform base, one 32-bit offset register
// per 16-column block, K advance in a scalar register), which leaves the
// accumulators and both operand buffers in registers.
template <typename TI, bool WIDE>
struct GemmTn {
    typedef GemmArgs Args;
    static constexpr int NTH = 256, WPE = WIDE ? 1 : 2;   // (64-bit addresses: 440 registers)
    static __device__ __forceinline__ void run(const GemmArgs& g, int bx, int by) { tile(g, bx, by, threadIdx.x); }
    static __device__ void tile(const GemmArgs& g, int bx, int by, int tid);   // (tid: the thread's index)
};

template <typename TI, bool WIDE>
__device__ __forceinline__ void GemmTn<TI, WIDE>::tile(const GemmArgs& g, int bx, int by, int tid)
{
    constexpr int BM = 64;
    constexpr int E = 16 / sizeof(TI);       // K values of a lane's 16 bytes
    constexpr int KS = 4 * E, KL = 2 * KS;   // K values per step (64 bytes of a column) and per turn of the loop
    constexpr int64_t SZ = sizeof(TI);
    typedef TI vin __attribute__((ext_vector_type(E), aligned(sizeof(TI))));
    typedef const __attribute__((address_space(1))) TI* gpi;
    typedef const __attribute__((address_space(1))) vin* gpvi;
    const int lane = tid & 63, r16 = lane & 15, g4 = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t M = g.M, N = g.N;
    const int64_t tiles_m = (M + BM - 1) / BM;
    if (g.xcd_remap) {
        // Work-group L of a launch runs on XCD L % 8: every XCD gets a
        // contiguous run of (K chunk, tile) work, whose tiles read their
        // operand panels through the same L2.
        const int64_t gxw = gridDim.x, T = gxw * gridDim.y;
        const int64_t L = bx + (int64_t)by * gxw;
        const int64_t x = L % 8, slot = L / 8, q = T / 8, r = T % 8;
        const int64_t v = x * q + (x < r ? x : r) + slot;
        bx = (int)(v % gxw);
        by = (int)(v / gxw);
    }
    int64_t ti, tj;
    if (g.lower) {
        tn_lower_tile(bx, ti, tj);
    } else {
        ti = bx % tiles_m;
        tj = bx / tiles_m;
    }
    const int64_t split = by;
    int64_t kbeg = split * g.kchunk;
    int64_t kend = (kbeg + g.kchunk < g.K) ? kbeg + g.kchunk : g.K;
    {
        const int64_t sub = ((kend - kbeg + 4 * KL - 1) / (4 * KL)) * KL;   // K share of a wavefront
        const int64_t ks = kbeg + w * sub;
        const int64_t ke = ks + sub;
        kend = ke < kend ? ke : kend;
        kbeg = ks;
    }
    // (into scalar registers, where the buffer descriptors have to be)
    ti = __builtin_amdgcn_readfirstlane((int)ti);
    tj = __builtin_amdgcn_readfirstlane((int)tj);
    const int64_t i0 = ti * BM, j0 = tj * BM;
    // which of the 16 MFMA blocks the product needs (bit 4 a + c: rows 16 a,
    // columns 16 c)
    unsigned mask = g.lower && ti == tj ? 0xf731u : 0xffffu;
    {
        int64_t na = (M - i0 + 15) / 16, nc = (N - j0 + 15) / 16;   // blocks inside the matrix
        na = na < 0 ? 0 : (na > 4 ? 4 : na);
        nc = nc < 0 ? 0 : (nc > 4 ? 4 : nc);
        mask &= (1u << (4 * na)) - 1u;
        mask &= ((1u << nc) - 1u) * 0x1111u;
    }
    mask = __builtin_amdgcn_readfirstlane(mask);
    const double* __restrict__ bv = (const double*)g.bvec;
    // op(A) bvec is formed beside the blocks on the diagonal (lower-triangle
    // products) or of the first tile column
    const bool fold = E == 2 && bv != nullptr && (g.lower ? (i0 == j0) : (j0 == 0));

    v4d acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = (v4d){0, 0, 0, 0};
    double cs[4] = {0, 0, 0, 0};

    if (mask != 0 && kbeg < kend) {
        const gpc pa = (gpc)((gpi)g.A + i0 * g.lda + kbeg), pb = (gpc)((gpi)g.B + j0 * g.ldb + kbeg);
        const gpc pv = (gpc)(gp64)(fold ? bv + kbeg : nullptr);
        // last column of each operand's 64 (columns past the matrix read it;
        // results not stored), and the lane's column and K offset in each
        // 16-column block, in bytes
        const int ila = (int)(M - 1 - i0 < 63 ? M - 1 - i0 : 63), ilb = (int)(N - 1 - j0 < 63 ? N - 1 - j0 : 63);
        const uint32_t lda8 = (uint32_t)(g.lda * SZ), ldb8 = (uint32_t)(g.ldb * SZ);
        auto oa = [&](int t) {
            const int c = t * 16 + r16;
            return (uint64_t)(c < ila ? c : ila) * g.lda * SZ + 16 * g4;
        };
        auto ob = [&](int t) {
            const int c = t * 16 + r16;
            return (uint64_t)(c < ilb ? c : ilb) * g.ldb * SZ + 16 * g4;
        };
        const uint32_t ov = 16 * g4;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)pa, 0, -1, 0x00027000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)pb, 0, -1, 0x00027000);
        vin xa[2][4], xb[2][4];
        auto load = [&](auto bufc, int64_t k) {
            constexpr int b = decltype(bufc)::value;
            if constexpr (WIDE) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    xa[b][t] = *(gpvi)(pa + SZ * k + oa(t));
                    xb[b][t] = *(gpvi)(pb + SZ * k + ob(t));
                }
            } else {
                // (column offsets formed anew from an opaque lane index:
                // kept in registers they would cost the last eight)
                const int so = (int)(SZ * k);
                int r = r16;
                asm volatile("" : "+v"(r));
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = t * 16 + r, ca = c < ila ? c : ila, cb = c < ilb ? c : ilb;
                    xa[b][t] = __builtin_bit_cast(vin, __builtin_amdgcn_raw_buffer_load_b128(
                                                            ra, (int)((uint32_t)ca * lda8 + 16 * g4), so, 0));
                    xb[b][t] = __builtin_bit_cast(vin, __builtin_amdgcn_raw_buffer_load_b128(
                                                            rb, (int)((uint32_t)cb * ldb8 + 16 * g4), so, 0));
                }
            }
        };
        // MASK 0: the wavefront's run-time mask
        auto mult = [&](auto bufc, auto maskc) {
            constexpr int b = decltype(bufc)::value;
            constexpr unsigned MASK = decltype(maskc)::value;
            const unsigned mk = MASK ? MASK : mask;
#pragma unroll
            for (int h = 0; h < E; ++h)
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if ((mk >> (4 * a + c)) & 1u)
                            acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xb[b][c][h], (double)xa[b][a][h],
                                                                             acc[a][c], 0, 0, 0);
        };
        auto fold_step = [&](auto bufc, int64_t k) {
            constexpr int b = decltype(bufc)::value;
            if constexpr (E == 2) {   // (only FP64 products fold)
                if (!fold) return;
                const v2d8 v = *(gpv2)(pv + 8 * k + ov);
#pragma unroll
                for (int t = 0; t < 4; ++t) cs[t] += xa[b][t][0] * v[0] + xa[b][t][1] * v[1];
            }
        };
        using B0 = std::integral_constant<int, 0>;
        using B1 = std::integral_constant<int, 1>;
        const int64_t len = kend - kbeg, main = len / KL * KL;
        // Two steps a turn: the loads of a step are issued ahead of the
        // multiplications of the step before it (the scheduling barriers keep
        // it so).
        auto loop = [&](auto maskc, auto foldc) {
            constexpr bool FOLD = decltype(foldc)::value;
            auto step = [&](auto bufc, int64_t k) {
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (FOLD) fold_step(bufc, k);
                mult(bufc, maskc);
                __builtin_amdgcn_sched_barrier(0);
            };
            load(B0{}, 0);
            for (int64_t k = 0; k < main; k += KL) {
                load(B1{}, k + KS);
                step(B0{}, k);
                load(B0{}, k + KL < main ? k + KL : k);   // (after the last turn: read again, unused)
                step(B1{}, k + KS);
            }
        };
        using F = std::false_type;
        using T = std::true_type;
        if (main > 0) {
            if (mask == 0xffffu) {
                if (fold) loop(std::integral_constant<unsigned, 0xffffu>{}, T{});
                else loop(std::integral_constant<unsigned, 0xffffu>{}, F{});
            } else if (mask == 0xf731u && fold) {
                loop(std::integral_constant<unsigned, 0xf731u>{}, T{});
            } else {
                loop(std::integral_constant<unsigned, 0>{}, T{});
            }
        }
        // the K values left over (less than a turn): zero past the end on
        // both sides
        for (int64_t k = main; k < len; k += KS) {
#pragma unroll
            for (int h = 0; h < E; ++h) {
                const bool in = k + E * g4 + h < len;
                const double v = (fold && in) ? *(gp64)(pv + 8 * (k + h) + ov) : 0.0;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    xa[0][t][h] = in ? *(gpi)(pa + SZ * (k + h) + oa(t)) : (TI)0;
                    xb[0][t][h] = in ? *(gpi)(pb + SZ * (k + h) + ob(t)) : (TI)0;
                    cs[t] += xa[0][t][h] * v;
                }
            }
            mult(B0{}, std::integral_constant<unsigned, 0>{});
        }
    }
    if (fold) {
        // sum over the four K values of a step (lane bits 4 and 5)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            cs[t] += lane_partner<32>(cs[t]);
            cs[t] += lane_partner<16>(cs[t]);
        }
    }

    {
        // sum of the four wavefronts' blocks, ((0 + 1) + (2 + 3)), in LDS
        __shared__ double sh[64 * 64];
        __shared__ double shc[3][64];
        auto put = [&]() {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) sh[((a * 4 + c) * 4 + r) * 64 + lane] = acc[a][c][r];
        };
        auto take = [&]() {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[a][c][r] += sh[((a * 4 + c) * 4 + r) * 64 + lane];
        };
        if (fold && w > 0 && g4 == 0)
#pragma unroll
            for (int t = 0; t < 4; ++t) shc[w - 1][t * 16 + r16] = cs[t];
        if (w == 1) put();
        __syncthreads();
        if (w == 0) {
            take();
            if (fold && g4 == 0)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    cs[t] = ((cs[t] + shc[0][t * 16 + r16]) + shc[1][t * 16 + r16]) + shc[2][t * 16 + r16];
        }
        __syncthreads();
        if (w == 3) put();
        __syncthreads();
        if (w == 2) {
            take();
            put();
        }
        __syncthreads();
        if (w == 0) take();
        __syncthreads();   // (keeps the last sums apart from the stores: mixed by the compiler, they spill 20 registers)
        if (w != 0) return;
    }

    // lane owns rows i = .. + r16 and columns j = .. + g4 + 4 r of each block
    typedef __attribute__((address_space(1))) double* gpw;
    const gpw P = (gpw)g.P + split * M * N;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int64_t i = i0 + a * 16 + r16;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (!((mask >> (4 * a + c)) & 1u) || i >= M) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j = j0 + c * 16 + g4 + 4 * r;
                if (j < N) {
                    double v = acc[a][c][r];
                    if (g.accumulate_partials) v += P[i + j * M];
                    P[i + j * M] = v;
                }
            }
        }
    }
    if (fold && g4 == 0)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t i = i0 + t * 16 + r16;
            if (i < M) ((double*)g.Pc)[split * M + i] = cs[t];
        }
}

}  // namespace pne
