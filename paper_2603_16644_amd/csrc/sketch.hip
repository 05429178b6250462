// Sketch A_s = Omega A (Algorithm 1, "Sketch"; Section 6.2), Omega an
// s x m Gaussian matrix with N(0, 1/s) entries drawn from the counter-based
// generator in philox.h.
//
// Pipeline per chunk of rows of A (bounded workspace for any m):
//   1. omega_gen: Omega(:, chunk) written once in the operand format, row
//      major (each sketch row contiguous over the chunk, zero padded to a
//      multiple of 64 columns).  VALU bound; every entry is drawn once.
//   2. quantize:  A(chunk, :) converted to the operand format, column major
//      (k contiguous), with per-(block, column) scales for FP16/FP8.
//   3. gemm_lp:   partial A_s += Omega_q A_q on MFMA 16x16 tiles with FP32
//      accumulation, split over K (rows of A) into fixed partial buffers.
// A final reduction sums the partials in a fixed order (bitwise
// reproducible) and applies 1/sqrt(s).
//
// Operand rounding (identical in the CPU reference): FP64 inputs go to FP32
// first, then RNE to BF16/FP16/E4M3.  FP16 uses power-of-two scales
// 2^(floor(log2 amax) - 14) per block of A, FP8 uses amax / 448 (FP32).
#include "common.h"
#include "convert.h"
#include "kernels.h"
#include "launch.h"
#include "philox.h"
#include "profile.h"

namespace pne {

template <int OP>
struct Op;
template <>
struct Op<OPK_F32> {
    typedef float T;
    static constexpr int KI = 4;   // K per MFMA
    static constexpr int EPL = 1;  // operand elements per lane
};
template <>
struct Op<OPK_BF16> {
    typedef uint16_t T;
    static constexpr int KI = 32;
    static constexpr int EPL = 8;
};
template <>
struct Op<OPK_F16> {
    typedef uint16_t T;
    static constexpr int KI = 32;
    static constexpr int EPL = 8;
};
template <>
struct Op<OPK_FP8> {
    typedef uint8_t T;
    static constexpr int KI = 32;
    static constexpr int EPL = 8;
};
template <>
struct Op<OPK_F64> {
    typedef double T;
    static constexpr int KI = 4;
    static constexpr int EPL = 1;
};

template <int OP>
__device__ __forceinline__ typename Op<OP>::T to_op(float x)
{
    if constexpr (OP == OPK_F32) return x;
    else if constexpr (OP == OPK_BF16) return f32_to_bf16_bits(x);
    else if constexpr (OP == OPK_F16) return f32_to_f16_bits(x);
    else if constexpr (OP == OPK_FP8) return f32_to_e4m3_bits(x);
    else return (double)x;
}

// ---------------------------------------------------------------- 1. Omega
// out[i * ldk + k] = Omega(i, k0 + k) in the operand format, i < s, k < kc;
// zero for kc <= k < ldk.
constexpr int OMEGA_QUADS = 8;   // row quads per thread
struct OmegaArgs {
    uint64_t seed;
    uint32_t pid;
    int64_t s, k0, kc, ldk;
    void* out;
};
template <int OP>
struct OmegaGen {
    typedef OmegaArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const OmegaArgs& a, int bx, int by);
};
template <int OP>
__device__ void OmegaGen<OP>::run(const OmegaArgs& a, int bx, int by)
{
    typedef typename Op<OP>::T T;
    const uint64_t seed = a.seed;
    const uint32_t pid = a.pid;
    const int64_t s = a.s, k0 = a.k0, kc = a.kc, ldk = a.ldk;
    T* __restrict__ out = (T*)a.out;
    const int64_t k = (int64_t)bx * 256 + threadIdx.x;
    if (k >= ldk) return;
    // OMEGA_QUADS quads of rows (4 rows each) per thread, same column k
    for (int qq = 0; qq < OMEGA_QUADS; ++qq) {
        const int64_t q = (int64_t)by * OMEGA_QUADS + qq;
        if (4 * q >= s) break;
        T v[4];
        if (k < kc) {
            Gauss4 g = omega_quad(seed, pid, (uint32_t)q, (uint32_t)(k0 + k));
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = to_op<OP>(g.z[t]);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = (T)0;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t i = 4 * q + t;
            if (i < s) out[i * ldk + k] = v[t];
        }
    }
}

// ---------------------------------------------------------------- 2. quantize A
constexpr int QUANT_PER = 4;     // rows per thread (unscaled formats)
// Unscaled formats: Aq[j * ldk + k] = op(A(k0 + k, j)); zero padding.
struct QuantArgs {
    const double* A;
    int64_t lda, k0, kc, ldk, br, n;
    void* Aq;
    float* sc;
};
template <int OP>
struct QuantizePlain {
    typedef QuantArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const QuantArgs& a, int bx, int by);
};
template <int OP>
__device__ void QuantizePlain<OP>::run(const QuantArgs& a, int bx, int by)
{
    typedef typename Op<OP>::T T;
    const double* __restrict__ A = a.A;
    const int64_t lda = a.lda, k0 = a.k0, kc = a.kc, ldk = a.ldk;
    T* __restrict__ Aq = (T*)a.Aq;
    const int64_t j = by;
    // QUANT_PER consecutive rows per thread: two 16-byte loads and one
    // 8-byte store when the column is aligned and the rows are all in range
    const int64_t kb = ((int64_t)bx * 256 + threadIdx.x) * QUANT_PER;
    if (kb >= ldk) return;
    const double* src = A + (k0 + kb) + j * lda;
    if (sizeof(T) == 2 && kb + QUANT_PER <= kc && (((uintptr_t)src) & 15) == 0) {
        const double2 v0 = *(const double2*)src, v1 = *(const double2*)(src + 2);
        const uint32_t q0 = (uint32_t)to_op<OP>((float)v0.x) | ((uint32_t)to_op<OP>((float)v0.y) << 16);
        const uint32_t q1 = (uint32_t)to_op<OP>((float)v1.x) | ((uint32_t)to_op<OP>((float)v1.y) << 16);
        *(uint2*)(Aq + j * ldk + kb) = make_uint2(q0, q1);
        return;
    }
#pragma unroll
    for (int t = 0; t < QUANT_PER; ++t) {
        const int64_t k = kb + t;
        if (k >= ldk) break;
        const float v = (k < kc) ? (float)A[(k0 + k) + j * lda] : 0.0f;
        Aq[j * ldk + k] = to_op<OP>(v);
    }
}

// Scaled formats: one scale per block of br rows of a column (br a multiple of
// 64).
template <int OP>
__device__ __forceinline__ float block_scale(float amax)
{
    if (amax == 0.0f) return 0.0f;
    if constexpr (OP == OPK_F16) {
        int E;
        frexpf(amax, &E);                   // amax = f 2^E, f in [0.5, 1)
        return ldexpf(1.0f, (E - 1) - 14);
    } else {
        return amax / 448.0f;
    }
}
template <int OP>
__device__ __forceinline__ typename Op<OP>::T scaled_op(float v, float scale)
{
    return to_op<OP>(scale != 0.0f ? v / scale : 0.0f);
}

// Blocks of up to 64 RPL rows: a wavefront takes QS_BLKS blocks of a column with
// their rows in registers, so A is read once and the work-groups are few: bound
// by memory (400,000 x 500 in blocks of 128 to FP8 0.45 ms; a work-group per block,
// 1.6e6 of them, 1.27 ms).
constexpr int QS_BLKS = 4;
template <int OP, int RPL>
struct QuantizeScaled {
    typedef QuantArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const Args& a, int bx, int by)
    {
        const int64_t kc = a.kc, ldk = a.ldk, br = a.br, n = a.n, j = by;
        const double* __restrict__ Aj = a.A + a.k0 + j * a.lda;
        typename Op<OP>::T* __restrict__ Qj = (typename Op<OP>::T*)a.Aq + j * ldk;
        const int lane = threadIdx.x & 63;
        const int64_t kb0 = ((int64_t)bx * 4 + (threadIdx.x >> 6)) * QS_BLKS;
        float v[QS_BLKS][RPL];
#pragma unroll
        for (int i = 0; i < QS_BLKS; ++i)
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int64_t r = (kb0 + i) * br + 64 * q + lane;
                v[i][q] = (64 * q < br && r < kc) ? (float)Aj[r] : 0.0f;
            }
#pragma unroll
        for (int i = 0; i < QS_BLKS; ++i) {
            float amax = 0.0f;
#pragma unroll
            for (int q = 0; q < RPL; ++q) amax = fmaxf(amax, fabsf(v[i][q]));
            const int64_t r0 = (kb0 + i) * br;
            const float scale = block_scale<OP>(wave_max(amax));
            if (r0 < ldk && lane == 0) a.sc[(kb0 + i) * n + j] = scale;
#pragma unroll
            for (int q = 0; q < RPL; ++q) {
                const int64_t r = r0 + 64 * q + lane;
                if (64 * q < br && r < ldk) Qj[r] = scaled_op<OP>(v[i][q], scale);
            }
        }
    }
};

// Longer blocks, and sketches with too few blocks to fill the machine: a
// work-group per block, its rows in registers up to 1024, else read twice.
template <int OP>
struct QuantizeBlock {
    typedef QuantArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const Args& a, int bx, int by)
    {
        __shared__ float red[4];
        const int64_t kc = a.kc, ldk = a.ldk, br = a.br, j = by, r0 = bx * br;
        const double* __restrict__ Aj = a.A + a.k0 + j * a.lda;
        typename Op<OP>::T* __restrict__ Qj = (typename Op<OP>::T*)a.Aq + j * ldk;
        const int tid = threadIdx.x;
        const bool held = br <= 1024;
        float v[4], amax = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t k = tid + 256 * q, r = r0 + k;
            v[q] = (k < br && r < kc) ? (float)Aj[r] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) amax = fmaxf(amax, fabsf(v[q]));
        if (!held)
            for (int64_t r = r0 + 1024 + tid; r < r0 + br && r < kc; r += NTH) amax = fmaxf(amax, fabsf((float)Aj[r]));
        amax = wave_max(amax);
        if ((tid & 63) == 0) red[tid >> 6] = amax;
        __syncthreads();
        const float scale = block_scale<OP>(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
        if (tid == 0) a.sc[bx * a.n + j] = scale;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t k = tid + 256 * q, r = r0 + k;
            if (k < br && r < ldk) Qj[r] = scaled_op<OP>(v[q], scale);
        }
        if (!held)
            for (int64_t r = r0 + 1024 + tid; r < r0 + br && r < ldk; r += NTH)
                Qj[r] = scaled_op<OP>(r < kc ? (float)Aj[r] : 0.0f, scale);
    }
};

// ---------------------------------------------------------------- 3. MFMA product
// P[i + j*M] (+)= sum_{k in split} Om[i*ldk + k] * Aq[j*ldk + k]  (per scale
// block multiplied by sc[kb*N + j] when SCALED).  128 x 128 output tile per
// work-group, 4 waves of 64 x 64, MFMA 16x16.  The MFMA A operand is the A
// side (columns j) and the B operand the Omega side (rows i), so lane l holds
// output rows i = l % 16 (contiguous in the column-major result).
constexpr int LP_BM = 128, LP_BN = 128, LP_BK = 64;

template <int OP>
__device__ __forceinline__ v4f mfma16(const typename Op<OP>::T* a, const typename Op<OP>::T* b,
                                      v4f c)
{
    if constexpr (OP == OPK_F32) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(*a, *b, c, 0, 0, 0);
    } else if constexpr (OP == OPK_BF16) {
        v8bf av = *(const v8bf*)a, bv = *(const v8bf*)b;
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
    } else if constexpr (OP == OPK_F16) {
        v8h av = *(const v8h*)a, bv = *(const v8h*)b;
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, c, 0, 0, 0);
    } else {
        long av = *(const long*)a, bv = *(const long*)b;
        return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(av, bv, c, 0, 0, 0);
    }
}

struct GemmLpArgs {
    const void* Om;
    const void* Aq;
    int64_t ldk, M, N;
    const float* sc;
    int64_t br;
    float* P;
    int64_t kchunk;
    int accumulate;
};
template <int OP, bool SCALED>
struct GemmLp {
    typedef GemmLpArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const GemmLpArgs& a, int bx, int by);
};
template <int OP, bool SCALED>
__device__ void GemmLp<OP, SCALED>::run(const GemmLpArgs& a, int bx, int by)
{
    typedef typename Op<OP>::T T;
    const T* __restrict__ Om = (const T*)a.Om;
    const T* __restrict__ Aq = (const T*)a.Aq;
    const int64_t ldk = a.ldk, M = a.M, N = a.N, br = a.br, kchunk = a.kchunk;
    const float* __restrict__ sc = a.sc;
    float* __restrict__ P = a.P;
    const int accumulate = a.accumulate;
    constexpr int E = sizeof(T);
    constexpr int PADE = 16 / E;                 // 16 bytes of padding per LDS row
    constexpr int LDR = LP_BK + PADE;            // LDS row length in elements
    constexpr int VPR = LP_BK * E / 16;          // 16-byte vectors per tile row
    constexpr int VPT = LP_BM * VPR / 256;       // vectors per thread per tile
    __shared__ __attribute__((aligned(16))) T As[LP_BM * LDR];
    __shared__ __attribute__((aligned(16))) T Bs[LP_BN * LDR];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w & 1, wn = w >> 1;
    const int64_t tiles_m = (M + LP_BM - 1) / LP_BM;
    const int64_t i0 = (int64_t)(bx % tiles_m) * LP_BM;
    const int64_t j0 = (int64_t)(bx / tiles_m) * LP_BN;
    const int64_t kbeg = (int64_t)by * kchunk;
    const int64_t kend = (kbeg + kchunk < ldk) ? kbeg + kchunk : ldk;

    v4f acc[4][4], tmp[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            acc[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
            tmp[a][b] = (v4f){0.f, 0.f, 0.f, 0.f};
        }

    uint4 ra[VPT], rb[VPT];
    auto gload = [&](int64_t k) {
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int v = tid + 256 * q;
            const int row = v / VPR, c = v % VPR;
            const int64_t gi = i0 + row, gj = j0 + row;
            const int64_t koff = k + (int64_t)c * (16 / E);
            ra[q] = (gi < M) ? *(const uint4*)(Om + gi * ldk + koff) : make_uint4(0, 0, 0, 0);
            rb[q] = (gj < N) ? *(const uint4*)(Aq + gj * ldk + koff) : make_uint4(0, 0, 0, 0);
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int v = tid + 256 * q;
            const int row = v / VPR, c = v % VPR;
            *(uint4*)(As + row * LDR + c * (16 / E)) = ra[q];
            *(uint4*)(Bs + row * LDR + c * (16 / E)) = rb[q];
        }
    };

    const int r16 = lane & 15, g4 = lane >> 4;
    int steps_in_block = 0;
    const int steps_per_block = SCALED ? (int)(br / LP_BK) : 1 << 30;
    if (kbeg < kend) gload(kbeg);
    for (int64_t k = kbeg; k < kend; k += LP_BK) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (k + LP_BK < kend) gload(k + LP_BK);
#pragma unroll
        for (int kk = 0; kk < LP_BK; kk += Op<OP>::KI) {
            const int ko = kk + g4 * Op<OP>::EPL;
            const T* pa[4];
            const T* pb[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                pb[t] = As + (wm * 64 + t * 16 + r16) * LDR + ko;   // Omega rows i
                pa[t] = Bs + (wn * 64 + t * 16 + r16) * LDR + ko;   // A columns j
            }
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
#pragma unroll
                for (int tj = 0; tj < 4; ++tj) {
                    if constexpr (SCALED) tmp[ti][tj] = mfma16<OP>(pa[tj], pb[ti], tmp[ti][tj]);
                    else acc[ti][tj] = mfma16<OP>(pa[tj], pb[ti], acc[ti][tj]);
                }
        }
        if constexpr (SCALED) {
            if (++steps_in_block == steps_per_block || k + LP_BK >= kend) {
                const int64_t kb = k / br;
#pragma unroll
                for (int tj = 0; tj < 4; ++tj)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int64_t j = j0 + wn * 64 + tj * 16 + 4 * g4 + r;
                        const float s = (j < N) ? sc[kb * N + j] : 0.0f;
#pragma unroll
                        for (int ti = 0; ti < 4; ++ti) {
                            acc[ti][tj][r] += tmp[ti][tj][r] * s;
                            tmp[ti][tj][r] = 0.0f;
                        }
                    }
                steps_in_block = 0;
            }
        }
    }
    float* Pp = P + (int64_t)by * M * N;
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
        const int64_t i = i0 + wm * 64 + ti * 16 + r16;
        if (i >= M) continue;
#pragma unroll
        for (int tj = 0; tj < 4; ++tj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j = j0 + wn * 64 + tj * 16 + 4 * g4 + r;
                if (j < N) {
                    float v = acc[ti][tj][r];
                    if (accumulate) v += Pp[i + j * M];
                    Pp[i + j * M] = v;
                }
            }
    }
}

// Wide variant for one large sketch: tiles of
// up to 256 x 256 per work-group of eight waves (2 x 4 waves of 16 TI x 16 TJ
// outputs), K tiles of 128 bytes per row, two LDS buffers (one barrier per
// K tile) and the next tile held in registers.  Twice the MFMA work of the
// 128 x 128 tile per byte brought in from L2.  Tile sizes: wide_tile.
//
// SCALED: a K tile lies in one scale block (br a multiple of the tile), its
// scales come to LDS with it, and the block's sum in tmp is scaled and added
// to acc at the block's end.  128 x 256 outputs then, for the two sets of
// accumulators; FP8 400,000 x 500 to 1500 rows 1.98 -> 0.66 ms against 128 x 128
// with two barriers per 64 rows and scales from memory.
template <int OP, int TI, int TJ, bool SCALED = false>
struct GemmLpW {
    typedef GemmLpArgs Args;
    static constexpr int NTH = 512, WPE = 2;
    static constexpr int LW_BM = 32 * TI, LW_BN = 64 * TJ;
    static __device__ void run(const GemmLpArgs& a, int bx, int by);
};
template <int OP, int TI, int TJ, bool SCALED>
__device__ void GemmLpW<OP, TI, TJ, SCALED>::run(const GemmLpArgs& a, int bx, int by)
{
    typedef typename Op<OP>::T T;
    const T* __restrict__ Om = (const T*)a.Om;
    const T* __restrict__ Aq = (const T*)a.Aq;
    const int64_t ldk = a.ldk, M = a.M, N = a.N, kchunk = a.kchunk;
    float* __restrict__ P = a.P;
    const int accumulate = a.accumulate;
    constexpr int E = sizeof(T);
    constexpr int BK = 128 / E;                  // K tile: 128 bytes per row
    constexpr int PADE = 16 / E;
    constexpr int LDR = BK + PADE;
    constexpr int VPR = 8;                       // 16-byte vectors per tile row
    constexpr int VA = (LW_BM * VPR + 511) / 512, VB = LW_BN * VPR / 512;   // vectors per thread
    __shared__ __attribute__((aligned(16))) T As[2][LW_BM * LDR];
    __shared__ __attribute__((aligned(16))) T Bs[2][LW_BN * LDR];
    __shared__ __attribute__((aligned(16))) float Ss[2][SCALED ? LW_BN : 1];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w & 1, wn = w >> 1;
    const int64_t tiles_m = (M + LW_BM - 1) / LW_BM;
    const int64_t i0 = (int64_t)(bx % tiles_m) * LW_BM;
    const int64_t j0 = (int64_t)(bx / tiles_m) * LW_BN;
    const int64_t kbeg = (int64_t)by * kchunk;
    const int64_t kend = (kbeg + kchunk < ldk) ? kbeg + kchunk : ldk;

    v4f acc[TI][TJ], tmp[SCALED ? TI : 1][SCALED ? TJ : 1];
#pragma unroll
    for (int x = 0; x < TI; ++x)
#pragma unroll
        for (int y = 0; y < TJ; ++y) {
            acc[x][y] = (v4f){0.f, 0.f, 0.f, 0.f};
            if constexpr (SCALED) tmp[x][y] = (v4f){0.f, 0.f, 0.f, 0.f};
        }

    uint4 ra[VA], rb[VB];
    float rs = 0.0f;
    auto gload = [&](int64_t k) {
        if constexpr (SCALED) rs = (tid < LW_BN && j0 + tid < N) ? a.sc[(int64_t)((uint32_t)k / (uint32_t)a.br) * N + j0 + tid] : 0.0f;
#pragma unroll
        for (int q = 0; q < VA; ++q) {
            const int v = tid + 512 * q;
            const int row = v / VPR, c = v % VPR;
            const int64_t gi = i0 + row;
            ra[q] = (row < LW_BM && gi < M) ? *(const uint4*)(Om + gi * ldk + k + c * (16 / E)) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < VB; ++q) {
            const int v = tid + 512 * q;
            const int row = v / VPR, c = v % VPR;
            const int64_t gj = j0 + row;
            rb[q] = (gj < N) ? *(const uint4*)(Aq + gj * ldk + k + c * (16 / E)) : make_uint4(0, 0, 0, 0);
        }
    };
    auto sstore = [&](int buf) {
        if constexpr (SCALED) {
            if (tid < LW_BN) Ss[buf][tid] = rs;
        }
#pragma unroll
        for (int q = 0; q < VA; ++q) {
            const int v = tid + 512 * q;
            const int row = v / VPR, c = v % VPR;
            if (row < LW_BM) *(uint4*)(As[buf] + row * LDR + c * (16 / E)) = ra[q];
        }
#pragma unroll
        for (int q = 0; q < VB; ++q) {
            const int v = tid + 512 * q;
            const int row = v / VPR, c = v % VPR;
            *(uint4*)(Bs[buf] + row * LDR + c * (16 / E)) = rb[q];
        }
    };

    const int r16 = lane & 15, g4 = lane >> 4;
    int buf = 0;
    if (kbeg < kend) {
        gload(kbeg);
        sstore(0);
        if (kbeg + BK < kend) gload(kbeg + BK);
    }
    for (int64_t k = kbeg; k < kend; k += BK) {
        __syncthreads();
        const T* as = As[buf];
        const T* bs = Bs[buf];
#pragma unroll
        for (int kk = 0; kk < BK; kk += Op<OP>::KI) {
            const int ko = kk + g4 * Op<OP>::EPL;
            const T* pa[TJ];
            const T* pb[TI];
#pragma unroll
            for (int t = 0; t < TI; ++t) pb[t] = as + (wm * 16 * TI + t * 16 + r16) * LDR + ko;   // Omega rows i
#pragma unroll
            for (int t = 0; t < TJ; ++t) pa[t] = bs + (wn * 16 * TJ + t * 16 + r16) * LDR + ko;   // A columns j
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) {
                    if constexpr (SCALED) tmp[ti][tj] = mfma16<OP>(pa[tj], pb[ti], tmp[ti][tj]);
                    else acc[ti][tj] = mfma16<OP>(pa[tj], pb[ti], acc[ti][tj]);
                }
        }
        if constexpr (SCALED) {
            if ((uint32_t)(k + BK) % (uint32_t)a.br == 0 || k + BK >= kend) {
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) {
                    const v4f sv = *(const v4f*)(Ss[buf] + wn * 16 * TJ + tj * 16 + 4 * g4);
#pragma unroll
                    for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[ti][tj][r] += tmp[ti][tj][r] * sv[r];
                        tmp[ti][tj] = (v4f){0.f, 0.f, 0.f, 0.f};
                    }
                }
            }
        }
        if (k + BK < kend) {
            sstore(buf ^ 1);
            if (k + 2 * BK < kend) gload(k + 2 * BK);
        }
        buf ^= 1;
    }
    float* Pp = P + (int64_t)by * M * N;
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
        const int64_t i = i0 + wm * 16 * TI + ti * 16 + r16;
        if (i >= M) continue;
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t j = j0 + wn * 16 * TJ + tj * 16 + 4 * g4 + r;
                if (j < N) {
                    float v = acc[ti][tj][r];
                    if (accumulate) v += Pp[i + j * M];
                    Pp[i + j * M] = v;
                }
            }
    }
}

// ---------------------------------------------------------------- 4. reduction
// As = scale * sum_split P[split]  (fixed order), written as FP32 and/or FP64.
struct SketchReduceArgs {
    const void* P;
    int64_t splits, M, N;
    double scale;
    float* o32;
    int64_t ld32;
    double* o64;
    int64_t ld64;
};
// (G threads per entry: as GemmReduce.)
template <typename TP, int G>
struct SketchReduce {
    typedef SketchReduceArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const SketchReduceArgs& a, int bx, int by);
};
template <typename TP, int G>
__device__ void SketchReduce<TP, G>::run(const SketchReduceArgs& a, int bx, int)
{
    __shared__ TP lds[G > 1 ? 256 : 1];
    constexpr int E = 256 / G;
    const TP* __restrict__ P = (const TP*)a.P;
    const int64_t splits = a.splits, M = a.M, N = a.N, ld32 = a.ld32, ld64 = a.ld64;
    const double scale = a.scale;
    float* __restrict__ o32 = a.o32;
    double* __restrict__ o64 = a.o64;
    const int64_t idx = (int64_t)bx * E + threadIdx.x % E;
    const bool in = idx < M * N;
    TP s = 0;
    if (in) s = slot_sum<G>(P + idx, M * N, splits, threadIdx.x / E);
    s = slot_total<G>(s, lds);
    if (!in || threadIdx.x >= E) return;
    const int64_t i = idx % M, j = idx / M;
    if (o32) o32[i + j * ld32] = (float)(s * (TP)scale);
    if (o64) o64[i + j * ld64] = (double)s * scale;
}

// ---------------------------------------------------------------- host driver
size_t sketch_workspace_bytes(int64_t m, int64_t n, int64_t s, int prec, int64_t br, int64_t kchunk_fixed)
{
    SketchPlan p = plan_sketch(m, n, s, prec, br, kchunk_fixed);
    return p.bytes;
}

// For a caller who has not given the block length yet: FP8 and FP16 sketches
// take the narrow product, with four times the partial sums, for some.
size_t sketch_workspace_bytes_any(int64_t m, int64_t n, int64_t s, int prec)
{
    const size_t wide = plan_sketch(m, n, s, prec, 128).bytes, narrow = plan_sketch(m, n, s, prec, 128, 0, true).bytes;
    return wide > narrow ? wide : narrow;
}

// Tile (32 wm x 64 wn) and split count of the wide kernel.  One work-group
// runs per CU, the largest split count whose work-groups fit the machine at
// once: the time is that of (rounds of 256 work-groups) x (tile) / (splits).
// 256 x 256 reads least from LDS and L2 per product, which BF16 is bound by;
// FP32 is bound by the matrix cores, where a smaller tile that leaves fewer
// CUs idle or pads less is faster: 6000 x 2000 is 192 tiles of 256 x 256 or
// 256 of 192 x 256, 771 x 257 is 8 of 256 x 256 (62% padding) or 15 of 160 x
// 128.  Measured: 6000 x 2000 x 1e6 257 -> 197 ms (122 TFLOP/s), 771 x 257 x
// 30011 0.28 -> 0.18 ms.  A smaller tile never takes more splits, so the partial sums stay
// within the space of 256 x 256.
static void wide_tile(int64_t s, int64_t n, int op, int64_t maxsplit, int* wm, int* wn, int64_t* splits)
{
    static const int tiles[][2] = {{8, 4}, {6, 4}, {6, 2}, {5, 3}, {5, 2}};
    double best = 0.0;
    for (const auto& t : tiles) {
        const int64_t nt = ceil_div(s, 32 * t[0]) * ceil_div(n, 64 * t[1]);
        int64_t sp = 256 / nt;
        sp = sp < 1 ? 1 : (sp < maxsplit ? sp : maxsplit);
        const double cost = (double)ceil_div(nt * sp, 256) * t[0] * t[1] / sp;
        if (best == 0.0 || cost < best) {
            best = cost;
            *wm = t[0];
            *wn = t[1];
            *splits = sp;
        }
        if (op != OPK_F32) return;
    }
}
// Split count of the narrow product: tiles x splits fill the machine.
static int64_t narrow_splits(int64_t s, int64_t n, int64_t maxsplit)
{
    const int64_t want = ceil_div(1024, ceil_div(s, LP_BM) * ceil_div(n, LP_BN));   // (FP64 tiles are as large)
    return want < maxsplit ? want : maxsplit;
}
// Scaled sketches for the wide kernel: blocks that hold whole K tiles (128 bytes
// per row).  Not FP16 where the splits are longer than 1024 rows (a split holds four
// blocks) and do not fill the machine even in the narrow product's tiles,
// whose K steps then take less time: 20,000 x 200 in blocks of 1024 to FP16 78
// us, wide 86; of 256 34 and 34; 20,000 x 1000 in blocks of 1024 315 and 212.
static bool wide_scaled(int64_t s, int64_t n, int op, int64_t br, int64_t maxsplit)
{
    if ((op != OPK_FP8 && op != OPK_F16) || br % (128 / opk_bytes(op)) != 0) return false;
    return op == OPK_FP8 || br <= 256 ||
           ceil_div(s, LP_BM) * ceil_div(n, LP_BN) * narrow_splits(s, n, maxsplit) >= 256;
}
template <int OP>
static void wide_launch(Exec& ex, const SketchPlan& p, int64_t s, int64_t n, const GemmLpArgs& a)
{
    const int64_t gx = ceil_div(s, 32 * p.wm) * ceil_div(n, 64 * p.wn);
    if constexpr (OP == OPK_F32) {
        if (p.wm == 6 && p.wn == 4) return launch<GemmLpW<OP, 6, 4>>(ex, gx, p.splits, a);
        if (p.wm == 6 && p.wn == 2) return launch<GemmLpW<OP, 6, 2>>(ex, gx, p.splits, a);
        if (p.wm == 5 && p.wn == 3) return launch<GemmLpW<OP, 5, 3>>(ex, gx, p.splits, a);
        if (p.wm == 5 && p.wn == 2) return launch<GemmLpW<OP, 5, 2>>(ex, gx, p.splits, a);
    }
    if constexpr (OP == OPK_FP8 || OP == OPK_F16) launch<GemmLpW<OP, 4, 4, true>>(ex, gx, p.splits, a);
    else launch<GemmLpW<OP, 8, 4>>(ex, gx, p.splits, a);
}

SketchPlan plan_sketch(int64_t m, int64_t n, int64_t s, int prec, int64_t br, int64_t kchunk_fixed, bool narrow)
{
    SketchPlan p{};
    const int op = prec_to_opk(prec);
    const int64_t E = opk_bytes(op);
    // rows of A per chunk: keep Omega_q of one chunk below ~1 GiB
    int64_t max_chunk = ((int64_t)1 << 30) / (E * (s > 0 ? s : 1));
    int64_t align = (op == OPK_FP8 || op == OPK_F16) ? (br > 64 ? br : 64) : 64;
    max_chunk = (max_chunk / align) * align;
    if (max_chunk < align) max_chunk = align;
    int64_t mpad = ceil_div(m, align) * align;
    p.chunk = mpad < max_chunk ? mpad : max_chunk;
    p.nchunks = ceil_div(m, p.chunk);
    p.ldk = p.chunk;  // multiple of 64
    if (kchunk_fixed > 0) {
        // batches: K chunks of a fixed length (a multiple of the alignment)
        int64_t kc = ceil_div(kchunk_fixed, align) * align;
        if (kc > p.ldk) kc = p.ldk;
        p.kchunk = kc;
        p.splits = ceil_div(p.ldk, kc);
    } else {
        int64_t maxsplit = p.ldk / (4 * align);
        if (maxsplit < 1) maxsplit = 1;
        if (op == OPK_BF16 || op == OPK_F32) {
            wide_tile(s, n, op, maxsplit, &p.wm, &p.wn, &p.splits);
        } else if (wide_scaled(s, n, op, br, maxsplit) && !narrow) {
            // the same with 128 x 256 tiles
            p.wm = 4;
            p.wn = 4;
            const int64_t want = 256 / (ceil_div(s, 128) * ceil_div(n, 256));
            p.splits = want < 1 ? 1 : (want < maxsplit ? want : maxsplit);
        } else {
            p.splits = narrow_splits(s, n, maxsplit);
        }
        p.kchunk = ceil_div(ceil_div(p.ldk, p.splits), align) * align;
        p.splits = ceil_div(p.ldk, p.kchunk);
    }
    p.op = op;
    Arena ar(nullptr, 0);
    ar.take<char>((size_t)s * p.ldk * E);                           // Omega_q
    if (op != OPK_F64) ar.take<char>((size_t)n * p.ldk * E);        // A_q
    if (op == OPK_FP8 || op == OPK_F16) ar.take<float>((size_t)ceil_div(p.ldk, br) * n);
    ar.take<char>((size_t)p.splits * s * n * (op == OPK_F64 ? 8 : 4));  // partials
    p.bytes = ar.used;
    return p;
}

// Generation of Omega (arithmetic-bound) and conversion of A (memory-bound)
// in one launch, their work-groups interleaved in proportion to their
// counts so that the two run side by side: work-group b is Omega work-group
// floor(b * G_o / G) when that index steps at b, otherwise conversion
// work-group b - floor(b * G_o / G).
struct SketchPrepArgs {
    OmegaArgs o;
    QuantArgs q;
    int64_t ogx, ogn, qgx, total;
};
template <int OP>
struct SketchPrep {
    typedef SketchPrepArgs Args;
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const SketchPrepArgs& a, int bx, int)
    {
        const int64_t b = bx;
        const int64_t oi = b * a.ogn / a.total, oi1 = (b + 1) * a.ogn / a.total;
        if (oi1 > oi) {
            OmegaGen<OP>::run(a.o, (int)(oi % a.ogx), (int)(oi / a.ogx));
        } else {
            const int64_t qi = b - oi;
            QuantizePlain<OP>::run(a.q, (int)(qi % a.qgx), (int)(qi / a.qgx));
        }
    }
};

template <int OP>
static void launch_chunk(Exec& ex, const SketchPlan& p, const double* A, int64_t lda, int64_t k0,
                         int64_t kc, int64_t n, int64_t s, uint64_t seed, uint32_t pid, int64_t br,
                         void* Omq, void* Aq, float* sc, void* P, int accumulate)
{
    const OmegaArgs oa{seed, pid, s, k0, kc, p.ldk, Omq};
    const int64_t ogx = ceil_div(p.ldk, 256), ogy = ceil_div(ceil_div(s, 4), OMEGA_QUADS);
    constexpr bool SC = (OP == OPK_FP8 || OP == OPK_F16);
    if constexpr (OP != OPK_F64 && !SC) {
        // Omega and the conversion of A in one launch
        const QuantArgs q{A, lda, k0, kc, p.ldk, br, n, Aq, sc};
        const int64_t qgx = ceil_div(p.ldk, 256 * QUANT_PER);
        const int64_t ogn = ogx * ogy, total = ogn + qgx * n;
        launch<SketchPrep<OP>>(ex, total, 1, SketchPrepArgs{oa, q, ogx, ogn, qgx, total});
        if (!ex.recording()) {
            prof_mark(PH_SK_OMEGA, ex.st);
            prof_mark(PH_SK_QUANT, ex.st);
        }
    } else {
        launch<OmegaGen<OP>>(ex, ogx, ogy, oa);
        if (!ex.recording()) prof_mark(PH_SK_OMEGA, ex.st);
    }
    if constexpr (OP == OPK_F64) {
        // C(s x n) = Omega_q (rows contiguous over k) * A(chunk rows)
        GemmArgs g{};
        g.M = s; g.N = n; g.K = kc;
        g.A = Omq; g.lda = p.ldk; g.transA = 1;
        g.B = A + k0; g.ldb = lda; g.transB = 0;
        g.splits = p.splits; g.kchunk = p.kchunk;
        g.P = (double*)P; g.accumulate_partials = accumulate;
        gemm_f64_partials(ex, g);
    } else {
        if constexpr (SC) {
            const QuantArgs q{A, lda, k0, kc, p.ldk, br, n, Aq, sc};
            // QuantizeScaled takes blocks of up to 384 rows (400,000 x 500 in
            // blocks of 320 0.62 ms, 0.69 with a work-group per block, of 512 0.57
            // and 0.48) where there are many: launching a work-group per block
            // costs 0.5 us per thousand, against the few that QuantizeScaled has
            // for few blocks, each for longer the longer its blocks are (scaled and
            // block, us: blocks of 128, 2000 x 30 4.6 and 2.2, 30,000 x 16 4.7 and
            // 4.0, 30,000 x 32 5.1 and 6.5; of 256, 30,000 x 100 12.4 and 10.9, x 160
            // 14.9 and 16.8; of 64, 4096 x 48 3.8 and 3.4, x 64 3.9 and 4.0)
            const int64_t blocks = ceil_div(p.ldk, br), wgs = ceil_div(blocks, 4 * QS_BLKS);
            const bool many = blocks * n >= 40 * br || ex.recording();
            if (many && br <= 256) launch<QuantizeScaled<OP, 4>>(ex, wgs, n, q);
            else if (many && br <= 384) launch<QuantizeScaled<OP, 8>>(ex, wgs, n, q);
            else launch<QuantizeBlock<OP>>(ex, blocks, n, q);
            if (!ex.recording()) prof_mark(PH_SK_QUANT, ex.st);
        }
        const GemmLpArgs ga{Omq, Aq, p.ldk, s, n, sc, br, (float*)P, p.kchunk, accumulate};
        if (p.wm) {
            wide_launch<OP>(ex, p, s, n, ga);
            if (!ex.recording()) prof_mark(PH_SK_GEMM, ex.st);
            return;
        }
        launch<GemmLp<OP, SC>>(ex, ceil_div(s, LP_BM) * ceil_div(n, LP_BN), p.splits, ga);
    }
    if (!ex.recording()) prof_mark(PH_SK_GEMM, ex.st);
}

// A_s = Omega A in precision `prec`; writes As32 (ld32) and/or As64 (ld64).
int sketch_run(Exec& ex, int64_t m, int64_t n, const double* A, int64_t lda, int64_t s, uint64_t seed,
               uint32_t pid, int prec, int64_t br, float* As32, int64_t ld32, double* As64,
               int64_t ld64, void* work, size_t work_bytes)
{
    SketchPlan p = plan_sketch(m, n, s, prec, br, ex.kchunk_fixed);
    if (work_bytes < p.bytes) return PNE_EWORKSPACE;
    ex.stage(ST_SKETCH);
    const int64_t E = opk_bytes(p.op);
    Arena ar(work, work_bytes);
    void* Omq = ar.take<char>((size_t)s * p.ldk * E);
    void* Aq = (p.op != OPK_F64) ? (void*)ar.take<char>((size_t)n * p.ldk * E) : nullptr;
    float* sc = (p.op == OPK_FP8 || p.op == OPK_F16) ? ar.take<float>((size_t)ceil_div(p.ldk, br) * n)
                                                      : nullptr;
    void* P = ar.take<char>((size_t)p.splits * s * n * (p.op == OPK_F64 ? 8 : 4));
    for (int64_t c = 0; c < p.nchunks; ++c) {
        const int64_t k0 = c * p.chunk;
        const int64_t kc = (m - k0 < p.chunk) ? m - k0 : p.chunk;
        const int acc = c > 0;
        ex.iter((uint32_t)c);
        switch (p.op) {
        case OPK_F64: launch_chunk<OPK_F64>(ex, p, A, lda, k0, kc, n, s, seed, pid, br, Omq, Aq, sc, P, acc); break;
        case OPK_F32: launch_chunk<OPK_F32>(ex, p, A, lda, k0, kc, n, s, seed, pid, br, Omq, Aq, sc, P, acc); break;
        case OPK_BF16: launch_chunk<OPK_BF16>(ex, p, A, lda, k0, kc, n, s, seed, pid, br, Omq, Aq, sc, P, acc); break;
        case OPK_F16: launch_chunk<OPK_F16>(ex, p, A, lda, k0, kc, n, s, seed, pid, br, Omq, Aq, sc, P, acc); break;
        case OPK_FP8: launch_chunk<OPK_FP8>(ex, p, A, lda, k0, kc, n, s, seed, pid, br, Omq, Aq, sc, P, acc); break;
        }
    }
    ex.stage(ST_SKETCH_REDUCE);
    const double scale = 1.0 / sqrt((double)s);
    const SketchReduceArgs ra{P, p.splits, s, n, scale, As32, ld32, As64, ld64};
    if (p.splits >= 32) {
        if (p.op == OPK_F64) launch<SketchReduce<double, 16>>(ex, ceil_div(s * n, 16), 1, ra);
        else launch<SketchReduce<float, 16>>(ex, ceil_div(s * n, 16), 1, ra);
    } else {
        if (p.op == OPK_F64) launch<SketchReduce<double, 1>>(ex, ceil_div(s * n, 256), 1, ra);
        else launch<SketchReduce<float, 1>>(ex, ceil_div(s * n, 256), 1, ra);
    }
    if (!ex.recording()) prof_mark(PH_SK_REDUCE, ex.st);
    return launch_status(ex);
}

}  // namespace pne
