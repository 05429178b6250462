// Split-K products C = A^T B in FP64 of two tall operands whose K direction
// is contiguous in memory (A: K x M, B: K x N, column-major), in 64 x 64
// output tiles: the Gram products A_p^T A_p and A_p^T A with A_p^T b, B^T A
// of the not-normal equations and small FP64 sketches (see tn_route for the
// sizes; larger products run in 128 x 128 tiles in gemm.hip), and the FP64
// Gram matrix of an FP32 sketch (gram_f32).
//
// An FP64 MFMA 16x16x4 keeps a SIMD's matrix core busy for 64 cycles and
// needs one operand value per lane and side.  A wavefront holds the 64 x 64
// block of C (4 x 4 MFMA blocks, 128 registers), and the four wavefronts of
// the work-group split its K chunk and are summed through LDS at the end.
// Lane (r, g) (r = lane % 16, g = lane / 16) takes 16 bytes of column r of
// each 16-column block, the K values k + 2 g, k + 2 g + 1, and MFMA h of the
// step multiplies the h-th value of every lane: its four K values are
// k + 2 g + h, g = 0..3, the same on both sides.  8 such loads per 32 MFMAs
// are little enough to load straight from memory into the MFMA registers: no
// LDS and no barriers in the loop, the wavefronts run free of each other;
// two register buffers, the next step loads while the current one multiplies
// (2048 cycles, twice that with two wavefronts per SIMD, against about 1000
// cycles of memory latency).  MFMA blocks outside the matrix, and above the
// diagonal of a lower-triangle product, are skipped (a 16-bit mask), so a
// ragged order pays for 16-column blocks instead of 64-column tiles.
//
// Measured against the LDS-staged 64 x 64 and 128 x 128 tiles of gemm.hip:
// the Gram products of 64 members (m 2000..50000, n 32..512) 6.67 -> 4.87 ms,
// of 30011 x 257 123 -> 72 us, A_p^T A of 32768 x 400 334 -> 260 us.
#include "common.h"
#include "gemm_tn_dev.h"
#include "kernels.h"
#include "launch.h"
#include "tune.h"

namespace pne {

// Products that run here: lower triangles in 64 x 64 tiles (tile_shape in
// gemm.hip), short K, and full products of order up to 512 whose operands
// together fit the 256 MB memory-side cache.  Beyond that the tiles'
// wavefronts, which nothing keeps in step, re-read the operands from HBM:
// A_p^T A of 400000 x 500 (3.2 GB) takes 4.8 ms here and 4.1 ms in 128 x 128
// tiles, of 32768 x 400 (0.2 GB) 0.26 and 0.33 ms.
bool tn_route(int64_t M, int64_t N, int64_t K, int lower)
{
    if (lower || K < 4096) return gemm_tile_is_64(M, N, K, lower);
    return M <= 512 && N <= 512 && 8 * K * (M + N) <= ((int64_t)256 << 20);
}

int64_t tn_tiles(int64_t M, int64_t N, int lower)
{
    const int64_t tm = ceil_div(M, 64), tn = ceil_div(N, 64);
    return lower ? tm * (tm + 1) / 2 : tm * tn;
}

void gemm_tn_partials(Exec& ex, const GemmArgs& g0)
{
    GemmArgs g = g0;
    if (g.splits < 1) g.splits = 1;
    if (g.kchunk <= 0) g.kchunk = ceil_div(ceil_div(g.K, g.splits), 16) * 16;
    g.xcd_remap = !ex.recording() && g.splits > 1;
    const int64_t tiles = tn_tiles(g.M, g.N, g.lower);
    if (g.lda >= ((int64_t)1 << 23) || g.ldb >= ((int64_t)1 << 23)) launch<GemmTn<double, true>>(ex, tiles, g.splits, g);
    else launch<GemmTn<double, false>>(ex, tiles, g.splits, g);
}

// Lower triangle of G = W^T W in FP64 for an FP32 W (rows x n, ld ldw < 2^23;
// the products are exact in FP64).  P: partials, room for pslots n x n FP64
// matrices; one K chunk is written straight into G.
void gram_f32(Exec& ex, int64_t rows, int64_t n, const float* W, int64_t ldw, double* G, double* P, int64_t pslots)
{
    GemmArgs g{};
    g.M = n; g.N = n; g.K = rows;
    g.A = W; g.lda = ldw; g.transA = 1;
    g.B = W; g.ldb = ldw; g.transB = 0;
    g.alpha = 1.0;
    g.C = G; g.ldc = n;
    g.lower = 1;
    // two work-groups per CU, chunks of 256 rows at least
    const int64_t tiles = tn_tiles(n, n, 1);
    int64_t sp = 512 / tiles;
    if (sp > rows / 256) sp = rows / 256;
    if (sp > pslots) sp = pslots;
    if (sp < 1) sp = 1;
    g.kchunk = ceil_div(ceil_div(rows, sp), 16) * 16;
    g.splits = ceil_div(rows, g.kchunk);
    g.P = g.splits > 1 ? (void*)P : (void*)G;
    g.xcd_remap = !ex.recording() && g.splits > 1;
    launch<GemmTn<float, false>>(ex, tiles, g.splits, g);
    if (g.splits > 1) gemm_f64_reduce(ex, g);
}

}  // namespace pne
