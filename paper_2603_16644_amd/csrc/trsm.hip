// A_p = A R_s^{-1} in FP64 (Algorithm 1, "Solve A_p = A R_s^{-1}", after
// R_s is promoted to double): block forward substitution
//   X_J = (A_J - sum_{I<J} X_I R_IJ) R_JJ^{-1}
// with every row of A handled by one wavefront from its first column to its
// last, in one launch.
//
// A wavefront owns 16 rows.  Its block of X sits in the accumulators of the
// FP64 MFMA 16x16x4: lane (r, g) (r = lane % 16, g = lane / 16) holds row r,
// register q of a 16-column block holds column g + 4 q.  Register q is at the
// same time exactly what an MFMA wants as its operand for the K values
// 4 q + g, so a finished block of X multiplies into the later ones straight
// from the accumulators, without a trip through LDS or memory.  Columns are
// taken in panels of up to 8 blocks (128 columns, 64 registers, which leaves
// room for three wavefronts per SIMD); a panel first subtracts the products
// with all earlier columns of X (read back from A_p by the lane that wrote
// them), then is solved block by block.
//
// Inside a block of 16 columns the substitution goes by groups of four: two
// MFMAs each, one with the inverse of the 4 x 4 diagonal block of R and one
// that removes the group from the columns right of it.  (An inverse of four
// columns changes rounding only, like the reciprocal of a pivot.)
//
// R is packed once (TrsmPack) in the order in which the MFMAs read it, with
// the sign changed.  The four wavefronts of a work-group (64 rows) share each
// 16-row strip of it through LDS, double-buffered, one barrier per strip: a
// strip is 32 MFMAs (2048 cycles) per wavefront.  HBM traffic is A once, X
// once and (n / 128 - 1) / 2 re-reads of X; the recursion of products and
// 64-column leaves this replaces read and wrote the right part of the matrix
// at every level (7.9 GB fetched at 100000 x 1000).
//
// Bound: FP64 MFMA (and, where the work-groups of 64 rows fill the machine's
// 768 places badly, its last round: 1563 work-groups at 100000 rows).
// Measured, recursion -> this: 1000 x 100 86 -> 21 us, 30011 x 257 250 -> 104
// us, 32768 x 400 0.39 -> 0.17 ms, 400000 x 500 3.9 -> 2.3 ms, 100000 x 1000
// 3.25 -> 2.38 ms, 1000000 x 2000 96 -> 73 ms (55 TFLOP/s), 64 members of
// m 2000..50000, n 32..512 9.5 -> 5.5 ms.  Panels of 12 and 16 blocks with two
// wavefronts per SIMD spilled registers (2.75 and 3.2 ms at 100000 x 1000; 8
// blocks with two wavefronts 2.50); a reload from scratch memory waits for
// every load in flight, so the loops must be free of them.
#include "common.h"
#include "kernels.h"
#include "launch.h"
#include "trsm_dev.h"

namespace pne {

size_t trsm_pack_bytes(int64_t n)
{
    const int64_t q = ceil_div(n, TB16);
    return (size_t)(q * (q + 1) / 2 * BLK + q * DTAB) * sizeof(double);
}

void trsm_right_upper(Exec& ex, int64_t m, int64_t n, const double* A, int64_t lda, const double* R,
                      int64_t ldr, double* Ap, int64_t ldap, double* pack)
{
    const int64_t nblk = ceil_div(n, TB16);
    launch<TrsmPack>(ex, nblk, nblk, TrsmPack::Args{n, R, ldr, pack});
    const TrsmArgs t{m, n, A, lda, pack, Ap, ldap};
    if (lda >= ((int64_t)1 << 26) || ldap >= ((int64_t)1 << 26)) launch<TrsmRows<true>>(ex, ceil_div(m, 64), 1, t);
    else launch<TrsmRows<false>>(ex, ceil_div(m, 64), 1, t);
}

}  // namespace pne
