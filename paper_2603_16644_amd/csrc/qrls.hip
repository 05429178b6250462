// FP64 Householder-QR least-squares solver on the GPU: the direct method the
// paper compares PNE/HPNE against (Section 7.4, a QR solver built from
// geqrf, orgqr and trsm).  Here Q is never formed: the QR of the augmented
// matrix [A b] yields R and Q^T b together, and
//   [A b] = Q [R_A  c; 0  rho]   =>   x = R_A^{-1} c
// (rho = ||b - A x|| is not formed: b takes A's reflectors and has none).
// The tall QR is the communication-avoiding FP64 Householder QR of caqr.hip;
// R_A x = c uses the block-parallel triangular solve.
#include "common.h"
#include "kernels.h"
#include "launch.h"

namespace pne {

namespace {

constexpr int64_t QRLS_NMAX = 3071;   // widest A

// W (h x (n + 1), ld h) = [A b], zero below row m.
struct AugCopy {
    struct Args {
        int64_t h, m, n, lda;
        const double* A;
        const double* b;
        double* W;
    };
    static constexpr int NTH = 256, WPE = 0;
    static __device__ void run(const Args& a, int bx, int by)
    {
        const int64_t i = (int64_t)bx * 256 + threadIdx.x;
        const int64_t j = by;   // column 0..n (n = b)
        if (i >= a.h) return;
        double v = 0.0;
        if (i < a.m) v = j < a.n ? a.A[i + j * a.lda] : a.b[i];
        a.W[i + j * a.h] = v;
    }
};

// rows of W: a square A has one row less than [A b] has columns
int64_t qrls_rows(int64_t m, int64_t n) { return m > n ? m : n + 1; }

struct QrlsBuffers {
    double *W, *R, *DR;
    int32_t* flags;
    char* qrws;
};

size_t qrls_layout(int64_t m, int64_t n, void* base, size_t cap, QrlsBuffers* out)
{
    QrlsBuffers b{};
    Arena ar(base, cap);
    const int64_t N1 = n + 1, h = qrls_rows(m, n);
    b.W = ar.take<double>((size_t)h * N1);
    b.R = ar.take<double>((size_t)N1 * N1);
    b.DR = ar.take<double>(dinv_elems(n));
    b.flags = ar.take<int32_t>(lb_flag_words(n));
    b.qrws = ar.take<char>(caqr_workspace_bytes(h));
    if (out) *out = b;
    return ar.used;
}

pne_status qrls_check(int64_t m, int64_t n, int64_t lda)
{
    if (n < 1 || m < n || lda < m) return PNE_EINVAL;
    if (n > QRLS_NMAX) return PNE_ENOTSUP;
    return PNE_OK;
}

}  // namespace

}  // namespace pne

using namespace pne;

extern "C" {

size_t qr_ls_workspace_size(int64_t m, int64_t n)
{
    if (qrls_check(m, n, m) != PNE_OK) return 0;
    return qrls_layout(m, n, nullptr, 0, nullptr);
}

pne_status qr_ls_solve(int64_t m, int64_t n, const double* dA, int64_t lda, const double* db, double* dx,
                       void* dwork, size_t work_bytes, int32_t* dinfo, pne_stream_t stream)
{
    pne_status chk = qrls_check(m, n, lda);
    if (chk) return chk;
    if (!dA || !db || !dx || !dinfo || !dwork) return PNE_EINVAL;
    QrlsBuffers b;
    if (work_bytes < qrls_layout(m, n, dwork, work_bytes, &b)) return PNE_EWORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    Exec ex;
    ex.st = st;
    zero_i32(ex, 1, dinfo);
    const int64_t h = qrls_rows(m, n);
    launch<AugCopy>(ex, ceil_div(h, 256), n + 1, AugCopy::Args{h, m, n, lda, dA, db, b.W});
    // R of [A b]: R_A = R(0:n, 0:n), c = R(0:n, n)
    const int64_t ldr = n + 1;
    const double* R = b.R;
    const int rc = qr_f64(ex, h, n + 1, n, b.W, h, b.R, ldr, dinfo, b.qrws, caqr_workspace_bytes(h));
    if (rc) return (pne_status)rc;
    inv_diag64(ex, n, InvTriMat{R, ldr, 0, 0, b.DR, nullptr});
    upper_solve_lb(ex, n, R, ldr, b.DR, R + n * ldr, dx, b.flags, dinfo);
    fill_nan_on_info(ex, n, dx, dinfo);
    return hipGetLastError() == hipSuccess ? PNE_OK : PNE_EHIP;
}

}  // extern "C"
