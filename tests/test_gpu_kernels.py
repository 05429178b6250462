"""Single kernels at the sizes where their tilings can go wrong, through the
C ABI, against FP64 products of the same inputs on the host."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def pne():
    import paper_2603_16644_amd as p
    p.lib()
    return p


def dev(a, lda=None):
    """Column-major device copy with leading dimension lda."""
    m, n = a.shape
    lda = m if lda is None else lda
    t = torch.empty(n, lda, dtype=torch.float64, device="cuda")
    t[:, :m] = torch.from_numpy(np.ascontiguousarray(a.T)).cuda()
    return t[:, :m].t()


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("m,n,lda", [
    (1, 1, 1), (17, 16, 17), (63, 17, 64), (100, 100, 101),      # less than one K turn per wavefront
    (4097, 64, 4097), (4801, 65, 4804), (5003, 130, 5003),       # tile edges, K remainders, odd columns
    (9000, 511, 9001), (20000, 512, 20000),                      # the largest order in 64 x 64 tiles
    (5000, 20, (1 << 23) + 2),                                   # 64-bit lane offsets
])
def test_gram_register_tiles(pne, hpne, m, n, lda):
    """C = A^T A and c = A^T b with R = I: the 64 x 64 split-K tiles whose
    wavefronts load their operands straight into registers.  A sum of m
    products in any order is within m u sum |a_ki| |a_kj| of the exact one,
    on both sides."""
    rng = np.random.default_rng(77 + m + n)
    A = rng.standard_normal((m, n))
    b = rng.standard_normal(m)
    Cg, cg, _, info = pne.pne_gram(dev(A, lda), torch.from_numpy(b).cuda(), dev(np.eye(n)), hpne=hpne)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    C, c = A.T @ A, A.T @ b
    tol = 2 * m * U
    sel = np.ones((n, n), bool) if hpne else np.tril(np.ones((n, n), bool))
    assert np.all(np.abs(Cg.cpu().numpy() - C)[sel] <= (tol * (np.abs(A).T @ np.abs(A)))[sel])
    assert np.all(np.abs(cg.cpu().numpy() - c) <= tol * (np.abs(A).T @ np.abs(b)))


def well_conditioned_r(n, rng):
    """Upper triangular with a diagonal in [1, 2] and small entries above it."""
    return np.triu(rng.standard_normal((n, n)), 1) * (0.5 / np.sqrt(n)) + np.diag(1.0 + rng.random(n))


@pytest.mark.parametrize("m,n,lda", [
    (1, 1, 1), (16, 16, 16), (65, 17, 65), (63, 63, 64), (1000, 100, 1001),   # blocks, rows past the tile
    (300, 128, 301), (300, 129, 300),             # one panel; two, packed R in the shared scratch
    (1000, 257, 1001), (777, 385, 777),           # panels of 6 and 7 blocks, odd column starts
    (1000, 3, 1 << 26),                           # 64-bit lane offsets
])
def test_right_substitution(pne, m, n, lda):
    """A_p = A R^{-1} seen through C = A_p^T A_p.  Substitution in blocks
    gives |dA_p| <= (n + 16) u |A_p| |R| |R^{-1}| elementwise (16: the group
    inverses), the product another m u |A_p|^T |A_p|; the reference on the
    host errs by no more."""
    from scipy.linalg import solve_triangular
    rng = np.random.default_rng(91 + m + n)
    A = rng.standard_normal((m, n))
    b = rng.standard_normal(m)
    R = well_conditioned_r(n, rng)
    Cg, cg, _, info = pne.pne_gram(dev(A, lda), torch.from_numpy(b).cuda(), dev(R))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    Ap = solve_triangular(R, A.T, trans="T", lower=False).T
    G = np.abs(Ap) @ np.abs(R) @ np.abs(np.linalg.inv(R))
    aAp = np.abs(Ap)
    tol = 2 * ((n + 16) * U * (G.T @ aAp + aAp.T @ G) + m * U * (aAp.T @ aAp))
    sel = np.tril(np.ones((n, n), bool))
    assert np.all((np.abs(Cg.cpu().numpy() - Ap.T @ Ap) <= tol)[sel])
    tolc = 2 * ((n + 16) * U * (G.T @ np.abs(b)) + m * U * (aAp.T @ np.abs(b)))
    assert np.all(np.abs(cg.cpu().numpy() - Ap.T @ b) <= tolc)


@pytest.mark.parametrize("col", [0, 2, 5, 15, 16, 40])
@pytest.mark.parametrize("val", [float("nan"), float("inf")])
def test_right_substitution_nonfinite_column(pne, col, val):
    """A non-finite entry of A reaches the columns of A_p from its own on, and
    none to the left of it."""
    m, n = 200, 48
    rng = np.random.default_rng(3)
    A = rng.standard_normal((m, n))
    A[77, col] = val
    R = well_conditioned_r(n, rng)
    Cg, _, _, _ = pne.pne_gram(dev(A), torch.zeros(m, dtype=torch.float64, device="cuda"), dev(R))
    d = np.diag(Cg.cpu().numpy())
    assert np.all(np.isfinite(d[:col])) and not np.any(np.isfinite(d[col:]))


@pytest.mark.parametrize("n", [1, 3, 5, 16, 17, 63, 64, 65, 81, 128, 130, 257, 700])
def test_cholesky_blocks(pne, n):
    """The factor of C = A^T A (R = I): groups of four, blocks of 16 and 64 and
    their remainders.  Cholesky's backward error |L L^T - C| <= (n + 1) u |L|
    |L|^T, widened by the inverses of four columns (16) and the rounding of
    the product (2)."""
    m = n + 300
    rng = np.random.default_rng(17 + n)
    A = rng.standard_normal((m, n)) * np.exp(rng.uniform(-3, 3, n))   # columns of unequal size
    b = np.zeros(m)
    C0, _, _, _ = pne.pne_gram(dev(A), torch.from_numpy(b).cuda(), dev(np.eye(n)))
    L, _, _, info = pne.pne_gram(dev(A), torch.from_numpy(b).cuda(), dev(np.eye(n)), factor=True)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    C, L = np.tril(C0.cpu().numpy()), np.tril(L.cpu().numpy())
    tol = (n + 19) * U * np.abs(L) @ np.abs(L).T
    assert np.all(np.abs(np.tril(L @ L.T) - C) <= np.tril(2 * tol))
    assert np.all(np.diag(L) > 0)


@pytest.mark.parametrize("sk,qr", [("fp32", "fp32"), ("bf16", "fp32"), ("fp16", "fp16")])
@pytest.mark.parametrize("n", [1, 15, 64, 65, 200])
def test_sketch_factor_nearly_dependent_columns(pne, sk, qr, n):
    """The factor from the sketch's Gram matrix where a column repeats an
    earlier one to 1e-9 (below FP32 roundoff: its pivot is raised) and columns
    differ in size by 1e6: the solve reaches the accuracy of its condition
    number, |x - x*| <= 10 kappa u |x*| for a consistent right-hand side, with
    kappa the one of A with its columns scaled to unit norm and the error
    taken in the same scaling.  (Not with R rounded to BF16: at this kappa of
    2e9 three refinement steps through a factor of 8 bits do not always
    converge, whichever way the factor is formed.)"""
    m = 40 * n + 60
    rng = np.random.default_rng(5 + n)
    A = rng.standard_normal((m, n))
    if n > 10:
        A[:, 7] = A[:, 3] + 1e-9 * rng.standard_normal(m)
    d = 10.0 ** rng.uniform(-3, 3, n)
    xs = rng.standard_normal(n) / d
    As = A * d
    o = pne.make_opts(seed=3, sketch_prec=sk, qr_prec=qr, refine_steps=3)
    x, info, _ = pne.pne_solve(dev(As), torch.from_numpy(As @ xs).cuda(), opts=o)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    kappa = np.linalg.cond(A)
    e = (x.cpu().numpy() - xs) * d
    assert np.linalg.norm(e) <= 10 * kappa * U * np.linalg.norm(xs * d)


@pytest.mark.parametrize("m,n,lda", [
    (1, 1, 1), (5, 5, 7), (16, 15, 16), (16, 16, 16), (40, 16, 41), (129, 17, 129),   # few chunks, last panel narrow
    (1024, 31, 1024), (1025, 33, 1025), (1041, 40, 1050), (2065, 64, 2065),           # one block, two, three
    (3000, 600, 3000), (6145, 150, 6145),                                             # blocks shrink with the panel
    (65537, 20, 65537), (1048593, 2, 1048593),                                        # three levels, last chunk of one row
])
def test_qr_blocks_and_levels(pne, m, n, lda):
    """Householder QR of [A b] at the edges of its 16-row chunks, 1024-row
    blocks and levels.  Backward error of a tree of Householder reflectors:
    columnwise c sqrt(m n) u with c = 8 (rounding errors of random sign), so
    |x - x*| <= c sqrt(m n) u kappa (1 + kappa |r| / (|A| |x*|)) |x*|."""
    rng = np.random.default_rng(m + 3 * n)
    A = rng.standard_normal((m, n)) + 2 * np.sqrt(m) * np.eye(m, n)
    xs = rng.standard_normal(n)
    Q, _ = np.linalg.qr(A)
    r = rng.standard_normal(m)
    r -= Q @ (Q.T @ r)
    r -= Q @ (Q.T @ r)
    r *= 1e-3
    b = A @ xs + r
    x, info = pne.qr_ls_solve(dev(A, lda), torch.from_numpy(b).cuda())
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    sv = np.linalg.svd(A, compute_uv=False)
    kappa = sv[0] / sv[-1]
    tol = 8 * np.sqrt(m * n) * U * kappa * (1 + kappa * np.linalg.norm(r) / (sv[0] * np.linalg.norm(xs)))
    # b itself is rounded: sqrt(n) u |A| |x*| per row, of random sign
    assert np.linalg.norm(x.cpu().numpy() - xs) <= 2 * tol * np.linalg.norm(xs)


def test_qr_zero_and_nonfinite_columns(pne):
    """A zero column and a NaN are reported (1000 + column) and x is NaN."""
    rng = np.random.default_rng(8)
    for bad, col in ((0.0, 18), (np.nan, 3)):
        A = rng.standard_normal((1100, 40))
        A[:, col] = bad
        x, info = pne.qr_ls_solve(dev(A), torch.from_numpy(A[:, 0] * 1.0).cuda())
        torch.cuda.synchronize()
        assert 1000 < int(info.item()) <= 1000 + col + 1
        assert bool(torch.isnan(x).all())


@pytest.mark.parametrize("n", [1, 5, 16, 17, 31, 32, 33, 63, 65, 128, 129, 257, 300, 513, 1000, 1025, 1100, 2060])
def test_lu_panels(pne, n):
    """P C = L U at the edges of panels, chunks and panel heights, for
    C = R^-T A^T A.  Backward error of Gaussian elimination
    |P C - L U| <= n u |L| |U|, with three roundings to a multiplier instead of
    one (3) and the rounding of the product (2); |l| <= 1 by pivoting."""
    m = n + 10
    rng = np.random.default_rng(31 + n)
    A = rng.standard_normal((m, n))
    R = np.triu(rng.standard_normal((n, n))) / np.sqrt(n) + np.diag(np.where(rng.random(n) < 0.5, -1.0, 1.0) * 2)
    b = torch.zeros(m, dtype=torch.float64, device="cuda")
    C0, _, _, _ = pne.pne_gram(dev(A), b, dev(R), hpne=True)
    LU, _, piv, info = pne.pne_gram(dev(A), b, dev(R), hpne=True, factor=True)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    C, LU, piv = C0.cpu().numpy().copy(), LU.cpu().numpy(), piv.cpu().numpy()
    for k, p in enumerate(piv):
        assert k <= p < n
        C[[k, p]] = C[[p, k]]
    L, Um = np.tril(LU, -1) + np.eye(n), np.triu(LU)
    assert np.abs(L).max() <= 1 + 4 * U
    assert np.all(np.abs(L @ Um - C) <= (3 * n + 2) * U * (np.abs(L) @ np.abs(Um)))


@pytest.mark.parametrize("n", [40, 200])
def test_lu_pivot_ties_zeros_and_nonfinite(pne, n):
    """Equal entries: the first row is the pivot.  A zero pivot and a NaN are
    reported at the first column that has one."""
    # C = 64 everywhere, 128 on the diagonal but for its first entry
    m = 64 + n
    A = np.zeros((m, n))
    A[:64, :] = 1.0
    A[64:, :] = 8.0 * np.eye(n)
    A[64, 0] = 0.0
    b = torch.zeros(m, dtype=torch.float64, device="cuda")
    I = dev(np.eye(n))
    _, _, piv, info = pne.pne_gram(dev(A), b, I, hpne=True, factor=True)
    assert int(info.item()) == 0 and piv.cpu().numpy().tolist() == list(range(n))
    Z = A.copy()
    Z[:, 20] = 0.0
    assert int(pne.pne_gram(dev(Z), b, I, hpne=True, factor=True)[3].item()) == 3021
    Z[70, 33] = np.nan      # row and column 33 of C: the first column has one
    assert int(pne.pne_gram(dev(Z), b, I, hpne=True, factor=True)[3].item()) == 3001


@pytest.mark.parametrize("s,n", [
    (305, 100), (1413, 471), (535, 107), (1140, 380), (405, 135), (1432, 716),   # 160 x 128, 192 x 128, 160 x 192
    (990, 198), (702, 702), (641, 212), (1334, 667)])                            # 256 x 256, 192 x 256
def test_sketch_tiles(pne, s, n):
    """FP32 sketches through every tile of the wide product against the FP64
    sketch of the same Omega: per entry the tolerance of the FP32 sketch, 1e-4
    of the size of a sum of m products, sqrt(m / s) for unit entries."""
    m = 20000
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, m, dtype=torch.float64, device="cuda", generator=g).t()
    got, ref = pne.pne_sketch(A, s, seed=4, prec="fp32"), pne.pne_sketch(A, s, seed=4, prec="fp64")
    torch.cuda.synchronize()
    assert float((got - ref).abs().max()) <= 1e-4 * np.sqrt(m / s)


@pytest.mark.parametrize("prec,u", [("fp8", 2.0 ** -4), ("fp16", 2.0 ** -11)])
@pytest.mark.parametrize("m,n,s,br", [
    (1, 1, 1, 128), (700, 3, 9, 64), (1000, 17, 130, 128), (2049, 257, 300, 128),    # blocks and tiles cut short
    (1500, 40, 120, 192), (3001, 65, 129, 256), (3001, 20, 70, 320), (5000, 30, 90, 1024),
])
def test_sketch_scaled_blocks(pne, prec, u, m, n, s, br):
    """Sketches with a scale per block of br rows (in registers up to 256 rows,
    read twice above; blocks that are no multiple of the product's K tile go
    to the narrow product) against the oracle.  Both operands are rounded
    (where Omega differs in its last bit, to neighbours): per entry at most 2 u
    of its sum of absolute products, on average the root of the sum of squares
    of the products, sqrt(pi / 2) |a|_2 / |a|_1 of that sum for a Gaussian
    Omega, times 2 u (sqrt(2 / 3) u expected)."""
    import oracle as orc
    rng = np.random.default_rng(m + n)
    A = rng.standard_normal((m, n)) * np.exp(rng.uniform(-4, 4, (m, 1)))
    A[:: 7, n // 2] = 0.0
    got = pne.pne_sketch(dev(A), s, seed=21, prec=prec, block_rows=br).cpu().numpy()
    ref, ab = orc.sketch(A, s, seed=21, prec=prec, block_rows=br, want_abs=True)
    err = np.abs(got - ref)
    assert np.all(err <= (2 * u + 1e-4) * ab + 1e-300)
    a1, a2 = np.abs(A).sum(axis=0), np.sqrt((A * A).sum(axis=0))
    mean = 2 * u * np.sqrt(np.pi / 2) * float((a2 / np.where(a1 > 0, a1, 1)).max())
    assert float(np.sum(err)) <= mean * float(np.sum(ab))


@pytest.mark.parametrize("n", [1, 5, 38, 130])
@pytest.mark.parametrize("m", [128 * 31, 128 * 32, 128 * 33 + 7, 70001])
@pytest.mark.parametrize("hpne", [False, True])
def test_partial_sums(pne, hpne, m, n):
    """Gram matrix and right-hand side from about 31, 32, 33 and several
    hundred partial sums: a thread per entry below 32, sixteen above.  Errors
    of sums of m rounded products in any order: (m + 2) u |A|^T |A|."""
    rng = np.random.default_rng(m + n)
    A, b = rng.standard_normal((m, n)), rng.standard_normal(m)
    C, c, _, info = pne.pne_gram(dev(A), torch.from_numpy(b).cuda(), dev(np.eye(n)), hpne=hpne)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    C, c = C.cpu().numpy(), c.cpu().numpy()
    tol = (m + 2) * U
    err = np.abs(C - A.T @ A)
    assert np.all((err if hpne else np.tril(err)) <= 2 * tol * (np.abs(A).T @ np.abs(A)))
    assert np.all(np.abs(c - A.T @ b) <= 2 * tol * (np.abs(A).T @ np.abs(b)))


@pytest.mark.parametrize("s,n", [
    (305, 100), (1413, 471), (535, 107), (1140, 380), (405, 135), (1432, 716),   # 160 x 128, 192 x 128, 160 x 192
    (990, 198), (702, 702), (641, 212), (1334, 667)])                            # 256 x 256, 192 x 256
def test_fp32_sketch_sums(pne, s, n):
    """FP32 sketches through every tile of the wide product, of a matrix that
    FP32 holds exactly, against the FP64 sketch of the same Omega: what is left
    is the rounding of FP32 sums.  Terms of size 1 leave partial sums of size
    sqrt(k), each rounded with an error uniform in u of it at most: after m of
    them u m / sqrt(6) root mean square (one chain; less where the sum is
    split), six times that for the largest of the entries."""
    m = 20000
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn(n, m, dtype=torch.float32, device="cuda", generator=g).double().t()
    got, ref = pne.pne_sketch(A, s, seed=4, prec="fp32"), pne.pne_sketch(A, s, seed=4, prec="fp64")
    torch.cuda.synchronize()
    err = (got - ref).abs()
    rms = 2.0 ** -24 * m / np.sqrt(6 * s)
    assert float(err.square().mean().sqrt()) <= rms
    assert float(err.max()) <= 6 * rms


@pytest.mark.parametrize("m", [50, 1100, 9000, 70000])                     # one block to three levels
@pytest.mark.parametrize("col", [0, 3, 15, 16, 18, 33, 39])
@pytest.mark.parametrize("bad", [0.0, np.nan, np.inf, -np.inf])
def test_qr_info_names_the_column(pne, m, col, bad):
    """A zero column stays exactly zero, and a NaN or infinity in one entry (of
    the first or the last row) stays in its column and those right of it: the
    info word is 1000 + that column, whatever the panel and the level."""
    rng = np.random.default_rng(m + col)
    b = torch.from_numpy(rng.standard_normal(m)).cuda()
    for row in (0, m - 1):
        A = rng.standard_normal((m, 40))
        A[slice(None) if bad == 0.0 else row, col] = bad
        x, info = pne.qr_ls_solve(dev(A), b)
        torch.cuda.synchronize()
        assert int(info.item()) == 1000 + col + 1
        assert bool(torch.isnan(x).all())


@pytest.mark.parametrize("m", [50, 1100, 9000, 70000])
@pytest.mark.parametrize("n", [31, 32, 40])
def test_qr_large_right_hand_side(pne, m, n):
    """x is linear in b, bit for bit under powers of two, also where b's norm
    overflows, and with one large entry."""
    rng = np.random.default_rng(m + n)
    A, b = dev(rng.standard_normal((m, n))), torch.from_numpy(rng.standard_normal(m)).cuda()
    x, info = pne.qr_ls_solve(A, b)
    big, binfo = pne.qr_ls_solve(A, b * 2.0 ** 900)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and int(binfo.item()) == 0
    assert torch.equal(big * 2.0 ** -900, x)
    b[m // 3] = 1e300
    x, info = pne.qr_ls_solve(A, b)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and bool(torch.isfinite(x).all())
