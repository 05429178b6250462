"""Rounding errors of the FP64 factorizations beside LAPACK's on the same
matrices: the sums that are taken from an entry are formed by themselves, so
that a block's update is one rounding of the entry and not one per product."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pne():
    import paper_2603_16644_amd as p
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.lib()
    return p


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t()


def geomean(e):
    return float(np.exp(np.mean(np.log(e))))


@pytest.mark.parametrize("n", [130, 400, 700])
def test_cholesky_backward_error(pne, n):
    """|L L^T - C| no more than twice LAPACK's (sums of 64 products in place of
    LAPACK's longer ones, inverses of four columns; product by product it is
    three to seven times)."""
    got, ref = [], []
    for s in range(3):
        A = np.random.default_rng(n + s).standard_normal((3 * n, n))
        b = torch.zeros(3 * n, dtype=torch.float64, device="cuda")
        I = dev(np.eye(n))
        low = np.tril(pne.pne_gram(dev(A), b, I)[0].cpu().numpy())
        L = np.tril(pne.pne_gram(dev(A), b, I, factor=True)[0].cpu().numpy())
        C = low + np.tril(low, -1).T
        for F, out in ((L, got), (np.linalg.cholesky(C), ref)):
            E = F.astype(np.longdouble) @ F.T.astype(np.longdouble) - C.astype(np.longdouble)
            out.append(np.linalg.norm(E.astype(np.float64)))
    assert geomean(got) <= 2 * geomean(ref)


@pytest.mark.parametrize("m,n", [(700, 600), (1500, 300)])
def test_qr_solver_error(pne, m, n):
    """The error of x over eight problems no more than 0.85 times that of LAPACK's
    QR of [A b], as its sums over rows are trees (product by product the
    updates bring the two level)."""
    got, ref = [], []
    for s in range(8):
        rng = np.random.default_rng(100 + s)
        V = np.linalg.qr(rng.standard_normal((n, n)))[0]
        Q = np.linalg.qr(rng.standard_normal((m, n)))[0]
        A = (Q * 10.0 ** (-3 * np.arange(n) / (n - 1))) @ V.T
        xs = rng.standard_normal(n)
        b = (A.astype(np.longdouble) @ xs.astype(np.longdouble)).astype(np.float64)
        x = pne.qr_ls_solve(dev(A), torch.from_numpy(b).cuda())[0].cpu().numpy()
        R = np.linalg.qr(np.c_[A, b])[1]
        got.append(np.linalg.norm(x - xs))
        ref.append(np.linalg.norm(np.linalg.solve(R[:n, :n], R[:n, n]) - xs))
    assert geomean(got) <= 0.85 * geomean(ref)
