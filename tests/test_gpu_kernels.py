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
