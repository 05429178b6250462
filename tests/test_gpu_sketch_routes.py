"""FP8 and FP16 sketches on every route of their dispatch, against the oracle."""
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


@pytest.mark.parametrize("prec,u", [("fp8", 2.0 ** -4), ("fp16", 2.0 ** -11)])
@pytest.mark.parametrize("m,n,s,br", [
    (1000, 1100, 8, 64), (777, 1100, 8, 128), (900, 1100, 8, 192), (1025, 1100, 8, 256),
    (700, 1100, 8, 320), (1025, 1100, 8, 384),                                             # blocks by wavefronts
    (777, 40, 8, 128), (1023, 20, 8, 256), (1000, 20, 8, 320), (1025, 1100, 8, 448), (3001, 20, 8, 1024),   # by work-groups
    (5000, 20, 8, 1088), (9001, 10, 8, 4096), (2000, 1100, 8, 2048),                       # read twice
    (20000, 200, 600, 256), (20000, 200, 600, 1024),                                       # wide product; narrow (FP16)
])
def test_scaled_sketch_routes(pne, prec, u, m, n, s, br):
    """Quantisation of a wavefront's or a work-group's blocks, rows held or read
    twice, and both products.  Both operands are rounded: per entry at most 2 u
    of its sum of absolute products; on average no more than 2 u |a|_2 / |a|_1
    sqrt(pi / 2) of it (root of the sum of squares, Gaussian Omega)."""
    import oracle as orc
    from paper_2603_16644_amd._lib import Workspace
    rng = np.random.default_rng(m + n + br)
    A = rng.standard_normal((m, n)) * np.exp(rng.uniform(-4, 4, (m, 1)))
    A[:: 7, n // 2] = 0.0
    A[:, n - 1] = 0.0
    ws = Workspace()
    ws.get(1 << 30, torch.device("cuda:0"))
    Ad = torch.from_numpy(np.ascontiguousarray(A.T)).cuda().t()
    got = pne.pne_sketch(Ad, s, seed=21, prec=prec, block_rows=br, workspace=ws).cpu().numpy()
    ref, ab = orc.sketch(A, s, seed=21, prec=prec, block_rows=br, want_abs=True)
    err = np.abs(got - ref)
    assert np.all(got[:, n - 1] == 0.0)
    assert np.all(err <= (2 * u + 1e-4) * ab + 1e-300)
    a1, a2 = np.abs(A).sum(axis=0), np.sqrt((A * A).sum(axis=0))
    mean = 2 * u * np.sqrt(np.pi / 2) * float((a2 / np.where(a1 > 0, a1, 1)).max())
    assert float(np.sum(err)) <= mean * float(np.sum(ab))


@pytest.mark.parametrize("prec,u", [("fp8", 2.0 ** -4), ("fp16", 2.0 ** -11)])
@pytest.mark.parametrize("m,n,s,br", [
    (63, 2560, 4, 64), (65, 1280, 4, 64), (1025, 569, 8, 128), (1500, 1100, 8, 192), (2700, 1100, 8, 256),
    (3700, 1100, 8, 320), (5500, 1100, 8, 384)])
def test_scaled_sketch_many_blocks(pne, prec, u, m, n, s, br):
    """As above, with blocks enough for wavefronts of several blocks each, for
    each length in registers (the first ones at the number of blocks where that
    begins)."""
    test_scaled_sketch_routes(pne, prec, u, m, n, s, br)
