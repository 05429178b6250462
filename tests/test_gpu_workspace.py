"""The workspace is the caller's memory and may hold anything: every entry
point returns bit for bit the same from one filled with 0xFF bytes (NaN in
every format) as from a zeroed one."""
import numpy as np
import pytest
import torch

from workloads import make_problem
from workloads.problems import pack_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pne():
    import paper_2603_16644_amd as p
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.lib()
    return p


class Filled:
    """A workspace of exactly the size asked for, every byte set."""

    def __init__(self, byte):
        self.byte = byte

    def get(self, nbytes, device):
        return torch.full((nbytes,), self.byte, dtype=torch.uint8, device=device)


def problem(m, n, kappa, seed):
    p = make_problem(m, n, kappa, 1e-6, seed=seed)
    A = torch.from_numpy(np.ascontiguousarray(p.numpy_A().T)).cuda().t()
    return A, torch.from_numpy(p.numpy_b()).cuda()


def both(call):
    """call(workspace) -> arrays; equal bits from the two fillings."""
    out = []
    for byte in (0x00, 0xFF):
        r = call(Filled(byte))
        torch.cuda.synchronize()
        out.append([t.cpu().numpy().copy() for t in r])
    for a, b in zip(*out):
        assert a.tobytes() == b.tobytes()
    return out[0]


OPTIONS = [("fp64", "fp64", 0, 0), ("fp32", "fp32", 0, 0), ("bf16", "fp32", 0, 0), ("fp16", "fp16", 0, 0),
           ("fp32", "bf16", 0, 0), ("fp8", "fp32", 0, 0), ("fp32", "fp32", 1, 0), ("auto", "auto", 0, 0),
           ("auto", "auto", 0, 1)]


@pytest.mark.parametrize("sk,qr,kind,cond", OPTIONS)
@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("m,n", [(40, 2), (900, 60), (3000, 200), (5000, 330), (4300, 600)])
def test_solves(pne, sk, qr, kind, cond, hpne, m, n):
    """Orders below and above one block of 64, sketch Gram matrices of one and
    of several partial sums (s = 3 n from 512 on)."""
    A, b = problem(m, n, 1e3, 50 + n)
    o = pne.make_opts(seed=3, sketch_prec=sk, qr_prec=qr, refine_steps=1, cond_method=cond,
                      sketch_kind="srft" if kind else "gaussian")
    fn = pne.hpne_solve if hpne else pne.pne_solve
    x, info = both(lambda ws: fn(A, b, opts=o, workspace=ws)[:2])
    assert int(info[0]) == 0 and np.all(np.isfinite(x))


@pytest.mark.parametrize("cond", [0, 1])
@pytest.mark.parametrize("hpne", [False, True])
def test_auto_picks(pne, hpne, cond):
    """Every precision that AUTO picks."""
    for kappa in (10.0, 1e6, 1e10):
        A, b = problem(3000, 190, kappa, 60)
        o = pne.make_opts(seed=4, sketch_prec="auto", qr_prec="auto", refine_steps=1, cond_method=cond)
        fn = pne.hpne_solve if hpne else pne.pne_solve
        x, info = both(lambda ws: fn(A, b, opts=o, workspace=ws)[:2])
        assert int(info[0]) == 0 and np.all(np.isfinite(x))


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("n", [1, 3, 64, 70, 260, 530])
def test_gram_and_factor(pne, hpne, n):
    A, b = problem(n + 700, n, 10.0, 70 + n)
    R = torch.eye(n, dtype=torch.float64, device="cuda").t()
    for factor in (False, True):
        def call(ws):
            C, c, piv, info = pne.pne_gram(A, b, R, hpne=hpne, factor=factor, workspace=ws)
            C = C if hpne else torch.tril(C)
            return (C, c, info) + ((piv,) if piv is not None else ())
        out = both(call)
        assert int(out[2][0]) == 0 and np.all(np.isfinite(out[0]))


def test_other_entry_points(pne):
    for m, n in ((700, 30), (5000, 210)):
        A, b = problem(m, n, 1e3, 80 + n)
        x, info = both(lambda ws: pne.qr_ls_solve(A, b, workspace=ws))
        assert int(info[0]) == 0 and np.all(np.isfinite(x))
        x, info = both(lambda ws: pne.nne_solve(A, A, b, refine_steps=1, workspace=ws))
        assert int(info[0]) == 0 and np.all(np.isfinite(x))
        both(lambda ws: pne.cond_est(A, workspace=ws))
        both(lambda ws: pne.cond_est_qr(A, workspace=ws))
        for qr in ("fp64", "fp32", "fp16"):
            R, info = both(lambda ws: pne.sketch_precond(A, opts=pne.make_opts(sketch_prec="fp32", qr_prec=qr),
                                                         workspace=ws)[:2])
            assert int(info[0]) == 0 and np.all(np.isfinite(R))
        for prec in ("fp64", "fp32", "bf16", "fp16", "fp8"):
            As, = both(lambda ws: (pne.pne_sketch(A, 3 * n, prec=prec, workspace=ws),))
            assert np.all(np.isfinite(As))


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("sk,qr", [("fp64", "fp64"), ("bf16", "fp32"), ("auto", "auto")])
def test_batch(pne, hpne, sk, qr):
    shapes = [(2000, 64, 1e2), (3100, 190, 1e5), (60, 3, 10.0), (6000, 520, 1e6)]
    probs = [make_problem(m, n, k, 1e-6, seed=900 + i) for i, (m, n, k) in enumerate(shapes)]
    A, b, x, descs = pack_batch(probs, "cuda")
    o = pne.make_opts(seed=5, sketch_prec=sk, qr_prec=qr, refine_steps=1)

    def call(ws):
        x.zero_()
        info = pne.pne_solve_batched(A, b, x, descs, opts=o, hpne=hpne, workspace=ws)
        return x, info
    xs, info = both(call)
    assert np.all(info == 0) and np.all(np.isfinite(xs))


@pytest.mark.parametrize("sk,qr", [("fp64", "fp64"), ("bf16", "fp32")])
@pytest.mark.parametrize("n", [50, 200])
def test_good_solve_after_a_bad_one(pne, sk, qr, n):
    """A solve of data with a NaN leaves nothing in the workspace, or in the
    static array of pne_solve_noalloc, that the next one could meet."""
    A, b = problem(4000, n, 1e3, 90 + n)
    bad = A.t().clone().t()
    bad[7, 3] = float("nan")
    o = pne.make_opts(seed=6, sketch_prec=sk, qr_prec=qr, refine_steps=1)
    want = pne.pne_solve(A, b, opts=o, workspace=Filled(0))[0].cpu().numpy()
    assert np.all(np.isfinite(want))
    from paper_2603_16644_amd._lib import Workspace
    ws = Workspace()
    x, info, _ = pne.hpne_solve(bad, b, opts=o, workspace=ws)
    assert int(info.item()) != 0 and bool(torch.isnan(x).all())
    x, info, _ = pne.pne_solve(A, b, opts=o, workspace=ws)
    assert int(info.item()) == 0 and x.cpu().numpy().tobytes() == want.tobytes()
    pne.pne_solve_noalloc(bad, b, opts=o, hpne=True)
    x, info, _ = pne.pne_solve_noalloc(A, b, opts=o)
    assert int(info.item()) == 0 and x.cpu().numpy().tobytes() == want.tobytes()
