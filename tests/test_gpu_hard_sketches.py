"""Solves whose sketch is rank deficient, or nearly so, in FP32: the factor of
the sketch must stay a preconditioner."""
import numpy as np
import pytest
import torch

from workloads import make_problem

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def pne():
    import paper_2603_16644_amd as p
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.lib()
    return p


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t()


def relerr(x, y):
    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


def solve(pne, hpne, A, b, **opts):
    fn = pne.hpne_solve if hpne else pne.pne_solve
    x, info, _ = fn(dev(A), torch.from_numpy(b).cuda(), opts=pne.make_opts(**opts))
    assert int(info.item()) == 0
    x = x.cpu().numpy()
    assert np.all(np.isfinite(x))
    return x


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("m,n", [(3000, 100), (4000, 600), (900, 200)])
@pytest.mark.parametrize("sk", ["fp64", "fp32"])
@pytest.mark.parametrize("kappa", [1e6, 1e7, 1e8, 1e10])
def test_large_condition_numbers(pne, orc, hpne, m, n, sk, kappa):
    """An FP32 factor of an FP64 or FP32 sketch, from condition numbers that
    FP32 resolves to ones whose smallest singular values it loses: the accuracy
    of the QR solve after one refinement step."""
    p = make_problem(m, n, kappa, 1e-10, seed=300 + n)
    A, b, xs = p.numpy_A(), p.numpy_b(), p.numpy_x_star()
    x = solve(pne, hpne, A, b, seed=7, sketch_prec=sk, qr_prec="fp32", refine_steps=1)
    assert relerr(x, xs) <= 10 * relerr(orc.qr_ls(A, b), xs)


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("kappa", [1e12, 1e14])
def test_beyond_fp32(pne, hpne, kappa):
    """No breakdown, whatever x is worth there (a BF16 sketch, wrong in its third
    digit, leaves A_p too ill-conditioned for PNE, whatever the factor)."""
    p = make_problem(3000, 100, kappa, 1e-10, seed=310)
    for sk in ("fp64", "fp32"):
        solve(pne, hpne, p.numpy_A(), p.numpy_b(), seed=7, sketch_prec=sk, qr_prec="fp32", refine_steps=1)


@pytest.mark.parametrize("hpne", [False, True])
@pytest.mark.parametrize("m,n", [(100, 100), (300, 257), (1000, 999), (700, 100)])
@pytest.mark.parametrize("sk,qr", [("fp32", "fp32"), ("bf16", "fp32"), ("fp32", "fp16")])
def test_sampled_rows(pne, hpne, m, n, sk, qr):
    """3 n rows drawn from m with replacement: of a square matrix one in twenty
    is missed, and the sketch loses as many directions.  Consistent right-hand
    side: |x - x*| <= 10 kappa u |x*| after three refinement steps."""
    kappa = 1e3
    p = make_problem(m, n, kappa, 1e-6, seed=320 + n)
    A, xs = p.numpy_A(), p.numpy_x_star()
    for seed in range(4):
        x = solve(pne, hpne, A, A @ xs, seed=seed, sketch_prec=sk, qr_prec=qr, refine_steps=3, sketch_kind="srft")
        assert relerr(x, xs) <= 10 * kappa * U


@pytest.mark.parametrize("n", [20, 64, 130, 300, 1000])
def test_many_repeated_columns(pne, n):
    """Half of the columns repeat the others to 1e-9 (below FP32 roundoff) and
    all differ in size by 1e6: |x - x*| <= 10 kappa u |x*| in the scaling of
    the columns, kappa that of the columns scaled to norm 1."""
    m = 6 * n + 300
    rng = np.random.default_rng(n)
    A = rng.standard_normal((m, n))
    A[:, n // 2:] = A[:, :n - n // 2] + 1e-9 * rng.standard_normal((m, n - n // 2))
    A /= np.linalg.norm(A, axis=0)
    d = 10.0 ** rng.uniform(-3, 3, n)
    xs = rng.standard_normal(n) / d
    x = solve(pne, False, A * d, (A * d) @ xs, seed=3, sketch_prec="fp32", qr_prec="fp32", refine_steps=3)
    assert np.linalg.norm((x - xs) * d) <= 10 * np.linalg.cond(A) * U * np.linalg.norm(xs * d)


@pytest.mark.parametrize("n", [2, 3, 16, 17, 33, 63, 65, 128, 129, 513, 700])
@pytest.mark.parametrize("qr", ["fp32", "fp16"])
def test_second_factor_sizes(pne, n, qr):
    """The last two columns (all but the first of three) repeat the first to
    1e-9, at the edges of the blocks of the second factor's steps; tolerance as
    above."""
    m = 6 * n + 900
    rng = np.random.default_rng(n)
    A = rng.standard_normal((m, n))
    k = min(2, n - 1)
    A[:, n - k:] = A[:, :1] + 1e-9 * rng.standard_normal((m, k))
    A /= np.linalg.norm(A, axis=0)
    xs = rng.standard_normal(n)
    x = solve(pne, False, A, A @ xs, seed=3, sketch_prec="fp32", qr_prec=qr, refine_steps=3)
    assert np.linalg.norm(x - xs) <= 10 * np.linalg.cond(A) * U * np.linalg.norm(xs)


@pytest.mark.parametrize("m,n,s", [
    (240, 70, 0), (400, 130, 0), (650, 257, 0), (800, 257, 0), (1100, 257, 0), (1300, 257, 0), (1560, 257, 0),
    (1088, 512, 0), (1600, 700, 0), (2600, 700, 0), (3800, 700, 0), (500, 257, 257), (700, 257, 300), (2150, 1000, 0)])
def test_second_factor_in_chunks(pne, m, n, s):
    """A_p's memory holds eighths to all of what the second factor works on (s =
    3 n where 0); inputs and tolerance as above, with the estimate of AUTO too."""
    rng = np.random.default_rng(m + n)
    A = rng.standard_normal((m, n))
    A[:, n - 2:] = A[:, :1] + 1e-9 * rng.standard_normal((m, 2))
    A /= np.linalg.norm(A, axis=0)
    xs = rng.standard_normal(n)
    for opts in (dict(sketch_prec="fp32", qr_prec="fp32"), dict(sketch_prec="auto", qr_prec="fp32", cond_method=1)):
        x = solve(pne, False, A, A @ xs, s=s, seed=3, refine_steps=3, **opts)
        assert np.linalg.norm(x - xs) <= 10 * np.linalg.cond(A) * U * np.linalg.norm(xs)


def test_second_factor_in_batches_and_replays(pne):
    """Members that need the second factor beside members that do not: each
    solves as it does alone, bit for bit, and a plan replayed from a graph, with
    other work between the replays, gives the same every time."""
    from workloads.problems import pack_batch
    shapes = [(3000, 100, 1e10), (2000, 64, 1e2), (4000, 300, 1e9), (900, 33, 1e8), (700, 100, 1e4)]
    probs = [make_problem(m, n, k, 1e-10, seed=330 + i) for i, (m, n, k) in enumerate(shapes)]
    A, b, x, descs = pack_batch(probs, "cuda")
    o = pne.make_opts(seed=5, sketch_prec="fp64", qr_prec="fp32", refine_steps=1)
    info = pne.pne_solve_batched(A, b, x, descs, opts=o)
    torch.cuda.synchronize()
    assert not bool(info.any())
    ref = x.clone()
    for i, (p, d) in enumerate(zip(probs, descs)):
        Ai = A[d["a_offset"]:d["a_offset"] + p.m * p.n].reshape(p.n, p.m).contiguous().t()
        bi = b[d["b_offset"]:d["b_offset"] + p.m].contiguous()
        one = torch.zeros_like(x[d["x_offset"]:d["x_offset"] + p.n])
        inf1 = pne.pne_solve_batched(Ai.t().reshape(-1), bi, one,
                                     [dict(m=p.m, n=p.n, lda=p.m, a_offset=0, b_offset=0, x_offset=0, problem_id=i)], opts=o)
        assert int(inf1.item()) == 0
        assert torch.equal(one, ref[d["x_offset"]:d["x_offset"] + p.n])
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        plan = pne.BatchPlan(A, b, x, descs, opts=o, stream=st)
        for _ in range(4):
            x.fill_(float("nan"))
            junk = torch.randn(1 << 20, device="cuda").sum()
            info = plan.execute_graph(st)
            st.synchronize()
            assert float(junk) == float(junk) and not bool(info.any())
            assert torch.equal(x, ref)
    plan.close()


@pytest.mark.parametrize("cols", [(0, 129), (5, 40, 97), (31, 32, 33), (64, 65), (128,), (129,)])
@pytest.mark.parametrize("bad", [0.0, np.nan])
def test_first_bad_column(pne, cols, bad):
    """Zero columns and columns with a NaN in several tiles of R: the first of
    them is reported."""
    A = np.random.default_rng(9).standard_normal((3000, 130))
    for c in cols:
        A[slice(None) if bad == 0.0 else 7 * c, c] = bad
    b = torch.ones(3000, dtype=torch.float64, device="cuda")
    for hpne in (False, True):
        fn = pne.hpne_solve if hpne else pne.pne_solve
        x, info, _ = fn(dev(A), b, opts=pne.make_opts(seed=3, sketch_prec="fp32", qr_prec="fp32"))
        assert int(info.item()) == 1000 + cols[0] + 1
        assert bool(torch.isnan(x).all())
