"""What a call launches: work that its result does not need."""
import numpy as np
import pytest
import torch

from workloads import make_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pne():
    import paper_2603_16644_amd as p
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    p.lib()
    return p


def kernels(call):
    """Names of the library's kernels that call() launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events() if "pne::" in e.name or "N3pne" in e.name]


@pytest.mark.parametrize("kappa,prec", [(1e2, "fp16"), (1e6, "fp32"), (1e10, "fp64")])
def test_auto_with_qr_estimate_does_nothing_twice(pne, kappa, prec):
    """AUTO with cond_method = 1 launches the estimate, one copy of the sketch
    and the solve in the precision it picks, less the sketch where that is
    FP32 (then the estimate's is used)."""
    p = make_problem(3000, 100, kappa, 1e-6, seed=96)
    A = torch.from_numpy(np.ascontiguousarray(p.numpy_A().T)).cuda().t()
    b = torch.from_numpy(p.numpy_b()).cuda()
    o = pne.make_opts(seed=6, sketch_prec="auto", qr_prec="auto", refine_steps=1, cond_method=1)
    assert pne.pne_solve(A, b, opts=o)[2]["qr_prec"] == prec
    auto = kernels(lambda: pne.pne_solve(A, b, opts=o))
    e = pne.make_opts(seed=6, sketch_prec=prec, qr_prec=prec, refine_steps=1)
    solve = kernels(lambda: pne.pne_solve(A, b, opts=e))
    est = kernels(lambda: pne.cond_est_qr(A, seed=6))
    sketch = kernels(lambda: pne.pne_sketch(A, 300, seed=6, prec="fp32")) if prec == "fp32" else []
    assert len(solve) > 10 and len(est) > 10
    assert len(auto) <= len(est) + 1 + len(solve) - len(sketch)
