"""The persistent form of the grouped MFMA products, on batches whose products
have one and are larger than the machine."""
import json
import math

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


def bucket(v):
    return int(math.floor(math.log2(v) + 0.5)) if v > 1 else 0


@pytest.mark.parametrize("hpne,sk,qr,codes", [(True, "bf16", "fp32", "sk4/qr2"), (False, "fp64", "fp64", "sk1/qr1")])
def test_persistent_products(pne, tmp_path, monkeypatch, hpne, sk, qr, codes):
    """LU updates (HPNE) and Gram products of order above 512 and FP64 sketches
    (PNE): persistent launches are what runs, and give the bits of the ordinary
    ones, called once and replayed."""
    from torch.profiler import ProfilerActivity, profile
    shapes = [(4200 + 37 * i, 520 + 11 * i) for i in range(20)]
    probs = [make_problem(m, n, 1e4, 1e-6, seed=1200 + i) for i, (m, n) in enumerate(shapes)]
    A, b, x, descs = pack_batch(probs, "cuda")
    cache = tmp_path / "tune.json"
    monkeypatch.setenv("PNE_TUNE_CACHE", str(cache))
    key = "batched/%s/%s/b2^%d/n2^%d/m2^%d" % ("hpne" if hpne else "pne", codes, bucket(len(shapes)),
                                               bucket(np.mean([n for _, n in shapes])),
                                               bucket(np.mean([m for m, _ in shapes])))
    o = pne.make_opts(seed=3, sketch_prec=sk, qr_prec=qr, refine_steps=1)
    out = {}
    for pe in (0, 1):
        entry = dict(batch_kchunk=8192, shortk_tile=64, lower_small_n=512, persistent=pe, ms=1.0)
        cache.write_text(json.dumps({key: entry}, indent=1 + 3 * pe))   # (another size: read again)
        x.zero_()
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            info = pne.pne_solve_batched(A, b, x, descs, opts=o, hpne=hpne)
            torch.cuda.synchronize()
        assert not bool(info.any())
        assert any("persistent_kernel" in e.name for e in prof.events()) == bool(pe)
        out[pe] = x.clone()
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            plan = pne.BatchPlan(A, b, x, descs, opts=o, hpne=hpne, stream=st)
            for _ in range(3):
                x.fill_(float("nan"))
                plan.execute_graph(st)
                st.synchronize()
                assert torch.equal(x, out[pe])
        plan.close()
    assert torch.equal(out[0], out[1])


def test_autotuner_times_equal_launches_once(pne, tmp_path, monkeypatch):
    """Orders up to 512 and 4096 rows and more, PNE: the tile and persistent
    settings reach none of the launches, so the tuner leaves them at their
    defaults instead of picking among equals."""
    shapes = [(4200 + 301 * i, 40 + 23 * i) for i in range(8)]
    probs = [make_problem(m, n, 1e3, 1e-6, seed=1300 + i) for i, (m, n) in enumerate(shapes)]
    A, b, x, descs = pack_batch(probs, "cuda")
    monkeypatch.setenv("PNE_TUNE_CACHE", str(tmp_path / "tune.json"))
    o = pne.make_opts(seed=3, sketch_prec="bf16", qr_prec="fp32", refine_steps=1)
    for _ in range(3):
        res = pne.autotune_batched(A, b, x, descs, opts=o)
        assert (res["shortk_tile"], res["lower_small_n"], res["persistent"]) == (64, 512, False)
