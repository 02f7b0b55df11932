"""Canonical FP64 batch traces at the edges of their kernels' forms: templates
of fewer and of more points than a wave has lanes (the subdivision reads the
signs one simplex ahead only for the former), boxes that cut the manifold (the
box test is skipped for simplices well inside), coarse stages of a few and of
many simplices, one and several batches, and refinement that starts from the
values the trace leaves.  Sets and points must equal the oracle's bit for bit."""
import numpy as np
import pytest

import oracle as O
from paper_2406_04795_amd import inputs as I
from test_gpu_trace import trace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ip():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2406_04795_amd import ip as _ip
    return _ip


@pytest.fixture(scope="module")
def ctx(ip):
    c = ip.Context(0)
    yield c
    c.close()


# d, k, lambda, cells: template points C(d + k, d) = 6, 66, 20, 56, 15, 70, 21, 56, 28, 84
@pytest.mark.parametrize("d,k,lam,cells", [
    (2, 2, 0.05, 300), (2, 10, 0.02, 500), (3, 3, 0.1, 1000), (3, 5, 0.06, 4000), (4, 2, 0.2, 3000),
    (4, 4, 0.12, 6000), (5, 2, 0.3, 6000), (5, 3, 0.25, 6000), (6, 2, 0.45, 8000), (6, 3, 0.3, 40000)])
def test_batch_fp64_matches_oracle(ip, ctx, d, k, lam, cells):
    wl = I.subbox_case(d, 60, lam, cells, seed=62 if d == 6 else d * 10 + k, k=k)
    print(f"batch d={d} k={k}", flush=True)
    ov, om = O.trace_batch(wl)[:2]
    assert len(ov) > 0
    opts, _ = O.points(wl, ov, om)
    for kw in ({}, {"budget": 1 << 20}):
        gv, gm, gp, st = trace(ip, ctx, wl, **kw)
        assert np.array_equal(gv, ov) and np.array_equal(gm, om)
        assert np.array_equal(gp.view(np.uint64), opts.view(np.uint64))
        assert kw == {} or st["n_batches"] >= 1
    gv, gm, gp, _ = trace(ip, ctx, wl, flags=ip.IP_REFINE(2))
    want = O.points_refined(wl, gv, gm, 2)
    assert np.array_equal(gv, ov) and np.array_equal(gp.view(np.uint64), want.view(np.uint64))
