"""Subdivision templates at the limit of one workgroup's LDS: the largest k of
each dimension is traced, in both modes, to the oracle's set and points, and
the next one is refused."""
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


def _case(d, k, lam):
    wl = I.sphere_case(d, 1.0, lam)
    wl.k = k
    return wl


@pytest.mark.parametrize("d,k,lam", [(2, 48, 0.02), (3, 15, 0.06), (4, 9, 0.2)])
@pytest.mark.parametrize("prec", ["IP_FP64", "IP_FP32_CERTIFY"])
def test_largest_template(ip, ctx, d, k, lam, prec):
    wl = _case(d, k, lam)
    print(f"template d={d} k={k} {prec}", flush=True)
    ov, om = O.trace_batch(wl)[:2]
    assert len(ov) > 0
    gv, gm, gp, _ = trace(ip, ctx, wl, precision=getattr(ip, prec))
    assert np.array_equal(gv, ov) and np.array_equal(gm, om)
    if prec == "IP_FP64":
        opts, _ = O.points(wl, ov, om)
        assert np.array_equal(gp.view(np.uint64), opts.view(np.uint64))


@pytest.mark.parametrize("d,k", [(2, 49), (3, 16), (4, 10), (5, 7), (6, 5), (7, 4)])
def test_template_too_large(ip, ctx, d, k):
    prob = ip.Problem(ctx, _case(d, k, 0.1 if d < 6 else 0.9))
    try:
        with pytest.raises(ip.IPError, match="does not fit"):
            ip.Cells(ctx, prob)
    finally:
        prob.close()
