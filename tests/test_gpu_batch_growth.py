"""Batch traces whose buffers turn out too small: the fine vertex table that
starts by coarse cells (spheres whose simplices share few vertices), the list
of owner-emitted keys and the set of shared-face keys (spheres with 1.8 to
2.6 times the projected cells), in one and in many batches.  Sets must equal
the oracle's, FP64 points too, and the counts of growths and batches show that
the case was reached."""
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


def _sphere(d, k, lam):
    wl = I.sphere_case(d, 1.0, lam)
    wl.k = k
    return wl


# growths in FP64 and in the certified mode, which has no vertex table
@pytest.mark.parametrize("d,k,lam,fp64,cert", [
    (6, 2, 0.9, 1, 0), (6, 2, 0.7, 2, 1), (7, 2, 0.6, 2, 1), (4, 4, 0.4, 1, 1), (5, 5, 0.3, 1, 1), (4, 9, 0.2, 1, 1)])
def test_growth(ip, ctx, d, k, lam, fp64, cert):
    wl = _sphere(d, k, lam)
    print(f"growth d={d} k={k} lam={lam}", flush=True)
    ov, om = O.trace_batch(wl)[:2]
    opts, _ = O.points(wl, ov, om)
    for prec, grows in ((ip.IP_FP64, fp64), (ip.IP_FP32_CERTIFY, cert)):
        gv, gm, gp, st = trace(ip, ctx, wl, precision=prec)
        assert np.array_equal(gv, ov) and np.array_equal(gm, om)
        if prec == ip.IP_FP64:
            assert np.array_equal(gp.view(np.uint64), opts.view(np.uint64))
        assert st["n_batches"] == 1 and st["regrows"] == grows


@pytest.mark.parametrize("d,k,lam", [(6, 2, 0.9), (6, 2, 0.7), (5, 5, 0.3), (4, 4, 0.4)])
def test_many_batches(ip, ctx, d, k, lam):
    wl = _sphere(d, k, lam)
    ov, om = O.trace_batch(wl)[:2]
    opts, _ = O.points(wl, ov, om)
    per = 12 + 16 * ((2 ** (d + 1) + 63) // 64)      # certified mode, bytes per coarse simplex
    for prec, budget in ((ip.IP_FP64, 1 << 17), (ip.IP_FP32_CERTIFY, 40 * per)):
        gv, gm, gp, st = trace(ip, ctx, wl, precision=prec, budget=budget)
        print(f"d={d} k={k}: {st['n_sigma']} coarse simplices in {st['n_batches']} batches", flush=True)
        assert np.array_equal(gv, ov) and np.array_equal(gm, om)
        if prec == ip.IP_FP64:
            assert np.array_equal(gp.view(np.uint64), opts.view(np.uint64))
            assert st["n_batches"] >= 3
        else:
            assert st["n_batches"] == -(-st["n_sigma"] // 40) > 1


@pytest.mark.parametrize("prec", ["IP_FP64", "IP_FP32_CERTIFY"])
def test_per_batch_mode(ip, ctx, prec):
    """The same growths with the owner list restarted at every batch."""
    wl = _sphere(5, 5, 0.3)
    sc = I.spatial_arm_scene(np.random.default_rng(3), 5, spheres_per_link=1, n_osph=3)
    prob = ip.Problem(ctx, wl)
    try:
        cells = ip.Cells(ctx, prob, precision=getattr(ip, prec))
        free, want, n = cells.check(sc), cells.digest(), cells.n
        cells.close()
        for budget in (0, 1 << 20):
            got, _ = prob.trace_check_batches(sc, budget=budget, precision=getattr(ip, prec))
            print(f"{prec} budget {budget}: {got['batches']} batches", flush=True)
            assert got["digest"] == want and got["n_cells"] == n and got["n_free"] == free
            assert (got["batches"] > 1) == (budget > 0)
    finally:
        prob.close()
