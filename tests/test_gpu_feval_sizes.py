"""ip_feval in canonical FP64 at the edges of its launch rules, bit for bit
against the oracle: vertex counts around the split kernel's group of 28, its
largest call (16 384) and the two steps of vertices per lane, support-vector
counts around the tile of 64, both kernels and a degree without its own
instantiation."""
import numpy as np
import pytest

import oracle as O
from paper_2406_04795_amd import inputs as I

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


@pytest.mark.parametrize("d,S,p,n", [
    (2, 1, 1, 1), (3, 63, 2, 27), (4, 64, 3, 28), (5, 65, 4, 29), (6, 130, 5, 57), (7, 129, 3, 16384),
    (6, 5, 3, 16385), (5, 66, 3, 20000), (3, 3, 2, 98304), (6, 2, 3, 98305), (4, 3, 5, 393216), (7, 2, 3, 393217),
    (4, 64, 0, 28), (5, 65, 0, 1000), (6, 3, 0, 16385), (2, 67, 0, 20001), (7, 130, 0, 29)])
def test_feval_fp64_launch_edges(ip, ctx, d, S, p, n):
    import torch
    rng = np.random.default_rng(1000 * d + S + n)
    dom = I.box(d)
    fm = I.rbf_manifold(d, S, rng, dom) if p == 0 else I.random_manifold(d, S, p, rng, dom)
    fm.bias = 0.125
    lat = I.make_lattice(d, 0.2, rng)
    wl = I.Workload("fe", fm, lat, dom, np.zeros((1, d)))
    V = rng.integers(-30, 30, size=(n, d)).astype(np.int32)
    print(f"feval d={d} S={S} p={p} n={n}", flush=True)
    want = O.feval(fm, lat, V)
    prob = ip.Problem(ctx, wl)
    try:
        vd = torch.from_numpy(V).cuda()
        fd = torch.full((n + 64,), 7.0, dtype=torch.float64, device="cuda")
        ip.ip_feval(ctx.h, prob.h, vd.data_ptr(), n, ip.IP_FP64, fd.data_ptr())
        torch.cuda.synchronize()
        got = fd.cpu().numpy()
    finally:
        prob.close()
    assert np.array_equal(got[:n].view(np.uint64), want.view(np.uint64))
    assert (got[n:] == 7.0).all()
