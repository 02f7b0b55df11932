"""ip_seed_search at the edges of its launch rule, bit for bit against the
oracle: start counts around the split kernel's group of 16 and its largest
call (12 288), support-vector counts around its tile of 48 and the other
kernel's tile of 64, degrees 1 to 5 and the Gaussian kernel."""
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


@pytest.mark.parametrize("d,S,p,n,iters", [
    (2, 1, 1, 1, 3), (3, 47, 2, 15, 4), (4, 48, 3, 16, 5), (5, 49, 4, 17, 6), (6, 97, 5, 33, 3), (7, 96, 3, 12288, 0),
    (3, 3, 3, 12288, 1), (6, 65, 3, 12289, 2), (2, 64, 1, 12289, 1), (7, 5, 4, 13000, 1), (4, 50, 0, 31, 4),
    (7, 48, 0, 16, 2), (5, 65, 0, 12289, 1), (2, 7, 2, 196608, 1), (2, 7, 2, 196609, 1)])
def test_seed_search_launch_edges(ip, ctx, d, S, p, n, iters):
    import torch
    rng = np.random.default_rng(100 * d + S)
    dom = I.box(d)
    fm = I.rbf_manifold(d, S, rng, dom) if p == 0 else I.random_manifold(d, S, p, rng, dom)
    fm.bias = -0.25
    wl = I.Workload("se", fm, I.make_lattice(d, 0.2, rng), dom, np.zeros((1, d)))
    q0 = rng.uniform(-4.0, 4.0, (n, d))
    print(f"seeds d={d} S={S} p={p} n={n} iters={iters}", flush=True)
    want_q, want_f = O.seed_search(wl, q0, iters)
    prob = ip.Problem(ctx, wl)
    try:
        q0d = torch.from_numpy(q0).cuda()
        qd = torch.full((n + 8, d), 7.0, dtype=torch.float64, device="cuda")
        fd = torch.full((n + 8,), 7.0, dtype=torch.float64, device="cuda")
        ip.ip_seed_search(ctx.h, prob.h, q0d.data_ptr(), n, iters, qd.data_ptr(), fd.data_ptr())
        torch.cuda.synchronize()
        q, f = qd.cpu().numpy(), fd.cpu().numpy()
    finally:
        prob.close()
    assert np.array_equal(q[:n].view(np.uint64), want_q.view(np.uint64))
    assert np.array_equal(f[:n].view(np.uint64), want_f.view(np.uint64))
    assert (q[n:] == 7.0).all() and (f[n:] == 7.0).all()
