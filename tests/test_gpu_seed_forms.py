"""ip_seed_search around the lines that its forms are chosen by, in starts and
in support vectors (few starts split their sums, others share the records
through LDS, many or with few records read them one lane each), bit for bit
against the oracle."""
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


def _problem(ip, ctx, d, S, p):
    rng = np.random.default_rng(100 * d + S)
    dom = I.box(d)
    fm = I.rbf_manifold(d, S, rng, dom) if p == 0 else I.random_manifold(d, S, p, rng, dom)
    fm.bias = -0.25
    wl = I.Workload("sf", fm, I.make_lattice(d, 0.2, rng), dom, np.zeros((1, d)))
    return wl, ip.Problem(ctx, wl)


@pytest.mark.parametrize("d,S,p,n,iters", [
    (3, 23, 2, 4096, 3), (3, 24, 2, 4096, 3), (6, 24, 3, 4097, 2), (4, 47, 4, 8192, 2), (5, 48, 3, 8192, 2),
    (2, 48, 1, 8193, 2), (7, 95, 3, 12288, 1), (3, 96, 5, 12288, 1), (4, 15, 0, 4096, 2), (4, 16, 0, 4096, 2),
    (5, 31, 0, 8192, 1), (5, 32, 0, 8192, 1), (2, 64, 0, 12288, 1), (6, 63, 0, 12288, 1), (3, 23, 3, 20001, 2),
    (6, 31, 2, 20001, 1), (6, 32, 2, 65536, 0), (6, 32, 2, 65537, 1), (2, 256, 2, 65537, 0), (3, 257, 2, 65537, 0), (2, 384, 1, 131073, 0),
    (2, 385, 1, 131073, 0), (2, 385, 1, 184321, 0), (3, 32, 0, 65536, 0), (3, 32, 0, 65537, 1),
    (2, 257, 0, 131073, 0), (2, 257, 0, 184321, 0)])
def test_lines_between_the_forms(ip, ctx, d, S, p, n, iters):
    import torch
    wl, prob = _problem(ip, ctx, d, S, p)
    q0 = np.random.default_rng(n).uniform(-4.0, 4.0, (n, d))
    print(f"seeds d={d} S={S} p={p} n={n} iters={iters}", flush=True)
    want_q, want_f = O.seed_search(wl, q0, iters)
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


def test_few_vectors_many_starts(ip, ctx):
    """With few support vectors 12 288 starts take what 20 000 take (a lane each
    on either side), and not a step of the split form for every 4096."""
    import torch
    _, prob = _problem(ip, ctx, 6, 20, 3)
    best = {}
    try:
        for n in (12288, 20000):
            q0 = torch.from_numpy(np.random.default_rng(n).uniform(-4.0, 4.0, (n, 6))).cuda()
            q, f = torch.empty_like(q0), torch.empty(n, dtype=torch.float64, device="cuda")
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            for _ in range(8):
                ev[0].record()
                for _ in range(10):
                    ip.ip_seed_search(ctx.h, prob.h, q0.data_ptr(), n, 30, q.data_ptr(), f.data_ptr())
                ev[1].record()
                torch.cuda.synchronize()
                best[n] = min(best.get(n, 1e9), ev[0].elapsed_time(ev[1]) * 100.0)
    finally:
        prob.close()
    print(f"12 288 starts {best[12288]:.0f} us, 20 000 {best[20000]:.0f}", flush=True)
    assert best[12288] < 1.25 * best[20000]
