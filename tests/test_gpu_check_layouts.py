"""ip_check around the line between its two layouts for robots of many
spheres, against the oracle; and no step in its time there."""
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


def _scene(d, per_link, obst):
    return I.spatial_arm_scene(np.random.default_rng(1), d, spheres_per_link=per_link, n_osph=obst[0], n_obox=obst[1],
                               n_ocyl=obst[2], obst_ball=((0.0, 0.0, 0.3), 0.9))


def _limit(spheres, obst):
    """Configurations from which one lane takes each (nsp lanes a sphere-parallel one)."""
    n, nsp = sum(obst), 1
    while nsp < spheres:
        nsp *= 2
    waves = max(8192, int((spheres * min(150.0 * n, 2000.0 + 10.0 * n) - 28000.0) / (1.4 + 0.045 * n)))
    return waves * 64 // nsp


@pytest.mark.parametrize("d,per_link,obst", [(7, 9, (8, 8, 0)), (7, 9, (1, 0, 0)), (6, 9, (4, 0, 3)), (4, 8, (8, 8, 0)),
                                             (7, 9, (20, 60, 40)), (6, 3, (8, 8, 0))])
def test_both_sides_of_the_line(ip, ctx, d, per_link, obst):
    import torch
    sc = _scene(d, per_link, obst)
    top = _limit(d * per_link, obst)
    q = np.random.default_rng(d).uniform(-I.PI, I.PI, (top, d))
    print(f"check d={d} spheres={d * per_link} obstacles={obst}: {top} configurations", flush=True)
    want = O.check(sc, q)
    for n in (top - 1, top):
        qd = torch.from_numpy(np.ascontiguousarray(q[:n].T)).cuda()
        vd = torch.full((n + 8,), 9, dtype=torch.uint8, device="cuda")
        ip.ip_check(ctx.h, sc, qd.data_ptr(), n, n, vd.data_ptr())
        got = vd.cpu().numpy()
        assert np.array_equal(got[:n], want[:n]) and (got[n:] == 9).all()


def test_no_step_in_time(ip, ctx):
    """63 spheres against 16 obstacles: 12 000 configurations take about half
    again what 8000 take, not three times."""
    import torch
    sc = _scene(7, 9, (8, 8, 0))
    best = {}
    for n in (8000, 12000):
        q = torch.from_numpy(np.random.default_rng(n).uniform(-I.PI, I.PI, (7, n))).cuda()
        v = torch.empty(n, dtype=torch.uint8, device="cuda")
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for _ in range(8):
            ev[0].record()
            for _ in range(14):
                ip.ip_check(ctx.h, sc, q.data_ptr(), n, n, v.data_ptr())
            ev[1].record()
            torch.cuda.synchronize()
            best[n] = min(best.get(n, 1e9), ev[0].elapsed_time(ev[1]) / 14.0 * 1e3)
    print(f"8000: {best[8000]:.1f} us, 12 000: {best[12000]:.1f}", flush=True)
    assert best[12000] < 1.8 * best[8000]
