"""ip_check at the edges of its launch rule and of its scene staging: counts
around 8192 waves of the sphere-parallel layout for 1 to 64 lanes per
configuration, scenes on both sides of what that kernel keeps in LDS and of an
upload slot, and more uploads in a row than there are slots, each with another
scene.  Verdicts must equal the oracle's."""
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


def _scene(d, per_link, n_osph, n_obox, n_ocyl, seed):
    return I.spatial_arm_scene(np.random.default_rng(seed), d, spheres_per_link=per_link, n_osph=n_osph,
                               n_obox=n_obox, n_ocyl=n_ocyl, obst_ball=((0.0, 0.0, 1.2), 1.5), osph_r=(0.02, 0.1),
                               obox_l=(0.05, 0.15), ocyl_r=(0.02, 0.08), ocyl_h=(0.05, 0.2))


def _run(ip, ctx, sc, q):
    import torch
    qd = torch.from_numpy(np.ascontiguousarray(q.T)).cuda()
    n = len(q)
    vd = torch.full((n + 8,), 9, dtype=torch.uint8, device="cuda")
    ip.ip_check(ctx.h, sc, qd.data_ptr(), n, n, vd.data_ptr())
    return vd


@pytest.mark.parametrize("d,per_link,obst,n", [
    (6, 3, (8, 8, 0), 1), (6, 3, (8, 8, 0), 16383), (6, 3, (8, 8, 0), 16384), (4, 2, (4, 4, 4), 65535),
    (4, 2, (4, 4, 4), 65536), (2, 1, (3, 0, 2), 300), (7, 9, (5, 1, 1), 8191), (7, 9, (5, 1, 1), 8192),
    (6, 3, (10, 180, 0), 500), (6, 3, (10, 181, 5), 500), (5, 2, (400, 100, 30), 700), (3, 0, (4, 2, 1), 200)])
def test_check_launch_edges(ip, ctx, d, per_link, obst, n):
    sc = _scene(d, per_link, *obst, seed=n % 97)
    if per_link == 9:            # 63 spheres: 64 lanes
        assert len(sc.lsph_r) == 63
    q = np.random.default_rng(n).uniform(-I.PI, I.PI, (n, d))
    print(f"check d={d} spheres={len(sc.lsph_r)} obstacles={obst} n={n}", flush=True)
    want = O.check(sc, q)
    got = _run(ip, ctx, sc, q).cpu().numpy()
    assert np.array_equal(got[:n], want) and (got[n:] == 9).all()


def test_many_scenes_in_flight(ip, ctx):
    """40 checks queued without a wait, each with its own scene."""
    import torch
    q = np.random.default_rng(1).uniform(-I.PI, I.PI, (333, 6))
    scenes = [_scene(6, 3, 5 + i % 3, 6, 2, seed=i) for i in range(40)]
    got = [_run(ip, ctx, sc, q) for sc in scenes]
    torch.cuda.synchronize()
    for sc, g in zip(scenes, got):
        assert np.array_equal(g.cpu().numpy()[:333], O.check(sc, q))
