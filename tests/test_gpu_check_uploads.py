"""ip_check's scene uploads: 40 checks, each with its own scene, queued behind
work that keeps the stream busy, so that the slots they go through are
written again while earlier ones are still to be read unless the upload waits;
and a check under stream capture, which is refused."""
import os
import subprocess
import sys

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


def _scene(seed, n_osph=6):
    return I.spatial_arm_scene(np.random.default_rng(seed), 6, spheres_per_link=3, n_osph=n_osph, n_obox=6, n_ocyl=2,
                               obst_ball=((0.0, 0.0, 1.2), 1.5), osph_r=(0.02, 0.1), obox_l=(0.05, 0.15),
                               ocyl_r=(0.02, 0.08), ocyl_h=(0.05, 0.2))


@pytest.mark.parametrize("own_stream", [False, True])
def test_scenes_queued_behind_work(ip, own_stream):
    import torch
    n, k = 333, 40
    q = np.random.default_rng(1).uniform(-I.PI, I.PI, (n, 6))
    qd = torch.from_numpy(np.ascontiguousarray(q.T)).cuda()
    vd = torch.full((k, n), 9, dtype=torch.uint8, device="cuda")
    a = torch.randn(4096, 4096, device="cuda")
    b = torch.empty_like(a)
    scenes = [_scene(i, 5 + i % 3) for i in range(k)]
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if own_stream else torch.cuda.default_stream()
    with ip.Context(0, stream.cuda_stream if own_stream else None) as ctx, torch.cuda.stream(stream):
        warm = torch.empty(n, dtype=torch.uint8, device="cuda")
        ip.ip_check(ctx.h, scenes[2], qd.data_ptr(), n, n, warm.data_ptr())   # the largest
        torch.cuda.synchronize()
        torch.mm(a, a, out=b)
        torch.cuda.synchronize()
        busy = torch.cuda.Event()
        for _ in range(40):          # some 50 ms of matrix products
            torch.mm(a, a, out=b)
        busy.record(stream)
        pending = []
        for i, sc in enumerate(scenes):
            ip.ip_check(ctx.h, sc, qd.data_ptr(), n, n, vd[i].data_ptr())
            pending.append(not busy.query())
        torch.cuda.synchronize()
    print(f"checks queued while the products ran: {sum(pending)}", flush=True)
    assert sum(pending) >= 12        # with the one before them, a wait at the 17th upload at the latest
    got = vd.cpu().numpy()
    for i, sc in enumerate(scenes):
        assert np.array_equal(got[i], O.check(sc, q)), i


# In a process of its own: HIP leaves the stream of a refused capture unusable.
_CAPTURE = r"""
import ctypes as C
import sys
import numpy as np
import torch
sys.path.insert(0, "tests")
from paper_2406_04795_amd import inputs as I
from paper_2406_04795_amd import ip
from test_gpu_check_uploads import _scene
paths = {line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line}
assert len(paths) == 1, paths
hip = C.CDLL(paths.pop())
n = 200
q = np.random.default_rng(2).uniform(-I.PI, I.PI, (n, 6))
qd = torch.from_numpy(np.ascontiguousarray(q.T)).cuda()
vd = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
torch.cuda.synchronize()
stream = torch.cuda.Stream()
ctx = ip.Context(0, stream.cuda_stream)
ip.ip_check(ctx.h, _scene(1), qd.data_ptr(), n, n, vd.data_ptr())
stream.synchronize()
assert hip.hipStreamBeginCapture(C.c_void_p(stream.cuda_stream), 2) == 0    # relaxed
try:
    ip.ip_check(ctx.h, _scene(2), qd.data_ptr(), n, n, vd.data_ptr())
    print("accepted", flush=True)
except ip.IPError as e:
    print("refused:", e, flush=True)
graph = C.c_void_p()
print("end of capture:", hip.hipStreamEndCapture(C.c_void_p(stream.cuda_stream), C.byref(graph)), flush=True)
"""


def test_check_under_capture_is_refused(ip):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _CAPTURE], cwd=root, capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert "refused:" in r.stdout and "accepted" not in r.stdout and r.returncode == 0
