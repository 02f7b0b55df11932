"""Device memory that calls take in a fresh context (the bytes that reached
hipMalloc), against what their sizes account for."""
import numpy as np
import pytest

from paper_2406_04795_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ip():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2406_04795_amd import ip as _ip
    return _ip


def _pow2(n):
    c = 1024
    while c < n:
        c *= 2
    return c


def _first_trace(ip, wl, **kw):
    with ip.Context(0) as ctx:
        prob = ip.Problem(ctx, wl)
        cells = ip.Cells(ctx, prob, **kw)
        st, dg = cells.stats(), cells.digest()
        cells.close()
        prob.close()
    return st, dg


def test_batch_trace(ip):
    """12.7 M cells.  The output lists are sized by the projected cells (12.8
    bytes of keys each and the set of shared edges at load 1/2 with its keys),
    points and their re-check list by the cells, the coarse stage by its
    cofaces; 64 MiB for the search's first buffers and everything small."""
    wl = I.subbox_case(4, 60, 0.004, 2.0e7, seed=7, k=6)
    st, _ = _first_trace(ip, wl, precision=ip.IP_FP32_CERTIFY, budget=64 << 20)
    assert st["regrows"] == 0
    est, n = st["n_coarse_edges"] * wl.k ** 3, st["n_cells"]
    want = (12.8 * est + 16 * _pow2(est / 2) + (8 * 4 + 8) * n + 8 * _pow2(2 * st["n_ncofaces"] + 2)
            + 8 * st["n_ncofaces"] + (12 + 16 + 40) * st["n_sigma"] + (64 << 20))
    print(f"{st['hip_malloc_bytes'] / 1e6:.1f} MB of {want / 1e6:.1f}", flush=True)
    assert st["hip_malloc_bytes"] <= want
