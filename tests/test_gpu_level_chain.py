"""The search's level chain where it has to stop and go on: a fresh context
starts with small buffers, so the vertex table, the edge list and the coface
slots run out in the middle of a search and are mended; a second trace in the
same context runs through.  Both must give the same cells, points and
counts, and a handful of cells must equal the oracle's f signs."""
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


def _d6():
    w = I.subbox_case(6, 40, 0.05, 8e6, seed=4, eps=0.05)
    return w


CASES = {
    "d5_growth": lambda: I.cubic_case(5, 60, 0.075, 2e-3, seed=3),
    "d6_wide_frontier": _d6,
    "d4": lambda: I.cubic_case(4, 50, 0.02, 0.01, seed=1),
}


@pytest.mark.parametrize("name,prec", [("d5_growth", "IP_FP64"), ("d5_growth", "IP_FP32_CERTIFY"),
                                       ("d6_wide_frontier", "IP_FP32_CERTIFY"), ("d4", "IP_FP64")])
def test_growth_in_the_middle_of_a_search(ip, name, prec):
    wl = CASES[name]()
    got = []
    with ip.Context(0) as ctx:
        prob = ip.Problem(ctx, wl)
        for run in range(2):
            cells = ip.Cells(ctx, prob, precision=getattr(ip, prec))
            st = cells.stats()
            print(f"{name} {prec} run {run}: cells {st['n_cells']} vertices {st['n_vertices']} levels {st['levels']} "
                  f"regrows {st['regrows']} mallocs {st['n_hip_malloc']}", flush=True)
            idx = np.linspace(0, cells.n - 1, 200).astype(np.int64)
            got.append((cells.digest(), st, cells.gather(idx)))
            cells.close()
        prob.close()
    (da, sa, ga), (db, sb, _) = got
    assert da == db
    for key in ("n_cells", "n_vertices", "n_cofaces", "levels"):
        assert sa[key] == sb[key], key
    assert sa["regrows"] > 0 and sb["regrows"] == 0
    v, m, _, _ = ga
    b = v + ((m[:, None] >> np.arange(wl.f.d)) & 1).astype(np.int32)
    fa, fb = O.feval(wl.f, wl.lat, v), O.feval(wl.f, wl.lat, b)
    assert ((fa < 0) != (fb < 0)).all()
