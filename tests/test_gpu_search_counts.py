"""The counts of a certified search: vertices whose sign only the canonical
FP64 sum settles, those of the seeds' own simplices among them, and the same
counts whether or not the search had to stop for larger buffers."""
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


def _zero(d, S, seeds):
    """f = 0 everywhere, exactly: no bound settles a sign, no edge crosses."""
    alpha = np.ones(S)
    alpha[1::2] = -1.0
    fm = I.Manifold(d=d, p=2, gamma=1.0, coef0=1.0, bias=0.0, sv=np.zeros((S, d)), alpha=alpha)
    return I.Workload("zero", fm, I.make_lattice(d, 0.2, np.random.default_rng(d)), I.box(d), seeds)


@pytest.mark.parametrize("d,n_seeds,k", [(2, 1, 1), (4, 3, 1), (6, 40, 1), (3, 2, 2)])
def test_vertices_of_the_seeds(ip, d, n_seeds, k):
    wl = _zero(d, 6, np.random.default_rng(n_seeds).uniform(-2.0, 2.0, (n_seeds, d)))
    wl.k = k
    with ip.Context(0) as ctx:
        prob = ip.Problem(ctx, wl)
        cells = ip.Cells(ctx, prob, precision=ip.IP_FP32_CERTIFY)
        st = cells.stats()
        cells.close()
        prob.close()
    print(f"d={d} k={k}: vertices {st['n_vertices']} fallback {st['n_fallback']}", flush=True)
    assert st["n_cells"] == 0 and d + 1 <= st["n_vertices"] <= n_seeds * (d + 1)
    assert st["n_fallback"] == st["n_vertices"] and st["n_settled64"] == 0


def test_counts_of_a_search_that_stops(ip):
    """11 M vertices, the first run in a fresh context: its vertex table grows
    three times.  A pair of support vectors that cancel leaves many
    signs open."""
    wl = I.cubic_case(5, 60, 0.075, 2e-3, seed=3)
    s = np.full((1, 5), 0.3)
    wl.f.sv = np.concatenate([s, s, wl.f.sv])
    wl.f.alpha = np.concatenate([[1e9, -1e9], wl.f.alpha])
    got = []
    with ip.Context(0) as ctx:
        prob = ip.Problem(ctx, wl)
        for _ in range(2):
            cells = ip.Cells(ctx, prob, precision=ip.IP_FP32_CERTIFY)
            got.append((cells.digest(), cells.stats()))
            cells.close()
        prob.close()
    (da, a), (db, b) = got
    print({q: (a[q], b[q]) for q in ("n_cells", "n_vertices", "n_fallback", "n_settled64", "regrows")}, flush=True)
    assert a["regrows"] > 0 and b["regrows"] == 0 and da == db
    assert a["n_fallback"] > 1000 and a["n_settled64"] > 100
    for key in ("n_cells", "n_vertices", "n_cofaces", "levels", "n_fallback", "n_settled64"):
        assert a[key] == b[key], key


def test_times_of_a_search_that_stops(ip):
    """What the stops cost (the host's reads, allocations and copies of a
    fresh context's first search: a third of it) is in neither of the search's
    times.  The vertex table does not grow here, so no pass runs twice and the
    passes take what they take in the runs that do not stop."""
    wl = I.subbox_case(6, 40, 0.05, 4e6, seed=4, eps=0.05)
    first, rest = [], []
    for _ in range(3):
        with ip.Context(0) as ctx:
            prob = ip.Problem(ctx, wl)
            for run in range(3):
                cells = ip.Cells(ctx, prob)
                st = cells.stats()
                cells.close()
                assert st["regrows"] == 0 and st["n_cells"] > 1 << 20     # a new context's edge list holds 2^20
                (first if run == 0 else rest).append(st["ms_feval"] + st["ms_expand"])
                print(f"run {run}: evaluation {st['ms_feval']:.2f} expansion {st['ms_expand']:.2f} "
                      f"total {st['ms_total']:.2f} ms, cells {st['n_cells']} vertices {st['n_vertices']} "
                      f"mallocs {st['n_hip_malloc']}", flush=True)
            prob.close()
    assert min(rest) > 0.0 and min(first) < 1.15 * min(rest)
