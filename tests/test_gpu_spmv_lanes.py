"""The solve's SpMV with several lanes per row, through the V-cycle and the solve.

Banded symmetric matrices of chosen row lengths put the levels on 4, 8, 16, 32 and 64 lanes
per row and on the row blocks, with ragged last rows (bands cut at the ends) and row counts
around the workgroup size; one problem has a row far longer than the rest, which stays with the
row blocks.  FP64 against the oracle: equal iterations and x within 1e-12 (the bound of every
parity test: the row sums differ from the oracle's by rounding only); the FP32 V-cycle against
the FP64 solve: 1e-8; grouped against standalone solves: bitwise, in both precisions.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb
from parity import compare_setup, compare_solve, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def banded(n, half, hub=False):
    """Rows couple to `half` neighbours on each side with decaying strength; with hub, row
    n // 2 also couples weakly to every fifth row."""
    d = np.arange(1, half + 1)
    i = np.repeat(np.arange(n), half)
    j = i + np.tile(d, n)
    w = 1.0 / np.tile(d, n) ** 2
    ok = j < n
    i, j, w = i[ok], j[ok], w[ok]
    if hub:
        far = np.arange(0, n, 5)
        far = far[np.abs(far - n // 2) > half]
        i = np.concatenate([i, np.minimum(far, n // 2)])
        j = np.concatenate([j, np.maximum(far, n // 2)])
        w = np.concatenate([w, np.full(far.size, 1e-3)])
    rows = np.concatenate([i, j, np.arange(n)])
    cols = np.concatenate([j, i, np.arange(n)])
    diag = np.bincount(np.concatenate([i, j]), weights=np.concatenate([w, w]), minlength=n)
    vals = np.concatenate([-w, -w, diag + 1e-3])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return pb.CsrProblem(n, rp, cols[o].astype(np.int32), vals[o], f"banded_{n}_{half}_{hub}")


CASES = [(1057, 7, False), (8191, 13, False), (40003, 13, False), (20011, 38, False),
         (9001, 70, False), (2049, 180, False), (40003, 13, True)]


@pytest.mark.parametrize("n,half,hub", CASES)
def test_lanes(n, half, hub):
    import torch
    from paper_2103_10476_amd import solver
    p = banded(n, half, hub)
    b = pb.random_rhs(p.n, 9)
    opts = dict(theta=0.1, max_coarse=40, variants=["offlmp", "1norm"], cheb_boost=1.1)
    g, h = run_both(p, **opts)
    compare_setup(g, h)
    compare_solve(g, h, b)
    x64, _, _, _ = g.solve(b)
    f = solver.Hierarchy.from_problem(p, options=solver.Options(**opts, precision="fp32"))
    x32, it32, _, st = f.solve(b)
    assert st == "SA_OK"
    assert float((x32 - x64).norm() / x64.norm()) <= 1e-8 * 1.1 + 2e-8
    both = solver.solve_many([g, f], [b, b])
    assert torch.equal(both[0][0], x64) and torch.equal(both[1][0], x32)
    assert both[1][1] == it32
    g.close()
    f.close()
