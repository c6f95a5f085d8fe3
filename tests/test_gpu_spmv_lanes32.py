"""The solve's SpMV with 32 lanes per row: a band of 201 entries per row, enough rows that the
rule takes the lanes for 8 to 12 entries each.  FP64 against the oracle as in every parity test,
grouped against standalone solves bitwise in both precisions.
"""
import pytest

from paper_2103_10476_amd import problems as pb
from parity import compare_setup, compare_solve, run_both
from test_gpu_spmv_lanes import banded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def test_lanes():
    import torch
    from paper_2103_10476_amd import solver
    p = banded(6001, 100)
    b = pb.random_rhs(p.n, 9)
    opts = dict(theta=0.1, max_coarse=40, variants=["offlmp", "1norm"], cheb_boost=1.1)
    g, h = run_both(p, **opts)
    compare_setup(g, h)
    compare_solve(g, h, b)
    f = solver.Hierarchy.from_problem(p, options=solver.Options(**opts, precision="fp32"))
    both = solver.solve_many([g, f], [b, b])
    for one, got in zip((g, f), both):
        x, it, _, _ = one.solve(b)
        assert torch.equal(got[0], x) and got[1] == it
    g.close()
    f.close()
