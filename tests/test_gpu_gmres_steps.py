"""The Gram-Schmidt passes of GMRES at their edges: cycles of more vectors than a block has
wavefronts, one and several blocks of the inner product, cycles that end with their last
vector, and each first smoother step that rides along.  Step counts equal the oracle's and
solutions agree to 1e-12, the bar of every solve test.
"""
import pytest

from paper_2103_10476_amd import problems as pb
from parity import run_both
from test_gpu_gmres import compare_gmres

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


SMOOTHERS = {"chebyshev 1": dict(degree=1), "chebyshev 3": dict(degree=3),
             "jacobi": dict(smoother="jacobi")}


@pytest.mark.parametrize("size", [9, 16, 21])  # 729, 4,096 and 9,261 unknowns
@pytest.mark.parametrize("smoother", list(SMOOTHERS))
def test_steps(size, smoother):
    p = pb.cd7_upwind(size, 1000.0, (4.0, 20.0, -10.0))
    g, h = run_both(p, coarse_solver="lu", rtol=1e-12, theta=0.3, max_coarse=60, max_iter=200,
                    **SMOOTHERS[smoother])
    b = pb.random_rhs(p.n, 21)
    its = compare_gmres(g, h, b, 60)
    for restart in (its, 2):
        compare_gmres(g, h, b, restart)
    g.close()
