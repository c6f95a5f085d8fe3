"""CG at the sizes where the inner products' stages change.

The kernels that use an inner product take its last stage (up to 4096 partials of 4096 terms)
themselves; beyond 4096 * 4096 unknowns a stage comes between.  A few iterations on grids
around one block, around several, and just past 4096 blocks: the recurrence residual that the
solver reports against the true residual of its x (1e-9 of it apart at most: three iterations
of rounding), and the grouped solve against the standalone one, bitwise.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


@pytest.mark.parametrize("nx,ny", [(64, 64), (64, 63), (4097, 3), (4097, 4096)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_stages(nx, ny, precision):
    import torch
    from paper_2103_10476_amd import solver
    p = pb.fd5_stretched(nx, ny, 1.0)
    b = torch.from_numpy(pb.random_rhs(p.n, 8)).cuda()
    h = solver.Hierarchy.from_problem(p, options=solver.Options(
        variants=["1norm"], precision=precision, max_iter=3, rtol=1e-14, max_coarse=100))
    x, it, rr, _ = h.solve(b)
    assert it == 3
    A = torch.sparse_csr_tensor(torch.from_numpy(p.rp).cuda(), torch.from_numpy(p.col).cuda(),
                                torch.from_numpy(p.val).cuda(), size=(p.n, p.n))
    true = float((b - A @ x).norm() / b.norm())
    assert abs(rr - true) <= 1e-9 * true
    y, it2, rr2, _ = solver.solve_many([h], [b])[0]
    assert it2 == it and rr2 == rr and torch.equal(x, y)
    h.close()
