"""GMRES at the sizes where the inner products' stages change.

The projection takes the last stage of its inner products itself up to 512 blocks of 4096
terms; beyond, one stage comes between, and past 4096 blocks two; the norm's stages change at
2048 and 4096 blocks.  Three steps with a restart after two, on grids just below and above each
of these: the residual that the rotations report against the true residual of x, 1e-9 of it
apart at most (three steps of rounding, as for CG).
"""
import pytest

from paper_2103_10476_amd import problems as pb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


@pytest.mark.parametrize("nx,ny", [(4096, 512), (4097, 512), (4096, 2048), (4097, 2048),
                                   (4097, 4096)])
def test_stages(nx, ny):
    import torch
    from paper_2103_10476_amd import solver
    p = pb.fd5_stretched(nx, ny, 1.0)
    A = [torch.from_numpy(v).cuda() for v in (p.rp, p.col, p.val)]
    b = torch.from_numpy(pb.random_rhs(p.n, 8)).cuda()
    h = solver.Hierarchy(p.n, *A, options=solver.Options(
        variants=["1norm"], max_iter=3, rtol=1e-14, max_coarse=100))
    x, it, rr, _ = h.solve_gmres(b, restart=2)
    assert it == 3
    M = torch.sparse_csr_tensor(*A, size=(p.n, p.n))
    true = float((b - M @ x).norm() / b.norm())
    assert abs(rr - true) <= 1e-9 * true
    h.close()
