"""The coarsest level's dense inverse at block and tile edges.

Matrices that stay on one level (max_coarse above their size), of 1 unknown up to several 64-
blocks with ragged last blocks, symmetric positive definite under Cholesky and nonsymmetric
diagonally dominant under LU, against numpy's inverse: the error is held to
16 n eps cond(A) relative to the largest entry of the inverse, the usual bound of a
factorisation and two triangular products.  An indefinite matrix is refused whichever of the 64
pivots is the bad one.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def inverse_error(A, lu):
    from paper_2103_10476_amd import solver
    n = A.shape[0]
    p = pb.from_dense(A)
    o = solver.Options(max_coarse=2000, coarse_solver="lu" if lu else "cholesky")
    g = solver.Hierarchy.from_problem(p, options=o)
    inv = g.export(0, "coarse_inv").reshape(n, n)
    g.close()
    ref = np.linalg.inv(A)
    return np.abs(inv - ref).max() / np.abs(ref).max()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 63, 64, 65, 127, 128, 129, 200, 321])
@pytest.mark.parametrize("lu", [False, True])
def test_inverse(n, lu):
    rng = np.random.Generator(np.random.PCG64(n))
    B = rng.uniform(-1.0, 1.0, size=(n, n))
    A = B / n + 2.0 * np.eye(n) if lu else B @ B.T / n + 0.05 * np.eye(n)
    assert inverse_error(A, lu) <= 16 * n * EPS * np.linalg.cond(A)


@pytest.mark.parametrize("at", [0, 1, 15, 16, 63, 64, 100])
def test_bad_pivot(at):
    from paper_2103_10476_amd import _lib, solver
    n = 101
    A = np.eye(n) + 0.01 * (np.eye(n, k=1) + np.eye(n, k=-1))
    if at:  # positive diagonal, negative pivot
        A[at, at - 1] = A[at - 1, at] = 2.0
    else:
        A[0, 0] = -1.0
    with pytest.raises(_lib.SaError):
        solver.Hierarchy.from_problem(pb.from_dense(A), options=solver.Options(max_coarse=2000))
