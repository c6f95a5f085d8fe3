"""The coarsest level's Cholesky factor and inverse on ill-conditioned operators.

Gaussian-kernel matrices exp(-|x_i - x_j|^2 / 2 w^2) + shift I: symmetric positive definite with
64-blocks as ill-conditioned as the whole, so a factor whose error grows with the condition of
its diagonal blocks loses pivots.  Every shift has to be accepted, and the inverse has to be as
near to the one from 80-bit arithmetic as that of substitution in 64 bits (LAPACK's Cholesky
and triangular solve of the same matrix): within 8 times its error, since both are one draw of
the same rounding errors (two orders of the same operations differ by up to 3 here).
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


def kernel_matrix(n, width, shift):
    x = np.linspace(0.0, 1.0, n)
    return np.exp(-((x[:, None] - x[None, :]) / width) ** 2 / 2) + shift * np.eye(n)


def extended_inverse(A):
    """A^-1 by Cholesky and triangular inversion in 80 bits."""
    n = A.shape[0]
    L = np.tril(A).astype(np.longdouble)
    for j in range(n):
        L[j:, j] /= np.sqrt(L[j, j])
        L[j + 1:, j + 1:] -= np.outer(L[j + 1:, j], L[j + 1:, j])
    L = np.tril(L)
    X = np.zeros_like(L)
    for i in range(n):
        X[i, :i] = -(L[i, :i] @ X[:i, :i]) / L[i, i]
        X[i, i] = 1.0 / L[i, i]
    return X.T @ X


def substitution_inverse(A):
    from scipy.linalg import cholesky, solve_triangular
    X = solve_triangular(cholesky(A, lower=True), np.eye(A.shape[0]), lower=True)
    return X.T @ X


def gpu_inverse(A):
    from paper_2103_10476_amd import solver
    n = A.shape[0]
    g = solver.Hierarchy.from_problem(pb.from_dense(A), options=solver.Options(max_coarse=2000))
    inv = g.export(0, "coarse_inv").reshape(n, n)
    g.close()
    return inv


def check_error(A):
    ref = extended_inverse(A)
    err = np.abs(gpu_inverse(A) - ref).max()
    assert err <= 8 * np.abs(substitution_inverse(A) - ref).max()


@pytest.mark.parametrize("shift", [1e-8, 1e-10, 1e-11, 1e-12])
@pytest.mark.parametrize("n", [512, 960])
def test_accepted(n, shift):
    assert np.isfinite(gpu_inverse(kernel_matrix(n, 0.05, shift))).all()


@pytest.mark.parametrize("shift", [1e-8, 1e-10, 1e-12])
def test_panels(shift):
    check_error(kernel_matrix(512, 0.05, shift))


@pytest.mark.parametrize("n,shift", [(200, 1e-12), (512, 1e-10), (512, 1e-12), (512, 1e-13)])
def test_diagonal_blocks(n, shift):
    # the narrower kernel: the 64-blocks' own inverses decide
    check_error(kernel_matrix(n, 0.02, shift))
