"""Setups on graphs of random neighbours, where nearly every neighbour lies in another aggregate.

The coarse operator is dense, so R (A P) has thousands of rows of more than 32,768 products (a
block each), and rows of 33 to 64 entries meet as many aggregates in P (the sparse product
where the average row has more than 32).  Every level's arrays against the oracle, bitwise, and again
after a numeric re-setup with the values doubled, which has to give the doubled operators.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb
from parity import assert_same, compare_setup, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def random_graph(n, degree, extra=0):
    """The union of degree / 2 random cycles through all n vertices, Laplacian weights; the
    first half of the vertices has `extra` more cycles."""
    rng = np.random.Generator(np.random.PCG64(2))
    i, j = [], []
    for k in range(degree // 2 + extra):
        q = rng.permutation(n if k < degree // 2 else n // 2)
        i.append(q)
        j.append(np.roll(q, 1))
    i, j = np.concatenate(i), np.concatenate(j)
    key = np.unique(np.minimum(i, j) * n + np.maximum(i, j))
    a, b = key // n, key % n
    rows = np.concatenate([a, b, np.arange(n)])
    cols = np.concatenate([b, a, np.arange(n)])
    deg = np.bincount(np.concatenate([a, b]), minlength=n)
    vals = np.concatenate([-np.ones(2 * a.size), deg + 0.01])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return pb.CsrProblem(n, rp, cols[o].astype(np.int32), vals[o], f"random_{n}_{degree}_{extra}")


def check(p):
    g, h = run_both(p, variants=["offlmp", "1norm"], cheb_boost=1.1, max_coarse=100,
                    theta=0.0)
    compare_setup(g, h)
    P = g.export(0, "P_val")
    g.resetup(2.0 * p.val)
    assert_same(g.export(0, "P_val"), P, "P after the re-setup")
    assert_same(g.export(1, "A_val"), 2.0 * h.levels[1].A[2], "A after the re-setup")
    g.close()
    return h


def products(X, Y):
    """Products of each row of X Y."""
    return np.add.reduceat(np.diff(Y[0])[X[1]].astype(np.int64), X[0][:-1])


def test_long_products():
    h = check(random_graph(120000, 14))
    L = h.levels[0]
    import scipy.sparse as sp
    AP = (sp.csr_matrix((L.A[2], L.A[1], L.A[0])) @ sp.csr_matrix((L.P[2], L.P[1], L.P[0])))
    T = products(L.R, (AP.indptr, AP.indices))
    assert 2048 < np.count_nonzero(T > 32768) <= 8192


@pytest.mark.parametrize("degree,extra", [(32, 0), (24, 4), (46, 0), (62, 0)])
def test_many_aggregates(degree, extra):
    p = random_graph(6000, degree, extra)
    assert np.diff(p.rp).max() > 32
    check(p)
