"""Setups at the sizes where the prefix sums change over and rows of each length by their
distance weights.

Grids of one to three tiles of 2,048 elements and their neighbours send the setup's scans to one
block, to two launches and to tiles that are full, nearly full and nearly empty; a random mesh
graph has rows of 1 to 40 neighbours, so the eight lanes of a row's weights meet every
remainder and the diagonal at every place.  Every level's arrays against the oracle, bitwise.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_2103_10476_amd import problems as pb
from parity import compare_setup, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4095, 4096, 4097, 6145])
def test_grid_sizes(n):
    nx = 1 if n % 2 else 32
    g, h = run_both(pb.fd5_stretched(nx, n // nx, 10.0), theta=0.02, max_coarse=20)
    compare_setup(g, h)
    g.close()


@pytest.mark.parametrize("power", [1, 2])
def test_distance_rows(power):
    n, rng = 1500, np.random.Generator(np.random.PCG64(8))
    X = rng.uniform(0.0, 1.0, size=(n, 3))
    deg = 1 + np.arange(n) % 40
    a = np.repeat(np.arange(n), deg)
    b = rng.integers(0, n, a.size)
    keep = a != b
    W = sp.coo_matrix((np.ones(int(keep.sum())), (a[keep], b[keep])), shape=(n, n)).tocsr()
    W = ((W + W.T) > 0).astype(float)
    A = (sp.diags(np.asarray(W.sum(axis=1)).ravel() + 0.1) - W).tocsr()
    A.sort_indices()
    p = pb.CsrProblem(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, "random")
    g, h = run_both(p, coords=X, theta=0.1, max_coarse=100, dist_power=power)
    compare_setup(g, h)
    g.close()
