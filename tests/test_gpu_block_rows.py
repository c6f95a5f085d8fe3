"""Systems setup on matrices whose nodes have rows of unlike block columns.

The node graph takes a node's neighbours from its first row where the node's rows agree entry
by entry and merges the rows otherwise; block norms look a block's start up again where a row
does not begin it where the row before did.  Here entries are dropped at random from a whole-
block elasticity matrix (symmetrically, diagonal blocks kept), from none to most of the nodes:
every level's arrays against the oracle, bitwise.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb
from parity import compare_setup, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


@pytest.mark.parametrize("share", [0.0, 0.002, 0.3])
@pytest.mark.parametrize("modes", [3, 6])
def test_ragged_blocks(share, modes):
    p, _, rbm = pb.elastic_beam(24, 5, 5)
    rows = np.repeat(np.arange(p.n), np.diff(p.rp))
    rng = np.random.Generator(np.random.PCG64(21))
    lo, hi = np.minimum(rows, p.col), np.maximum(rows, p.col)
    _, pair = np.unique(lo.astype(np.int64) * p.n + hi, return_inverse=True)
    drop = (rng.uniform(size=pair.max() + 1) < share)[pair] & (rows // 3 != p.col // 3)
    keep = ~drop
    diag = rows == p.col
    val = p.val.copy()
    # keep the matrix safely positive definite: what is dropped stays as a diagonal weight
    val[diag] += np.bincount(rows[drop], weights=np.abs(p.val[drop]), minlength=p.n)
    rp = np.zeros(p.n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows[keep], minlength=p.n))
    q = pb.CsrProblem(p.n, rp, p.col[keep], val[keep], f"ragged_{share}")
    g, h = run_both(q, nullspace=rbm[:, :modes].copy(), block_size=3, max_coarse=100,
                    cheb_boost=1.1)
    compare_setup(g, h)
    g.close()
