"""Galerkin products whose rows have the product counts where the product's bins change over.

A forest of stars (a centre tied to its leaves) gives A P rows of the centres' lengths plus a
few products: every count around 16, 32, 64, 128, 256, 512, 1024 and 2048 occurs.  Grids with
weakly tied far vertices give rows past the column tiles and ranges of the long rows' kernel.
Every level's arrays against the oracle, bitwise, the stars with 32-bit sort keys and without.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import test_gpu_row_lengths as rows
from paper_2103_10476_amd import problems as pb
from parity import compare_setup, run_both

pytestmark = pytest.mark.gpu

BOUNDS = [16, 32, 64, 128, 256, 512, 1024, 2048]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def counts(lv):
    A = sp.csr_matrix((np.ones(len(lv.A[1])), lv.A[1], lv.A[0]), shape=(lv.n, lv.n))
    return (A @ np.diff(lv.P[0]).astype(float)).astype(np.int64)


@pytest.mark.parametrize("key64", [None, "1"])
def test_rows_around_the_bins(key64, monkeypatch):
    monkeypatch.setattr(rows, "LENGTHS", [b + d for b in BOUNDS for d in range(-5, 3)])
    if key64:
        monkeypatch.setenv("SAAMG_SPGEMM_KEY64", key64)
    else:
        monkeypatch.delenv("SAAMG_SPGEMM_KEY64", raising=False)
    g, h = run_both(rows.stars(False), theta=0.0, max_coarse=10, max_levels=3,
                    variants=["offlmp", "1norm"])
    seen = set(counts(h.levels[0]).tolist())
    assert all(b in seen and b + 1 in seen for b in BOUNDS), sorted(seen)
    compare_setup(g, h)
    g.close()


def far_coupled(side, hubs, entries, seed=5):
    """A five-point Laplacian with `hubs` vertices weakly tied to `entries` others each."""
    n = side * side
    g = np.arange(n).reshape(side, side)
    rng = np.random.Generator(np.random.PCG64(seed))
    h = rng.permutation(n)[:hubs]
    a = [g[:, :-1].ravel(), g[:-1].ravel(), np.repeat(h, entries)]
    b = [g[:, 1:].ravel(), g[1:].ravel(), rng.integers(0, n, hubs * entries)]
    w = np.concatenate([np.ones(a[0].size + a[1].size), np.full(hubs * entries, 0.01)])
    a, b = np.concatenate(a), np.concatenate(b)
    w[a == b] = 0.0
    W = sp.coo_matrix((w, (a, b)), shape=(n, n)).tocsr()
    W = W + W.T
    A = (sp.diags(np.asarray(W.sum(axis=1)).ravel() + 0.05) - W).tocsr()
    A.sort_indices()
    return pb.CsrProblem(n, A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data,
                         f"far_{side}_{hubs}")


# more than 2048 long rows take a wavefront each (over two column tiles), fewer a block (the
# wide grid's over two tiles); all have more columns than one range of ranks
@pytest.mark.parametrize("side, hubs, entries, tile", [(330, 2200, 440, 16384),
                                                       (640, 40, 700, 65536),
                                                       (330, 3, 9000, 16384)])
def test_long_rows(side, hubs, entries, tile):
    g, h = run_both(far_coupled(side, hubs, entries), theta=0.02, max_coarse=500)
    lv = h.levels[0]
    t = counts(lv)
    assert lv.nc > tile and int(np.sum(t > 1024)) >= hubs, (lv.nc, np.sum(t > 1024))
    compare_setup(g, h)
    g.close()
