"""Galerkin products whose rows have the product counts where the product's bins change over.

A forest of stars (a centre tied to its leaves) gives A P rows of the centres' lengths plus a
few products: every count around 16, 32, 64, 128, 256, 512, 1024 and 2048 occurs.  Every
level's arrays against the oracle, bitwise, with 32-bit sort keys and without them.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import test_gpu_row_lengths as rows
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
