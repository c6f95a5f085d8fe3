"""The aggregates' QR with nullspaces of one to sixteen columns.

A wavefront runs the sums of one aggregate's columns side by side, eight products ahead, a row
per lane in the updates: aggregates of fewer than 8 and of more than 64 rows, a single column,
as many as are allowed, and a column that is zero on a part of the nodes (no reflection there).
Every level's arrays against the oracle, bitwise.
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


def nullspace(n, k, zeros):
    B = np.random.Generator(np.random.PCG64(k)).uniform(0.5, 1.5, size=(n, k))
    if zeros:
        B[: n // 2, k - 1] = 0.0
    return B


@pytest.mark.parametrize("k,zeros", [(1, False), (2, True), (5, False), (6, True), (16, False)])
def test_columns(k, zeros):
    p, _, _ = pb.elastic_beam(24, 5, 5)
    g, h = run_both(p, nullspace=nullspace(p.n, k, zeros), block_size=3, max_coarse=100,
                    max_levels=3, cheb_boost=1.1)
    compare_setup(g, h)
    g.close()


def test_short_aggregates():
    p = pb.fd7_stretched(12, 1000.0)
    g, h = run_both(p, nullspace=np.ones((p.n, 1)), block_size=1, max_coarse=60)
    compare_setup(g, h)
    g.close()
