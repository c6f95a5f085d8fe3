"""Sorting rows of 257 to 1024 entries by a block that counts smaller keys, next to longer ones.

Stars whose centres' rows take every length around 256, 512 and 1024, with and without rows
beyond 1024 beside them (those go to the block's bitonic sort), on shuffled vertices: the
strength graph, the aggregates' members and R are sorted this way.  Every level's arrays against
the oracle, bitwise.
"""
import pytest

import test_gpu_row_lengths as row_lengths
from parity import compare_setup, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


@pytest.mark.parametrize("lengths", [
    list(range(253, 259)) + list(range(508, 516)) + list(range(1016, 1021)),
    list(range(1019, 1028)) + [1500, 5000],
], ids=["to_1024", "beyond"])
def test_lengths(lengths, monkeypatch):
    monkeypatch.setattr(row_lengths, "LENGTHS", lengths)
    g, h = run_both(row_lengths.stars(True), theta=0.0, max_coarse=10, max_levels=3,
                    variants=["offlmp", "1norm"])
    compare_setup(g, h)
    g.close()
