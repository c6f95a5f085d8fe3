"""GPU parity of the root selection's looks and stamps at their edges.

A chain decides three vertices a round, so its round stamps wrap and are aged many times over;
its round count is known: roots 0, 3, 6, ..., T of them, one a round, and the reported count is
2 T - 1, plus 1 if the last root has a vertex after it to mark.  Combs of hubs have balls of
one, several and many steps of the looking lanes (rows of 1, 8, 9, 32, 33, 64, 65, 300 and 700
neighbours).  Both run on the grid with one and with four vertices per thread and in one
workgroup, in natural and hashed order, against the oracle: aggregates, roots and every setup
array bitwise.
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


def from_edges(n, a, b):
    """Graph Laplacian plus 0.01 I of the edges (a, b), all couplings strong."""
    rows = np.concatenate([a, b, np.arange(n)])
    cols = np.concatenate([b, a, np.arange(n)])
    deg = np.bincount(np.concatenate([a, b]), minlength=n)
    vals = np.concatenate([-np.ones(2 * a.size), deg + 0.01])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return pb.CsrProblem(n, rp, cols[o].astype(np.int32), vals[o], "graph")


def chain(n):
    return from_edges(n, np.arange(n - 1), np.arange(1, n))


def comb():
    """Hubs of the listed degrees spread over the index range, tied to their leaves and to the
    next hub; leaves are chained in index order."""
    rng = np.random.Generator(np.random.PCG64(11))
    deg = [1, 8, 9, 32, 33, 64, 65, 300, 700]
    n = 4000
    hubs = rng.choice(n, size=len(deg), replace=False)
    pairs = set()
    for h, d in zip(hubs, deg):
        for v in rng.choice(n, size=d, replace=False):
            if v != h:
                pairs.add((min(h, v), max(h, v)))
    for h, g in zip(hubs[:-1], hubs[1:]):
        pairs.add((min(h, g), max(h, g)))
    for v in range(n - 1):
        pairs.add((v, v + 1))
    e = np.array(sorted(pairs))
    return from_edges(n, e[:, 0], e[:, 1])


MODES = {"grid": ("0", None), "grid, four": ("0", "0"), "workgroup": ("1073741824", None)}


@pytest.mark.parametrize("order", ["natural", "hashed"])
@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("name", ["chain 4999", "chain 5120", "chain 379", "comb"])
def test_looks(name, mode, order, monkeypatch):
    for var, v in zip(("SAAMG_MIS_WG_MAX_N", "SAAMG_MIS_V_MIN_N"), MODES[mode]):
        if v is None:
            monkeypatch.delenv(var, raising=False)
        else:
            monkeypatch.setenv(var, v)
    n = int(name.split()[1]) if name.startswith("chain") else 0
    p = chain(n) if n else comb()
    # theta 0: every coupling strong; one level of aggregation is what is looked at
    g, h = run_both(p, theta=0.0, max_levels=2, max_coarse=10, agg_order=order, seed=5)
    compare_setup(g, h)
    if n and order == "natural":
        roots = -(-n // 3)
        assert g.info()["mis_rounds"][0] == 2 * roots - 1 + (1 if 3 * (roots - 1) < n - 1 else 0)
    g.close()
