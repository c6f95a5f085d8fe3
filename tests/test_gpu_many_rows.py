"""Setups of more rows than one launch has wavefronts (2^26 of 64 lanes within 2^32 threads).

Nearly all rows are alone; the last ones hold two hubs, h0 and h1, that share their 40
neighbours.  h0 is the only root among them, so the shared ones join it, and h1, two steps from
it, joins through its neighbours: the join of a row of more than 32 neighbours, and in the
systems setup the node graph, block norms, labels and smoothing, all of them beyond the rows
that one launch of a wavefront per row reaches.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = (1 << 26) + 1000
SHARED = 40


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def matrix():
    """(n, rp, col, val) on the GPU: h0 = N - 500, its neighbours after it, then h1."""
    import torch
    h0 = N - 500
    h1 = h0 + SHARED + 1
    length = torch.ones(N, dtype=torch.int64, device="cuda")
    length[h0] += SHARED
    length[h1] += SHARED
    length[h0 + 1:h1] += 2
    rp = torch.zeros(N + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(length, 0)
    nnz = int(rp[-1])
    tail_rows, tail_vals = [], []
    shared = list(range(h0 + 1, h1))
    for i in range(h0, h1 + 1):
        if i in (h0, h1):
            cols = sorted(shared + [i])
        else:
            cols = [h0, i, h1]
        tail_rows += cols
        tail_vals += [float(SHARED + 1) if c == i else -1.0 for c in cols]
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    val = torch.full((nnz,), float(SHARED + 1), dtype=torch.float64, device="cuda")
    b, e = int(rp[h0]), int(rp[h1 + 1])
    col[:b] = torch.arange(h0, dtype=torch.int32, device="cuda")
    col[e:] = torch.arange(h1 + 1, N, dtype=torch.int32, device="cuda")
    col[b:e] = torch.tensor(tail_rows, dtype=torch.int32, device="cuda")
    val[b:e] = torch.tensor(tail_vals, dtype=torch.float64, device="cuda")
    return (N, rp.int(), col, val), h0, h1


@pytest.mark.parametrize("system", [False, True])
def test_last_rows(system):
    import torch
    from paper_2103_10476_amd import solver
    A, h0, h1 = matrix()
    extra = {}
    if system:
        extra = dict(block_size=1, nullspace=torch.ones(N, 1, dtype=torch.float64, device="cuda"))
    h = solver.Hierarchy(*A, options=solver.Options(max_levels=2), **extra)
    assert h.info()["n"] == [N, 1]
    agg = h.export(0, "agg")
    want = np.full(N, -1, dtype=np.int32)
    want[h0:h1 + 1] = 0
    assert np.array_equal(agg, want)
    prp = h.export(0, "P_rp")
    assert prp[h0] == 0 and prp[-1] == SHARED + 2
    # one aggregate of a constant: the smoothed P = (I - omega D^-1 Abar) Pt, row by row
    omega = h.info()["omega"][0]
    pt = 1.0 / np.sqrt(SHARED + 2.0) if system else 1.0
    d = SHARED + 1.0
    rowsum = np.full(SHARED + 2, d - 2.0)
    rowsum[[0, -1]] = d - SHARED
    np.testing.assert_allclose(h.export(0, "P_val"), pt * (1.0 - omega * rowsum / d), rtol=1e-13)
    h.close()
