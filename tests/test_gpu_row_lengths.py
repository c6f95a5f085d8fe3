"""Setup arrays on rows of the lengths where the setup's row kernels change over.

A forest of stars (a centre tied to its leaves, the first leaf of a star to the next centre):
the rows of the strength graph and of R take the lengths 1 ... 700 around 8, 16, 32, 64 and
256, so the per-row sorts (8 lanes, a wavefront, a block), the transposes, the strength graph
and the product counts meet each length and a mix of them in one block.  27-point cubes put
filtered rows of 27 entries on the thread-per-row kernels with every lumping.  Every level's
arrays against the oracle, bitwise.
"""
import numpy as np
import pytest

from paper_2103_10476_amd import problems as pb
from parity import compare_setup, run_both

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 128, 255, 256, 257, 300, 700]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def stars(shuffle):
    a, b, at, last = [], [], 0, None
    for k in LENGTHS + LENGTHS[::-1]:
        centre = at
        a += [centre] * k
        b += list(range(at + 1, at + 1 + k))
        if last is not None:
            a.append(last)
            b.append(centre)
        last = at + 1
        at += k + 1
    a, b, n = np.array(a), np.array(b), at
    if shuffle:
        perm = np.random.Generator(np.random.PCG64(3)).permutation(n)
        a, b = perm[a], perm[b]
    rows = np.concatenate([a, b, np.arange(n)])
    cols = np.concatenate([b, a, np.arange(n)])
    deg = np.bincount(np.concatenate([a, b]), minlength=n)
    w = 1.0 + (np.arange(a.size) % 7) / 8.0
    diag = np.bincount(np.concatenate([a, b]), weights=np.concatenate([w, w]), minlength=n)
    vals = np.concatenate([-w, -w, diag + 0.01 * deg])
    o = np.lexsort((cols, rows))
    rp = np.zeros(n + 1, dtype=np.int32)
    rp[1:] = np.cumsum(np.bincount(rows, minlength=n))
    return pb.CsrProblem(n, rp, cols[o].astype(np.int32), vals[o], f"stars_{shuffle}")


@pytest.mark.parametrize("shuffle", [False, True])
@pytest.mark.parametrize("theta", [0.0, 0.08])
def test_stars(shuffle, theta):
    g, h = run_both(stars(shuffle), theta=theta, max_coarse=10, max_levels=3,
                    variants=["offlmp", "1norm"])
    compare_setup(g, h)
    g.close()


@pytest.mark.parametrize("variants", [["1norm"], ["offlmp"], ["offlmp", "1norm", "cnstrnt"],
                                      ["sprsfy", "offlmp", "1norm"]])
def test_27_point(variants):
    p = pb.q1_random_kappa(13, seed=9)
    g, h = run_both(p, theta=0.02, variants=variants, max_coarse=30)
    compare_setup(g, h)
    g.close()
