"""Graph creation where the size of its chunks of entries changes: 64 entries
below 131,072, twice as many from each doubling on, up to 1024.  Stars of
exactly those sizes (one row over half the entries, rows of one entry between
runs of empty rows) and R-MAT graphs inside each range; walks at 1/p = 4 follow
the reverse positions and must equal the oracle's."""
import numpy as np
import pytest

import oracle as O
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, torch_cuda

pytestmark = pytest.mark.gpu


def star(edges):
    # hub 1, leaves 4, 7, 10, ...: two empty rows before every row
    n = 3 * edges + 3
    leaf = np.arange(4, 3 * edges + 3, 3, dtype=np.uint32)
    off = np.zeros(n + 1, dtype=np.uint64)
    deg = np.zeros(n, dtype=np.int64)
    deg[1], deg[leaf] = edges, 1
    off[1:] = np.cumsum(deg)
    return O.CSR(off, np.concatenate([leaf, np.ones(edges, dtype=np.uint32)]), None)


@pytest.mark.parametrize("edges", [31, 32, 33, 65_535, 65_536, 65_537, 131_071, 131_072, 262_144, 524_287, 524_288])
def test_stars(edges):
    torch_cuda()
    og = star(edges)
    g = gpu_graph_from_oracle(og, validate=2)
    starts = np.concatenate([[0, 1, 4, og.n - 2, og.n - 1], np.arange(1, og.n, 3 * (1 + edges // 500))])
    starts = starts.astype(np.uint32)
    want = oracle_walk(og, starts, 9, 0.25, 0.5, 3)
    got = gpu_walk(g, starts, 9, 0.25, 0.5, 3)
    assert first_mismatch(got, want) is None, first_mismatch(got, want)


@pytest.mark.parametrize("scale,ef,weighted", [(9, 16, True), (12, 16, False), (13, 16, True), (12, 50, False),
                                               (15, 16, False), (16, 16, True)])
def test_rmat(scale, ef, weighted):
    torch_cuda()
    og = oracle_rmat(scale, ef, 0.57, 0.19, 0.19, scale, weighted)
    g = gpu_graph_from_oracle(og, validate=2, d_rule=100)
    starts = np.arange(0, og.n, 1 + og.n // 4000, dtype=np.uint32)
    want = oracle_walk(og, starts, 10, 0.25, 2.0, 4, d_rule=100)
    got = gpu_walk(g, starts, 10, 0.25, 2.0, 4)
    assert first_mismatch(got, want) is None, first_mismatch(got, want)
