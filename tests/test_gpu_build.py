"""Graph creation at the edges of its work split: rows and runs of empty rows
against chunks of 1024 entries.  Walks at 1/p = 4 follow the reverse positions
that creation derives, and must equal the oracle's."""
import numpy as np
import pytest

import oracle as O
import paper_1805_00280_amd as P
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, say, torch_cuda, u32

pytestmark = pytest.mark.gpu


def _spread(n, ids, edges, rng):
    a = ids[rng.integers(0, len(ids), edges)]
    b = ids[rng.integers(0, len(ids), edges)]
    return O.CSR.from_edges(n, list(zip(a.tolist(), b.tolist())))


def _graph(name):
    rng = np.random.default_rng(11)
    if name == "runs of empty rows":  # long runs at the front, between rows and at the end
        ids = np.concatenate([np.arange(5_000, 5_040), np.arange(90_000, 250_000, 977)]).astype(np.int64)
        return _spread(300_000, ids, 6_000, rng), ids
    if name == "one row over many chunks":
        n = 6_000
        hub = [(2_999, v) for v in range(n) if v != 2_999]
        extra = list(zip(rng.integers(0, n, 4_000).tolist(), rng.integers(0, n, 4_000).tolist()))
        return O.CSR.from_edges(n, hub + extra), np.arange(n)
    if name == "rows of exactly a chunk":  # complete graph of 1025 vertices: m = 1025 * 1024
        n = 1025
        i, j = np.triu_indices(n, 1)
        return O.CSR.from_edges(n, list(zip(i.tolist(), j.tolist()))), np.arange(n)
    if name == "one edge":
        return O.CSR.from_edges(70_000, [(3, 69_999)]), np.array([3, 69_999, 0])
    raise ValueError(name)


@pytest.mark.parametrize("name", ["runs of empty rows", "one row over many chunks", "rows of exactly a chunk",
                                  "one edge"])
def test_reverse_positions(name):
    torch_cuda()
    say(f"[build] {name}")
    og, ids = _graph(name)
    g = gpu_graph_from_oracle(og, validate=2)
    starts = np.tile(np.asarray(ids, dtype=np.uint32), 2)[:4_000]
    want = oracle_walk(og, starts, 12, 0.25, 4.0, 17)
    got = gpu_walk(g, starts, 12, 0.25, 4.0, 17)
    assert first_mismatch(got, want) is None, first_mismatch(got, want)


def test_entries_without_a_partner():
    # each entry of a symmetric graph dropped with probability 1/4, so that most
    # rows hold entries with and without a reverse entry
    torch_cuda()
    og = oracle_rmat(12, 16, 0.65, 0.15, 0.15, 5, False)
    keep = np.random.default_rng(3).random(len(og.adj)) < 0.75
    row = np.repeat(np.arange(og.n), np.diff(og.off.astype(np.int64)))[keep]
    off = np.zeros(og.n + 1, dtype=np.uint64)
    off[1:] = np.cumsum(np.bincount(row, minlength=og.n))
    dg = O.CSR(off, og.adj[keep].copy(), None)
    starts = np.arange(og.n, dtype=np.uint32)
    g = gpu_graph_from_oracle(dg, d_rule=200)
    want = oracle_walk(dg, starts, 12, 0.25, 2.0, 23, d_rule=200)
    for mode in (P.MODE_PERSISTENT, P.MODE_PLAIN):
        got = gpu_walk(g, starts, 12, 0.25, 2.0, 23, mode=mode)
        assert first_mismatch(got, want) is None, (mode, first_mismatch(got, want))
    with pytest.raises(P.N2VError) as e:
        gpu_graph_from_oracle(dg, validate=2)
    assert e.value.code == -3


@pytest.mark.parametrize("scale,ef,abc", [(9, 50, (0.18, 0.25, 0.25)), (11, 40, (0.9, 0.04, 0.04)), (1, 3, (0.25, 0.25, 0.25))])
def test_row_lengths_of_dense_and_skewed_graphs(scale, ef, abc):
    torch = torch_cuda()
    off, adj, wt = P.Graph.generate_rmat(scale, ef, *abc, 4, weighted=True)
    torch.cuda.synchronize()
    og = oracle_rmat(scale, ef, *abc, 4, True)
    assert np.array_equal(off.cpu().numpy().view(np.uint64), og.off)
    assert np.array_equal(u32(adj), og.adj)
    assert np.array_equal(wt.cpu().numpy().view(np.uint16), og.wt)
