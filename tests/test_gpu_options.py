"""Execution options on launches of few walks: they never change results, and
the autotuner keeps what a small sample cannot tell."""
import numpy as np
import pytest

import oracle as O
import paper_1805_00280_amd as P
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    # no hub rows: a walk call with a wavefront per walk
    torch_cuda()
    og = oracle_rmat(12, 5, 0.25, 0.25, 0.25, 4, False)
    return og, gpu_graph_from_oracle(og)


@pytest.mark.parametrize("t_wave", [0, 5, 12, 1023, 1024, 1025])
def test_t_wave_of_lone_walks(graph, t_wave):
    og, g = graph
    for n in (1, 200):
        starts = (np.arange(n, dtype=np.uint64) * 37 % og.n).astype(np.uint32)
        want = oracle_walk(og, starts, 20, 0.5, 2.0, 9)
        got = gpu_walk(g, starts, 20, 0.5, 2.0, 9, mode=P.MODE_PERSISTENT, t_wave=t_wave)
        assert first_mismatch(got, want) is None, (n, first_mismatch(got, want))


def test_autotune_of_lone_walks_keeps_the_default_t_wave():
    torch_cuda()
    og = oracle_rmat(12, 5, 0.25, 0.25, 0.25, 4, False)
    for n in (1, 50, 1000):
        g = gpu_graph_from_oracle(og)
        g.autotune(n, 20, 0.5, 2.0)
        assert P.exec_opts(g).t_wave == 1024, n


@pytest.mark.parametrize("t_wg", [0, 1100, 65535, 65536])
def test_t_wg_where_hub_rows_are_few(t_wg):
    # two adjacent hubs with common neighbours hold 7% of the entries; every hub
    # move takes the dense merge, in the step's launch or by a workgroup
    torch_cuda()
    rng = np.random.default_rng(2)
    n = 3000
    e = rng.integers(2, n, (40_000, 2))
    hubs = [(h, int(v)) for h in (0, 1) for v in rng.choice(n - 2, 1500, replace=False) + 2] + [(0, 1)]
    og = O.CSR.from_edges(n, [(int(a), int(b)) for a, b in e if a != b] + hubs)
    g = gpu_graph_from_oracle(og)
    for count in (3, 500, 9000):
        starts = np.zeros(count, dtype=np.uint32)
        starts[1::2] = np.arange(count // 2, dtype=np.uint32) % n
        want = oracle_walk(og, starts, 12, 0.25, 4.0, 21)
        got = gpu_walk(g, starts, 12, 0.25, 4.0, 21, mode=P.MODE_PLAIN, t_wg=t_wg, sparse_ratio=1 << 20)
        assert first_mismatch(got, want) is None, (count, first_mismatch(got, want))
