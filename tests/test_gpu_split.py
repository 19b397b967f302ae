"""How a persistent launch splits its walks: by wavefront index, to part of the
lanes, and from the shared counter, around the sizes where the rule changes (on
a 256-CU device a weighted graph's grid has 5120 wavefronts, an unweighted
one's 6144), on graphs without hub rows, with
some, and with most entries in them; and the membership filter on rows whose
words several rows share."""
import numpy as np
import pytest

import oracle as O
import paper_1805_00280_amd as P
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, say, torch_cuda, u32

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 255, 2049, 5119, 5121, 10_241, 40_961, 330_001, 1_400_003]


@pytest.mark.parametrize("d_rule", [1024, 100, 12])  # no entries in hub rows, part of them, most
@pytest.mark.parametrize("weighted", [False, True])
def test_split_covers_every_walk(d_rule, weighted):
    torch = torch_cuda()
    og = oracle_rmat(10, 8, 0.57, 0.19, 0.19, 6, weighted)
    g = gpu_graph_from_oracle(og, d_rule=d_rule)
    for n in SIZES:
        say(f"[split] d_rule={d_rule} weighted={weighted} walks={n}")
        starts = (np.arange(n, dtype=np.uint64) * 7 % og.n).astype(np.uint32)
        L = 7 if n < 100_000 else 3
        want = oracle_walk(og, starts, L, 0.5, 2.0, 12, d_rule=d_rule)
        got = gpu_walk(g, starts, L, 0.5, 2.0, 12, mode=P.MODE_PERSISTENT)
        assert first_mismatch(got, want) is None, (n, first_mismatch(got, want))
        cnt = torch.zeros(og.n, dtype=torch.int32, device="cuda")
        cs = torch.zeros(1, dtype=torch.int64, device="cuda")
        g.walk_counts(torch.from_numpy(starts.view(np.int32)).cuda(), L, 0.5, 2.0, 12, cnt, cs)
        torch.cuda.synchronize()
        live = want[want != 0xFFFFFFFF]
        assert np.array_equal(u32(cnt), np.bincount(live, minlength=og.n).astype(np.uint32)), n


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 6, 7, 95])
def test_rows_stored_four_entries_at_a_time(L):
    # dead ends (a directed graph) end rows at every column; entries before and
    # after them come in groups cut by the rows' own ends
    torch = torch_cuda()
    rng = np.random.default_rng(L)
    n = 3000
    deg = rng.integers(0, 9, n) * (rng.random(n) < 0.97)
    off = np.zeros(n + 1, dtype=np.uint64)
    off[1:] = np.cumsum(deg)
    adj = np.concatenate([np.sort(rng.choice(n - 1, d, replace=False)) for d in deg]) if off[-1] else np.zeros(0)
    row = np.repeat(np.arange(n), deg)
    adj = (adj + (adj >= row)).astype(np.uint32)  # no self-loops
    og = O.CSR(off, adj, None)
    g = gpu_graph_from_oracle(og)
    starts = np.tile(np.arange(n, dtype=np.uint32), 3)
    want = oracle_walk(og, starts, L, 2.0, 0.5, 8)
    got = gpu_walk(g, starts, L, 2.0, 0.5, 8)
    assert first_mismatch(got, want) is None, first_mismatch(got, want)
    # an output that is only 4-byte aligned
    out = torch.zeros(len(starts) * (L + 1) + 1, dtype=torch.int32, device="cuda")[1:].view(len(starts), L + 1)
    g.walk(torch.from_numpy(starts.view(np.int32)).cuda(), L, 2.0, 0.5, 8, out=out)
    torch.cuda.synchronize()
    assert np.array_equal(u32(out), want)


@pytest.mark.parametrize("p,q", [(1.0, 0.25), (4.0, 4.0)])
def test_large_graph_of_short_rows(p, q):
    # 2^18 vertices of mean degree 10: the entries carry their neighbours' rows
    torch_cuda()
    og = oracle_rmat(18, 5, 0.25, 0.25, 0.25, 18, False)
    g = gpu_graph_from_oracle(og)
    starts = np.arange(0, og.n, 5, dtype=np.uint32)
    want = oracle_walk(og, starts, 15, p, q, 77)
    for mode in (P.MODE_PERSISTENT, P.MODE_PLAIN):
        got = gpu_walk(g, starts, 15, p, q, 77, mode=mode)
        assert first_mismatch(got, want) is None, (mode, first_mismatch(got, want))
    # capped moves and hub rows on the same kind of entries
    g2 = gpu_graph_from_oracle(og, d_rule=22, a_cap=2)
    g2.attach_memo()
    want = oracle_walk(og, starts, 15, p, q, 77, d_rule=22, a_cap=2)
    for mode in (P.MODE_PERSISTENT, P.MODE_PLAIN):
        got = gpu_walk(g2, starts, 15, p, q, 77, mode=mode)
        assert first_mismatch(got, want) is None, (mode, first_mismatch(got, want))


@pytest.mark.parametrize("d_rule,a_cap", [(1024, 1024), (100, 1024), (12, 3)])  # few hub moves, many, and capped ones
def test_plain_supersteps_of_every_size(d_rule, a_cap):
    # 1, 4, 8 or 64 lanes make a walk's attempts, by the number of walks; hub
    # and capped moves in the same launch or queued
    torch_cuda()
    og = oracle_rmat(10, 8, 0.57, 0.19, 0.19, 6, False)
    g = gpu_graph_from_oracle(og, d_rule=d_rule, a_cap=a_cap)
    for n in (1, 7, 65, 8192, 8193, 32_769, 65_537, 262_145):
        say(f"[plain] d_rule={d_rule} walks={n}")
        starts = (np.arange(n, dtype=np.uint64) * 5 % og.n).astype(np.uint32)
        L = 6 if n < 100_000 else 3
        want = oracle_walk(og, starts, L, 0.25, 2.0, 12, d_rule=d_rule, a_cap=a_cap)
        got = gpu_walk(g, starts, L, 0.25, 2.0, 12, mode=P.MODE_PLAIN)
        assert first_mismatch(got, want) is None, (n, first_mismatch(got, want))
