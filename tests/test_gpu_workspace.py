"""Graph workspaces from the least that a graph needs to the queried size: the
parts left out of a smaller one (membership filters, rows in the entry records)
never change a walk."""
import ctypes as C

import numpy as np
import pytest

import paper_1805_00280_amd as P
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, say, torch_cuda, u32

pytestmark = pytest.mark.gpu


def query(n, m, weighted):
    ws = C.c_size_t()
    assert P.lib().n2v_graph_workspace(n, m, weighted, C.byref(ws)) == 0
    return ws.value


def sized(monkeypatch, nbytes):
    alloc = P._alloc
    monkeypatch.setattr(P, "_alloc", lambda _, device: alloc(nbytes, device))


def graph_with(og, nbytes, **kw):
    with pytest.MonkeyPatch.context() as mp:
        sized(mp, nbytes)
        return gpu_graph_from_oracle(og, **kw)


def least(og, **kw):
    """Smallest accepted workspace, in steps of 256 bytes; N2V_ENOMEM below."""
    lo, hi = 0, query(og.n, len(og.adj), int(og.wt is not None)) // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            graph_with(og, mid * 256, **kw).close()
            hi = mid
        except P.N2VError as e:
            assert e.code == -2
            lo = mid
    return hi * 256


@pytest.mark.parametrize("name,args,kw", [
    ("no hubs, rows in the entries", (18, 5, 0.25, 0.25, 0.25, 18, False), dict(d_rule=1024)),
    ("hubs, large enough for them", (18, 5, 0.57, 0.19, 0.19, 18, False), dict(d_rule=40)),
    ("weighted", (12, 16, 0.57, 0.19, 0.19, 12, True), dict(d_rule=64)),
])
def test_smaller_workspaces(name, args, kw):
    torch = torch_cuda()
    og = oracle_rmat(*args)
    n, m, weighted = og.n, len(og.adj), int(og.wt is not None)
    full, wfull, low = query(n, m, weighted), query(n, m, 1), least(og, **kw)
    # what a graph needs: 16 bytes of record, 8 of sketch index (weighted 8 of weight sum) per vertex, 8 per entry
    assert low <= 8 * m + (32 if weighted else 24) * n + 65536
    assert low + 2 * m <= full
    starts = np.arange(0, n, 1 + n // 30_000, dtype=np.uint32)
    want = oracle_walk(og, starts, 12, 2.0, 0.5, 5, **kw)
    visits = np.bincount(want[want != 0xFFFFFFFF], minlength=n).astype(np.uint32)
    for nbytes in (low, low + 2 * m + 512, wfull, full):
        say(f"[workspace] {name}: {nbytes} of {full}")
        g = graph_with(og, nbytes, validate=2, **kw)
        g.attach_memo()
        for mode in (P.MODE_PERSISTENT, P.MODE_PLAIN):
            got = gpu_walk(g, starts, 12, 2.0, 0.5, 5, mode=mode)
            assert first_mismatch(got, want) is None, (nbytes, mode, first_mismatch(got, want))
        cnt = torch.zeros(n, dtype=torch.int32, device="cuda")
        cs = torch.zeros(1, dtype=torch.int64, device="cuda")
        g.walk_counts(torch.from_numpy(starts.view(np.int32)).cuda(), 12, 2.0, 0.5, 5, cnt, cs)
        torch.cuda.synchronize()
        assert np.array_equal(u32(cnt), visits), nbytes
        g.close()


def test_a_large_graph_with_hubs_takes_no_more_than_it_uses(monkeypatch):
    # 2^21 vertices of edge factor 16: the rows could lie in the entry records by size
    torch = torch_cuda()
    assert P.TRIM_ENTRIES == 1 << 30
    monkeypatch.setattr(P, "TRIM_ENTRIES", 1 << 25)
    off, adj, _ = P.Graph.generate_rmat(21, 16, 0.57, 0.19, 0.19, 3)
    n, m = 1 << 21, adj.numel()
    assert m >= 1 << 25 and query(n, m, 1) < query(n, m, 0)
    hubs = P.Graph(off, adj, None, n=n)
    assert hubs.ws.numel() == query(n, m, 1)
    none = P.Graph(off, adj, None, n=n, d_rule=1 << 20)
    assert none.ws.numel() == query(n, m, 0)
    sized(monkeypatch, query(n, m, 0))
    whole = P.Graph(off, adj, None, n=n)
    st = torch.arange(0, n, 37, dtype=torch.int32, device="cuda")
    a, b = hubs.walk(st, 10, 0.5, 2.0, 8), whole.walk(st, 10, 0.5, 2.0, 8, ws=None)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
