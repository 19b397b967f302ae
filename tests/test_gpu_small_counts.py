"""Visit counts and checksums where their path changes: counters in LDS up to
4096 vertices and from 64 visits a vertex on, and per-workgroup checksums of the
plain form's fused supersteps; with and without rows, weighted and not.  And the
persistent launch at the edges of its split on this device: a wavefront per
walk, filled lanes, every lane of the largest grid."""
import numpy as np
import pytest

import oracle as O
import paper_1805_00280_amd as P
from gpuhelp import first_mismatch, gpu_graph_from_oracle, gpu_walk, oracle_rmat, oracle_walk, say, starts_tensor
from gpuhelp import torch_cuda, u32

pytestmark = pytest.mark.gpu


def check_counts(og, g, starts, L, p, q, seed, mode, d_rule, rows):
    torch = torch_cuda()
    want = O.walk(og, starts, L, p, q, seed, d_rule=d_rule, want_counts=True, nthreads=16)
    cnt = torch.zeros(og.n, dtype=torch.int32, device="cuda")
    cs = torch.zeros(1, dtype=torch.int64, device="cuda")
    out = torch.empty((len(starts), L + 1), dtype=torch.int32, device="cuda") if rows else None
    g.walk_counts(starts_tensor(torch, starts), L, p, q, seed, cnt, cs, out=out, mode=mode)
    torch.cuda.synchronize()
    assert np.array_equal(u32(cnt), want["cnt"])
    assert int(cs.cpu().numpy().view(np.uint64)[0]) == want["checksum"]
    if rows:
        assert first_mismatch(u32(out), want["out"]) is None, first_mismatch(u32(out), want["out"])


@pytest.mark.parametrize("n", [4095, 4096, 4097])
@pytest.mark.parametrize("weighted", [False, True])
def test_counters_in_lds_at_their_limits(n, weighted):
    rng = np.random.default_rng(n)
    edges = rng.integers(0, n, (9 * n, 2))
    edges = [(int(a), int(b)) for a, b in edges if a != b] + [(0, int(v)) for v in range(1, n, 2)]
    weights = {(min(a, b), max(a, b)): 1 + (a + b) * 7 % 1000 for a, b in edges} if weighted else None
    og = O.CSR.from_edges(n, edges, weights)
    g = gpu_graph_from_oracle(og, d_rule=100)
    L = 16
    for count in (4 * n - 1, 4 * n, 4 * n + 1):  # count * L around 64 n
        starts = (np.arange(count, dtype=np.uint64) * 11 % n).astype(np.uint32)
        for rows in (False, True):
            say(f"[counts] n={n} weighted={weighted} walks={count} rows={rows}")
            check_counts(og, g, starts, L, 0.25, 2.0, 6, P.MODE_PERSISTENT, 100, rows)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("d_rule", [1024, 200])  # no hub rows; rows above 200 hold 3% of the entries
def test_counts_of_fused_plain_supersteps(weighted, d_rule):
    torch = torch_cuda()
    og = oracle_rmat(10, 8, 0.57, 0.19, 0.19, 6, weighted)
    deg = np.diff(og.off.astype(np.int64))
    assert deg[deg > d_rule].sum() * 10 < len(og.adj)
    g = gpu_graph_from_oracle(og, d_rule=d_rule)
    slots = torch.cuda.get_device_properties(0).multi_processor_count * 32 * 64
    for count in (1, 63, slots // 512, slots // 512 + 1, slots // 64 + 1, slots // 8 + 1, slots // 2, slots // 2 + 1):
        starts = (np.arange(count, dtype=np.uint64) * 5 % og.n).astype(np.uint32)
        L = 6 if count < 100_000 else 2
        for rows in (False, True):
            say(f"[fused] weighted={weighted} d_rule={d_rule} walks={count} rows={rows}")
            check_counts(og, g, starts, L, 0.5, 2.0, 12, P.MODE_PLAIN, d_rule, rows)


@pytest.mark.parametrize("d_rule", [1024, 40, 12])  # no entries in hub rows, part of them, most
@pytest.mark.parametrize("weighted", [False, True])
def test_split_at_the_edges_of_this_devices_grids(d_rule, weighted):
    torch = torch_cuda()
    og = oracle_rmat(10, 8, 0.57, 0.19, 0.19, 6, weighted)
    g = gpu_graph_from_oracle(og, d_rule=d_rule)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = {cus * 8 * 9, cus * 8 * 54 + 1494, cus * 8 * 64 + 1}
    for per_cu in (5, 6):  # workgroups of four wavefronts: weighted, unweighted
        waves = cus * per_cu * 4
        sizes |= {waves - 1, waves, waves + 1, 2 * waves + 1, 8 * waves - 1, 8 * waves + 1, 64 * waves - 1, 64 * waves,
                  64 * waves + 1}
    for n in sorted(sizes):
        say(f"[edges] d_rule={d_rule} weighted={weighted} walks={n}")
        starts = (np.arange(n, dtype=np.uint64) * 7 % og.n).astype(np.uint32)
        L = 5 if n < 60_000 else 2
        want = oracle_walk(og, starts, L, 0.5, 2.0, 12, d_rule=d_rule)
        got = gpu_walk(g, starts, L, 0.5, 2.0, 12, mode=P.MODE_PERSISTENT)
        assert first_mismatch(got, want) is None, (n, first_mismatch(got, want))
        check_counts(og, g, starts, L, 0.5, 2.0, 12, P.MODE_PERSISTENT, d_rule, False)
