"""Solves that leave out rows which cannot change the result: the last bucket's, and,
for compact copies, those from which every open vertex is within the smallest
weight.  Distances, predecessors, settled counts and rounds stay the oracle's."""
import numpy as np
import pytest

import oracle
from tests.graphs import INF, random_dense

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


def graphs():
    """(name, matrix, source): last buckets of one vertex and of most, everything at one
    distance, zero-weight edges into and inside the last levels, unreachable rests,
    smallest weights of 1, 5 and the largest code of a compact copy."""
    rng = np.random.default_rng(4242)
    out = []
    for n in (1, 2, 5, 64, 257, 1030, 2051, 4099):
        for lo, hi, zero in ((1, 3, 0.0), (5, 9, 0.0), (2, 2, 0.0), (250, 254, 0.0), (65000, 65534, 0.0), (1, 2, 0.05)):
            p = min(1.0, 0.3 if hi < 1000 else 6.0 / n)
            out.append(("n%d w%d-%d z%g" % (n, lo, hi, zero),
                        random_dense(rng, n, p, lo, hi, directed=n % 2 == 1, zero_prob=zero), n // 3))
    for n in (300, 1500):
        star = np.full((n, n), INF, np.int32)
        np.fill_diagonal(star, 0)
        star[7, :] = 4
        star[7, 7] = 0
        out.append(("star n%d" % n, star, 7))
        cut = random_dense(rng, n, 0.4, 1, 3)
        cut[:n // 2, n // 2:] = INF
        cut[n // 2:, :n // 2] = INF
        out.append(("two halves n%d" % n, cut, 3))
        # the last level reached only through zero-weight edges of its own bucket
        late = np.full((n, n), INF, np.int32)
        np.fill_diagonal(late, 0)
        late[0, 1:n - 5] = 3
        for k in range(n - 5, n):
            late[n - 5 - k % 3 - 1, k] = 0
        out.append(("zero tail n%d" % n, late, 0))
    return out


GRAPHS = graphs()


def same(name, what, dist, pred, dr, pr):
    assert np.array_equal(dist.cpu().numpy(), dr), (name, what)
    assert np.array_equal(pred.cpu().numpy(), pr), (name, what)


@pytest.mark.parametrize("case", range(len(GRAPHS)), ids=[g[0] for g in GRAPHS])
def test_last_buckets(sp, case):
    name, W, src = GRAPHS[case]
    n = W.shape[0]
    dr, pr, relaxed = oracle.dijkstra(W, src)
    levels = len({int(x) for x in dr if x != INF})
    Wt = torch.from_numpy(W).cuda()
    dist = torch.full((n,), -9, dtype=torch.int32, device="cuda")
    pred = torch.full((n,), -9, dtype=torch.int32, device="cuda")
    # the default solve and its whole-GPU and one-workgroup forms that read every row
    for flags in (0, sp.SSSP_FLAG_GRID, sp.SSSP_FLAG_SINGLE):
        sp.sssp_dense_solve_ex(Wt, n, n, src, dist, pred, flags)
        status, stats = sp.sssp_last_status()
        assert status & 3 == 0
        same(name, flags, dist, pred, dr, pr)
        assert stats[1] == relaxed, (name, flags, stats, relaxed)
        if not status & sp.SSSP_STATUS_ZERO_FALLBACK:
            assert stats[0] == levels, (name, flags, stats, levels)
        rows = [r for _, r in sp.sssp_last_trace()[:-1]]
        if stats[0] <= 256 and not status & sp.SSSP_STATUS_ZERO_FALLBACK:
            assert sum(rows) == relaxed, (name, flags)
    # one workgroup and gangs, from the int32 matrix and from a compact copy
    items = [(Wt, src, dist, pred)]
    for flags in (0, sp.SSSP_FLAG_COMPACT):
        for tuning in (dict(single_max_n=16384), dict(single_max_n=1, gang_columns=64),
                       dict(single_max_n=1, gang_columns=1024)):
            dist.fill_(-9)
            pred.fill_(-9)
            with sp.BatchPlan(items, flags, **tuning) as plan:
                plan.launch()
                status, stats = plan.status()
                assert status & 3 == 0
                same(name, (flags, tuning), dist, pred, dr, pr)
                assert stats[1] == relaxed, (name, flags, tuning, stats)
                if not status & sp.SSSP_STATUS_ZERO_FALLBACK:
                    assert stats[0] == levels, (name, flags, tuning, stats, levels)


def test_server_queries(sp):
    with sp.Server(single_max_n=512, gang_columns=256) as srv:
        todo = []
        for name, W, src in GRAPHS:
            n = W.shape[0]
            Wt = torch.from_numpy(W).cuda()
            torch.cuda.current_stream().synchronize()
            out = [torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2)]
            torch.cuda.current_stream().synchronize()
            gid = srv.add_graph(Wt, sp.SSSP_FLAG_COMPACT)
            todo.append((name, W, src, out, srv.submit(gid, src, *out)))
        for name, W, src, (dist, pred), t in todo:
            srv.wait(t, timeout_s=60)
            dr, pr, _ = oracle.dijkstra(W, src)
            same(name, "served", dist, pred, dr, pr)
