"""Whole-GPU, batched and served rounds that read no row, or few column groups, of a
slice: with pauses (libsssp_stress.so) of workgroups before an exchange and of their
waves after it.  dist and pred against the oracle bit for bit."""
import os

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
    from paper_2504_03667_amd import build, sssp
    if not os.path.exists(build.SO_STRESS):
        pytest.fail("libsssp_stress.so is not built (run the package build first)")
    prev = sssp.use_library(build.SO_STRESS)
    yield m
    sssp._lib = prev


def block_graph(rng, n, block, levels):
    """Vertices in `levels` ranges of neighbours, one range after the other: a slice's
    vertices settle together, early ones many rounds before the end."""
    W = np.full((n, n), INF, np.int32)
    np.fill_diagonal(W, 0)
    step = n // levels
    for k in range(levels):
        a, b = k * step, n if k == levels - 1 else (k + 1) * step
        W[a, a:b] = rng.integers(1, 4, size=b - a)
        W[a, a] = 0
        if k + 1 < levels:
            W[b - 1, b] = block
            W[b - 2, b] = block + 1
    return W


def check(sp, W, src, workgroups, tag):
    Wt = torch.from_numpy(np.ascontiguousarray(W)).cuda()
    print("skipped rows", tag, "n", W.shape[0], "workgroups", workgroups, flush=True)
    d, p = sp.solve(Wt, src, workgroups=workgroups)
    status, stats = sp.sssp_last_status()
    dr, pr, relaxed = oracle.dijkstra(W, src)
    assert status & 3 == 0, (tag, status)
    assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), tag
    assert stats[1] == relaxed, tag
    return stats


@pytest.mark.parametrize("workgroups", [0, 7, 40])
def test_finished_slices(sp, workgroups):
    rng = np.random.default_rng(5200)
    check(sp, block_graph(rng, 3000, 5, 30), 0, workgroups, "ranges")
    check(sp, random_dense(rng, 2500, 0.002, 1, 1000), 3, workgroups, "sparse")
    check(sp, random_dense(rng, 2500, 0.3, 1, 3), 3, workgroups, "dense")
    # a hazard in a round that some slices take no part in
    Z = block_graph(rng, 2400, 4, 24)
    for k in range(0, 24, 3):
        Z[k * 100, k * 100 + 50:k * 100 + 60] = 0
        Z[k * 100 + 50, k * 100 + 70] = 0
    assert check(sp, Z, 0, workgroups, "zero")[2] > 0


def test_finished_slices_of_gangs(sp):
    rng = np.random.default_rng(5201)
    graphs = [block_graph(rng, n, 5, 20) for n in (700, 1900, 2600)] + [random_dense(rng, 1500, 0.01, 1, 500)]
    items, want = [], []
    for W in graphs:
        n = W.shape[0]
        d, p = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2))
        items.append((torch.from_numpy(W).cuda(), 0, d, p))
        want.append(oracle.dijkstra(W, 0)[:2])
    for flags in (0, sp.SSSP_FLAG_COMPACT):
        with sp.BatchPlan(items, flags, single_max_n=512, gang_columns=128) as plan:
            for _ in range(3):
                plan.launch()
                assert plan.status()[0] & 3 == 0
                for (_, _, d, p), (dr, pr) in zip(items, want):
                    assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr)
                    d.fill_(-9)
    torch.cuda.current_stream().synchronize()
    with sp.Server(single_max_n=512, gang_columns=128) as srv:
        jobs = [(srv.submit(srv.add_graph(W), src, d, p), d, p, ref) for (W, src, d, p), ref in zip(items, want)]
        for t, d, p, (dr, pr) in jobs:
            srv.wait(t, timeout_s=60)
            assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr)
