"""Batches of few instances split over the whole GPU: sizes at the edges of a slice,
shared matrices, counts from one instance to more workgroups than the GPU holds."""
import numpy as np
import pytest

import oracle
from tests.graphs import random_dense

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("sizes,copies", [([1], 1), ([64], 1), ([65], 1), ([4100], 1), ([127, 128, 129], 3),
                                          ([1, 2, 3, 4, 63, 1000, 3001], 2), ([513], 40), ([700, 900], 150),
                                          ([1500], 300)])
def test_one_shot_and_plan(sp, sizes, copies):
    rng = np.random.default_rng(sum(sizes) + copies)
    items, refs = [], []
    for n in sizes:
        W = random_dense(rng, n, min(1.0, 0.05 + 3.0 / n), 1, 30, zero_prob=0.02 if n == 1000 else 0.0)
        Wt = torch.from_numpy(W).cuda()
        want = {}
        for _ in range(copies):
            s = int(rng.integers(0, n))
            if s not in want:
                want[s] = oracle.dijkstra(W, s)
            items.append((Wt, s, torch.full((n,), -9, dtype=torch.int32, device="cuda"),
                          torch.full((n,), -9, dtype=torch.int32, device="cuda")))
            refs.append(want[s])

    def check(what, stats):
        for (_, s, d, p), (dr, pr, _) in zip(items, refs):
            assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), (what, s)
            d.fill_(-9)
            p.fill_(-9)
        assert stats[1] == sum(r for _, _, r in refs), what

    for flags in (0, sp.SSSP_FLAG_LITERAL):
        sp.sssp_dense_solve_batched(items, flags=flags)
        status, stats = sp.sssp_last_status()
        assert status & 3 == 0
        check(("one-shot", flags), stats)
    for flags in (0, sp.SSSP_FLAG_COMPACT):
        with sp.BatchPlan(items, flags) as plan:
            if plan.info()["lc_instances"]:
                continue  # label-correcting counts rows, not vertices
            for _ in range(2):
                plan.launch()
                status, stats = plan.status()
                assert status & 3 == 0
                check(("plan", flags), stats)


@pytest.mark.parametrize("sizes,copies", [([769], 1), ([1026, 1025], 2), ([2049], 40), ([4100, 300, 1500], 5),
                                          ([5001], 30), ([6001, 768], 16), ([9000], 3)])
def test_one_shot_splits(sp, sizes, copies):
    """Gangs of the one-shot call: slices of 64 to 2048 columns whose last is partial,
    beside instances that are not split; few rounds and many; zero weights."""
    rng = np.random.default_rng(sum(sizes) * copies)
    items, refs = [], []
    for n in sizes:
        for p, hi, zero in ((0.05, 30, 0.0), (5.0 / n, 1000, 0.02)):
            W = random_dense(rng, n, p, 1, hi, zero_prob=zero)
            Wt, want = torch.from_numpy(W).cuda(), {}
            for _ in range(copies):
                s = int(rng.integers(0, 5))
                want[s] = want.get(s) or oracle.dijkstra(W, s)
                items.append((Wt, s, *(torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2))))
                refs.append(want[s])
    sp.sssp_dense_solve_batched(items)
    status, stats = sp.sssp_last_status()
    assert status & 3 == 0
    for (_, s, d, p), (dr, pr, _) in zip(items, refs):
        assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), (d.numel(), s)
    assert stats[1] == sum(r for _, _, r in refs)
