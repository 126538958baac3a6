"""Matrices whose rows start at any multiple of 4 bytes: odd n, odd row strides and
base addresses off a 16-byte boundary, through every kernel that streams rows
(16-byte loads at any alignment; the last column group of a row is read as the
four columns that end with it)."""
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


def offset_matrix(W, ld, off):
    """W on the GPU with row stride ld, `off` entries past an aligned address; nothing
    follows the last row's n-th entry but the end of the buffer."""
    n = W.shape[0]
    buf = torch.full((off + (n - 1) * ld + n,), 12345, dtype=torch.int32, device="cuda")
    view = buf.as_strided((n, n), (ld, 1), off)
    view.copy_(torch.from_numpy(W))
    return view


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 9, 63, 255, 258, 1021, 1031, 2050, 5003])
def test_any_row_alignment(sp, n):
    rng = np.random.default_rng(7000 + n)
    W = random_dense(rng, n, min(1.0, 0.05 + 4.0 / n), 1, 40, directed=True)
    src = int(rng.integers(0, n))
    dr, pr, _ = oracle.dijkstra(W, src)
    for ld, off in ((n, 0), (n, 1), (n + 1, 3), (n + 3, 2)):
        Wt = offset_matrix(W, ld, off)
        dist = torch.empty(n, dtype=torch.int32, device="cuda")
        pred = torch.empty(n, dtype=torch.int32, device="cuda")

        def same(what):
            torch.cuda.synchronize()
            assert np.array_equal(dist.cpu().numpy(), dr), (what, n, ld, off)
            assert np.array_equal(pred.cpu().numpy(), pr), (what, n, ld, off)
            dist.fill_(-9)
            pred.fill_(-9)

        for flags in (0, sp.SSSP_FLAG_SINGLE, sp.SSSP_FLAG_GRID, sp.SSSP_FLAG_LABEL_CORRECTING,
                      sp.SSSP_FLAG_GRID | sp.SSSP_FLAG_LITERAL):
            sp.sssp_dense_solve_ex(Wt, ld, n, src, dist, pred, flags)
            same(flags)
        items = [(Wt, src, dist, pred)]
        sp.sssp_dense_solve_batched(items)
        same("batched")
        sp.sssp_dense_solve_batched(items, flags=sp.SSSP_FLAG_LABEL_CORRECTING)
        same("batched label-correcting")
        for tuning in (dict(single_max_n=2, gang_columns=64), dict(single_max_n=2, gang_columns=1024)):
            with sp.BatchPlan(items, **tuning) as plan:
                plan.launch()
                same(tuning)


@pytest.mark.parametrize("n", [5, 514, 1031])
def test_shared_matrix_groups(sp, n):
    """Lockstep groups (32 sources of one matrix) on odd strides."""
    rng = np.random.default_rng(7100 + n)
    W = random_dense(rng, n, 0.2, 1, 40)
    Wt = offset_matrix(W, n + 1, 1)
    srcs = [int(s) for s in rng.integers(0, n, 32)]
    items = [(Wt, s, torch.empty(n, dtype=torch.int32, device="cuda"),
              torch.empty(n, dtype=torch.int32, device="cuda")) for s in srcs]
    with sp.BatchPlan(items, group_sources=4, group_columns=512) as plan:
        assert plan.info()["group_items"] > 0
        plan.launch()
        torch.cuda.synchronize()
        for _, s, d, p in items:
            dr, pr, _ = oracle.dijkstra(W, s)
            assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), s
