"""GPU tests of the one-workgroup solve at the sizes where its number of threads changes,
with every number forced: dist, pred and statistics equal Algorithm 1's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INF = 2 ** 31 - 1


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("threads", [0, 256, 512, 1024])
@pytest.mark.parametrize("n", [1, 127, 128, 129, 767, 768, 769, 1024, 2047, 2048, 2049])
def test_thread_counts(sp, n, threads):
    rng = np.random.default_rng(n)
    for p, lo, hi in ((0.3, 1, 9), (min(1.0, 6 / n), 1, 400), (0.2, 0, 3)):
        W = np.where(rng.random((n, n)) < p, rng.integers(lo, hi, (n, n)), INF).astype(np.int32)
        np.fill_diagonal(W, 0)
        d, q = sp.solve(torch.from_numpy(W).cuda(), n // 2, flags=sp.SSSP_FLAG_SINGLE, threads=threads)
        status, stats = sp.sssp_last_status()
        dr, pr = oracle.dijkstra(W, n // 2)[:2]
        assert status & 3 == 0
        assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(q.cpu().numpy(), pr)
        assert stats[1] == np.count_nonzero(dr != INF)
