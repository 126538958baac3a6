"""GPU tests of the label-correcting sweeps' exchange and of pred kept beside dist, at the
frontiers where their paths change: one entry a member (staged at once), more (read from
the lists), all vertices at once, many sweeps; ties for pred, tight and slack zero-weight
edges, negative weights; matrices on both sides of the size that is cached.  dist and pred
equal Algorithm 1's bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

INF = 2 ** 31 - 1
ZERO_FALLBACK = 4
NEG = 2


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


def solve(sp, W, src, workgroups):
    n = W.shape[0]
    d, p = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    sp.sssp_dense_solve_ex(W, n, n, src, d, p, sp.SSSP_FLAG_LABEL_CORRECTING, workgroups=workgroups)
    status, stats = sp.sssp_last_status()
    return d.cpu().numpy(), p.cpu().numpy(), status, stats


def check(sp, W, src, workgroups, zero=False):
    d, p, status, stats = solve(sp, torch.from_numpy(W).cuda(), src, workgroups)
    dr, pr = oracle.dijkstra(W, src)[:2]
    assert np.array_equal(d, dr) and np.array_equal(p, pr)
    assert status & 3 == 0
    assert bool(status & ZERO_FALLBACK) == zero
    if not zero:
        assert tuple(stats[:2]) == tuple(x + y for x, y in
                                         zip(oracle.label_correcting(W, src)[1:3], (0, np.count_nonzero(dr != INF))))


def empty(n):
    W = np.full((n, n), INF, dtype=np.int32)
    np.fill_diagonal(W, 0)
    return W


@pytest.mark.parametrize("workgroups", [0, 1, 2, 3, 64, 65])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 63, 257, 1000])
def test_frontiers(sp, n, workgroups):
    rng = np.random.default_rng(n)
    chain = empty(n)  # a sweep a vertex, in an order that jumps between members
    order = rng.permutation(n)
    chain[order[:-1], order[1:]] = 3
    check(sp, chain, int(order[0]), workgroups)
    star = empty(n)  # all at once, then again through vertex 0 for less
    star[n - 1, :] = 100
    star[n - 1, 0] = 1
    star[0, :] = 50 + np.arange(n) % 7
    np.fill_diagonal(star, 0)
    check(sp, star, n - 1, workgroups)
    ties = np.where(rng.random((n, n)) < 0.3, rng.integers(1, 4, (n, n)), INF).astype(np.int32)
    np.fill_diagonal(ties, 0)
    check(sp, ties, n // 2, workgroups)


@pytest.mark.parametrize("workgroups", [0, 1, 7])
@pytest.mark.parametrize("n", [6, 100, 301])
def test_zero_and_negative_weights(sp, n, workgroups):
    rng = np.random.default_rng(n)
    W = np.where(rng.random((n, n)) < 0.2, rng.integers(2, 90, (n, n)), INF).astype(np.int32)
    np.fill_diagonal(W, 0)
    W[0, 1:5] = [2, 3, 4, 90]
    W[:, 5] = INF
    W[5, 5] = 0
    W[4, 5] = 0      # 5 is reached from 4 alone, over weight 0
    check(sp, W, 0, workgroups, zero=True)
    W[1, 5] = 1      # ... and now over 1 for less: the edge of weight 0 is not tight
    check(sp, W, 0, workgroups, zero=False)
    W[3, 3] = 7      # a diagonal entry plays no part
    check(sp, W, 0, workgroups, zero=False)
    W[2, 4] = -1
    assert solve(sp, torch.from_numpy(W).cuda(), 0, workgroups)[2] & NEG


@pytest.mark.parametrize("n", [8191, 8192, 8193])
def test_cached_and_streamed_matrices(sp, n):
    g = torch.Generator(device="cuda").manual_seed(n)
    W = torch.randint(1, 1001, (n, n), generator=g, device="cuda", dtype=torch.int32)
    W[torch.rand(n, n, generator=g, device="cuda") > 0.002] = INF
    W.fill_diagonal_(0)
    d, p, status, _ = solve(sp, W, 17, 0)
    ref = sp.solve(W, 17)
    assert status == 0
    assert np.array_equal(d, ref[0].cpu().numpy()) and np.array_equal(p, ref[1].cpu().numpy())
