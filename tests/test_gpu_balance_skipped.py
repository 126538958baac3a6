"""Balanced rounds (at least 8 chunks of bucket rows) of the default solve, which leaves
out rows that can lower nothing: members with no open column or a few open groups give
their rows up while partners claim and stream.  With the plain library and with the
stress build's pauses; dist and pred against the oracle bit for bit."""
import os

import numpy as np
import pytest

import oracle
from tests.graphs import INF, random_dense

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", params=["plain", "stress"])
def sp(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    from paper_2504_03667_amd import build, sssp
    so = build.SO if request.param == "plain" else build.SO_STRESS
    if not os.path.exists(so):
        pytest.fail("%s is not built (run the package build first)" % so)
    prev = sssp.use_library(so)
    yield m
    sssp._lib = prev


def check(sp, Wt, W, src, workgroups, tag, ref={}):
    print("balance", tag, "n", W.shape[0], "src", src, "workgroups", workgroups, flush=True)
    d, p = sp.solve(Wt, src, workgroups=workgroups, balance=1)
    status, stats = sp.sssp_last_status()
    if ref.get("of") != (tag, src):
        ref.update(of=(tag, src), want=oracle.dijkstra(W, src))
    dr, pr, relaxed = ref["want"]
    assert status & 3 == 0, (tag, status)
    bad = np.nonzero((d.cpu().numpy() != dr) | (p.cpu().numpy() != pr))[0]
    assert bad.size == 0, (tag, workgroups, bad[:5].tolist())
    assert stats[1] == relaxed, (tag, stats, relaxed)
    return stats


def test_rounds_of_most_vertices(sp):
    rng = np.random.default_rng(3200)
    for tag, W, src, wgs in (("unit", random_dense(rng, 9000, 0.97, 1, 1), 4321, (0, 64, 7, 255)),
                             ("one-two", random_dense(rng, 12000, 0.9, 1, 2, directed=True), 5, (0, 33)),
                             ("many", random_dense(rng, 14000, 0.7, 1, 2), 13999, (0, 63))):
        Wt = torch.from_numpy(W).cuda()
        for wg in wgs:
            check(sp, Wt, W, src, wg, tag)


def test_zero_weights(sp):
    rng = np.random.default_rng(3201)
    W = random_dense(rng, 9000, 0.95, 0, 1, zero_prob=0.2)
    Wt = torch.from_numpy(W).cuda()
    for wg in (0, 9, 64):
        assert check(sp, Wt, W, 11, wg, "zero")[2] > 0


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("blocks", [1, 2, 9, 0])
def test_few_open_columns_in_a_large_round(sp, blocks, zero):
    """The second round holds about 8400 vertices.  The rest, a twelfth in blocks of 64 (or
    a handful in all), keeps some slices open, wide or by single groups, while those beside
    them have nothing left to lower."""
    n = 9003
    rng = np.random.default_rng(3300 + blocks)
    late = np.zeros(n, bool)
    if blocks:
        for k in range(blocks):
            a = 64 * (7 + 15 * k)
            late[a:a + (540 // blocks if blocks < 9 else 60)] = True
    else:
        late[[1030, 1031, 5000, 8999, 9002]] = True
    near, far = np.nonzero(~late)[0], np.nonzero(late)[0]
    src = int(near[17])
    W = np.full((n, n), INF, np.int32)
    W[src, near] = 1
    for v in far:
        tails = rng.choice(near, size=40, replace=False)
        W[tails, v] = rng.integers(2, 6, size=40)
    W[near[:200], near[300:500]] = 1
    if zero:  # a late vertex joins the large round's distance: single steps, then a fused round again
        W[near[1], far[0]] = 0
        W[far[0], far[-1]] = 1
    np.fill_diagonal(W, 0)
    Wt = torch.from_numpy(W).cuda()
    for wg in (0, 64, 63, 7, 2):
        stats = check(sp, Wt, W, src, wg, "late%d-%d" % (blocks, zero))
        assert (stats[2] > 0) == zero
