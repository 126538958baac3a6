"""GPU tests of edge list conversions and hop counts at the sizes where their paths change:
adjacency lists sorted by eight lanes, by a wave, in place, and by the prefix sums' two
forms; the dense matrix at every alignment of rows, with what lies between rows left
alone; pred chains beyond what one pass of the hop count follows."""
import numpy as np
import pytest

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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).astype(np.int32)).cuda()


def lists(eu, ev, ew, n, directed):
    """(row_ptr, col, w): lists sorted by (head, weight), without self-loops."""
    if not directed:
        eu, ev, ew = np.concatenate([eu, ev]), np.concatenate([ev, eu]), np.concatenate([ew, ew])
    keep = eu != ev
    eu, ev, ew = eu[keep], ev[keep], ew[keep]
    order = np.lexsort((ew, ev, eu))
    return np.concatenate([[0], np.cumsum(np.bincount(eu, minlength=n))]), ev[order], ew[order]


def check_lists(sp, eu, ev, ew, n, directed):
    got = sp.csr_from_edges(dev(eu), dev(ev), dev(ew), n, directed)
    assert got[3] == 0
    for a, b in zip(got[:3], lists(eu, ev, ew, n, directed)):
        assert a.numel() == max(1, b.size)  # empty lists: one entry without meaning
        assert np.array_equal(a.cpu().numpy()[:b.size], b)


@pytest.mark.parametrize("directed", [True, False])
def test_lists_of_every_length(sp, directed):
    """Lists of 0 to 70 entries side by side, then 128, 129, 1000, 5000; heads repeat."""
    rng = np.random.default_rng(7)
    lens = np.concatenate([rng.permutation(71), [128, 129, 1000, 5000, 1, 8, 9, 64, 65, 0, 3]])
    n = lens.size
    eu = rng.permutation(np.repeat(np.arange(n), lens))
    ev = rng.integers(0, n, size=eu.size)
    check_lists(sp, eu, ev, rng.integers(0, 5, size=eu.size), n, directed)


@pytest.mark.parametrize("n", [1, 2, 7, 31, 1023, 1024, 1025, 4096 * 1024, 4096 * 1024 + 1])
def test_lists_of_many_vertices(sp, n):
    rng = np.random.default_rng(n)
    eu, ev = rng.integers(0, n, size=(2, 4000))
    eu[:9], ev[9:20] = n - 1, n - 1
    check_lists(sp, eu, ev, rng.integers(0, INF, size=eu.size), n, False)


@pytest.mark.parametrize("n, ld", [(1, 1), (1, 5), (2, 3), (5, 5), (5, 8), (63, 65), (1023, 1023), (1025, 1026),
                                   (4096, 4096), (4097, 4097), (4099, 4103)])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_dense_rows_at_any_alignment(sp, n, ld, shift):
    rng = np.random.default_rng(n)
    eu, ev = rng.integers(0, n, size=(2, 3 * n))
    ew = rng.integers(0, 100, size=3 * n)
    buf = torch.full((n * ld + 8,), -7, dtype=torch.int32, device="cuda")
    W = buf[shift:shift + n * ld]
    assert sp.sssp_edges_to_dense(dev(eu), dev(ev), dev(ew), n, W, ld, True) == 0
    ref = np.full((n, n), INF)
    np.fill_diagonal(ref, 0)
    off = eu != ev
    np.minimum.at(ref, (eu[off], ev[off]), ew[off])
    want = np.full(n * ld + 8, -7)
    rows = np.full((n, ld), -7)
    rows[:, :n] = ref
    want[shift:shift + n * ld] = rows.ravel()
    assert np.array_equal(buf.cpu().numpy(), want)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 65, 1000, 65535, 65536, 65537, 131073])
@pytest.mark.parametrize("depth", ["chain", "random"])
def test_hops(sp, n, depth):
    """Chains through all vertices in random order, and random trees; the last vertex of
    three or more is unreachable.  hops may take pred's place."""
    rng = np.random.default_rng(n)
    order = rng.permutation(n)
    reach = n - 1 if n > 2 else n
    before = np.arange(-1, reach - 1)
    if depth == "random":
        before = np.concatenate([[-1], (rng.random(reach - 1) * np.arange(1, reach)).astype(int)])
    pred, dist, hops = np.full(n, -1), np.full(n, INF), np.full(n, -1)
    count = np.zeros(reach, int)
    for i in range(1, reach):
        count[i] = count[before[i]] + 1
    pred[order[1:reach]] = order[before[1:]]
    dist[order[:reach]] = 3 * count
    hops[order[:reach]] = count
    p, d = dev(pred), dev(dist)
    out = torch.full((n,), 99, dtype=torch.int32, device="cuda")
    sp.sssp_hops(p, d, out)
    assert np.array_equal(out.cpu().numpy(), hops)
    sp.sssp_hops(p, d, p)
    assert np.array_equal(p.cpu().numpy(), hops)
