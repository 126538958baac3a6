"""GPU tests of the CSR solve's sweeps at the sizes where their paths change: frontiers
that workgroup 0 keeps in LDS, those it hands back, appends beyond the LDS buffers, and
graphs solved a range of distances at a time (empty ranges, distances up to the largest
representable, zero weights).  dist and pred equal Algorithm 1's bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RANGE_N = 131072     # vertices from which ranges are used (with 4 list entries a vertex)
SOLO = 512           # frontier that workgroup 0 takes alone
CAP = 4096           # appends that a workgroup gathers in LDS (half of it while alone)
MAX_DIST = 2 ** 31 - 2


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


def check(sp, eu, ev, ew, n, src=0, workgroups=0, directed=True):
    rp, col, w = oracle.edges_to_csr(eu.astype(np.int32), ev.astype(np.int32), ew.astype(np.int32), n, directed)
    ref = oracle.dijkstra_csr(rp, col, w, src)
    got = sp.csr_solve(*(torch.from_numpy(a).cuda() for a in (rp, col, w)), src, workgroups=workgroups)
    status, stats = sp.sssp_last_status()
    assert status & 3 == 0
    assert stats[1] >= np.count_nonzero(ref[0] != 2 ** 31 - 1)
    assert np.array_equal(got[0].cpu().numpy(), ref[0])
    assert np.array_equal(got[1].cpu().numpy(), ref[1])


@pytest.mark.parametrize("workgroups", [0, 1, 2])
@pytest.mark.parametrize("width", [1, SOLO - 1, SOLO, SOLO + 1, CAP // 2, CAP // 2 + 1, CAP, CAP + 1, 3 * CAP])
def test_frontier_of_given_width(sp, width, workgroups):
    """The source reaches `width` vertices at once, each of them one more, those a common
    end: frontiers of 1, width, width, 1 whatever the order of the relaxations."""
    a, b, end = 1 + np.arange(width), 1 + width + np.arange(width), 1 + 2 * width
    eu = np.concatenate([np.zeros(width, int), a, b])
    ev = np.concatenate([a, b, np.full(width, end)])
    ew = np.concatenate([1 + np.arange(width) % 7, 1 + np.arange(width) % 3, 5 - np.arange(width) % 5])
    check(sp, eu, ev, ew, end + 1, workgroups=workgroups)


@pytest.mark.parametrize("degree", [16, 17])
def test_lists_too_long_for_one_workgroup(sp, degree):
    rng = np.random.default_rng(degree)
    n = 3000
    eu = np.repeat(np.arange(n), degree)
    ev = (eu + rng.integers(1, n, size=eu.size)) % n
    check(sp, eu, ev, rng.integers(0, 60, size=eu.size), n)


@pytest.mark.parametrize("n, lo, hi", [(RANGE_N - 1, 1, 1000), (RANGE_N, 1, 1000), (RANGE_N + 1, 1, 1000),
                                       (RANGE_N, 0, 3), (RANGE_N, 0, 0), (RANGE_N, 10 ** 8, 3 * 10 ** 8)])
def test_ranges(sp, n, lo, hi):
    rng = np.random.default_rng(n + hi)
    eu, ev = rng.integers(0, n, size=(2, 3 * n))
    check(sp, eu, ev, rng.integers(lo, hi + 1, size=eu.size), n, src=5, directed=False)


@pytest.mark.parametrize("degree", [3, 4])
def test_empty_ranges_and_largest_distances(sp, degree):
    """Two dense parts of light edges joined by one heavy edge (a gap of many ranges), and
    a tail that ends at the largest representable distance; one further is unreachable."""
    n, half = RANGE_N, RANGE_N // 2
    rng = np.random.default_rng(3)
    m = degree * n - 4
    eu = rng.integers(0, half, size=m)
    ev = rng.integers(0, half, size=m)
    eu[m // 2:] += half
    ev[m // 2:] += half
    keep = (ev != n - 1) & (ev != n - 2) & (eu != n - 1) & (eu != n - 2)
    eu, ev = eu[keep], ev[keep]
    pad = degree * n - eu.size - 4  # list entries without effect: repeats of one edge
    bridge = 10 ** 6
    eu = np.concatenate([eu, np.full(pad, 1), [0, half, n - 2, half]])
    ev = np.concatenate([ev, np.full(pad, 2), [half, n - 2, n - 1, n - 1]])
    ew = np.concatenate([rng.integers(1, 20, size=eu.size - pad - 4), np.full(pad, 20),
                         [bridge, MAX_DIST - bridge, 1, MAX_DIST - bridge + 1]])
    check(sp, eu, ev, ew, n)


def test_ranges_much_narrower_than_the_paths_edges(sp):
    """A long chain of heavy edges beside many light ones, which set the width of the
    ranges; hubs whose lists are long while the average one is short."""
    n, chain = RANGE_N, 3000
    rng = np.random.default_rng(9)
    eu, ev = rng.integers(chain, n, size=(2, 4 * n))
    ew = rng.integers(1, 4, size=eu.size)
    c = np.arange(chain - 1)
    hub = np.arange(chain, n)
    eu = np.concatenate([eu, c, np.full(hub.size, 7)])
    ev = np.concatenate([ev, c + 1, hub])
    ew = np.concatenate([ew, rng.integers(10 ** 5, 10 ** 6, size=chain - 1), rng.integers(1, 10 ** 6, size=hub.size)])
    check(sp, eu, ev, ew, n)


@pytest.mark.parametrize("workgroups", [1, 2, 3])
@pytest.mark.parametrize("spread", [1, 7, 64])
def test_appends_of_one_workgroup_beyond_the_buffer(sp, spread, workgroups):
    """Lists of 20 entries on average (no workgroup runs alone): sweeps that append many
    times what fits the buffer, by waves whose appends end, begin or lie beyond it."""
    width, fan = 5 * CAP // spread, spread
    a = 1 + np.arange(width)
    b = 1 + width + np.arange(width * fan)
    n = 1 + width + width * fan
    pad = 20 * n
    eu = np.concatenate([np.zeros(width, int), np.repeat(a, fan), np.full(pad, n - 1)])
    ev = np.concatenate([a, b, np.full(pad, 0)])
    ew = np.concatenate([1 + np.arange(width) % 7, 1 + np.arange(width * fan) % 3, np.full(pad, 9)])
    check(sp, eu, ev, ew, n, workgroups=workgroups)


@pytest.mark.parametrize("length", [63, 64, 65, 66, 300])
@pytest.mark.parametrize("hubs", [1, 7, SOLO - 1, SOLO])
def test_long_lists_in_a_short_frontier(sp, hubs, length):
    """The source reaches `hubs` vertices, each of them `length` others (shared by two
    hubs), those a common end: lists that workgroup 0 relaxes and lists that it hands back,
    beside short ones, in a graph whose lists are short on average."""
    h = 1 + np.arange(hubs)
    leaves = hubs * length // 2 + length
    first = 1 + hubs
    leaf = first + np.arange(leaves)
    end = first + leaves
    eu = np.concatenate([np.zeros(hubs, int), np.repeat(h, length), leaf])
    ev = np.concatenate([h, (first + (np.repeat((h - 1) * length // 2, length) + np.tile(np.arange(length), hubs))),
                         np.full(leaves, end)])
    ew = np.concatenate([1 + np.arange(hubs) % 5, 1 + np.arange(hubs * length) % 4, 9 - np.arange(leaves) % 9])
    mixed = np.arange(0, hubs, 3) + 1  # every third hub has a short list
    keep = ~(np.isin(eu, mixed) & (ev >= first + 5) & (hubs > 1)) | (eu >= first)
    check(sp, eu[keep], ev[keep], ew[keep], end + 1)
    check(sp, eu, ev, ew, end + 1)


@pytest.mark.parametrize("n", [300, 505, SOLO, SOLO + 2])
def test_hubs_where_every_vertex_is_lowered_in_every_sweep(sp, n):
    """Frontiers of all vertices, long lists among them: together more than a list holds."""
    v = np.arange(1, n)
    hubs = np.arange(40, 40 + 5)
    eu = np.concatenate([np.zeros(n - 1, int), v[1:], np.repeat(hubs, 70)])
    ev = np.concatenate([v, v[1:] - 1, np.tile(100 + np.arange(70), hubs.size)])
    ew = np.concatenate([10 ** 6 - 2 * v, np.ones(n - 2, int), np.full(70 * hubs.size, 10 ** 6)])
    check(sp, eu, ev, ew, n)
