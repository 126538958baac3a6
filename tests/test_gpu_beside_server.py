"""Other calls while a server's kernel stays on the GPU (it leaves a few compute units
free): their workgroups find room or are done without, and nothing waits for the server
to leave."""
import time

import numpy as np
import pytest

import oracle
from tests.graphs import random_dense

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STAY_MS = 8000  # the server's kernel leaves after this long without queries


@pytest.fixture(scope="module")
def sp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2504_03667_amd as m
    m.lib()
    return m


class Busy:
    """A server whose kernel has just answered a query and stays.  (With much more than
    three quarters of the compute units held, the hardware keeps most other kernels
    waiting although some units are free.)"""

    def __init__(self, sp, workgroups, idle_park_ms=STAY_MS):
        n = 40
        W = torch.from_numpy(random_dense(np.random.default_rng(1), n, 0.5, 1, 9)).cuda()
        self.out = [torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2)]
        torch.cuda.synchronize()
        self.srv = sp.Server(workgroups=workgroups, idle_park_ms=idle_park_ms)
        self.gid = self.srv.add_graph(W)
        self.touch()

    def touch(self):
        self.srv.wait(self.srv.submit(self.gid, 0, *self.out), timeout_s=60)
        self.since = time.perf_counter()

    def stayed(self):
        assert time.perf_counter() - self.since < STAY_MS / 2e3, "a call waited for the server to leave"


def lists(n, seed, directed=False):
    rng = np.random.default_rng(seed)
    eu, ev = rng.integers(0, n, size=(2, 3 * n)).astype(np.int32)
    ew = rng.integers(1, 1000, size=3 * n).astype(np.int32)
    rp, col, w = oracle.edges_to_csr(eu, ev, ew, n, directed)
    return [torch.from_numpy(a).cuda() for a in (rp, col, w)], oracle.dijkstra_csr(rp, col, w, 0)


@pytest.mark.parametrize("held", [128, 192])
def test_csr_solve(sp, held):
    cases = [(n, *lists(n, n)) for n in (900, 5000, 20000)]
    full = {n: sp.sssp_csr_grid(n)[0] for n, _, _ in cases}
    for n, csr, _ in cases:
        sp.csr_solve(*csr, 0)  # code and scratch are there when the server starts
    cus = sp.sssp_csr_grid(900)[2]
    busy = Busy(sp, held)
    with busy.srv:
        for n, csr, (dr, pr, _) in cases:
            for workgroups in (0, 1024):
                busy.touch()
                grid, per_cu, _ = sp.sssp_csr_grid(n, workgroups)
                assert grid <= per_cu * (cus - held)
                d, p = sp.csr_solve(*csr, 0, workgroups=workgroups)
                status, _ = sp.sssp_last_status()
                busy.stayed()
                assert status & 3 == 0, (n, status)
                assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), n
    assert {n: sp.sssp_csr_grid(n)[0] for n, _, _ in cases} == full


def test_csr_grid_beside_a_server_on_most_of_the_gpu(sp):
    """The solve starts when the server leaves, with the whole GPU."""
    full = sp.sssp_csr_grid(40000)[0]
    csr, (dr, pr, _) = lists(20000, 6)
    busy = Busy(sp, 248, idle_park_ms=50)
    with busy.srv:
        assert sp.sssp_csr_grid(40000)[0] == full
        d, p = sp.csr_solve(*csr, 0)
        assert sp.sssp_last_status()[0] & 3 == 0
        assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr)


def test_csr_grid_beside_a_parked_server(sp):
    full = sp.sssp_csr_grid(40000)[0]
    csr, (dr, pr, _) = lists(20000, 3)
    busy = Busy(sp, 192, idle_park_ms=1)
    with busy.srv:
        for _ in range(200):
            if sp.sssp_csr_grid(40000)[0] == full:
                break
            time.sleep(0.01)
        assert sp.sssp_csr_grid(40000)[0] == full
        d, p = sp.csr_solve(*csr, 0)
        busy.touch()  # comes back while the solve may still run
        assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr)
        assert sp.sssp_last_status()[0] & 3 == 0


def test_csr_solve_beside_a_batch_on_half_the_gpu(sp):
    """The batch holds half of the compute units for some milliseconds: the solve's
    workgroups that find no room take no part, whatever their number."""
    rng = np.random.default_rng(5)
    n = 1000
    W = torch.from_numpy(random_dense(rng, n, 0.005, 1, 1000)).cuda()
    items = [(W, int(s), *(torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2)))
             for s in rng.integers(0, n, size=640)]
    csr, (dr, pr, _) = lists(30000, 4)
    streams = [torch.cuda.Stream() for _ in range(2)]
    with sp.BatchPlan(items, single_max_n=16384, workgroups=128, group_sources=1) as plan:
        for workgroups in (0, 4, 128, 129, 1024):
            torch.cuda.synchronize()
            d, p = (torch.full((30000,), -9, dtype=torch.int32, device="cuda") for _ in range(2))
            torch.cuda.synchronize()
            plan.launch(stream=streams[0])
            sp.sssp_csr_solve(*csr, 30000, 0, d, p, workgroups=workgroups, stream=streams[1])
            assert sp.sssp_last_status(stream=streams[1])[0] & 3 == 0
            assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), workgroups
            assert plan.status(stream=streams[0])[0] & 3 == 0


def batch(rng, sizes):
    items, refs = [], []
    for n in sizes:
        W = random_dense(rng, n, min(1.0, 0.05 + 3.0 / n), 1, 30)
        s = int(rng.integers(0, n))
        d, p = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2))
        items.append((torch.from_numpy(W).cuda(), s, d, p))
        refs.append(oracle.dijkstra(W, s)[:2])
    return items, refs


def compare(items, refs):
    for (_, _, d, p), (dr, pr) in zip(items, refs):
        assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr), d.numel()
        d.fill_(-9)
        p.fill_(-9)


@pytest.mark.parametrize("held", [128, 192])
def test_one_shot_batch(sp, held):
    items, refs = batch(np.random.default_rng(7), [70, 300, 1500, 2500, 4000])
    sp.sssp_dense_solve_batched(items)
    compare(items, refs)
    busy = Busy(sp, held)
    with busy.srv:
        for _ in range(3):
            busy.touch()
            sp.sssp_dense_solve_batched(items)
            assert sp.sssp_last_status()[0] & 3 == 0
            busy.stayed()
            compare(items, refs)


def test_plan_with_gangs_larger_than_what_is_free(sp):
    """Made while the GPU is free; a gang that cannot form is given up, and one workgroup
    solves its item.  Both kinds of matrices, and launches before and after."""
    items, refs = batch(np.random.default_rng(8), [40, 900, 1500, 2000, 2000])
    for flags in (0, sp.SSSP_FLAG_COMPACT):
        with sp.BatchPlan(items, flags, single_max_n=64, gang_columns=16) as plan:
            assert plan.info()["max_parts"] > 64
            plan.launch()
            compare(items, refs)
            busy = Busy(sp, 192)
            with busy.srv:
                for _ in range(3):
                    busy.touch()
                    plan.launch()
                    assert plan.status()[0] & 3 == 0
                    busy.stayed()
                    compare(items, refs)
            plan.launch()
            assert plan.status()[0] & 3 == 0
            compare(items, refs)


def test_batches_beside_whole_gpu_solves(sp):
    """On two streams at once: split batches and solves that need all of their workgroups."""
    rng = np.random.default_rng(9)
    items, refs = batch(rng, [300, 1500, 2500, 4000, 6000])
    n = 6000
    W = random_dense(rng, n, 0.01, 1, 100)
    dr, pr, _ = oracle.dijkstra(W, 5)
    Wt = torch.from_numpy(W).cuda()
    d, p = (torch.full((n,), -9, dtype=torch.int32, device="cuda") for _ in range(2))
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(30):
        sp.sssp_dense_solve_batched(items, stream=a)
        sp.sssp_dense_solve_ex(Wt, n, n, 5, d, p, 0, stream=b)
    assert sp.sssp_last_status(stream=a)[0] & 3 == 0
    assert sp.sssp_last_status(stream=b)[0] & 3 == 0
    compare(items, refs)
    assert np.array_equal(d.cpu().numpy(), dr) and np.array_equal(p.cpu().numpy(), pr)
