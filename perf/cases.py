"""The work that users of this framework have it do, as measurable cases.

Each case is a dict of plain values.  `prepare` makes what a program holds before
the call (matrices in HBM, edge lists, a plan, a server with resident graphs),
`run` is one pass through the public entry points, `exact` the same answer from
plain torch in 64 bits, and `work` the bytes and operations a pass cannot do
without (each input read once, each output written once; one addition and one
comparison per matrix entry or list edge and source).

Graphs are seeded random ones: G(n, p) matrices with integer weights in [1, hi]
(INT32_MAX = no edge, zero diagonal), or edge lists of m = 3n edges, the paper's
sparse family.
"""
import math
import random
import weakref

import torch

import paper_2504_03667_amd as sp

INF = 0x7FFFFFFF
DEV = "cuda"


def listed():
    return [
        # Smallest calls: launch and round latency of one solve.
        dict(name="solve_n256", kind="solve", n=256, p=0.1, hi=100, directed=False, lc=False),
        # The latency workload: n=1024, p=0.1, weights in [1, 100].
        dict(name="solve_n1024", kind="solve", n=1024, p=0.1, hi=100, directed=False, lc=False),
        # An odd size in a contiguous matrix, as a program that reads a graph file gets it.
        dict(name="solve_n5001", kind="solve", n=5001, p=0.05, hi=100, directed=False, lc=False),
        # The medium workload: n=16384, p=0.01, weights in [1, 100], directed.
        dict(name="solve_n16384_directed", kind="solve", n=16384, p=0.01, hi=100, directed=True, lc=False),
        # The headline workload: n=65536, p=0.5, weights in [1, 1000] (16 GiB).
        dict(name="solve_n65536", kind="solve", n=65536, p=0.5, hi=1000, directed=False, lc=False),
        # Many distinct distances: a sparse matrix with wide weights, label-correcting.
        dict(name="solve_lc_n8192", kind="solve", n=8192, p=0.001, hi=1000, directed=False, lc=True),
        # Graphs of uneven size, all different, solved once in one launch.
        dict(name="batch_24_graphs", kind="batch", graphs=24, n_lo=512, n_hi=6000, p_lo=0.005, p_hi=0.5, hi=100,
             sources=1, compact=False, plan=False),
        # A plan kept by the program: many sources of one graph beside single ones of others.
        dict(name="plan_80_compact", kind="batch", graphs=16, n_lo=512, n_hi=4096, p_lo=0.005, p_hi=0.5, hi=100,
             sources=64, compact=True, plan=True),
        # Serving: a burst of queries over resident graphs (compact copies).
        dict(name="serve_64_queries", kind="serve", graphs=8, n_lo=256, n_hi=8192, p_lo=0.01, p_hi=0.5, hi=1000,
             queries=64, compact=True),
        # Adjacency lists far beyond what a matrix holds: m = 3n, n = 10^6.
        dict(name="csr_solve_n1000000", kind="csr", n=1000000, hi=1000, directed=False),
        # Edge list to matrix, the input step of a dense solve.
        dict(name="edges_to_dense_n16000", kind="todense", n=16000, hi=1000, directed=False),
        # A whole sparse query at the paper's largest size: edges, lists, solve, 100 routes.
        dict(name="route_n40000", kind="route", n=40000, hi=1000, directed=False, targets=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "batch", "serve", "csr", "todense", "route"])
    hi = rng.choice([10, 100, 1000])
    directed = rng.random() < 0.5
    if kind == "solve":
        n = _log_int(rng, 100, 40000)
        lc = n >= 2000 and rng.random() < 0.25
        lo_p = max(0.0005, 8.0 / n)  # mostly connected graphs
        p = math.exp(rng.uniform(math.log(lo_p), math.log(max(lo_p, 0.02 if lc else 0.5))))
        return dict(kind=kind, n=n, p=p, hi=hi, directed=directed, lc=lc)
    if kind == "batch":
        plan = rng.random() < 0.5
        return dict(kind=kind, graphs=rng.randint(2, 32), n_lo=_log_int(rng, 64, 1000), n_hi=_log_int(rng, 1500, 6000),
                    p_lo=0.005, p_hi=0.5, hi=hi, sources=rng.choice([1, 8, 32, 64]),
                    compact=plan and rng.random() < 0.6, plan=plan)
    if kind == "serve":
        return dict(kind=kind, graphs=rng.randint(2, 12), n_lo=256, n_hi=_log_int(rng, 1024, 12000), p_lo=0.01,
                    p_hi=0.5, hi=1000, queries=_log_int(rng, 4, 128), compact=rng.random() < 0.6)
    if kind == "csr":
        return dict(kind=kind, n=_log_int(rng, 1000, 1000000), hi=hi, directed=directed)
    if kind == "todense":
        return dict(kind=kind, n=_log_int(rng, 100, 20000), hi=hi, directed=directed)
    return dict(kind=kind, n=_log_int(rng, 1000, 200000), hi=hi, directed=directed, targets=_log_int(rng, 1, 1000))


# ---- inputs ----

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed & 0x7FFFFFFFFFFF)
    return g


def _matrix(n, p, hi, directed, g):
    """A contiguous int32 [n, n] G(n, p) matrix, made in row blocks."""
    W = torch.empty((n, n), dtype=torch.int32, device=DEV)
    step = max(1, (1 << 27) // n)
    for r in range(0, n, step):
        rows = W[r:r + step]
        rows.random_(1, hi + 1, generator=g)
        rows.masked_fill_(torch.rand(rows.shape, generator=g, device=DEV) >= p, INF)
    if not directed:
        t = 8192
        for i in range(0, n, t):
            d = W[i:i + t, i:i + t]
            up = torch.triu(d, 1)
            d.copy_(up + up.t())
            for j in range(i + t, n, t):
                W[j:j + t, i:i + t].copy_(W[i:i + t, j:j + t].t())
    W.fill_diagonal_(0)
    return W


def _edges(n, hi, g):
    m = 3 * n
    eu = torch.randint(0, n, (m,), generator=g, device=DEV, dtype=torch.int32)
    ev = torch.randint(0, n, (m,), generator=g, device=DEV, dtype=torch.int32)
    ew = torch.randint(1, hi + 1, (m,), generator=g, device=DEV, dtype=torch.int32)
    return eu, ev, ew


def _host_rng(seed):
    return random.Random(seed)


def _shapes(case):
    """(n, p) of each matrix of a batch or server, the first of the largest size: they
    belong to the case, the entries to the seed."""
    r = random.Random(case["graphs"] * 1000003 + case["n_lo"] * 1009 + case["n_hi"])
    out = [(case["n_hi"], 0.05)]
    while len(out) < case["graphs"]:
        out.append((_log_int(r, case["n_lo"], case["n_hi"]), r.uniform(case["p_lo"], case["p_hi"])))
    return out


def _solves(case):
    """Matrix index of each solve of a batch or server."""
    if case["kind"] == "serve":
        r = random.Random(case["queries"])
        return [r.randrange(case["graphs"]) for _ in range(case["queries"])]
    return [0] * case["sources"] + list(range(1, case["graphs"]))


def _instances(case, seed):
    """(matrices, [(matrix index, source)])."""
    g, r = _gen(seed), _host_rng(seed)
    mats = [_matrix(n, p, case["hi"], False, g) for n, p in _shapes(case)]
    return mats, [(i, r.randrange(mats[i].shape[0])) for i in _solves(case)]


def _outputs(mats, inst):
    """One dist and one pred buffer for all solves, and each solve's part of them."""
    sizes = [mats[i].shape[0] for i, _ in inst]
    dist, pred = _empty(sum(sizes)), _empty(sum(sizes))
    return dist, pred, list(zip(dist.split(sizes), pred.split(sizes)))


def _empty(n):
    return torch.empty(n, dtype=torch.int32, device=DEV)


# room for the vertices of one route; shortest paths of these graphs have a few dozen
ROUTE = 256


def _targets(case, seed):
    r = _host_rng(seed + 1)
    return [r.randrange(case["n"]) for _ in range(case["targets"])]


def prepare(case, seed):
    k = case["kind"]
    if k == "solve":
        W = _matrix(case["n"], case["p"], case["hi"], case["directed"], _gen(seed))
        return dict(case=case, W=W, src=_host_rng(seed).randrange(case["n"]))
    if k == "batch":
        mats, inst = _instances(case, seed)
        dist, pred, parts = _outputs(mats, inst)
        items = [(mats[i], s, d, p) for (i, s), (d, p) in zip(inst, parts)]
        state = dict(case=case, items=items, outs=(dist, pred))
        if case["plan"]:
            plan = sp.BatchPlan(items, sp.SSSP_FLAG_COMPACT if case["compact"] else 0)
            state["plan"] = plan
            weakref.finalize(plan, sp.sssp_batch_plan_destroy, plan.h)
        return state
    if k == "serve":
        mats, inst = _instances(case, seed)
        dist, pred, parts = _outputs(mats, inst)
        torch.cuda.synchronize()  # the server reads the matrices from its own stream
        # leaves the GPU soon after a burst, so that the program's own device waits end
        srv = sp.Server(idle_park_ms=1)
        weakref.finalize(srv, sp.sssp_server_destroy, srv.h)
        gids = [srv.add_graph(W, sp.SSSP_FLAG_COMPACT if case["compact"] else 0) for W in mats]
        queries = [(gids[i], s, d, p) for (i, s), (d, p) in zip(inst, parts)]
        return dict(case=case, srv=srv, queries=queries, outs=(dist, pred))
    eu, ev, ew = _edges(case["n"], case["hi"], _gen(seed))
    state = dict(case=case, eu=eu, ev=ev, ew=ew, src=_host_rng(seed).randrange(case["n"]))
    if k == "csr":
        state["csr"] = sp.csr_from_edges(eu, ev, ew, case["n"], case["directed"])[:3]
    elif k == "todense":
        state["W"] = torch.empty((case["n"], case["n"]), dtype=torch.int32, device=DEV)
    elif k == "route":
        t = _targets(case, seed)
        state["targets"] = torch.tensor(t, dtype=torch.int32, device=DEV)
        state["offsets"] = torch.arange(len(t), dtype=torch.int64, device=DEV) * ROUTE
        state["hops"] = _empty(case["n"])
        # a longer route would run on into what follows, at most n vertices
        state["routes"] = _empty(len(t) * ROUTE + case["n"])
    return state


def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "solve":
        return sp.solve(state["W"], state["src"], sp.SSSP_FLAG_LABEL_CORRECTING if case["lc"] else 0)
    if k == "batch":
        if case["plan"]:
            state["plan"].launch()
        else:
            sp.sssp_dense_solve_batched(state["items"])
        return state["outs"]
    if k == "serve":
        srv = state["srv"]
        tickets = [srv.submit(g, s, d, p) for g, s, d, p in state["queries"]]
        for t in tickets:
            srv.wait(t, timeout_s=60)
        srv.poll()
        return state["outs"]
    if k == "csr":
        return sp.csr_solve(*state["csr"], state["src"])
    if k == "todense":
        sp.sssp_edges_to_dense(state["eu"], state["ev"], state["ew"], case["n"], state["W"],
                               directed=case["directed"])
        return state["W"]
    rp, col, w, _ = sp.csr_from_edges(state["eu"], state["ev"], state["ew"], case["n"], case["directed"])
    dist, pred = sp.csr_solve(rp, col, w, state["src"])
    routes = state["routes"].fill_(-1)
    sp.sssp_hops(pred, dist, state["hops"])
    sp.sssp_paths(pred, state["hops"], state["targets"], state["offsets"], routes)
    return dist, pred, state["hops"], routes


# ---- what a pass cannot do without ----

def work(case):
    k = case["kind"]
    if k == "solve":
        n = case["n"]
        return dict(bytes=4 * n * n + 8 * n, flops=2 * n * n)
    if k in ("batch", "serve"):
        shapes = _shapes(case)
        elem = 4 if not case["compact"] else 1 if case["hi"] <= 254 else 2
        solves = [shapes[i][0] for i in _solves(case)]
        return dict(bytes=elem * sum(n * n for n, _ in shapes) + 8 * sum(solves), flops=2 * sum(n * n for n in solves))
    n, m = case["n"], 3 * case["n"]
    entries = m if case["directed"] else 2 * m
    csr = 8 * (n + 1) + 8 * entries
    if k == "csr":
        return dict(bytes=csr + 8 * n, flops=2 * entries)
    if k == "todense":
        return dict(bytes=12 * m + 4 * n * n, flops=entries)
    return dict(bytes=12 * m + csr + 12 * n, flops=3 * entries)


# ---- the same answers from plain torch, in 64 bits ----

def _exact_dense(W, src):
    """Shortest distances by levels: all vertices of the smallest unsettled distance at
    once (weights are at least 1); pred is the lowest (dist, index) among the tails
    that give a vertex its distance."""
    n = W.shape[0]
    big = 1 << 62
    dist = torch.full((n,), INF, dtype=torch.int64, device=DEV)
    pred = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    done = torch.zeros(n, dtype=torch.bool, device=DEV)
    dist[src] = 0
    step = max(1, (1 << 25) // n)
    while True:
        open_dist = torch.where(done, torch.full_like(dist, INF), dist)
        d = int(open_dist.min())
        if d >= INF:
            break
        level = torch.nonzero(open_dist == d).flatten()
        done[level] = True
        if bool(done.all()):
            break
        best = torch.full((n,), big, dtype=torch.int64, device=DEV)
        for c in range(0, level.numel(), step):
            u = level[c:c + step]
            w = W[u].to(torch.int64)
            k = (w << 20) | u[:, None]
            k.masked_fill_(w >= INF, big)
            best = torch.minimum(best, k.min(0).values)
        cand = d + (best >> 20)
        take = ~done & (best < big) & (cand < dist)
        dist = torch.where(take, cand, dist)
        pred = torch.where(take, best & ((1 << 20) - 1), pred)
    return dist, pred


def _all_edges(eu, ev, ew, directed):
    eu, ev, ew = eu.to(torch.int64), ev.to(torch.int64), ew.to(torch.int64)
    if not directed:
        eu, ev, ew = torch.cat([eu, ev]), torch.cat([ev, eu]), torch.cat([ew, ew])
    keep = eu != ev
    return eu[keep], ev[keep], ew[keep]


def _exact_edges(n, u, v, w, src):
    dist = torch.full((n,), 1 << 40, dtype=torch.int64, device=DEV)
    dist[src] = 0
    while True:
        new = dist.scatter_reduce(0, v, dist[u] + w, "amin")
        if torch.equal(new, dist):
            break
        dist = new
    tight = (dist[u] + w == dist[v]) & (dist[v] < (1 << 40))
    key = torch.full((n,), 1 << 62, dtype=torch.int64, device=DEV)
    key = key.scatter_reduce(0, v[tight], (dist[u[tight]] << 21) | u[tight], "amin")
    pred = torch.where(key < (1 << 62), key & ((1 << 21) - 1), torch.full_like(key, -1))
    pred[src] = -1
    return torch.where(dist >= (1 << 40), torch.full_like(dist, INF), dist), pred


def exact(case, seed):
    k = case["kind"]
    if k == "solve":
        W = _matrix(case["n"], case["p"], case["hi"], case["directed"], _gen(seed))
        return _exact_dense(W, _host_rng(seed).randrange(case["n"]))
    if k in ("batch", "serve"):
        mats, inst = _instances(case, seed)
        got = [_exact_dense(mats[i], s) for i, s in inst]
        return torch.cat([d for d, _ in got]), torch.cat([p for _, p in got])
    n = case["n"]
    eu, ev, ew = _edges(n, case["hi"], _gen(seed))
    u, v, w = _all_edges(eu, ev, ew, case["directed"])
    if k == "todense":
        W = torch.full((n * n,), INF, dtype=torch.int64, device=DEV)
        W.scatter_reduce_(0, u * n + v, w, "amin")
        W = W.view(n, n)
        W.fill_diagonal_(0)
        return W
    src = _host_rng(seed).randrange(n)
    dist, pred = _exact_edges(n, u, v, w, src)
    if k == "csr":
        return dist, pred
    par, reach = pred.tolist(), (dist < INF).tolist()
    hops = [-1] * n
    for v in torch.argsort(dist, stable=True).tolist():  # a tail comes before its heads
        if reach[v]:
            hops[v] = 0 if v == src else hops[par[v]] + 1
    routes = [-1] * (case["targets"] * ROUTE + n)
    for i, t in enumerate(_targets(case, seed)):
        while t >= 0 and reach[t]:
            routes[i * ROUTE + hops[t]] = t
            t = par[t]
    return dist, pred, torch.tensor(hops, device=DEV), torch.tensor(routes, device=DEV)
