"""The work that users of this framework have it do, as cases that can be timed.

A case is a dict of plain values.  ``listed()`` gives the fixed ones, ``draw()``
more of the same ranges; ``prepare(case, seed)`` makes what a user's program
holds before the call (timetable on the GPU, queries, result slabs, the prepared
batch or session), ``run(state)`` makes one pass through the public entry
points, ``work(case)`` says what a pass cannot do without, ``exact(case, seed)``
gives the same answers by plain relaxation over the connection list in torch.

Values of a case:
  kind     query | journey | profile | batch | goal | oneshot | serve (see run())
  sizes    stops of each timetable, as text ("10000,50000")
  network  city | towns | lines
  layout   hybrid | flat
  queries  queries of a pass; they leave at uniform times of the day, those of
           the single calls (query, journey) between 06:00 and 18:00, so that
           one draw is not an empty evening
  k        profile: departures of the source between 06:00 and 08:00
"""
import math

import numpy as np
import torch

from paper_1912_00966_amd import eat, synth

DAY = 86400
LAYOUTS = {"hybrid": eat.EAT_LAYOUT_HYBRID, "flat": eat.EAT_LAYOUT_FLAT}
PROFILE_FROM, PROFILE_TO = 6 * 3600, 8 * 3600


def _case(kind, sizes, queries, network="city", layout="hybrid", k=0, name=None):
    c = {"kind": kind, "sizes": sizes, "network": network, "layout": layout, "queries": queries, "k": k}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one rider's question in a small town: the smallest call, launch and host cost count
        _case("query", "1000", 1, name="query-1k"),
        # the same in a city of 50,000 stops: one query alone on the GPU
        _case("query", "50000", 1, name="query-50k"),
        # a trip planner that also shows the way: the arrival times and the connection behind each
        _case("journey", "50000", 1, name="journey-50k"),
        # a timetable poster: every sensible departure of one stop in the morning peak
        _case("profile", "50000", 1, k=32, name="profile-50k"),
        # a small prepared batch on a small town
        _case("batch", "1000", 16, name="batch-1k-16"),
        # the city's batch: one query per compute unit
        _case("batch", "50000", 256, name="batch-50k-256"),
        # point-to-point questions of many riders, answered together
        _case("goal", "50000", 1000, name="goal-50k-1000"),
        # several cities of uneven size in one launch, far more queries than work-groups
        _case("batch", "2000,5000,10000,20000,50000,100000,200000", 3584, name="batch-mixed-3584"),
        # a region of towns joined by a few long lines: the largest timetable, long queries, few of them
        _case("batch", "500000", 64, network="towns", name="batch-region-64"),
        # a list of questions that comes once: created, run, waited for and freed in one call; ragged sizes
        _case("oneshot", "10007", 100, name="oneshot-10k-100"),
        # vehicles on lines, with sub-trip shortcuts: long chains of short hops
        _case("batch", "5000", 256, network="lines", name="batch-lines-256"),
        # a server's burst over its resident cities: admitted, launched, copied out and released
        _case("serve", "10000,50000", 96, name="serve-96"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "journey", "profile", "batch", "batch", "batch", "goal", "oneshot", "serve"])
    network = "city"
    if kind == "profile":  # every size here has sources with that many departures
        return _case(kind, str(_log_int(rng, 20_000, 100_000)), 1, k=rng.randint(24, 48))
    if kind in ("query", "journey"):
        return _case(kind, str(_log_int(rng, 700, 200_000)), 1, layout=rng.choice(["hybrid", "hybrid", "hybrid", "flat"]))
    if kind == "serve":
        return _case(kind, "%d,%d" % (_log_int(rng, 1_000, 20_000), _log_int(rng, 10_000, 100_000)), _log_int(rng, 4, 300))
    if kind == "batch":
        network = rng.choice(["city", "city", "city", "towns", "lines"])
    if network == "lines":
        return _case(kind, str(_log_int(rng, 1_000, 6_000)), _log_int(rng, 16, 600), network)
    if network == "towns":
        return _case(kind, str(_log_int(rng, 20_000, 400_000)), _log_int(rng, 8, 200), network)
    if kind == "batch" and rng.random() < 0.4:
        n = rng.randint(2, 5)
        return _case(kind, ",".join(str(_log_int(rng, 1_000, 100_000)) for _ in range(n)), n * _log_int(rng, 64, 512))
    return _case(kind, str(_log_int(rng, 700, 200_000)), _log_int(rng, 4, 2000),
                 layout=rng.choice(["hybrid", "hybrid", "hybrid", "flat"]))


# ---------------------------------------------------------------------------
# Timetables, drawn on the GPU at the densities of the package's generator:
# stops on a jittered grid (towns: one patch each), linked both ways to their
# nearest neighbours; a few connection types per edge; departures of a type in
# a progression from the early morning on, and a share of irregular ones.
# ---------------------------------------------------------------------------
def _ints(g, lo, hi, n):
    """n integers uniform in [lo, hi]; lo and hi are numbers or tensors."""
    r = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    return (lo + r * (hi - lo + 1)).long()


def _near_edges(g, n, k):
    """Directed edges of a patch of n stops: each with its k nearest, both ways."""
    side = max(1, math.isqrt(n - 1) + 1)
    i = torch.arange(n, device="cuda")
    x, y = i % side, i // side
    p = torch.stack([x, y], 1) + torch.rand(n, 2, generator=g, device="cuda")
    at, far = [], []
    for dy in range(-2, 3):
        for dx in range(-2, 3):
            if dx == 0 and dy == 0:
                continue
            j = i + dy * side + dx
            ok = (x + dx >= 0) & (x + dx < side) & (j >= 0) & (j < n)
            j = j.clamp(0, n - 1)
            at.append(j)
            far.append(torch.where(ok, ((p - p[j]) ** 2).sum(1), torch.inf))
    far, at = torch.stack(far, 1), torch.stack(at, 1)
    d, w = far.topk(k, dim=1, largest=False)
    src, dst, ok = i.repeat_interleave(k), at.gather(1, w).reshape(-1), torch.isfinite(d).reshape(-1)
    src, dst = src[ok], dst[ok]
    key = torch.unique(torch.cat([src * n + dst, dst * n + src]))
    return key // n, key % n


def _network(n, network, g):
    """(u, v, shortest and longest duration) of every edge, and the recipe."""
    small = n < 10_000
    k, recipe = (3, (1, 3, 0.10, 200)) if small else (5, (1, 4, 0.15 if network == "city" else 0.25, 240))
    lam = (60, 1800) if small else (30, 3600)
    towns = 20 if network == "towns" else 1
    us, vs, first = [], [], 0
    for t in range(towns):
        size = n // towns + (1 if t < n % towns else 0)
        u, v = _near_edges(g, size, k)
        us.append(u + first)
        vs.append(v + first)
        first += size
    u, v = torch.cat(us), torch.cat(vs)
    lo, hi = torch.full_like(u, lam[0]), torch.full_like(u, lam[1])
    if towns > 1:  # a few long lines from each town to three others
        a = torch.arange(towns, device="cuda").repeat_interleave(3 * 8)
        b = (a + torch.arange(3, device="cuda").repeat_interleave(8).repeat(towns) + 1) % towns
        size = n // towns
        su, sv = a * size + _ints(g, 0, size - 1, len(a)), b * size + _ints(g, 0, size - 1, len(a))
        u, v = torch.cat([u, su, sv]), torch.cat([v, sv, su])
        lo = torch.cat([lo, torch.full((2 * len(a),), 1800, device="cuda")])
        hi = torch.cat([hi, torch.full((2 * len(a),), 7200, device="cuda")])
    names = torch.randperm(n, generator=g, device="cuda")  # a stop's number says nothing about its place
    return names[u], names[v], lo, hi, small, recipe


def _timetable(n, network, seed):
    """Connections (u, v, t, lam, trip or None) as int32 host arrays."""
    if network == "lines":
        tt = synth.lines_city(n, seed)
        return tt.u, tt.v, tt.t, tt.lam, tt.trip
    g = torch.Generator(device="cuda").manual_seed(seed)
    u, v, lo, hi, small, (few, many, irregular, per_stop) = _network(n, network, g)
    e = torch.arange(len(u), device="cuda").repeat_interleave(_ints(g, few, many, len(u)))
    types = len(e)
    lam = _ints(g, lo[e], hi[e], types)
    start = _ints(g, synth.AP_START_LO, synth.AP_START_HI, types)
    if small:
        h = torch.tensor(synth.SMALL_HEADWAYS, device="cuda")[_ints(g, 0, len(synth.SMALL_HEADWAYS) - 1, types)]
    else:
        h = _ints(g, 120, 3600, types)
    mean = per_stop * n / (types * (1 + irregular))
    terms = torch.minimum(_ints(g, 1, max(1, round(2 * mean - 1)), types), (synth.AP_END_CAP - start) // h + 1)
    of = torch.arange(types, device="cuda").repeat_interleave(terms)
    term = torch.arange(len(of), device="cuda") - (terms.cumsum(0) - terms)[of]
    t = start[of] + term * h[of]
    odd = of[torch.rand(len(of), generator=g, device="cuda") < irregular]
    of, t = torch.cat([of, odd]), torch.cat([t, _ints(g, 0, DAY - 1, len(odd))])
    host = [a.to(torch.int32).cpu().numpy() for a in (u[e[of]], v[e[of]], t, lam[of])]
    return host[0], host[1], host[2], host[3], None


def _sizes(case):
    return [int(x) for x in case["sizes"].split(",")]


def _timetables(case, seed):
    return [_timetable(n, case["network"], seed * 16 + i) for i, n in enumerate(_sizes(case))]


def _questions(case, seed, tts):
    """Graph, source and departure time of every query, and a destination each."""
    rng = np.random.default_rng([seed, 7])
    sizes, n = np.array(_sizes(case)), case["queries"]
    graph = (np.arange(n) % len(sizes)).astype(np.int32)
    src = rng.integers(0, sizes[graph]).astype(np.int32)
    dst = rng.integers(0, sizes[graph]).astype(np.int32)
    ts = rng.integers(0, DAY, n).astype(np.int32)
    if case["kind"] in ("query", "journey"):
        ts = rng.integers(6 * 3600, 18 * 3600, n).astype(np.int32)
    if case["kind"] == "profile":  # a source with k departures in the interval
        u, _, t, _, _ = (torch.from_numpy(a).cuda() if a is not None else None for a in tts[0])
        inside = (t >= PROFILE_FROM) & (t <= PROFILE_TO)
        key = torch.unique(u[inside].long() * DAY + t[inside])
        count = torch.bincount(key // DAY, minlength=int(sizes[0]))
        fit = torch.nonzero(count == case["k"]).reshape(-1)
        src[0] = int(fit[int(rng.integers(0, len(fit)))])
    return graph, src, ts, dst


def prepare(case, seed):
    tts = _timetables(case, seed)
    graphs = []
    for n, (u, v, t, lam, trip) in zip(_sizes(case), tts):
        if trip is None:
            graphs.append(eat.eat_graph_build(u, v, t, lam, n, layout=LAYOUTS[case["layout"]]))
        else:
            graphs.append(eat.eat_graph_build_trips(u, v, t, lam, trip, n))
    graph, src, ts, dst = _questions(case, seed, tts)
    s = {"kind": case["kind"], "graphs": graphs, "graph": graph, "src": src, "ts": ts}
    if case["kind"] == "profile":
        return s
    # one result slab per query; the queries of one timetable share a tensor
    s["slabs"] = [torch.empty((int((graph == i).sum()), g.n_vertices), dtype=torch.int32, device="cuda") for i, g in enumerate(graphs)]
    place, s["outs"] = [0] * len(graphs), []
    for i in graph:
        s["outs"].append(s["slabs"][i][place[i]])
        place[i] += 1
    if case["kind"] == "batch":
        s["batch"] = eat.Batch(graphs, graph, src, ts, s["outs"])
    elif case["kind"] == "goal":
        s["batch"] = eat.Batch(graphs, graph, src, ts, s["outs"], q_dst=dst)
        s["cell"] = torch.from_numpy(np.arange(len(dst)) * graphs[0].n_vertices + dst).cuda()
    elif case["kind"] == "journey":
        s["par"] = torch.empty((graphs[0].n_vertices, 3), dtype=torch.int32, device="cuda")
    elif case["kind"] == "serve":
        s["session"] = eat.Session(graphs, n_streams=4)
        s["arrival"] = np.zeros(len(src))
    return s


def run(state):
    kind, g = state["kind"], state["graphs"][0]
    if kind == "query":  # one earliest-arrival query, every stop
        return g.query(int(state["src"][0]), int(state["ts"][0]), out=state["outs"][0])
    if kind == "journey":  # the same, and the connection behind every arrival
        arr = g.query(int(state["src"][0]), int(state["ts"][0]), out=state["outs"][0])
        return {"arr": arr, "par": g.parents(int(state["src"][0]), arr, out=state["par"])}
    if kind == "profile":  # every Pareto departure of the source in the morning peak, every stop
        dep, arr = g.profile(int(state["src"][0]), PROFILE_FROM, PROFILE_TO)
        return {"dep": dep, "arr": arr}
    if kind == "batch":  # a prepared batch
        state["batch"].run()
        return state["slabs"]
    if kind == "goal":  # a prepared batch with a destination each: the arrival there is the answer
        state["batch"].run()
        return state["slabs"][0].view(-1)[state["cell"]]
    if kind == "oneshot":  # a batch made, run, waited for and freed in one call
        eat.eat_query_batch(state["graphs"], state["graph"], state["src"], state["ts"], state["outs"])
        return state["slabs"]
    state["session"].serve(state["graph"], state["src"], state["ts"], state["arrival"], copy_dst=state["outs"])
    return state["slabs"]


def work(case):
    """The result slabs written once, and per query the records of the
    connection types it has to look at read once: those leaving the stops that
    it reaches (some 600 on average over the day), 32 bytes and about 20 integer
    operations each."""
    sizes, n = _sizes(case), case["queries"]
    slab = reach = 0.0
    for v in sizes:
        q = n / len(sizes)
        if case["kind"] == "profile":
            q = case["k"] + 1
        per_stop = 7 if v < 10_000 else 15
        slab += q * 4 * v if case["kind"] != "goal" else q * 4
        reach += q * min(v, 600) * per_stop
        if case["kind"] == "journey":
            slab += 12 * v
    return {"bytes": slab + 32 * reach, "flops": 20 * reach}


# ---------------------------------------------------------------------------
# The same answers by plain relaxation: every connection tried until no arrival
# improves, 64-bit integers.
# ---------------------------------------------------------------------------
def _arrivals(conn, n, s, ts):
    u, v, t, lam = conn
    arr = torch.full((n,), int(eat.EAT_INF), dtype=torch.int64, device="cuda")
    arr[s] = ts
    while True:
        ok = arr[u] <= t
        new = arr.scatter_reduce(0, v[ok], (t + lam)[ok], "amin")
        if torch.equal(new, arr):
            return arr
        arr = new


def exact(case, seed):
    sizes = _sizes(case)
    if sum(240 * v * case["queries"] / len(sizes) for v in sizes) > 1.5e10:
        return None  # takes over about 20 seconds
    tts = _timetables(case, seed)
    graph, src, ts, dst = _questions(case, seed, tts)
    conns = [tuple(torch.from_numpy(a).cuda().long() for a in tt[:4]) for tt in tts]
    inf = int(eat.EAT_INF)
    if case["kind"] == "profile":
        u, v, t, lam = conns[0]
        s = int(src[0])
        dep = torch.unique(t[(u == s) & (t >= PROFILE_FROM)])
        k = int((dep <= PROFILE_TO).sum())
        rows = torch.stack([_arrivals(conns[0], sizes[0], s, int(d)) for d in dep[:k + 1]])
        if len(rows) == k:
            rows = torch.cat([rows, torch.full_like(rows[:1], inf)])
        arr = torch.where(rows[:k] < rows[1:], rows[:k], inf)
        arr[:, s] = inf
        return {"dep": dep[:k].cpu().numpy(), "arr": arr}
    rows = [_arrivals(conns[i], sizes[i], int(s), int(x)) for i, s, x in zip(graph, src, ts)]
    if case["kind"] == "query":
        return rows[0]
    if case["kind"] == "goal":
        return torch.stack([r[d] for r, d in zip(rows, dst)])
    if case["kind"] == "journey":
        u, v, t, lam = conns[0]
        arr, s = rows[0], int(src[0])
        real = (arr[u] <= t) & (t + lam == arr[v]) & (v != s)
        none = torch.iinfo(torch.int64).max
        key = torch.full_like(arr, none).scatter_reduce(0, v[real], (u[real] << 32) | lam[real], "amin")
        lam_p = key & 0xFFFFFFFF
        par = torch.stack([key >> 32, arr - lam_p, lam_p], 1)
        return {"arr": arr, "par": torch.where((key == none)[:, None], -1, par)}
    return [torch.stack([r for r, i in zip(rows, graph) if i == k]) for k in range(len(sizes))]
