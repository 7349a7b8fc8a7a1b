"""Table rounds of more connection types than the windows hold and sweeps of more
stops than the list takes, bit-exact against the CPU oracle."""
import functools

import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
LAYOUTS = {"grid": {}, "compact": {"header_grid": -1}, "flat": {"layout": eat.EAT_LAYOUT_FLAT}}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    eat.lib()


@functools.lru_cache(maxsize=None)
def _case(types, layout):
    """Stop 0 leaves for the stops 1 .. len(types) at once; stop i has types[i - 1]
    connection types to the stops after those.  Every third of these leads nowhere
    (improved, but with no types to list); the others lead on and back."""
    rng = np.random.default_rng([len(types), sum(types)])
    k, n_out = len(types), max(types) + 11
    u, v, t, lam = [np.zeros(k, np.int64)], [1 + np.arange(k)], [np.full(k, 3600)], [1 + rng.integers(0, 9, k)]
    for i, m in enumerate(types):
        u.append(np.full(m, 1 + i))
        v.append(1 + k + (np.arange(m) + 5 * i) % n_out)
        t.append(3700 + rng.integers(0, 7000, m))
        lam.append(1 + rng.integers(0, 3000, m))
    on = np.arange(n_out)[np.arange(n_out) % 3 > 0]
    for to in (1 + k + rng.integers(0, n_out, len(on)), 1 + rng.integers(0, k, len(on))):
        u.append(1 + k + on)
        v.append(to)
        t.append(rng.integers(5000, 40000, len(on)))
        lam.append(1 + rng.integers(0, 900, len(on)))
    cat = [np.concatenate(x).astype(np.int32) for x in (u, v, t, lam)]
    keep = cat[0] != cat[1]
    cat = [c[keep] for c in cat]
    n = 1 + k + n_out
    return eat.eat_graph_build(*cat, n, **LAYOUTS[layout]), oracle.Csa(*cat, n), n


# types of the second round: as many as 80 windows of 64 hold, one more, as many as
# two and three times that, one more; in one entry, in entries that end at a window's
# edge and one past it, in more entries than a list of 64 or of 704 takes
ROUNDS = [(5120,), (5121,), (5119, 1), (1, 5119, 1), (10240,), (10241,), (64,) * 80, (64,) * 81, (65,) * 79, (1,) * 63,
          (1,) * 64, (1,) * 65, (127, 1, 64, 65) * 40, (30, 5000, 30, 7000, 1), (9,) * 703, (9,) * 704, (9,) * 1500]


@pytest.mark.parametrize("types", ROUNDS, ids=lambda t: "%dx%d" % (len(t), max(t)))
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_large_rounds(types, layout):
    g, csa, n = _case(types, layout)
    topo = {"mode": eat.EAT_MODE_TOPOLOGY}
    opts = [{}, {"threads_per_query": 768}, {"threads_per_query": 256}, {"frontier_cap": 64}, {"time_window": -1}, topo,
            {"frontier_cap": 64, "threads_per_query": 512}, dict(topo, time_window=-1), dict(topo, time_window=60),
            dict(topo, threads_per_query=384), dict(topo, frontier_cap=64)]
    for s, ts in ((0, 0), (n - 1, 4000)):
        exp = csa.query(s, ts)
        for o in opts:
            print(len(types), max(types), layout, s, ts, o, flush=True)
            out, st = g.query(s, ts, options=o, stats=True)
            assert np.array_equal(out.cpu().numpy(), exp)
            assert st["status"] == 0 and st["reached"] == int((exp < oracle.INF).sum())
    d = int(np.argmax(np.where(exp < oracle.INF, exp, -1)))
    for o in ({}, {"threads_per_query": 768}, topo):
        assert g.query_goal(s, ts, d, options=o).cpu().numpy()[d] == exp[d], o
