"""GPU parity of the table rounds (one connection type per lane) at the edges of
their lists, windows and far list, bit-exact against the CPU oracle."""
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


def _fan(n_mid, types_per_mid, lam_spread, seed):
    """Stop 0 leaves for n_mid stops at once; each of them has types_per_mid
    connection types to a layer of 997 stops, and those lead on and back."""
    rng = np.random.default_rng(seed)
    n_out = 997
    mid = 1 + np.arange(n_mid)
    out = 1 + n_mid + np.arange(n_out)
    u, v, t, lam = [], [], [], []

    def add(uu, vv, tt, ll):
        u.append(uu), v.append(vv), t.append(tt), lam.append(ll)

    add(np.zeros(n_mid), mid, np.full(n_mid, 3600), 1 + rng.integers(0, lam_spread, n_mid))
    for k in range(3):  # a few departures of every type
        m = np.repeat(mid, types_per_mid)
        r = np.random.default_rng([seed, 1])  # the same types every time
        add(m, out[r.integers(0, n_out, len(m))], 3600 + 9000 * k + rng.integers(0, 9000, len(m)),
            1 + r.integers(0, 5000, len(m)))
    a = rng.integers(0, n_out, 4000)
    add(out[a], out[rng.integers(0, n_out, 4000)], rng.integers(0, 80000, 4000), 1 + rng.integers(0, 900, 4000))
    add(out[a[:500]], mid[rng.integers(0, n_mid, 500)], rng.integers(0, 80000, 500), 1 + rng.integers(0, 900, 500))
    cat = [np.concatenate(x).astype(np.int32) for x in (u, v, t, lam)]
    return cat + [1 + n_mid + n_out]


# (stops listed at once, their types, spread of their arrivals): a wave's worth
# and one more; stops of more than 64 types; exactly and just over the 80 windows
# of 64 types; more than the windows hold in fewer entries than the list; an
# overflowing list; arrivals past the window, fewer and many more than the far
# list holds
FANS = [(1, 1, 1), (64, 1, 1), (65, 3, 100), (3, 65, 10), (5, 200, 10), (64, 80, 1), (40, 129, 1), (100, 80, 1),
        (900, 4, 1), (300, 5, 60000), (700, 3, 80000), (1500, 2, 80000)]


@functools.lru_cache(maxsize=None)
def _case(fan, layout):
    u, v, t, lam, n = _fan(*fan, seed=11)
    return eat.eat_graph_build(u, v, t, lam, n, **LAYOUTS[layout]), oracle.Csa(u, v, t, lam, n), n


@pytest.mark.parametrize("fan", FANS, ids=str)
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_table_rounds_at_their_edges(fan, layout):
    g, csa, n = _case(fan, layout)
    opts = [{"threads_per_query": th} for th in (1024, 768, 512, 384, 256)]
    opts += [{"frontier_cap": 64}, {"threads_per_query": 384, "frontier_cap": 64}, {"time_window": -1},
             {"time_window": 300, "frontier_cap": 64}, {"table_cap": 64}, {"mode": eat.EAT_MODE_TOPOLOGY}]
    starts = [(0, 0), (0, 3600), (min(1, n - 1), 3000), (n - 1, 40000)]
    for s, ts in starts:
        exp = csa.query(s, ts)
        for o in opts:
            print(fan, layout, s, ts, o, flush=True)
            out, st = g.query(s, ts, options=o, stats=True)
            assert np.array_equal(out.cpu().numpy(), exp)
            assert st["reached"] == int((exp < oracle.INF).sum()) and st["status"] == 0
        for d in (int(np.argmax(np.where(exp < oracle.INF, exp, -1))), n - 1, 0):
            for th in (1024, 768):
                out, _ = g.query_goal(s, ts, d, options={"threads_per_query": th}, stats=True)
                assert out.cpu().numpy()[d] == exp[d], (s, ts, d)


def test_table_rounds_repeat_and_batch_agree():
    """One launch of many queries with overflowing lists: the lists, marks and
    counters of one query leave nothing behind for the next on its work-group."""
    g, csa, n = _case((700, 3, 80000), "grid")
    rng = np.random.default_rng(5)
    q = 600
    s = np.where(rng.random(q) < 0.3, 0, rng.integers(0, n, q)).astype(np.int32)
    ts = rng.integers(0, 80000, q).astype(np.int32)
    exp = csa.query_many(s, ts)
    for o in ({"threads_per_query": 768}, {"threads_per_query": 256}, {"frontier_cap": 64}, {"table_cap": 256}):
        out = torch.full((q, n), -1, dtype=torch.int32, device="cuda")
        eat.eat_query_batch([g], np.zeros(q, np.int32), s, ts, [out[i] for i in range(q)], options=o)
        assert np.array_equal(out.cpu().numpy(), exp), o


# entries of a list of 64 whose last is spare: one fewer than fit, as many, and
# more by one or two; and of its far list of 32 (arrivals 300 s to 60,000 s apart)
@pytest.mark.parametrize("fan", [(n, 3, s) for s, sizes in ((1, (62, 63, 64, 65)), (60000, (31, 32, 33, 34, 97)))
                                 for n in sizes], ids=str)
def test_table_rounds_with_lists_full_to_the_spare_entry(fan):
    g, csa, n = _case(fan, "grid")
    for s, ts in ((0, 0), (0, 3600), (n - 1, 40000)):
        exp = csa.query(s, ts)
        for o in ({"frontier_cap": 64}, {"frontier_cap": 64, "time_window": 300},
                  {"frontier_cap": 64, "threads_per_query": 768, "time_window": 20000}):
            print(fan, s, ts, o, flush=True)
            assert np.array_equal(g.query(s, ts, options=o).cpu().numpy(), exp), (s, ts, o)
