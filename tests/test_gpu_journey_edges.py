"""GPU parity of journeys and profiles at the edges of their kernels (stops per
wave, lanes per stop, departure chunks, rows in flight), bit-exact against the
CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
LAYOUTS = {"grid": {"cluster_seconds": 7200}, "compact": {"cluster_seconds": 7200, "header_grid": -1},
           "flat": {"layout": eat.EAT_LAYOUT_FLAT}}
DAY = 86400


def _scan(u, v, t, lam, n):
    """The oracle without self-loops, which a graph does not keep (they can be
    in no journey, but their departures would be listed)."""
    k = u != v
    return oracle.Csa(u[k], v[k], t[k], lam[k], n)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    eat.lib()


def _timetable(n, m, days, seed, hub=0):
    """m random connections over n stops and some days; stop 0 also has `hub`
    connection types of its own."""
    rng = np.random.default_rng([seed, n, m])
    u, v = rng.integers(0, n, m), rng.integers(0, n, m)
    t, lam = rng.integers(0, days * DAY, m), 1 + rng.integers(0, 4000, m)
    if hub:
        u, v = np.r_[u, np.zeros(hub, np.int64)], np.r_[v, rng.integers(0, n, hub)]
        t, lam = np.r_[t, rng.integers(0, days * DAY, hub)], np.r_[lam, 1 + np.arange(hub)]
    return [x.astype(np.int32) for x in (u, v, t, lam)]


# stops: below, at and just over what one wave and one work-group take; types of
# one stop: below, at and over its 16 lanes, and over a work-group's 256 threads
@pytest.mark.parametrize("n,m,hub", [(1, 0, 0), (2, 9, 0), (15, 200, 15), (16, 300, 16), (17, 300, 17), (63, 900, 40),
                                     (64, 900, 300), (65, 2000, 0), (1001, 20000, 700)])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_parents_at_their_edges(n, m, hub, layout):
    u, v, t, lam = _timetable(n, m, 1, 3, hub)
    g, csa = eat.eat_graph_build(u, v, t, lam, n, **LAYOUTS[layout]), oracle.Csa(u, v, t, lam, n)
    for s, ts in ((0, 0), (n - 1, 20000), (n // 2, 80000)):
        print(n, m, hub, layout, s, ts, flush=True)
        arr = g.query(s, ts)
        exp = np.stack(oracle.parents(u, v, t, lam, n, s, csa.query(s, ts)), 1)
        room = torch.full((3 * n + 8,), 7, dtype=torch.int32, device="cuda")
        for off in (0, 1, 2, 3):  # any 4-byte alignment of the answer
            room.fill_(7)
            par = room[off:off + 3 * n].view(n, 3)
            g.parents(s, arr, out=par)
            assert np.array_equal(par.cpu().numpy(), exp), off
            rest = torch.cat([room[:off], room[off + 3 * n:]])
            assert int((rest != 7).sum()) == 0  # nothing beside it


# intervals: one second, within a chunk of departures, over several chunks, over
# a gap of days without departures, up to the end of time
@pytest.mark.parametrize("lo,hi", [(0, 0), (5000, 5000), (0, 131071), (0, 131072), (1, 3 * DAY), (100000, 400000),
                                   (0, 2**31 - 1), (5 * DAY, 2**31 - 1)])
@pytest.mark.parametrize("layout", list(LAYOUTS))
def test_profiles_at_their_edges(lo, hi, layout):
    n = 40
    u, v, t, lam = _timetable(n, 1500, 2, 9)
    late = _timetable(n, 60, 1, 10)  # the same stops again on the fifth day
    u, v, t, lam = (np.r_[a, b] for a, b in zip((u, v, t, lam), (late[0], late[1], late[2] + 4 * DAY, late[3])))
    g, csa = eat.eat_graph_build(u, v, t, lam, n, **LAYOUTS[layout]), _scan(u, v, t, lam, n)
    for s in (0, 7, n - 1):
        print(lo, hi, layout, s, flush=True)
        dep, arr = g.profile(s, lo, hi)
        e_dep, e_arr = csa.profile(s, lo, hi)
        assert np.array_equal(dep, e_dep)
        assert np.array_equal(arr.cpu().numpy(), e_arr)


@pytest.mark.parametrize("k", [1, 7, 8, 9, 16, 17, 1023, 1024, 1025])
def test_profile_of_exactly_k_departures(k):
    """As many departures as the filter's rows in flight, and as the kept scratch
    takes, one fewer and one more; with and without a departure after them."""
    n, rng = 50, np.random.default_rng(k)
    t0 = 1000 + 3 * np.arange(k)
    u = np.r_[np.zeros(k, np.int64), rng.integers(1, n, 3000)].astype(np.int32)
    v = np.r_[rng.integers(1, n, k), rng.integers(1, n, 3000)].astype(np.int32)
    t = np.r_[t0, rng.integers(0, 9000, 3000)].astype(np.int32)
    lam = np.r_[1 + rng.integers(0, 50, k), 1 + rng.integers(0, 500, 3000)].astype(np.int32)
    for extra in (0, 1):
        uu, vv, tt, ll = (np.r_[a, b].astype(np.int32) for a, b in zip((u, v, t, lam), ([0], [1], [9500], [10])))
        if not extra:
            uu, vv, tt, ll = u, v, t, lam
        g, csa = eat.eat_graph_build(uu, vv, tt, ll, n), _scan(uu, vv, tt, ll, n)
        dep, arr = g.profile(0, 1000, 1000 + 3 * (k - 1))
        e_dep, e_arr = csa.profile(0, 1000, 1000 + 3 * (k - 1))
        assert len(dep) == k and np.array_equal(dep, e_dep)
        assert np.array_equal(arr.cpu().numpy(), e_arr)
