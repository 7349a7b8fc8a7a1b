"""One-shot batches and profiles that a graph's scratch does not take in part or at
all, bit-exact against the CPU oracle: more departures than it holds, and graphs
whose activity bitmap is in HBM."""
import ctypes
import functools

import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    eat.lib()


@functools.lru_cache(maxsize=None)
def _dense():
    """A departure of stop 0 every minute, 1,200 of them, to stops that lead on."""
    n, k = 64, 1200
    i = np.arange(k)
    rng = np.random.default_rng(3)
    u = np.concatenate([np.zeros(k, int), rng.integers(1, n, 900)])
    v = np.concatenate([1 + i % (n - 1), rng.integers(1, n, 900)])
    t = np.concatenate([60 * i, rng.integers(0, 80000, 900)])
    lam = 1 + rng.integers(0, 4000, k + 900)
    keep = u != v
    args = [x[keep].astype(np.int32) for x in (u, v, t, lam)] + [n]
    return eat.eat_graph_build(*args), oracle.Csa(*args)


# departures: with the query after the interval 1,023 to 1,026 queries, and all 1,200
# (no query after them); cap as many, or more than the scratch takes
@pytest.mark.parametrize("k", [1, 1022, 1023, 1024, 1025, 1200])
@pytest.mark.parametrize("spare", [0, 2000])
def test_profiles_around_the_scratch(k, spare):
    g, csa = _dense()
    hi = 60 * (k - 1) + 30
    e_dep, e_arr = csa.profile(0, 0, hi)
    dep = np.full(k + spare, -1, np.int32)
    n = np.zeros(1, np.int32)
    arr = torch.full((k + spare, g.n_vertices), -3, dtype=torch.int32, device="cuda")
    for _ in range(2):
        st = eat.lib().eat_profile(g.handle, 0, 0, hi, k + spare, eat._ptr32(dep), eat._ptr32(n), arr.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream, None)
        assert st == 0 and n[0] == k
        assert np.array_equal(dep[:k], e_dep) and np.all(dep[k:] == -1)
        assert np.array_equal(arr[:k].cpu().numpy(), e_arr) and bool((arr[k:] == -3).all())
    if k > 1:  # one departure too many for the arrays
        st = eat.lib().eat_profile(g.handle, 0, 0, hi, k - 1, eat._ptr32(dep), eat._ptr32(n), arr.data_ptr(), None, None)
        assert st == eat.EAT_ERR_UNSUPPORTED and n[0] == k


def test_graphs_whose_bitmap_is_in_hbm():
    n = 1_300_000
    rng = np.random.default_rng(1)
    u = np.repeat(np.arange(n, dtype=np.int32), 2)
    v = ((u + rng.integers(1, 40, 2 * n)) % n).astype(np.int32)
    t, lam = rng.integers(0, 86400, 2 * n).astype(np.int32), rng.integers(1, 900, 2 * n).astype(np.int32)
    g, csa = eat.eat_graph_build(u, v, t, lam, n), oracle.Csa(u, v, t, lam, n)
    src, ts = np.array([0, 7, n - 1, 650_000], np.int32), np.array([0, 40_000, 86_000, 20_000], np.int32)
    out = torch.empty((4, n), dtype=torch.int32, device="cuda")
    for o in (None, {"table_cap": -1}, {"table_cap": 64}):
        eat.eat_query_batch([g], np.zeros(4, np.int32), src, ts, [out[i] for i in range(4)], options=o)
        for i in range(4):
            assert np.array_equal(out[i].cpu().numpy(), csa.query(int(src[i]), int(ts[i]))), (o, i)
    dep, arr = g.profile(5, 0, 86_400)
    e_dep, e_arr = csa.profile(5, 0, 86_400)
    assert np.array_equal(dep, e_dep) and np.array_equal(arr.cpu().numpy(), e_arr)


def _device_bytes(g):
    gi = eat.GraphInfo()
    assert eat.lib().eat_graph_info(g.handle, ctypes.byref(gi)) == 0
    return gi.device_bytes


@pytest.mark.parametrize("first", ["batch", "profile"])
def test_the_scratch_is_made_by_the_first_call_and_counted(first):
    n = 500_000
    u, t = np.arange(4, dtype=np.int32), np.full(4, 50, np.int32)
    g = eat.eat_graph_build(u, u + 1, t, t, n)
    out = torch.empty((1, n), dtype=torch.int32, device="cuda")
    held = _device_bytes(g)
    assert 8 * n <= held < 10 * n  # the stops' type ranges: no result row
    g.query(0, 0, out=out[0])
    assert _device_bytes(g) == held
    for _ in range(2):
        if first == "batch":
            eat.eat_query_batch([g], np.zeros(1, np.int32), np.zeros(1, np.int32), np.zeros(1, np.int32), [out[0]])
        else:
            g.profile(0, 0, 100)
        assert held + 4 * n <= _device_bytes(g) < held + 5 * n
