"""Which graphs a launch plan takes, and what its options promise, bit-exact
against the CPU oracle."""
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
def _ring(n):
    """n stops, two connections each to stops a little further on."""
    rng = np.random.default_rng(n)
    u = np.repeat(np.arange(n, dtype=np.int32), 2)
    v = ((u + rng.integers(1, 40, 2 * n)) % n).astype(np.int32)
    t, lam = rng.integers(0, 86400, 2 * n).astype(np.int32), rng.integers(1, 900, 2 * n).astype(np.int32)
    return eat.eat_graph_build(u, v, t, lam, n), oracle.Csa(u, v, t, lam, n)


# stops whose activity bitmap leaves two queries a CU their 320 list entries, one
# stop more, and the most that 256 entries leave room for
@pytest.mark.parametrize("n", [532_480, 532_481, 552_960])
def test_two_queries_a_cu_on_graphs_near_the_limit(n):
    g, csa = _ring(n)
    for threads in (768, 512):
        for s, ts in ((0, 0), (n - 1, 30_000)):
            print(n, threads, s, ts, flush=True)
            out = g.query(s, ts, options={"threads_per_query": threads})
            assert np.array_equal(out.cpu().numpy(), csa.query(s, ts))
    q = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    out = torch.empty((q, n), dtype=torch.int32, device="cuda")
    src, ts = (np.arange(q) * 997 % n).astype(np.int32), np.full(q, 70_000, np.int32)
    b = eat.Batch([g], np.zeros(q, np.int32), src, ts, [out[i] for i in range(q)])
    assert b.options()["threads_per_query"] == 768  # more queries than CUs
    b.run()
    b.wait()
    for i in (0, 1, q - 1):
        assert np.array_equal(out[i].cpu().numpy(), csa.query(int(src[i]), 70_000)), i


def test_a_bitmap_past_the_smaller_lists_is_refused():
    g, _ = _ring(552_961)
    with pytest.raises(eat.EatError) as ei:
        g.query(0, 0, options={"threads_per_query": 768})
    assert ei.value.status == eat.EAT_ERR_UNSUPPORTED


@functools.lru_cache(maxsize=None)
def _line(hops, lam, layout):
    """A line of hops connections of lam seconds each, and a side branch at every stop."""
    i = np.arange(hops, dtype=np.int32)
    u, v = np.concatenate([i, i]), np.concatenate([i + 1, hops + 1 + i])
    t = np.concatenate([1000 + i * (lam + 5)] * 2)
    args = (u, v, t.astype(np.int32), np.full(2 * hops, lam, np.int32), 2 * hops + 1)
    kw = {"grid": {}, "flat": {"layout": eat.EAT_LAYOUT_FLAT}}[layout]
    return eat.eat_graph_build(*args, cluster_seconds=30000, **kw), oracle.Csa(*args)


# hops shorter than the window, longer, and longer than any window asked for; one
# round for every hop and one that finds nothing more to do
@pytest.mark.parametrize("lam", [300, 9000, 50_000])
@pytest.mark.parametrize("layout", ["grid", "flat"])
def test_a_round_limit_of_one_per_hop_is_enough(lam, layout):
    hops = 30
    g, csa = _line(hops, lam, layout)
    exp = csa.query(0, 0)
    for o in ({}, {"threads_per_query": 768}, {"time_window": 60}, {"time_window": -1}, {"time_window": 20_000},
              {"types_per_lane": 2}, {"table_cap": -1}, {"threads_per_vertex": 16}, {"mode": eat.EAT_MODE_TOPOLOGY}):
        print(lam, layout, o, flush=True)
        out, st = g.query(0, 0, options=dict(o, max_rounds=hops + 1), stats=True)
        assert np.array_equal(out.cpu().numpy(), exp) and st["rounds"] <= hops + 1
        with pytest.raises(eat.EatError) as ei:  # the last stop is out of reach
            g.query(0, 0, options=dict(o, max_rounds=hops - 1), stats=True)
        assert ei.value.status == eat.EAT_ERR_NOT_CONVERGED
    n = 40
    outs = torch.empty((n, g.n_vertices), dtype=torch.int32, device="cuda")
    eat.eat_query_batch([g], np.zeros(n, np.int32), np.arange(n) % 5, np.zeros(n, np.int32), [outs[i] for i in range(n)],
                        options={"max_rounds": hops + 1})
    for i in range(5):
        assert np.array_equal(outs[i].cpu().numpy(), csa.query(i, 0))
