"""One-shot batches and profiles from the scratch a graph keeps, bit-exact against
the CPU oracle: sizes around what it takes, calls in a row, on several streams
and from several threads at once, and a failed call followed by a good one."""
import threading

import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def towns():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tts = [synth.scaled_city(700 + 13 * i, seed=60 + i) for i in range(3)]
    return [eat.graph_from_timetable(t) for t in tts], [oracle.Csa(t.u, t.v, t.t, t.lam, t.n_vertices) for t in tts]


def _questions(graphs, which, n, seed):
    rng = np.random.default_rng(seed)
    gi = rng.integers(0, len(which), n).astype(np.int32)
    nv = np.array([graphs[w].n_vertices for w in which])[gi] if n else np.zeros(0, np.int64)
    return gi, rng.integers(0, np.maximum(nv, 1)).astype(np.int32), rng.integers(0, 86400, n).astype(np.int32), nv


def _run(towns, which, n, seed, stream=None, check=True, **kw):
    graphs, csa = towns
    gi, src, ts, nv = _questions(graphs, which, n, seed)
    with torch.cuda.stream(stream or torch.cuda.current_stream()):
        outs = [torch.full((int(v),), -3, dtype=torch.int32, device="cuda") for v in nv]
        eat.eat_query_batch([graphs[w] for w in which], gi, src, ts, outs, **kw)
    if check:  # the call has waited: no synchronisation here
        for i in range(n):
            exp = csa[which[gi[i]]].query(int(src[i]), int(ts[i]))
            assert np.array_equal(outs[i].cpu().numpy(), exp), i


# queries: none, one, fewer and more than the XCDs' buckets, the scratch's 1,024 and
# one more; graphs: one, several, its 16 and one more
@pytest.mark.parametrize("n,graphs", [(0, 1), (1, 1), (7, 3), (9, 3), (100, 2), (1024, 1), (1025, 1), (40, 16), (40, 17)])
def test_one_shot_batches_around_the_scratch(towns, n, graphs):
    which = [i % 3 for i in range(graphs)]
    for seed in (1, 2):  # twice in a row, other questions
        _run(towns, which, n, seed)
    _run(towns, which, min(n, 5), 3)
    _run(towns, which, min(n, 5), 4, stats=True)


def test_a_failed_call_leaves_nothing_behind(towns):
    for rnd in range(2):
        with pytest.raises(eat.EatError) as ei:
            _run(towns, [0], 50, 7, check=False, options={"max_rounds": 1})
        assert ei.value.status == eat.EAT_ERR_NOT_CONVERGED
        _run(towns, [0], 50, 8 + rnd)
    with pytest.raises(eat.EatError):
        towns[0][0].profile(0, 0, 86400, options={"max_rounds": 1})
    _run(towns, [0], 50, 10)


def test_threads_and_streams_share_a_graph(towns):
    graphs, csa = towns
    errors = []

    def work(k):
        try:
            torch.cuda.set_device(0)
            stream = torch.cuda.Stream()
            for rnd in range(6):
                _run(towns, [0, 1], 30 + 11 * k, 100 * k + rnd, stream=stream)
                s = (37 * k + rnd) % graphs[0].n_vertices
                with torch.cuda.stream(stream):
                    dep, arr = graphs[0].profile(s, 6 * 3600, 9 * 3600)
                stream.synchronize()
                e_dep, e_arr = csa[0].profile(s, 6 * 3600, 9 * 3600)
                assert np.array_equal(dep, e_dep) and np.array_equal(arr.cpu().numpy()[:len(e_dep)], e_arr)
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
