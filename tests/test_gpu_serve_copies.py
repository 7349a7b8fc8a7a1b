"""Result copies of the native request loop, bit-exact against the CPU oracle:
destinations of any 4-byte alignment and in host memory, requests without one,
slabs of odd sizes, and pools that force waits for slots whose copies are still
pending."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cities():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    tts = [synth.scaled_city(1001, seed=31), synth.scaled_city(4097, seed=32), synth.scaled_city(20003, seed=33)]
    return [eat.graph_from_timetable(t) for t in tts], [oracle.Csa(t.u, t.v, t.t, t.lam, t.n_vertices) for t in tts]


# requests: one, about a copy launch's 64 slabs, several launches' worth; pools of
# every slot at once and of only a few
@pytest.mark.parametrize("n,pool", [(1, 0), (63, 0), (64, 0), (65, 0), (300, 0), (300, 400_000)])
@pytest.mark.parametrize("on_stream", [False, True])
def test_serve_copies(cities, n, pool, on_stream):
    graphs, csa = cities
    rng = np.random.default_rng([n, pool])
    gi = rng.integers(0, 3, n).astype(np.int32)
    nv = np.array([g.n_vertices for g in graphs])[gi]
    src = rng.integers(0, nv).astype(np.int32)
    ts = rng.integers(0, 86400, n).astype(np.int32)
    room = torch.full((int((nv + 8).sum()),), -5, dtype=torch.int32, device="cuda")
    place = np.cumsum(nv + 8) - (nv + 8) + np.arange(n) % 4
    kind = rng.integers(0, 8, n)  # 0: no copy, 1: host memory, else device memory
    host = {i: torch.full((int(nv[i]),), -5, dtype=torch.int32, pin_memory=True) for i in range(n) if kind[i] == 1}
    dst = (ctypes.c_void_p * n)()
    for i in range(n):
        if kind[i] == 1:
            dst[i] = host[i].data_ptr()
        elif kind[i] > 1:
            dst[i] = room.data_ptr() + 4 * int(place[i])
    sess = eat.Session(graphs, pool_bytes=pool, n_streams=4)
    lat, arrival = np.zeros(n), np.sort(rng.uniform(0, 300e-6, n))
    f64 = ctypes.POINTER(ctypes.c_double)
    i32 = ctypes.POINTER(ctypes.c_int32)
    stream = torch.cuda.Stream() if on_stream else torch.cuda.current_stream()
    torch.cuda.synchronize()
    for rnd in range(2):  # slots and marks of the first round are used again
        print(n, pool, on_stream, rnd, flush=True)
        room.fill_(-5)
        torch.cuda.synchronize()
        st = eat.lib().eat_session_serve(sess._h, n, gi.ctypes.data_as(i32), src.ctypes.data_as(i32),
                                         ts.ctypes.data_as(i32), arrival.ctypes.data_as(f64), 16, 20e-6, dst,
                                         ctypes.c_void_p(stream.cuda_stream), lat.ctypes.data_as(f64), None)
        assert st == 0
        torch.cuda.synchronize()
        got = room.cpu().numpy()
        left = np.ones(len(got), bool)
        for i in range(n):
            exp = csa[gi[i]].query(int(src[i]), int(ts[i]))
            if kind[i] == 1:
                assert np.array_equal(host[i].numpy(), exp), i
            elif kind[i] > 1:
                assert np.array_equal(got[place[i]:place[i] + nv[i]], exp), i
                left[place[i]:place[i] + nv[i]] = False
        assert np.all(got[left] == -5)  # nothing beside the destinations
