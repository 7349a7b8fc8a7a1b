"""Table slots that every wave writes while others probe them, bit-exact against
the CPU oracle: stops whose slots lie side by side, each improved by hundreds of
connections of one round."""
import numpy as np
import pytest

import oracle
from paper_1912_00966_amd import eat

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# stops of the contended layer: one pair of slots, a few, more than a wave has lanes
@pytest.mark.parametrize("narrow", [1, 2, 7, 65])
@pytest.mark.parametrize("threads", [1024, 768, 256])
def test_contended_slots(narrow, threads):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(narrow)
    wide = 400  # 0 -> wide -> narrow -> wide, departures and durations at random
    a, b = 1 + np.arange(wide), 1 + wide + np.arange(narrow)
    aa, bb = (x.ravel() for x in np.meshgrid(a, b))
    u = np.concatenate([np.zeros(wide), aa, bb])
    v = np.concatenate([a, bb, aa])
    t = np.concatenate([np.full(wide, 100), rng.integers(200, 9000, len(aa)), rng.integers(200, 20000, len(bb))])
    lam = np.concatenate([1 + rng.integers(0, 50, wide), 1 + rng.integers(0, 5000, 2 * len(aa))])
    conn = [x.astype(np.int32) for x in (u, v, t, lam)]
    n = 1 + wide + narrow
    g, csa = eat.eat_graph_build(*conn, n), oracle.Csa(*conn, n)
    q = 512
    s, ts = np.where(np.arange(q) % 2, rng.integers(0, n, q), 0).astype(np.int32), rng.integers(0, 101, q).astype(np.int32)
    exp = csa.query_many(s, ts)
    for table in (0, 1024):
        out = torch.empty((q, n), dtype=torch.int32, device="cuda")
        eat.eat_query_batch([g], np.zeros(q, np.int32), s, ts, [out[i] for i in range(q)],
                            options={"threads_per_query": threads, "table_cap": table})
        assert np.array_equal(out.cpu().numpy(), exp)
