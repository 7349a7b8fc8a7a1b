"""The serving session's host code (session.cpp) against a stand-in for the device
(native/fake_device.cpp): what the request loop does with slots that are not its
own, and what it leaves behind when a call fails half way."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_00966_amd", "csrc")
i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
OK, BUSY = 0, 5  # eat_status


class SessionOptions(ctypes.Structure):
    _fields_ = [("pool_bytes", i64), ("n_streams", i32), ("max_step", i32), ("run", i32 * 13), ("reserved", i32 * 4)]


class Report(ctypes.Structure):
    _fields_ = [("steps", i64), ("launched", i64), ("busy_waits", i64), ("wall_s", ctypes.c_double)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libsession_fake.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-w",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "session.cpp"), os.path.join(ROOT, "tests", "native", "fake_device.cpp"),
                    "-o", so, "-lpthread"], check=True)
    lib = ctypes.CDLL(so)
    lib.fake_alloc.restype, lib.fake_alloc.argtypes = vp, [ctypes.c_size_t]
    lib.fake_graph.restype = vp
    lib.fake_get.restype, lib.fake_get.argtypes = ctypes.c_long, [ctypes.c_char_p]
    lib.fake_set.argtypes = [ctypes.c_char_p, ctypes.c_long]
    lib.fake_error.restype = ctypes.c_char_p
    return lib


V = 100  # stops: two 64-word units of the pool
CALLER = vp(0x1000)  # a caller's stream


def answer(s, ts):
    return 1000 * s + ts


class Fake:
    def __init__(self, lib, slots, **ctl):
        self.lib = lib
        for k in ("hold", "finish", "fail_record", "fail_relax", "fail_copies", "attributes_us", "stream_device", "memcpys",
                  "copy_launches", "overlaps", "stream_syncs", "attributes"):
            lib.fake_set(k.encode(), ctl.get(k, 0))
        g = (vp * 1)(lib.fake_graph(V))
        o = SessionOptions(pool_bytes=slots * 128 * 4, n_streams=4)
        self.h = vp()
        assert lib.eat_session_create(g, 1, ctypes.byref(o), ctypes.byref(self.h)) == OK

    def get(self, name):
        return self.lib.fake_get(name.encode())

    def admit(self, s, ts):
        slot = i32()
        st = self.lib.eat_session_admit(self.h, 0, s, ts, ctypes.byref(slot))
        return slot.value if st == OK else None

    def step(self):
        assert self.lib.eat_session_step(self.h, None) == OK

    def poll(self):
        a, n = (i32 * 4096)(), i32()
        assert self.lib.eat_session_poll(self.h, a, 4096, ctypes.byref(n)) == OK
        return list(a[:n.value])

    def result(self, slot):
        p, n = ctypes.POINTER(i32)(), i32()
        assert self.lib.eat_session_result(self.h, slot, ctypes.byref(p), ctypes.byref(n)) == OK
        return list(p[:n.value])

    def buffers(self, n):
        return [self.lib.fake_alloc(V) for _ in range(n)]

    def serve(self, n, dst=None, arrival=None, min_batch=1000):
        """(status, latency, report); a guard word on each side of every array."""
        def arr(x, dt):
            a = np.full(n + 2, -77, dt)
            a[1:n + 1] = x
            return a
        src, ts = arr(np.arange(n) % V, np.int32), arr(10 + np.arange(n), np.int32)
        gr, at = arr(np.zeros(n), np.int32), arr(np.zeros(n) if arrival is None else arrival, np.float64)
        lat, rep = arr(np.full(n, -5.0), np.float64), Report()
        d = (vp * (n + 2))(*([None] + list(dst) + [None])) if dst is not None else None
        at_ = lambda a: vp(a.ctypes.data + a.itemsize)  # noqa: E731
        st = self.lib.eat_session_serve(self.h, n, at_(gr), at_(src), at_(ts), at_(at), min_batch,
                                        ctypes.c_double(0.0), vp(ctypes.addressof(d) + 8) if d is not None else None,
                                        CALLER, at_(lat), ctypes.byref(rep))
        assert lat[0] == -77 and lat[-1] == -77
        return st, lat[1:-1], rep

    def room(self):
        """Slots that can be admitted now (they are given back)."""
        got = []
        while (s := self.admit(0, 0)) is not None:
            got.append(s)
        for s in got:
            assert self.lib.eat_session_release(self.h, s) == OK
        return len(got)


def holds(p, n, value):
    a = ctypes.cast(p, ctypes.POINTER(i32))
    return all(a[k] == value for k in range(n))


def test_serve_answers_and_copies(lib):
    f = Fake(lib, 300)
    dst = f.buffers(200)
    st, lat, rep = f.serve(200, dst)
    assert st == OK and rep.launched == 200 and np.all(lat >= 0)
    assert all(holds(d, V, answer(i % V, 10 + i)) for i, d in enumerate(dst))
    assert f.room() == 300 and f.poll() == []


def test_results_stay_listed_when_their_copies_fail(lib):
    f = Fake(lib, 100, fail_copies=1)
    st, lat, _ = f.serve(40, f.buffers(40))
    assert st != OK and np.all(lat >= 0)
    got = f.poll()
    assert sorted(f.result(s)[0] for s in got) == sorted(answer(i, 10 + i) for i in range(40))
    for s in got:
        assert f.lib.eat_session_release(f.h, s) == OK
    assert f.room() == 100


def test_results_that_wait_for_a_copy_stay_listed_when_a_step_fails(lib):
    # three bursts of 10, 5 of each finish: the first five are being copied, the second
    # five wait for that copy, the third burst's step fails
    f = Fake(lib, 100, hold=1, finish=5, fail_relax=3)
    dst = f.buffers(30)
    st, lat, _ = f.serve(30, dst, arrival=np.repeat([0, 0.01, 0.02], 10), min_batch=10)
    assert st != OK
    f.lib.fake_drain()
    assert all(holds(d, V, answer(i, 10 + i)) for i, d in enumerate(dst[:5]))
    assert sorted(f.result(s)[0] for s in f.poll()) == [answer(i, 10 + i) for i in range(10, 15)]


@pytest.mark.parametrize("own", [1, 3])
@pytest.mark.parametrize("n", [1, 70])
def test_finished_slots_of_the_caller_are_left_alone(lib, own, n):
    f = Fake(lib, 100)
    mine = [f.admit(90 + i, 5) for i in range(own)]
    f.step()
    assert f.lib.eat_session_sync(f.h) == OK
    dst = f.buffers(n)
    st, lat, rep = f.serve(n, dst)
    assert st == OK and rep.launched == n and np.all(lat >= 0)
    assert all(holds(d, V, answer(i, 10 + i)) for i, d in enumerate(dst))
    assert f.poll() == mine  # finished, not polled yet: as before the call
    assert [f.result(s)[0] for s in mine] == [answer(90 + i, 5) for i in range(own)]
    assert f.room() == 100 - own


@pytest.mark.parametrize("polled", [False, True])
def test_requests_that_can_never_get_a_slot_are_refused(lib, polled):
    f = Fake(lib, 3)
    mine = [f.admit(90 + i, 5) for i in range(3)]  # all of the pool
    f.step()
    assert f.lib.eat_session_sync(f.h) == OK
    if polled:
        assert f.poll() == mine
    st, lat, _ = f.serve(4, f.buffers(4))
    assert st == BUSY
    for s in mine:
        assert f.lib.eat_session_release(f.h, s) == OK
    assert f.serve(4, f.buffers(4))[0] == OK and f.room() == 3


# the first copy launch of 64 results is under way when the next one, or the event
# behind one, fails: no slab may be given out while it is still being copied
@pytest.mark.parametrize("n,ctl", [(100, {"fail_copies": 2}), (150, {"fail_copies": 3}), (40, {"fail_record": 1}),
                                   (100, {"fail_record": 1}), (100, {"fail_record": 2})], ids=str)
def test_slabs_under_copy_are_kept_when_a_copy_fails(lib, n, ctl):
    f = Fake(lib, 200, hold=1, **ctl)
    dst = f.buffers(n)
    assert f.serve(n, dst)[0] != OK
    for s in f.poll():
        assert f.lib.eat_session_release(f.h, s) == OK
    taken = 0
    while f.admit(99, 7) is not None:  # take all that is free, and overwrite it
        taken += 1
        f.step()
        assert f.lib.eat_session_sync(f.h) == OK
    launched = f.get("copy_launches") - (1 if "fail_copies" in ctl else 0)
    assert taken == 200 - 64 * launched or f.get("stream_syncs") > 0  # kept, or waited for
    f.lib.fake_drain()
    for i, d in enumerate(dst[:64 * launched]):
        assert holds(d, V, answer(i % V, 10 + i)), i
    assert not any(holds(d, V, answer(99, 7)) for d in dst)


# requests with one destination, or with destinations that overlap in part: copies one
# after the other, the one that finished last on top
@pytest.mark.parametrize("shift", [0, 1, V - 1])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 130])
def test_destinations_that_overlap_are_written_one_after_the_other(lib, n, shift):
    f = Fake(lib, 200)
    room = f.lib.fake_alloc(V + n * shift)
    st, _, _ = f.serve(n, [room + 4 * shift * i for i in range(n)])
    assert st == OK and f.get("overlaps") == 0
    a = ctypes.cast(room, ctypes.POINTER(i32))
    assert holds(room + 4 * shift * (n - 1), V, answer((n - 1) % V, 9 + n))
    if shift > 0:
        assert all(a[shift * i] == answer(i % V, 10 + i) for i in range(n))
    # destinations side by side still share launches
    f.lib.fake_set(b"copy_launches", 0)
    room = f.lib.fake_alloc(V * n)
    assert f.serve(n, [room + 4 * V * i for i in range(n)])[0] == OK
    assert f.get("copy_launches") == (n + 63) // 64 and f.get("overlaps") == 0


def test_the_time_of_a_call_counts_from_its_start(lib):
    n = 50
    f = Fake(lib, 100, attributes_us=2000)
    st, lat, rep = f.serve(n, f.buffers(n))
    assert st == OK and f.get("attributes") == n  # the destinations are looked at once
    assert rep.wall_s >= n * 2e-3  # "from the call until the last query finished"


def test_requests_do_not_queue_up_while_destinations_are_looked_at(lib):
    # 200 destinations of 1 ms each; the first request has its answer before that
    n = 200
    f = Fake(lib, 300, attributes_us=1000)
    st, lat, _ = f.serve(n, f.buffers(n), arrival=np.concatenate([[0], np.full(n - 1, 0.02)]), min_batch=1)
    assert st == OK and lat[0] < 0.02


def test_a_copy_stream_of_another_device_gets_plain_copies(lib):
    f = Fake(lib, 100, stream_device=1)
    dst = f.buffers(70)
    assert f.serve(70, dst)[0] == OK
    assert f.get("copy_launches") == 0 and f.get("memcpys") == 70  # a kernel cannot be launched there
    assert all(holds(d, V, answer(i % V, 10 + i)) for i, d in enumerate(dst))
