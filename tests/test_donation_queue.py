"""The queue of donated tasks on the CPU: its slot arithmetic compiled for the
host, and a model of the waves' steps on the control words (one atomic access a
step, steps of all waves interleaved at random).  Every donated task is taken
exactly once, with the words its donor wrote, slots are used again, and no wave
leaves while an entry has nobody left to take it."""
import ctypes
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("donate") / "donate_host.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(HERE, "native", "donate_host.cpp"), "-o", out])
    L = ctypes.CDLL(out)
    for f in (L.t_slot, L.t_published, L.t_read, L.t_last):
        f.restype = ctypes.c_uint32
    for f in (L.t_slot, L.t_published, L.t_read):
        f.argtypes = [ctypes.c_uint32] * 2
    L.t_fits.argtypes = [ctypes.c_uint32] * 4
    return L


@pytest.mark.parametrize("cap", [4, 2048, 4096])
def test_ready_words_never_repeat_and_the_numbers_end(lib, cap):
    last = lib.t_last()
    for s in (0, 1, cap - 1, cap, 2 * cap + 3, last - cap, last):
        assert lib.t_slot(s, cap) == s % cap
        use = s // cap
        assert (lib.t_published(s, cap), lib.t_read(s, cap)) == (3 * use + 1, 3 * use + 3)
        if s + cap <= last:  # the next use starts where this one ended, and its words are larger
            assert lib.t_published(s + cap, cap) == lib.t_read(s, cap) + 1
    assert lib.t_fits(0, 0, min(64, cap), cap)
    assert lib.t_fits(5, 5 + cap - 3, 3, cap) and not lib.t_fits(5, 5 + cap - 3, 4, cap)
    assert lib.t_fits(last - 64, last - 64, min(64, cap), cap)
    assert not lib.t_fits(last, last, 1, cap) and not lib.t_fits(last - 2, last - 2, 3, cap)


@pytest.mark.parametrize("cap, head, tail", [(4, 0, 0), (4, 0, 3), (4, 6, 10), (2048, 4095, 4097), (2048, 5000, 6100)])
def test_an_entry_left_behind_is_found(lib, cap, head, tail):
    """The check at the end of a launch: 256 threads, each over its share of the
    entries from the head on."""
    W = 9
    don = (ctypes.c_uint32 * (W * cap))()

    def left():
        return any(lib.t_left(don, W, cap, head, tail, t, 256) for t in range(256))

    for s in range(tail):
        don[W * lib.t_slot(s, cap) + 1] = lib.t_read(s, cap)
    assert not left()
    for s in sorted({head, (head + tail) // 2, tail - 1}):
        if head <= s < tail:
            for state in (0, 1, 2):  # reserved, published, claimed
                don[W * lib.t_slot(s, cap) + 1] = lib.t_read(s, cap) - 3 + state
                assert left()
            don[W * lib.t_slot(s, cap) + 1] = lib.t_read(s, cap)
    assert not left()


class Model:
    """waves[i] starts with work[i] units; a wave with several units left hands
    some to the queue while waves wait, as many as wait beyond the queue."""

    def __init__(self, lib, rng, cap, max_waiters, work):
        self.lib, self.rng, self.cap, self.max_waiters = lib, rng, cap, max_waiters
        self.head = self.tail = self.idle = 0
        self.active = 0
        self.ready = [0] * cap
        self.payload = [None] * cap
        self.done = 0
        self.taken = set()
        self.waves = [self.wave(i, w) for i, w in enumerate(work)]

    def wave(self, me, units):
        L, cap = self.lib, self.cap
        self.active += 1
        given = 0  # the sequence number after this wave's last donated task
        while True:
            # ---- work, donating between units
            while units:
                units -= 1
                self.done += 1
                yield
                if units < 2 or self.rng.random() < 0.3:
                    continue
                idle = self.idle
                yield
                if idle == 0:
                    continue
                head = self.head
                yield
                tail = self.tail
                yield
                room = idle - (tail - head) if tail >= head else 0
                k = min(units // 2, room, cap)
                if k <= 0 or not L.t_fits(head, tail, k, cap) or self.tail != tail:
                    continue
                self.tail = given = tail + k  # (the compare-and-swap above)
                yield
                share = units // (2 * k)
                for s in range(tail, tail + k):
                    assert self.ready[L.t_slot(s, cap)] == L.t_read(s, cap) - 3, "a slot in use was reserved"
                    self.payload[L.t_slot(s, cap)] = (s, share)
                    yield
                    self.ready[L.t_slot(s, cap)] = L.t_published(s, cap)
                    yield
                units -= share * k
            # ---- drained
            self.active -= 1
            yield
            wait = self.idle < self.max_waiters
            yield
            got = None
            if wait or given:
                if wait:
                    self.idle += 1
                    yield
                for poll in range(10 ** 6):
                    h = self.head
                    yield
                    t = self.tail
                    yield
                    if h < t:
                        s = self.rng.randrange(h, t) if self.rng.random() < 0.75 else h
                        pub = L.t_published(s, cap)
                        seen = self.ready[L.t_slot(s, cap)]
                        yield
                        if seen == pub and self.ready[L.t_slot(s, cap)] == pub:
                            self.ready[L.t_slot(s, cap)] = pub + 1
                            got = s
                            yield
                        i = 0
                        while s == h and h < t and i < 8:
                            word = self.ready[L.t_slot(h, cap)]
                            yield
                            if word != L.t_read(h, cap):
                                break
                            if self.head == h:
                                self.head = h + 1
                            yield
                            h += 1
                            i += 1
                        if got is not None:
                            break
                    if not wait and h >= given:
                        break
                    if h >= t:
                        act = self.active
                        yield
                        if act == 0:
                            break
                if wait:
                    self.idle -= 1
                    yield
            if got is None:
                return
            self.active += 1
            yield
            s, units = self.payload[L.t_slot(got, cap)]
            yield
            assert s == got and got not in self.taken
            self.taken.add(got)
            self.ready[L.t_slot(got, cap)] = L.t_read(got, cap)
            yield

    def run(self):
        live = list(self.waves)
        steps = 0
        while live:
            i = self.rng.randrange(len(live))
            # now and then one wave runs on for a while, or is held back
            for _ in range(self.rng.choice([1, 1, 1, 40])):
                steps += 1
                try:
                    next(live[i])
                except StopIteration:
                    live.pop(i)
                    break
            assert steps < 10 ** 7, "no end"


@pytest.mark.parametrize("cap, waiters, waves", [(4, 1, 3), (4, 2, 6), (8, 3, 12), (16, 40, 12)])
def test_every_donated_task_is_taken_once(lib, cap, waiters, waves):
    used = 0
    for seed in range(30):
        rng = random.Random(100 * seed + cap + waiters)
        work = [rng.choice([0, 1, 3, 200, 600]) for _ in range(waves)] + [1500]
        m = Model(lib, rng, cap, waiters, work)
        m.run()
        assert m.done == sum(work)
        assert m.taken == set(range(m.tail))
        assert all(m.ready[lib.t_slot(s, cap)] == lib.t_read(s, cap) for s in range(m.head, m.tail))
        used += m.tail > cap
    assert used  # slots were used again
