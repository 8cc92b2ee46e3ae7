"""The pools that jobs of a CountingServer share, taken from and given back to
by several threads at once. No GPU: streams and buffers are stand-ins."""
import sys
import threading
from types import SimpleNamespace

import pytest

from paper_1607_06618_amd import serve


class Item:
    def __init__(self, *args, **kw):
        self.users = 0

    def numel(self):
        return 1 << 20


fake_torch = SimpleNamespace(cuda=SimpleNamespace(Stream=Item), empty=Item, uint8=None)


class Racing(list):
    """A list whose emptiness is asked by every thread before any of them takes its last item."""

    def __init__(self, items, threads):
        super().__init__(items)
        self.barrier = threading.Barrier(threads)

    def __bool__(self):
        some = len(self) > 0
        try:
            self.barrier.wait(timeout=0.2)
        except threading.BrokenBarrierError:
            pass   # (they cannot meet where one holds a lock)
        return some


@pytest.mark.parametrize("kind", ["streams", "buffers"])
def test_the_last_item_goes_to_one_thread(kind):
    n = 3
    if kind == "streams":
        pool = serve._StreamPool(fake_torch, "cuda:0", 8)
        pool.free = Racing([Item()], n)
        take = pool.take
    else:
        pool = serve._PinnedPool(fake_torch)
        pool.free[1 << 20] = Racing([Item()], n)
        take = lambda: pool.take(100)
    got, errors = [], []

    def run():
        try:
            got.append(take())
        except Exception as e:   # noqa: BLE001 -- the test reports whatever came
            errors.append(e)

    threads = [threading.Thread(target=run) for _ in range(n)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not errors
    assert len(set(map(id, got))) == n


def test_streams_are_handed_to_one_job_at_a_time_and_bounded():
    pool = serve._StreamPool(fake_torch, "cuda:0", 4)
    old, bad = sys.getswitchinterval(), []
    sys.setswitchinterval(1e-6)

    def run():
        for _ in range(2000):
            s = pool.take()
            s.users += 1
            if s.users != 1:
                bad.append(s)
            s.users -= 1
            pool.give(s)

    try:
        threads = [threading.Thread(target=run) for _ in range(8)]
        [t.start() for t in threads]
        [t.join() for t in threads]
    finally:
        sys.setswitchinterval(old)
    assert not bad and len(pool.free) <= 4
