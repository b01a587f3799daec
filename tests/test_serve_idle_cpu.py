"""The server's idle moments: what it collects in them has to fit."""
import gc

from paper_2210_01465_amd import serve
from test_serve_cpu import FakeBackend, make_requests


def test_no_long_collection_in_a_short_gap(monkeypatch):
    """A busy spell leaves many objects behind; the gaps of about 2 ms after it
    are too short to collect them, those between few objects are not."""
    kept, collected = [], []
    real = gc.collect

    def collect(generation=2):
        collected.append(gc.get_count()[0])
        return real(generation)

    class Busy(FakeBackend):
        def step(self):
            if len(self.built) >= 3 and not kept:   # the spell
                kept.extend([] for _ in range(300_000))
            return super().step()

    reqs = make_requests(60, seed=6, rate=500.0)
    fb = Busy()
    srv = serve.Server(fb, hbm_budget=1 << 30, clock=fb.clock, sleep=fb.sleep)
    real()
    monkeypatch.setattr(serve.gc, "collect", collect)
    done = srv.run(reqs)
    monkeypatch.undo()
    assert len(done) == len(reqs) and len(kept) == 300_000
    # before the spell it did collect; 0.1 us per object: none took 10 ms
    assert collected and max(collected) < 100_000
