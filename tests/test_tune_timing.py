"""The tuner's clock, on a simulated device: candidates timed again are timed
over more launches, with rows from HBM as with rows just produced."""
import contextlib

import pytest

from paper_2603_27569_amd import tune


class _Device:
    """Counts launches; each takes `us` of simulated time when it runs."""

    def __init__(self, us):
        self.us, self.now, self.capturing, self.replayed = us, 0.0, None, 0
        device = self

        class Graph:
            launches = 0

            def replay(self):
                device.replayed += self.launches
                device.now += self.launches * device.us

        class Event:
            def __init__(self, enable_timing):
                pass

            def record(self, stream):
                self.at = device.now

            def elapsed_time(self, other):
                return (other.at - self.at) / 1e3

        @contextlib.contextmanager
        def graph(g, stream):
            device.capturing = g
            yield
            device.capturing = None

        self.cuda = type("cuda", (), {"CUDAGraph": Graph, "Event": Event, "graph": staticmethod(graph),
                                      "stream": staticmethod(lambda s: contextlib.nullcontext()),
                                      "synchronize": staticmethod(lambda: None)})

    def launch(self, *_):
        if self.capturing is not None:
            self.capturing.launches += 1


@pytest.mark.parametrize("us", [2.0, 5.0, 40.0, 400.0])
@pytest.mark.parametrize("ring", [3, 15, 400])
def test_second_timing_is_longer(us, ring):
    def launches(factor):
        d = _Device(us)
        buffers = list(range(ring))
        got = tune._time_both(d, None, d.launch, buffers, buffers, 30, factor)
        assert got == pytest.approx(us)
        return d.replayed

    # every timed repeat is `factor` times as long; the two untimed replays of
    # each graph that probe the duration are not
    assert launches(tune.FINAL_FACTOR) >= 0.8 * tune.FINAL_FACTOR * launches(1) * 3 / 5


@pytest.mark.parametrize("us", [2.0, 40.0])
def test_a_repeat_covers_its_time(us):
    d = _Device(us)
    tune._time(d, None, d.launch, 30)
    once = d.replayed
    d = _Device(us)
    tune._time(d, None, d.launch, 30, tune.FINAL_FACTOR)
    per = 30
    assert d.replayed - 2 * per == tune.FINAL_FACTOR * (once - 2 * per)
    assert (once - 2 * per) / 3 * us >= min(tune.REPEAT_US, 2000 * us)
