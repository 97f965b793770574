"""A lookup without the cache's lock never meets a plan that is being closed."""
import paper_2603_27569_amd as sf


class _Stub:
    def __init__(self):
        self.closed = False
        self.seen_while_closing = None

    def close(self):
        self.closed = True
        self.seen_while_closing = list(sf._plan_cache.values())


def test_clear_takes_plans_out_before_closing_them(monkeypatch):
    stubs = [_Stub(), _Stub()]
    monkeypatch.setattr(sf, "_plan_cache", {(256, i, -1, 0, 0, None, 0): s for i, s in enumerate(stubs)})
    assert sf._plan_for(256, 1, -1, 0, 0, None, 0) is stubs[1]
    sf.clear_plan_cache()
    for s in stubs:
        assert s.closed and s.seen_while_closing == []
    assert sf._plan_cache == {}
