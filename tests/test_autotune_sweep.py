"""Which launch shapes the autotuner times (no GPU: the step and the timer are
stand-ins)."""
import json
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture
def sweep(monkeypatch):
    """tune() with a step that takes cost(cfg) ms; returns its choice and the
    shapes (tile, lds_batch, persistent, lds_batch_bwd) it timed."""
    from paper_2603_27781_amd import autotune, batched
    state = SimpleNamespace(ms=0.0)

    class Step:
        def __init__(self, g, views, cfg, *a, **kw):
            self.cfg = cfg

        def ensure_capacity(self):
            pass

        def run(self):
            state.ms = state.cost(self.cfg)
            state.seen.append((self.cfg.tile, self.cfg.lds_batch, self.cfg.persistent, self.cfg.lds_batch_bwd))

    class Event:
        def __init__(self, **kw):
            pass

        def record(self):
            pass

        def elapsed_time(self, other):
            return state.ms

    monkeypatch.setattr(batched, "MappingStep", Step)
    monkeypatch.setattr(torch.cuda, "Event", Event)
    for f in ("synchronize", "empty_cache"):
        monkeypatch.setattr(torch.cuda, f, lambda: None)
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda i: "stand-in")

    def run(cost, cache=None):
        state.cost, state.seen = cost, []
        g = SimpleNamespace(n=10, n_feat=16)
        cfg = autotune.tune(g, [SimpleNamespace(width=8, height=8)], None, None, None, None, None, cache=cache)
        return cfg, list(dict.fromkeys(state.seen))

    return run


@pytest.mark.parametrize("best", [(16, 256, 0), (16, 128, 1), (8, 64, 0), (32, 256, 1)])
def test_every_backward_batch_is_timed_by_name(sweep, best):
    def cost(c):  # the backward is fastest with the batch that is not the forward's
        return 1.0 * ((c.tile, c.lds_batch, c.persistent) != best) + (0.1 if c.lds_batch_bwd == c.lds_batch else 0.0)

    cfg, seen = sweep(cost)
    assert (cfg.tile, cfg.lds_batch, cfg.persistent) == best
    assert cfg.lds_batch_bwd in (64, 128, 256) and cfg.lds_batch_bwd != best[1]
    assert all(s[3] in (64, 128, 256) for s in seen)
    most = 128 if best[0] == 8 else 256
    assert {s[3] for s in seen if s[:3] == best} == {b for b in (64, 128, 256) if b <= most}


def test_entries_of_the_old_meaning_are_not_read(sweep, tmp_path):
    """Before, an entry's lds_batch_bwd = 0 stood for lds_batch."""
    import dataclasses
    from paper_2603_27781_amd import raster
    path = tmp_path / "cache.json"
    old = dataclasses.asdict(raster.Config(tile=32, lds_batch=256))
    path.write_text(json.dumps({"stand-in|n=10|F=16|8x8|params=1|pose=0": {"config": old}}))
    cfg, seen = sweep(lambda c: float(c.tile != 16), cache=str(path))
    assert cfg.tile == 16 and seen
    again, seen = sweep(lambda c: 1.0, cache=str(path))
    assert again == cfg and not seen
