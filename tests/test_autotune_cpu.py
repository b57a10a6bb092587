"""What the tuner chooses and applies, on a model of a handle whose step times are given."""
import json

import pytest

from paper_1808_08555_amd import autotune, lbm3


class _Handle:
    """Records the calls that shape a batch or a lattice; ms() is the model's time of its step."""

    def __init__(self, times):
        self.times, self.shape, self.rows, self.mode = times, None, {}, 0

    def ms(self):
        kind = "default" if self.shape is None and not self.rows and self.mode == 0 else \
            "pairs" if self.mode == 2 else "march"
        return self.times[kind] + (0.0 if self.shape in (None, 128) else 1.0)


@pytest.fixture
def tuner(monkeypatch, tmp_path):
    monkeypatch.setenv("LBM3_AUTOTUNE_CACHE", str(tmp_path / "cache.json"))
    monkeypatch.setattr(autotune, "_arch", lambda torch: "gfx950")

    def set_tile(b, side, threads, rows):
        if side == 0:
            b.shape = threads
        else:
            assert threads == b.shape
            b.rows[side] = rows

    def clear(b):
        b.shape, b.rows = None, {}

    monkeypatch.setattr(lbm3, "lbm3_batch_set_tile", set_tile)
    monkeypatch.setattr(lbm3, "lbm3_batch_clear_tile", clear)
    monkeypatch.setattr(lbm3, "lbm3_batch_set_steps_per_launch", lambda b, mode: setattr(b, "mode", mode))
    monkeypatch.setattr(lbm3, "lbm3_batch_get_pair_launch", lambda b: (b.mode, 0, 0, 0))
    monkeypatch.setattr(lbm3, "lbm3_batch_step", lambda b, n: None)
    return tmp_path / "cache.json"


@pytest.mark.parametrize("times,want", [(dict(default=7.5, march=18.2, pairs=13.6), (None, 0)),
                                        (dict(default=20.0, march=18.2, pairs=23.6), (128, 1)),
                                        (dict(default=20.0, march=18.2, pairs=13.6), (128, 2))])
def test_batch_without_a_shape_is_a_candidate(tuner, monkeypatch, times, want):
    """A batch whose default launches are fastest (blocks, which no shape gives) is left without a
    shape, whatever it had before; otherwise it gets the fastest shape and steps per launch.  The
    second call applies the same from the cache, where an entry of before this candidate is not
    taken."""
    tuner.write_text(json.dumps({"batch3/gfx950/fp64/64,96": {"threads": 512, "rows": {}, "steps_per_launch": 1}}))
    b = _Handle(times)
    b.shape, b.mode = 256, 1
    monkeypatch.setattr(autotune, "_time", lambda torch, fn, steps: b.ms())
    first = autotune.tune_batch(b, [64, 96], "fp64")
    assert (b.shape, b.mode) == want
    again = _Handle(times)
    again.shape = 512
    monkeypatch.setattr(autotune, "_time", None)
    assert autotune.tune_batch(again, [64, 96], "fp64") == first
    assert (again.shape, again.mode, again.rows) == (b.shape, b.mode, b.rows)


@pytest.mark.parametrize("default_ms,shaped", [(3.6, False), (9.0, True)])
def test_lattice_without_a_shape_is_a_candidate(tuner, monkeypatch, default_ms, shaped):
    class Lattice(_Handle):
        def __init__(self, *a, **k):
            super().__init__(dict(default=default_ms, march=5.0, pairs=9.0))

        def init(self, rho):
            return self

        def step(self, n):
            return self

        def set_tile(self, t, r):
            self.shape = t
            return self

        def clear_tile(self):
            self.shape = None
            return self

        def tile(self):
            return self.shape, 0

        def close(self):
            pass

    made = []
    monkeypatch.setattr(lbm3, "Lattice", lambda *a, **k: made.append(Lattice()) or made[-1])
    monkeypatch.setattr(autotune, "_time", lambda torch, fn, steps: made[-1].ms())
    import torch
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: None)
    for again in (False, True):
        target = Lattice()
        target.shape = 512
        t, r = autotune.tune_lattice(64, 64, "fp64", lattice=target)
        assert t == 128 and r in autotune.ROWS
        assert target.shape == (128 if shaped else None)
        monkeypatch.setattr(autotune, "_time", None)  # the second call is served from the cache
