"""Host: the autotuner times the library's own choice and keeps it where it is fastest."""
import json

import pytest

from paper_1008_2865_amd import autotune as A
from paper_1008_2865_amd import binding as B


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tiles.json"
    monkeypatch.setenv("LB_TUNE_CACHE", str(path))
    return path


def fake_timer(monkeypatch, default, others):
    calls = []

    def time_shape(nx, ny, storage, tile_x, tile_y, tile_rows, steps=100, warmup=20, steps_per_launch=1):
        calls.append((tile_x, tile_y, tile_rows, steps_per_launch))
        return default if calls[-1] == (0, 0, 0, 0) else others + 0.001 * tile_y

    monkeypatch.setattr(A, "time_shape", time_shape)
    return calls


@pytest.mark.parametrize("storage", ["f32", "f64"])
def test_the_default_is_timed_and_kept(cache, monkeypatch, storage):
    calls = fake_timer(monkeypatch, default=4.5, others=7.5)
    assert A.tune(512, 512, storage) == (0, 0, 0)
    assert (0, 0, 0, 0) in calls and len(calls) > 1
    calls.clear()
    assert A.tune(512, 512, storage) == (0, 0, 0) and calls == []
    # Zeros are the library's choice: no shape of the caller's.
    p = B.make_params(512, 512, storage=B.LB_F32)
    assert (p.tile_x, p.tile_y, p.tile_rows) == (0, 0, 0)


def test_a_faster_shape_still_wins(cache, monkeypatch):
    fake_timer(monkeypatch, default=9.0, others=7.5)
    assert A.tune(512, 512, "f32") == (256, 2, 1)


def test_entries_that_the_default_took_no_part_in_are_not_answers(cache, monkeypatch):
    cache.write_text(json.dumps({"f32:512x512": {"tile_x": 128, "tile_y": 16, "tile_rows": 1, "us_per_step": 7.0}}))
    fake_timer(monkeypatch, default=4.5, others=7.5)
    assert A.tune(512, 512, "f32") == (0, 0, 0)
    # A list of the caller's is timed as given and keeps its own entry.
    assert A.tune(512, 512, "f32", candidates=[(64, 4, 1)]) == (128, 16, 1)


def test_two_step_tuner_times_the_default_height_wherever_it_has_one(cache, monkeypatch):
    dx, dy, _ = B.lb_two_step_shape(B.make_params(1100, 1100, storage=B.LB_F32, steps_per_launch=2))
    assert dy >= 8
    calls = fake_timer(monkeypatch, default=0.0, others=2.0)
    A.tune(1100, 1100, "f32", steps_per_launch=2)
    assert (dx, dy, 1, 2) in calls


class FakeBatch:
    """A batch whose own height is 28 and whose time is least there."""
    storage, shapes, default = "f32", [(96, 96)], 28

    def __init__(self):
        self.height, self.set = self.default, []

    def two_step_shape(self):
        return 128, self.height, 1

    def set_two_step_tile(self, ty):
        self.height = ty or self.default
        self.set.append(ty)

    def step(self, n):
        pass


class FakeEvent:
    batch = None

    def __init__(self, enable_timing):
        pass

    def record(self):
        pass

    def elapsed_time(self, other):
        return abs(self.batch.height - 28) + 1.0


def test_batch_height_tuner_times_the_batch_s_own_height(cache, monkeypatch):
    torch = pytest.importorskip("torch")
    batch = FakeEvent.batch = FakeBatch()
    monkeypatch.setattr(torch.cuda, "Event", FakeEvent)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    assert A.tune_batch_two_step(batch) == 28 and batch.height == 28
    assert set(A.BATCH_TWO_STEP_HEIGHTS) < set(batch.set)
    # A list of the caller's is timed as given.
    assert A.tune_batch_two_step(batch, heights=(16, 32)) == 32
