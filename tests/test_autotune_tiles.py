"""The batch tuner on a stand-in batch whose larger tiles are the faster ones: it
takes tiles past the default only from a caller who lists them, since the
fixed-point quantum of a tile grows with the records it holds."""
import json
import time

import pytest
import torch

from paper_1706_08575_amd import autotune


class Stand:
    W, sigma, R, sizes = 6, 2.0, 8.0, [256]

    def set_tuning(self, tile=32, chunk=4096):
        self.tile, self.chunk = tile, chunk

    def set_points(self, m, k):
        pass

    def execute(self, fhat, out=None):
        time.sleep(2e-3 * 64 / self.tile + (0.0 if self.chunk == 4096 else 5e-3))


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("FTCG_TUNING_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    return path


def test_default_candidates_stop_at_the_default_tile(cache):
    B = Stand()
    best, ms = autotune.tune_batch(B, [1000], None, None, reps=1)
    assert best == (32, 4096) and (B.tile, B.chunk) == best
    assert max(t for t, _ in ms) == 32
    assert autotune.tune_batch(B, [1000], None, None)[0] == best     # from the cache


def test_listed_candidates_are_taken(cache):
    B = Stand()
    best, _ = autotune.tune_batch(B, [1000], None, None, tiles=(32, 64), reps=1)
    assert best == (64, 4096) and B.tile == 64
    # remembered for callers who list it, not for the others
    assert autotune.tune_batch(B, [1000], None, None, tiles=(32, 64))[0] == best
    best, _ = autotune.tune_batch(B, [1000], None, None, reps=1)
    assert best == (32, 4096) and B.tile == 32


def test_entry_of_another_tile_is_measured_again(cache):
    key = autotune.batch_key(6, 2.0, 8.0, [256], [1000])
    cache.write_text(json.dumps({key: {"tile": 64, "chunk": 16384}}))
    best, ms = autotune.tune_batch(Stand(), [1000], None, None, reps=1)
    assert best == (32, 4096) and ms
