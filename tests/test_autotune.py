"""The tile tuner's choices, with the timings given: it also times the automatic
setting, so that a tuned call is never slower than an untuned one, and takes no
result from a cache file that another build of the library wrote."""
import json
import types

import pytest
import torch

from paper_2609_10816_amd import autotune, ctmhd


@pytest.fixture
def tuner(monkeypatch):
    """tune(kind, ms, cache) with ms(tile) the time of a setting."""
    monkeypatch.setattr(autotune, "_cache", {})
    tried = []

    class Stepper:
        def __init__(self, params, state):
            tried.append(params.tile)

    monkeypatch.setattr(ctmhd, "Stepper", Stepper)
    monkeypatch.setattr(ctmhd, "BatchedStepper", Stepper)
    state = types.SimpleNamespace(cons=[torch.zeros(1)], bface=[], n=(16, 16, 16),
                                  shapes=[(16, 16, 16), (8, 32, 8)])

    def tune(kind, ms, cache_file=None):
        monkeypatch.setattr(autotune, "_time_calls", lambda prepare, fn, reps: ms(tried[-1]))
        f = autotune.tune_single if kind == "single" else autotune.tune_batched
        return f(ctmhd.make_params(recon="ppm"), state, steps=1, reps=1, cache_file=cache_file)[0]

    return tune


@pytest.mark.parametrize("kind", ["single", "batched"])
def test_automatic_chunk_is_tried(tuner, kind):
    # the automatic chunk is the fastest: below the shortest explicit one
    assert tuner(kind, lambda tile: 1.0 + (tile & 255) + 0.1 * (tile >> 8)) & 255 == 0


@pytest.mark.parametrize("kind", ["single", "batched"])
def test_explicit_chunk_still_wins_where_it_is_faster(tuner, kind):
    assert tuner(kind, lambda tile: 1.0 + abs((tile & 255) - 16)) & 255 == 16


@pytest.mark.parametrize("kind", ["single", "batched"])
def test_cache_of_another_library_is_not_used(tuner, kind, tmp_path, monkeypatch):
    cache = str(tmp_path / "tiles.json")
    assert tuner(kind, lambda tile: 1.0 + abs((tile & 255) - 64), cache) & 255 == 64
    autotune._cache.clear()
    # the same library: served from the file, whatever the timings are now
    assert tuner(kind, lambda tile: 1.0 + (tile & 255), cache) & 255 == 64
    autotune._cache.clear()
    other = tmp_path / "libctmhd.so"
    other.write_bytes(b"another build")
    monkeypatch.setattr(ctmhd, "LIB_PATH", str(other))
    assert tuner(kind, lambda tile: 1.0 + (tile & 255), cache) & 255 == 0
    assert len(json.load(open(cache))) == 2
