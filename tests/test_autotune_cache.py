"""The autotuner's cache: a stored choice holds for the library and the candidates that it was measured with (no GPU)."""
import json

import pytest

from paper_2411_02703_amd import autotune, scenes


class Measured(Exception):
    pass


def _step(opts):
    raise Measured


def _tune(**kw):
    return autotune.tune_batched(_step, 1000, [scenes.identity_camera(50.0, 50.0, 32.0, 24.0, 64, 48)], 0, **kw)


@pytest.fixture
def store(tmp_path, monkeypatch):
    path = tmp_path / "autotune.json"
    monkeypatch.setattr(autotune, "_CACHE", str(path))
    key = autotune.cache_key(1000, [scenes.identity_camera(50.0, 50.0, 32.0, 24.0, 64, 48)], 0)
    return lambda entry: path.write_text(json.dumps({key: entry}))


def test_a_choice_of_this_library_and_these_candidates_is_taken(store):
    best = autotune.CANDIDATES[1]
    store([list(best), {}, autotune.identity(autotune.CANDIDATES)])
    assert _tune() == (best, {})


@pytest.mark.parametrize("entry", [
    [[16, 8, 1, 8, 512], {}],                                   # stored before entries named their library
    [[16, 8, 1, 4, 512], {}, "another library"],
    [], "text", [[16, 8, 1, 4, 512]],
])
def test_other_choices_are_measured_again(store, entry):
    store(entry)
    with pytest.raises(Measured):
        _tune()


def test_a_choice_among_other_candidates_is_measured_again(store):
    some = autotune.CANDIDATES[:2]
    store([list(some[0]), {}, autotune.identity(some)])
    assert _tune(candidates=some) == (some[0], {})
    with pytest.raises(Measured):
        _tune()


def test_the_identity_follows_the_library_file(tmp_path, monkeypatch):
    from paper_2411_02703_amd import binding

    ids = []
    for text in (b"one", b"two", b"one"):
        lib = tmp_path / "libgs.so"
        lib.write_bytes(text)
        monkeypatch.setattr(binding, "LIB_PATH", str(lib))
        ids.append(autotune.identity(autotune.CANDIDATES))
    assert ids[0] == ids[2] != ids[1]
