"""What the tuner makes of its probes' times, with made-up times and no device: the
faster class mappings are applied only where the whole ensemble, timed as it runs, is
faster with them; probes keep the chains' elements; earlier choices are reused."""
import json

import numpy as np
import pytest

pytest.importorskip("torch")

from paper_1106_2899_amd import autotune  # noqa: E402


class FakeEnsemble:
    precision, device, sample_every = "fp32", "cpu", 10

    def __init__(self, N, E):
        self.N = np.asarray(N, dtype=np.int32)
        self.n_elements = E
        self.element_offsets = np.arange(E + 1) * self.N.size // E
        self.maps = {}

    def set_mapping(self, lo, hi, w, b):
        self.maps[lo, hi] = (w, b)


DEFAULTS = {(9, 16): (16, 1), (17, 32): (32, 1), (33, 64): (64, 1)}


def _tuned(monkeypatch, class_times, whole, E=4, flow=False, **kw):
    """class_times: {mapping: ns} that differ from 1.0; whole: (defaults, chosen)."""
    e = FakeEnsemble(np.resize(np.arange(9, 65), 5600), E)
    calls = []

    def fake(lengths, elements, mappings, *args):
        calls.append((np.array(lengths), np.array(elements), list(mappings)))
        if len(lengths) == e.N.size:
            return whole[1] if mappings else whole[0]
        (lo, hi, w, b), = mappings
        return class_times.get((w, b), 1.0 if (w, b) in DEFAULTS.values() else 2.0)

    monkeypatch.setattr(autotune, "_time_mappings", fake)
    kap = np.tile([0, 0.1, 0, 0, 0, 0, 0, 0, 0], (E, 1)) if flow else None
    return e, autotune.tune(e, kap, **kw), calls


def test_defaults_stay_when_the_whole_is_faster_with_them(monkeypatch):
    e, res, calls = _tuned(monkeypatch, {(32, 2): 0.8}, (1.0, 1.2))
    assert res.choices == DEFAULTS and e.maps == {(9, 16): (16, 1), (17, 32): (32, 1), (33, 64): (64, 1)}
    whole = [c for c in calls if len(c[0]) == e.N.size]
    assert [bool(c[2]) for c in whole] == [False, True]  # as created, then with the choices set


def test_choices_are_applied_when_the_whole_gains(monkeypatch):
    e, res, _ = _tuned(monkeypatch, {(32, 2): 0.8}, (1.0, 0.9))
    assert res.choices == {(9, 16): (32, 2), (17, 32): (32, 2), (33, 64): (32, 2)}
    assert e.maps == res.choices


def test_probes_keep_the_elements(monkeypatch):
    e, res, calls = _tuned(monkeypatch, {}, (1.0, 1.0), E=7, flow=True, probe_chains=600)
    elem = np.repeat(np.arange(7), np.diff(e.element_offsets))
    assert len(calls) == sum(len(autotune.candidates(c[1])) for c in DEFAULTS)  # nothing to compare as a whole
    for lengths, elements, _ in calls:
        assert len(lengths) == 600 and set(elements) == set(elem) and np.all(np.diff(elements) >= 0)


def test_cache_holds_what_was_decided(monkeypatch, tmp_path):
    path = str(tmp_path / "cache.json")
    with open(path, "w") as f:
        json.dump({"fp32:33-64": [32, 2]}, f)  # of an earlier form, without the comparison
    e, res, calls = _tuned(monkeypatch, {(32, 2): 0.8}, (1.0, 1.2), cache=path)
    assert calls and res.choices == DEFAULTS
    e, res, calls = _tuned(monkeypatch, {(32, 2): 0.8}, (1.0, 0.5), cache=path)
    assert not calls and res.choices == DEFAULTS and e.maps
    e, res, calls = _tuned(monkeypatch, {(32, 2): 0.8}, (1.0, 0.5), flow=True, cache=path)
    assert calls and res.choices != DEFAULTS
