"""The ensemble tuner's cache (paper_1912_02457_amd/tune.py) on the CPU, with a
stand-in for the ensemble: an entry is used again for the same members and
candidates only, and one from before the present launch scheme never."""

import hashlib
import json
from types import SimpleNamespace

import pytest


@pytest.fixture
def tuner(monkeypatch):
    import torch
    from paper_1912_02457_amd import swe, tune
    tried = []

    class FakeEnsemble:
        def __init__(self, members, *, rows_per_wave=0, chunk=0):
            tried.append((rows_per_wave, chunk))

        def use_graphs(self, on):
            pass

        def step(self, n):
            pass

        def close(self):
            pass

    monkeypatch.setattr(swe, "Ensemble", FakeEnsemble)
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda dev=None: "card")
    monkeypatch.setattr(torch.cuda, "synchronize", lambda dev=None: None)

    def run(cache, **kw):
        tried.clear()
        members = [SimpleNamespace(nx=nx, ny=ny, device="cuda:0", wind_field=kw.get("wind"),
                                   params=SimpleNamespace(north_projection=kw.get("north", 0),
                                                          compensated_state=kw.get("comp", 1)))
                   for nx, ny in kw.get("sizes", [(300, 200), (100, 50)])]
        args = {k: kw[k] for k in ("rows", "chunks") if k in kw}
        rows, chunk, rep = tune.autotune_ensemble(members, steps=1, cache=str(cache), **args)
        assert rep["cached"] == (not tried)
        return rep["cached"], list(tried)

    return run


def test_only_the_same_members_and_candidates_share_an_entry(tuner, tmp_path):
    cache = tmp_path / "tune.json"
    kinds = [dict(), dict(comp=0), dict(north=1), dict(wind=object()), dict(sizes=[(300, 200)]), dict(rows=(8,)),
             dict(chunks=(2,)), dict(rows=(8, 16))]
    for kw in kinds:
        assert not tuner(cache, **kw)[0], kw
    for kw in kinds:
        assert tuner(cache, **kw)[0], kw
    # the order of the members does not matter, nor does how the candidates are given
    assert tuner(cache, sizes=[(100, 50), (300, 200)])[0]
    assert tuner(cache, rows=iter([8, 16]))[0]


def test_entries_of_the_earlier_launch_scheme_are_not_used(tuner, tmp_path):
    cache = tmp_path / "tune.json"
    old = hashlib.sha1(json.dumps(["card", False, [(100, 50), (300, 200)]]).encode()).hexdigest()[:20]
    cache.write_text(json.dumps({old: {"rows": 64, "chunk": 4}}))
    cached, tried = tuner(cache)
    assert not cached and len(tried) > 1
    assert old in json.loads(cache.read_text())


def test_the_built_in_choice_is_a_candidate(tuner, tmp_path):
    cached, tried = tuner(tmp_path / "tune.json")
    assert not cached and (0, 1) in tried
