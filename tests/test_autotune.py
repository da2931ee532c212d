"""Installing the autotuner's cached choices (autotune.apply_cache).  CPU only:
the calls on the library are recorded."""
import json

import pytest

from paper_2407_18304_amd import autotune, mgrhd


@pytest.fixture
def calls(monkeypatch, tmp_path):
    """apply_cache of a record for N_g groups; returns the set_variant calls."""
    monkeypatch.setattr(autotune, "arch", lambda: "gfx950")
    made = []
    monkeypatch.setattr(mgrhd, "set_variant", lambda *a: made.append(a))

    def apply(ng, lanes, groups, waves):
        made.clear()
        path = tmp_path / "cache.json"
        path.write_text(json.dumps({"gfx950": {"single": {f"{ng}:1": dict(
            lanes_per_cell=lanes, groups_per_lane=groups, waves_per_simd=waves)}}}))
        autotune.apply_cache(str(path))
        return list(made)
    return apply


@pytest.mark.parametrize("ng,lanes,groups,waves", [(16, 8, 2, 3), (16, 8, 2, 4), (64, 32, 2, 4),
                                                   (11, 8, 2, 3)])
def test_the_librarys_own_choice_is_left_to_it(calls, ng, lanes, groups, waves):
    """A set variant holds for every launch size; the library's own choice
    splits the cells of small launches over more lanes."""
    assert calls(ng, lanes, groups, waves) == [(ng, 0, 0)]


@pytest.mark.parametrize("ng,lanes,groups,waves", [(16, 4, 4, 2), (16, 16, 1, 4), (11, 8, 2, 4)])
def test_other_choices_are_installed(calls, ng, lanes, groups, waves):
    assert calls(ng, lanes, groups, waves) == [(ng, 0, 0), (ng, lanes, groups, waves)]


def test_shipped_choices_are_variants_of_the_library():
    for rec in autotune.load_cache()["gfx950"]["single"].values():
        assert (rec["lanes_per_cell"], rec["groups_per_lane"],
                rec["waves_per_simd"]) in mgrhd.variants()
