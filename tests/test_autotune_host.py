"""The autotuner's choices on the host (no GPU work): the timing calls are replaced."""
import json

import pytest

import paper_2302_13524_amd as tm


class Times:
    def __init__(self, monkeypatch):
        self.timed, self.set = [], []
        monkeypatch.setattr(tm, "tm_tune_time", lambda ctx, n1, n2, K, P, v, *a: self._time(("digits", v)))
        monkeypatch.setattr(tm, "tm_tune_config",
                            lambda ctx, n1, n2, K, P, cfg, *a: (self._time(("full", cfg)), 10.0))
        monkeypatch.setattr(tm, "tm_set_config", lambda ctx, n1, n2, cfg: self.set.append(cfg))
        monkeypatch.setattr(tm, "tm_set_variant", lambda ctx, n1, n2, v: self.set.append(v))

    def _time(self, what):
        self.timed.append(what)
        return 100.0 - len(self.timed)  # each call faster than the last, as on a ramping clock


@pytest.mark.parametrize("n1,n2", [(32, 32), (64, 32), (64, 64), (128, 64), (8, 8)])
def test_one_kernel_is_timed_once(monkeypatch, n1, n2):
    # both digit orders of these grids run the same kernels
    t = Times(monkeypatch)
    e = tm.autotune(None, n1, n2, 4, 16)
    assert t.timed == [("digits", 0)] and e["variant"] == 0 and len(e["us"]) == 2
    t = Times(monkeypatch)
    e = tm.autotune(None, n1, n2, 4, 16, space="full")
    assert ("full", 1) not in t.timed
    assert e["candidates"]["1"] == e["candidates"]["0"] and e["config"] != 1
    assert set(e["candidates"]) == {str(c) for c in range(8) if tm.tm_config_info(n1, n2, c)}


def test_two_kernels_are_both_timed(monkeypatch):
    t = Times(monkeypatch)
    e = tm.autotune(None, 64, 128, 4, 16)
    assert t.timed == [("digits", 0), ("digits", 1)] and e["variant"] == 1 and t.set == [1]


@pytest.mark.parametrize("space", ["digits", "full"])
def test_entry_of_other_kernels_is_timed_anew(monkeypatch, tmp_path, space):
    cache = str(tmp_path / "tune.json")
    key = "gfx950:128x64:K4:f32" + (":full" if space == "full" else "")
    old = {"config": 3, "variant": 1, "candidates": {}, "rows": 16} if space == "full" else {"variant": 1, "us": [2.0, 1.0]}
    json.dump({key: old, "other": {"variant": 0}}, open(cache, "w"))
    t = Times(monkeypatch)
    e = tm.autotune(None, 128, 64, 4, 16, cache=cache, space=space)
    assert t.timed and json.load(open(cache)) == {key: e, "other": {"variant": 0}}
    t = Times(monkeypatch)
    assert tm.autotune(None, 128, 64, 4, 16, cache=cache, space=space) == e and not t.timed
    monkeypatch.setattr(tm, "_kernels_revision", lambda: "another library")
    tm.autotune(None, 128, 64, 4, 16, cache=cache, space=space)
    assert t.timed


def test_shape_of_the_kernels_that_run():
    # mixed-axis kernels of configurations 0 and 1: one row of N / 16 threads
    for n1, n2 in [(32, 32), (64, 32), (64, 64), (128, 64)]:
        for cfg in (0, 1):
            assert tm.tm_config_kernel(n1, n2, cfg) == (0, n1 * n2 // 16, 1, 16)
    # one axis per pass: as tm_config_info; the digit order changes axes of 32 and 128 points alone
    for n1, n2, cfg, kernel in [(8, 8, 1, 0), (16, 16, 1, 0), (8, 32, 1, 1), (32, 64, 1, 1), (64, 128, 1, 1),
                                (128, 64, 3, 3), (64, 64, 3, 2), (64, 64, 4, 4), (64, 64, 5, 4)]:
        assert tm.tm_config_kernel(n1, n2, cfg) == (kernel, *tm.tm_config_info(n1, n2, cfg))
    for bad in [(-1, 32, 32), (8, 32, 32), (0, 3, 8), (4, 128, 64)]:
        assert tm.tm_config_kernel(bad[1], bad[2], bad[0]) is None
