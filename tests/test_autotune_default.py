"""The autotuner's answer holds the time of a plan without a hint, which takes
kernels that hinted plans leave out; entries cached before it was timed are
timed again.  On the CPU: launches are replaced by a table of times."""
import json
import types

import pytest

from paper_1307_5700_amd import autotune

KW = dict(nchans=1024, f_ch0_mhz=398.0, df_mhz=0.02, tsamp_s=51.2e-6, ndms=640, dm_start=0.0, dm_step=0.2)


@pytest.fixture
def times(monkeypatch):
    t = {0: 0.49, 1: 1.75, 2: 2.0, 3: None}
    asked = []

    def time_tiling(kw, dtype, rfi, nsamps, hint, x=None):
        asked.append(hint)
        return t[hint]
    monkeypatch.setattr(autotune, "time_tiling", time_tiling)
    monkeypatch.setattr(autotune, "_synthetic_chunk", lambda *a: None)
    monkeypatch.setattr(autotune.A, "num_tilings", lambda: 3)
    monkeypatch.setattr(autotune.torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(autotune.torch.cuda, "get_device_properties",
                        lambda d: types.SimpleNamespace(gcnArchName="gfx950", name="gpu"))
    return asked


def test_default_time_stands_beside_the_fastest_tiling(times, tmp_path):
    path = str(tmp_path / "t.json")
    r = autotune.best_tiling(KW, "u8", False, 65536, path=path)
    assert sorted(times) == [0, 1, 2, 3]
    assert r == {"hint": 1, "ms": 1.75, "all": {"1": 1.75, "2": 2.0, "3": None}, "default_ms": 0.49}
    assert autotune.best_tiling(KW, "u8", False, 65536, path=path) == r and len(times) == 4
    assert autotune.best_shared_tiling([KW, KW], "u8", False, [65536, 65536], path) == 1


def test_entries_without_it_are_timed_again(times, tmp_path):
    path = str(tmp_path / "t.json")
    old = {"hint": 2, "ms": 1.0, "all": {"1": 1.5, "2": 1.0, "3": None}}
    with open(path, "w") as f:
        json.dump({autotune._key(KW, "u8", False, 65536): old}, f)
    r = autotune.best_tiling(KW, "u8", False, 65536, path=path)
    assert r["default_ms"] == 0.49 and r["hint"] == 1 and len(times) == 4
    assert list(json.load(open(path)).values()) == [r]
