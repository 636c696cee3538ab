"""What the autotuner keeps, on the CPU with made-up times: a knob set only
where it beats the launch that a call without knobs and tuned entries has."""
import json
import types

import pytest

from paper_1502_02389_amd import tune

ARCH, CUS = "gfx950", 256


def _operands(own_us, best_us):
    class Operands:
        bytes = 1 << 22

        def __init__(self, op, storage, elements, m=None, n=None, seed=11):
            pass

        def time_us(self, acc, k, reps=40, trials=5):
            if k is None:
                return own_us
            return best_us if (k.block, k.vec_bytes, k.unroll) == (256, 16, 4) else 2 * best_us

    return Operands


@pytest.fixture
def cache(tmp_path, monkeypatch):
    import torch

    path = tmp_path / "tuning.json"
    path.write_text(json.dumps({"device": {"arch": ARCH, "cus": CUS}, "entries": {
        "asum/f32/f32/20": {"knobs": {"block": 64}, "us": 9.0}, "asum/f32/f32/30": {"knobs": {"block": 128}, "us": 8.0}}}))
    monkeypatch.setenv("LIFT_TUNE_CACHE", str(path))
    monkeypatch.setenv("LIFT_IGNORE_TUNED", "1")     # main() sets it: put back after the test
    monkeypatch.setattr(tune, "_CACHE", None)
    monkeypatch.setattr(tune, "current_device", lambda: (ARCH, CUS))
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda i: types.SimpleNamespace(name="x"))
    return path


@pytest.mark.parametrize("own, best, kept", [(3.0, 2.5, True), (3.0, 2.99, False), (3.0, 3.4, False)])
def test_an_entry_has_to_beat_the_librarys_own_launch(cache, monkeypatch, capsys, own, best, kept):
    monkeypatch.setattr(tune, "Operands", _operands(own, best))
    tune.main(["--ops", "asum", "--sizes", "20", "--quick", "--write"])
    entries = json.loads(cache.read_text())["entries"]
    assert "asum/f32/f32/30" in entries                  # others stay
    assert ("asum/f32/f32/20" in entries) == kept        # the old one goes where the launch is faster
    if kept:
        assert entries["asum/f32/f32/20"]["knobs"]["unroll"] == 4
        assert entries["asum/f32/f32/20"]["own_us"] == own
