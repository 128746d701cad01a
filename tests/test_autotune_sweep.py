"""The autotuner's coordinate descent on the host: a knob that moves the time is kept, one without effect never is, even
when its trial happens to be faster; every trial is recorded; a changed output stops the sweep."""
import time

import pytest

torch = pytest.importorskip("torch")

import paper_2311_10337_amd as ce
from paper_2311_10337_amd import autotune


@pytest.fixture
def no_device(monkeypatch):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)


def sweep(seconds, digest=lambda out: (1,)):
    """A call that takes seconds(knobs)."""
    def run():
        time.sleep(seconds(ce.current_tuning() or {}))
    return autotune.sweep(run, digest, reps=3,
                          candidates={"krt_level_bits": (3, 6), "list_grid": (1024, 2048)})


def test_knob_without_effect_is_never_kept(no_device):
    res = sweep(lambda k: 0.004 if k.get("krt_level_bits") == 6 else 0.02)
    assert res["knobs"] == {} and len(res["trials"]) == 5


def test_knob_with_effect_is_kept(no_device):
    res = sweep(lambda k: 0.004 if k.get("list_grid") == 2048 else 0.02)
    assert res["knobs"] == {"list_grid": 2048} and res["tuned_ms"] < res["default_ms"]


def test_changed_output_stops(no_device):
    with pytest.raises(RuntimeError):
        sweep(lambda k: 0.0, lambda out: (len(ce.current_tuning() or {}),))
