"""The committed table of tuned configurations and the tuner's record."""
import pytest

import paper_1704_08657_amd as d
from paper_1704_08657_amd import autotune


@pytest.fixture
def gfx950(monkeypatch):
    monkeypatch.setattr(autotune, "_arch", "gfx950")
    monkeypatch.setattr(autotune, "_cache", None)
    monkeypatch.setattr(d, "_tuned", {})


@pytest.mark.parametrize("h,w", [(5000, 300), (64, 8192), (4100, 4100), (8192, 8192), (256, 256)])
@pytest.mark.parametrize("levels", [1, 5])
def test_table_leaves_the_choice_to_the_library(gfx950, h, w, levels):
    """An entry covers a whole size class by the longer side, where the library's own
    choice goes by the level's samples: the committed table has none."""
    for direction in ("fwd", "inv", "adj"):
        for dtype in (d.DWT2_F32, d.DWT2_BF16, d.DWT2_F16):
            assert d.tuned_config(direction, "cdf97", dtype, h, w, levels) is None


def _timer(ms):
    """A _time that runs the call once and takes its time from `ms`."""
    def time(torch, fn, steps=0, warm=0):
        return ms[fn(0)]
    return time


def test_tune_case_times_the_given_configurations(gfx950, monkeypatch):
    """run(config, i) is called with indices; they alone are returned, and the fastest is recorded."""
    monkeypatch.setattr(autotune, "_time", _timer({0: 3.0, 2: 1.0, 4: 2.0}))
    seen = []

    def run(config, i):
        seen.append(config)
        return (d.DWT2_FLAG_KERNEL(config) >> d.DWT2_FLAG_KERNEL_SHIFT) - 1     # an index, or a TypeError

    best, times = autotune.tune_case("fwd", "cdf97", "f32", 512, 512, 1, run, configs=[0, 2, 4])
    assert best == 2 and times == {0: 3.0, 2: 1.0, 4: 2.0} and sorted(times) == [0, 2, 4]
    assert seen[:3] == [0, 2, 4]
    assert d.tuned_config("fwd", "cdf97", d.DWT2_F32, 512, 512, 1) == 2


@pytest.mark.parametrize("own,recorded", [(0.5, None), (1.5, 2)])
def test_tune_case_leaves_a_faster_choice_of_the_library(gfx950, monkeypatch, own, recorded):
    monkeypatch.setattr(autotune, "_time", _timer({0: 3.0, 2: 1.0, None: own}))
    best, times = autotune.tune_case("fwd", "cdf97", "f32", 512, 512, 5, lambda config, i: config, configs=[0, 2])
    assert best == 2 and times == {0: 3.0, 2: 1.0}
    assert d.tuned_config("fwd", "cdf97", d.DWT2_F32, 512, 512, 5) == recorded


@pytest.mark.gpu
def test_calls_after_tune_use_its_result(tmp_path, monkeypatch):
    """Calls of the process that ran tune() go by what it found, not by what its timed calls used."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ms = iter(range(1000, 0, -1))       # every configuration faster than the one before

    def time(torch, fn, steps=0, warm=0):
        fn(0)
        return next(ms)

    monkeypatch.setattr(autotune, "_time", time)
    monkeypatch.setattr(autotune, "_cache", {})
    monkeypatch.setattr(d, "_tuned", {})
    result = autotune.tune(sizes=(64,), levels=(1,), quick=True, out=str(tmp_path / "t.json"),
                           log=lambda line: None, dtypes=("i32",))
    for direction in ("fwd", "inv"):
        best = result[autotune.key(autotune.arch_name(), direction, "cdf53", "i32", 64, 64, 1)]
        assert best is not None and d.tuned_config(direction, "cdf53", d.DWT2_I32, 64, 64, 1) == best
