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
