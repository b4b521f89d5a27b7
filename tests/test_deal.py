"""How the tile kernels' grids deal their tiles over the XCDs: tests/host/deal_check.cpp,
compiled against the library's header."""
from test_batch_plan import build_and_run, needs_tools


@needs_tools
def test_every_tile_is_dealt_once_and_evenly(tmp_path):
    r = build_and_run(tmp_path, "deal_check")
    assert r.returncode == 0, r.stdout + r.stderr
    assert "bad 0" in r.stdout
