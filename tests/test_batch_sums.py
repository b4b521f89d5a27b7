"""What a batched call sums over its images before it launches: tests/host/batch_sums_check.cpp,
compiled against the library's headers."""
from test_batch_plan import build_and_run, needs_tools


@needs_tools
def test_one_pass_sums(tmp_path):
    r = build_and_run(tmp_path, "batch_sums_check")
    assert r.returncode == 0, r.stdout + r.stderr
    assert "bad 0" in r.stdout
