"""Infinities and NaN through the multi-level tiles, their border planes above all: the same
samples are non-finite, and all others equal, as with one launch a level (configuration 0; DD
13/7: the levels one by one)."""
import pytest

import workloads
from test_gpu_taps4 import one_by_one

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402


def image(h, w, tdt, seed):
    """An image with a NaN and infinities at a corner, on two edges and inside."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(workloads.planes(1, h, w, seed=seed)[0])
    x[0, 0], x[h - 1, w // 2], x[h // 2, w - 1], x[h // 3, w // 3] = float("inf"), float("nan"), -float("inf"), float("inf")
    return x.to("cuda").to(tdt)


def same(y, z):
    return torch.equal(torch.isnan(y), torch.isnan(z)) and torch.equal(torch.nan_to_num(y, nan=0.0, posinf=7.0, neginf=-7.0),
                                                                      torch.nan_to_num(z, nan=0.0, posinf=7.0, neginf=-7.0))


SHAPES = [(40, 224, 2), (83, 450, 2), (64, 192, 3), (33, 193, 3), (200, 1000, 4), (1501, 1499, 3), (3001, 2050, 2)]


@pytest.mark.parametrize("wavelet", ["cdf97", "cdf53f"])
@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("h,w,levels", SHAPES)
def test_two_tap(wavelet, tdt, h, w, levels):
    x = image(h, w, tdt, 111)
    print("nonfinite", wavelet, tdt, h, w, levels, flush=True)
    for direction in (d.fwd, d.inv):
        assert same(direction(x, wavelet, levels), direction(x, wavelet, levels, config=0)), direction.__name__
    if wavelet == "cdf97":
        assert same(d.adj(x, levels), d.adj(x, levels, config=0))


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("h,w,levels", SHAPES)
def test_four_tap(tdt, h, w, levels):
    x = image(h, w, tdt, 112)
    print("nonfinite dd137", tdt, h, w, levels, flush=True)
    for direction in (d.fwd, d.inv):
        assert same(direction(x, "dd137", levels), one_by_one(direction, x, levels)), direction.__name__
