"""Stacks of planes less high than a tile: the waves whose rows lie below the image leave
before the first step.  Bit for bit the streaming kernel's results (configuration 5, which
has no tiles), at the heights where one wave more stays, for one launch a level and for
two and three levels in one."""
import pytest

import workloads
from oracle import lifting

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402

STREAM_CONFIG = 5


@pytest.mark.parametrize("wavelet,tdt", [("cdf97", torch.float32), ("cdf53", torch.int32), ("cdf53f", torch.float32)])
@pytest.mark.parametrize("n", [3, 700])
def test_low_planes(wavelet, tdt, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for h in (2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 21, 24, 25, 28, 29, 33, 41, 48, 49, 57, 64, 65, 73):
        w = 10 + h % 7
        x = torch.from_numpy(workloads.planes(n, h, w, seed=h)).to("cuda")
        x = (x * 255).round().to(tdt) if tdt == torch.int32 else x.to(tdt)
        for levels in range(1, min(3, lifting.max_levels(h, w)) + 1):
            print("low planes", wavelet, n, h, w, levels, flush=True)
            y = d.fwd(x, wavelet, levels, config=STREAM_CONFIG)
            for config in (None, 0, 1, 3):
                assert torch.equal(d.fwd(x, wavelet, levels, config=config), y)
                assert torch.equal(d.inv(y, wavelet, levels, config=config),
                                   d.inv(y, wavelet, levels, config=STREAM_CONFIG))
                if wavelet == "cdf97":
                    assert torch.equal(d.adj(y, levels, config=config), d.adj(y, levels, config=STREAM_CONFIG))


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16])
def test_low_images_in_a_batch(tdt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    xs = [torch.from_numpy(workloads.planes(1, h, 9 + h % 5, seed=h)[0]).to("cuda").to(tdt) for h in range(4, 80)] * 10
    for levels in (1, 2):
        print("low batch", tdt, levels, flush=True)
        for x, y in zip(xs, d.fwd_batched(xs, levels)):
            assert torch.equal(y, d.fwd(x, "cdf97", levels, config=0)), tuple(x.shape)
