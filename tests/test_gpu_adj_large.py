"""The adjoint of cotangents near the largest FP32 number, on the end samples of the axes
above all: border tiles hold those doubled, which must not overflow where the transform
does not.  Against the streaming kernel (configuration 5), whose steps weight the ends."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402

STREAM_CONFIG = 5
MAX = torch.finfo(torch.float32).max


def positions(h, w, levels):
    """The corners, the middles of the edges and the middle of every detail band."""
    out = []
    for _ in range(levels):
        he, we = (h + 1) // 2, (w + 1) // 2
        for r0, r1, c0, c1 in ((0, he, we, w), (he, h, 0, we), (he, h, we, w)):
            out += [(r, c) for r in (r0, (r0 + r1) // 2, r1 - 1) for c in (c0, (c0 + c1) // 2, c1 - 1)]
        h, w = he, we
    return out


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("h,w,levels", [(40, 60, 1), (41, 61, 1), (40, 60, 2), (43, 227, 2), (64, 192, 3), (67, 201, 3),
                                        (700, 900, 2)])
def test_one_large_coefficient(tdt, h, w, levels):
    """Wherever the weighted steps give a finite image, the same image; never fewer finite samples."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    finite = 0
    for r, c in positions(h, w, levels):
        for part in (0.25, 0.4):
            x = torch.zeros((h, w), device=dev, dtype=tdt)
            x[r, c] = part * MAX
            want = d.adj(x, levels, config=STREAM_CONFIG)
            ok = torch.isfinite(want)
            finite += int(ok.all()) * (part > 0.3)
            for config in (None, 0):
                y = d.adj(x, levels, config=config)
                assert torch.equal(y[ok], want[ok]), (r, c, part, config)
    print("adj large", tdt, h, w, levels, "whole images finite at 0.4:", finite, flush=True)
    assert finite


@pytest.mark.parametrize("h,w,levels", [(41, 61, 1), (43, 227, 2), (67, 201, 3)])
def test_small_and_ordinary_values(h, w, levels):
    """The same at ordinary magnitudes and down to 2^-100, bit for bit; infinities stay where they were."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(workloads.planes(1, h, w, seed=5)[0]).to("cuda") - 0.5
    for scale in (1.0, 2.0 ** -100, 2.0 ** 90, 2.0 ** 110):
        print("adj scale", h, w, levels, scale, flush=True)
        y = d.adj(x * scale, levels)
        assert torch.equal(y, d.adj(x * scale, levels, config=STREAM_CONFIG))
        assert torch.equal(y, d.adj(x, levels) * scale)
