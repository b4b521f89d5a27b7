"""Batched calls that name no configuration take two levels in a launch where
that pays: bit for bit one launch per level (configuration 0), on batches whose
tiles all run at once and larger ones, with image sides at the ends of the
two-level tiles (224 pixels wide, 40 or 72 high), odd and even level counts."""
import random

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1704_08657_amd as d  # noqa: E402


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("count,lo,hi", [(5, 40, 230), (24, 64, 700), (40, 200, 1300), (1100, 16, 60)])
def test_two_level_launches(tdt, count, lo, hi):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    r = random.Random(count)
    shapes = [(40, 224), (41, 225), (72, 223), (73, 450)] + [(r.randint(lo, hi), r.randint(lo, hi)) for _ in range(count)]
    g = torch.Generator(device=dev).manual_seed(7)
    xs = [torch.rand(s, device=dev, generator=g).to(tdt) for s in shapes]
    for levels in (2, 3, 4):
        print("batched pair", tdt, count, levels, flush=True)
        for y, z in zip(d.fwd_batched(xs, levels), d.fwd_batched(xs, levels, config=0)):
            assert torch.equal(y, z), (levels, tuple(y.shape))


@pytest.mark.parametrize("tdt", [torch.float32, torch.bfloat16])
def test_three_level_tall_tiles(tdt):
    """150 small images: three levels in tiles 64 pixels high."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda", 0)
    r = random.Random(3)
    shapes = [(64, 192), (65, 193), (63, 194)] + [(r.randint(33, 80), r.randint(20, 200)) for _ in range(150)]
    g = torch.Generator(device=dev).manual_seed(8)
    xs = [torch.rand(s, device=dev, generator=g).to(tdt) for s in shapes]
    print("batched triple", tdt, flush=True)
    for y, z in zip(d.fwd_batched(xs, 3), d.fwd_batched(xs, 3, config=0)):
        assert torch.equal(y, z), tuple(y.shape)
